"""The launch shapes of sweeps that are not tuned: what the rule picks, by the
kernel instances a solve's timing report names."""
import re

import numpy as np
import pytest

import lattice_inputs as li
from gpu_util import note

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def wd():
    from paper_1207_2223_amd import wd
    wd.lib()
    return wd


def random_links(V, seed):
    """[V][4][3][3] random SU(3) links made on the device."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    a, b = (torch.randn((V, 4, 3), dtype=torch.complex128, device="cuda", generator=g) for _ in range(2))
    a = a / torch.linalg.vector_norm(a, dim=-1, keepdim=True)
    b = b - (a.conj() * b).sum(-1, keepdim=True) * a
    b = b / torch.linalg.vector_norm(b, dim=-1, keepdim=True)
    return torch.stack([a, b, torch.linalg.cross(a, b, dim=-1).conj()], dim=-2).contiguous()


@pytest.mark.parametrize("dims,nrhs", [((24, 24, 24, 24), 3), ((24, 24, 24, 24), 5), ((24, 24, 24, 24), 6), ((24, 24, 24, 24), 7),
                                       ((24, 24, 24, 24), 8), ((16, 12, 16, 18), 5), ((24, 24, 24, 48), 5)])
@pytest.mark.parametrize("recon", [12, 18])
def test_few_slots_of_an_fp64_batch_stay_empty(wd, recon, dims, nrhs):
    """On lattices that only take z slabs of 32-site tiles, with two lanes a
    site: an odd batch leaves a lane without a right-hand side in every site's
    last group, so small odd batches take another shape."""
    import torch
    V = li.volume(dims)
    lat = wd.Lattice(dims)
    lat.gauge_load(random_links(V, 5), recon=recon)
    g = torch.Generator(device="cuda")
    g.manual_seed(6)
    b = torch.randn((nrhs, V // 2, 4, 3), dtype=torch.complex128, device="cuda", generator=g)
    wd.wd_timing_enable(lat.ctx, True)
    lat.cg_solve(torch.empty_like(b), b, np.full(nrhs, 0.1), wd.solver_params(maxiter=3, poll=3, tol=1e-14))
    names = sorted(wd.wd_timing_report(lat.ctx))
    note(f"{dims} {nrhs} RHS, {recon}-real: {names}")
    assert names
    for n in names:
        nr, rl = (int(v) for v in re.match(r"dslash_kernel<0, \d+, (\d+), (\d+),", n).groups())
        slots = -(-nrhs // (nr * rl)) * nr * rl
        assert (slots - nrhs) / slots <= 0.125
    lat.close()
