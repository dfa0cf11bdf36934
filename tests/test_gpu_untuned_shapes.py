"""The launch shapes of sweeps that are not tuned: what the rule picks, by the
kernel instances a solve's timing report names, and that each branch gives a
right-hand side of a batch the bits of its single solve."""
import re

import numpy as np
import pytest

import lattice_inputs as li
from gpu_util import note, random_links

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def wd():
    from paper_1207_2223_amd import wd
    wd.lib()
    return wd


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


def same_bits(a, b):
    import torch
    return torch.equal(torch.view_as_real(a).view(torch.int64), torch.view_as_real(b).view(torch.int64))


def solves(wd, dims, recon, code, nrhs, maxiter):
    """A batch, and the single solves of its first and last right-hand side."""
    import torch
    V = li.volume(dims)
    lat = wd.Lattice(dims)
    lat.gauge_load(random_links(V, 7), recon=recon)
    g = torch.Generator(device="cuda")
    g.manual_seed(8)
    b = torch.randn((nrhs, V // 2, 4, 3), dtype=torch.complex128, device="cuda", generator=g)
    kap = np.linspace(0.08, 0.1, nrhs)
    p = wd.solver_params(prec=code, maxiter=maxiter, tol=1e-14, delta=0.3)
    x = torch.empty_like(b)
    lat.cg_solve(x, b, kap, p)
    for j in (0, nrhs - 1):
        y = torch.empty_like(b[:1])
        lat.cg_solve(y, b[j:j + 1].contiguous(), kap[j:j + 1], p)
        note(f"{dims} recon {recon} code {code:#x} rhs {j} of {nrhs}")
        assert same_bits(y[0], x[j])
    lat.close()


@pytest.mark.parametrize("dims,nrhs", [((18, 14, 18, 18), 37),  # beyond the caches, no slabs: two RHS a lane
                                       ((16, 16, 16, 8), 7),    # t slabs
                                       ((16, 16, 18, 16), 42),  # t slabs, beyond the caches
                                       ((16, 16, 16, 16), 48),  # z slabs, two RHS a lane
                                       ((16, 12, 16, 18), 8),   # z slabs of 32 sites, two lanes a site and two RHS a lane
                                       ((16, 12, 16, 18), 6),   # ... one RHS a lane
                                       ((16, 12, 16, 18), 7),   # an odd batch: dispatch order
                                       ((16, 12, 16, 18), 11),  # ... with few sites in flight
                                       ((16, 12, 16, 18), 31)]) # ... in z slabs again
@pytest.mark.parametrize("recon", [12, 18])
def test_fp64_batches_equal_single_solves(wd, recon, dims, nrhs):
    solves(wd, dims, recon, wd.WD_F64, nrhs, 12)


@pytest.mark.parametrize("dims,prec,recon", [((32, 32, 32, 32), "f64", 12), ((32, 32, 32, 32), "f32", 12), ((32, 32, 32, 32), "f16", 12),
                                             ((32, 32, 32, 64), "f32r8", 12), ((32, 32, 32, 64), "f16r8", 12)])
def test_single_solves_with_streamed_links_equal_a_batch(wd, prec, recon, dims):
    """One right-hand side over links beyond the last-level cache (FP64 and FP32
    12-real, FP32 8-real) reads them non-temporally; a batch of two does not."""
    code = {"f64": wd.WD_F64, "f32": wd.WD_F32, "f16": wd.WD_F16, "f32r8": wd.WD_F32 | wd.WD_LINKS_R8,
            "f16r8": wd.WD_F16 | wd.WD_LINKS_R8}[prec]
    solves(wd, dims, recon, code, 2, 6)
