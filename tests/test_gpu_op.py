"""Operator calls that read the caller's field in the sweep itself against the
same call through a packed copy (taken when input and output overlap), and
against the launch-shape entry point, which packs, sweeps and unpacks: the
same bits in every storage format, on lattices with a partial last
work-group, with a single tile, and with extents of 2."""
import numpy as np
import pytest

import lattice_inputs as li
from gpu_util import dev, empty_like_dev, host, note, rel_err

pytestmark = pytest.mark.gpu

# the relative 2-norm bounds of tests/test_gpu_dslash.py (the packed links of the
# last, partial work-group of the packing kernel are among those read here)
TOL = {"f64": 1e-12, "f32": 2e-7, "f32l16": 4.5e-4, "f32r18": 2e-7, "f32r8": 6e-7, "f16": 6e-4, "f16l16": 9e-4,
       "f16r18": 6e-4, "f16r8": 6e-4, "i16": 6e-5, "i16l16": 4.5e-4}
CODES = {"f64": 0, "f32": 1, "f32l16": 1 | 0x10, "f32r18": 1 | 0x20, "f32r8": 1 | 0x40, "f16": 2, "f16l16": 2 | 0x10,
         "f16r18": 2 | 0x20, "f16r8": 2 | 0x40, "i16": 3, "i16l16": 3 | 0x10}


@pytest.fixture(scope="module")
def wd():
    from paper_1207_2223_amd import wd
    wd.lib()
    return wd


def bits(t):
    return host(t).view(np.uint64)


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 4, 10, 2), (10, 14, 6, 6)])
@pytest.mark.parametrize("prec", sorted(CODES))
def test_canonical_and_packed_input_give_the_same_bits(wd, oracle, prec, dims):
    V = li.volume(dims)
    U = li.random_su3_field(dims, 0.5, seed=51)
    for recon in ((12, 18) if prec == "f64" else (12,)):
        lat = wd.Lattice(dims)
        lat.gauge_load(dev(U), recon=recon)
        for part, n in ((wd.WD_EVEN, V // 2), (wd.WD_ODD, V // 2), (wd.WD_FULL, V)):
            psi = li.gaussian_spinor(n, seed=60 + part)
            psi[n // 2] = 0.0  # a site whose norm is zero
            for dag in (0, 1):
                out = empty_like_dev(psi)
                lat.dslash(out, dev(psi), part, dag, CODES[prec])
                same = dev(psi)
                lat.dslash(same, same, part, dag, CODES[prec])
                note(f"op {prec} {dims} recon {recon} part {part} dag {dag}")
                assert np.array_equal(bits(out), bits(same))
                if part != wd.WD_FULL:
                    shaped = empty_like_dev(psi)
                    wd.wd_dslash_shaped(lat.ctx, shaped, dev(psi), part, dag, CODES[prec])
                    assert np.array_equal(bits(out), bits(shaped))
                ref = oracle.hop(dims, U, psi, dagger=bool(dag)) if part == wd.WD_FULL else oracle.hop_eo(
                    dims, U, psi, 1 if part == wd.WD_ODD else 0, dagger=bool(dag))
                assert rel_err(host(out), ref) <= TOL[prec]
        lat.close()


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (10, 14, 6, 6), (48, 16, 32, 18)])
@pytest.mark.parametrize("recon", [12, 18])
def test_normal_operator_in_place_and_from_an_unaligned_field(wd, oracle, recon, dims):
    """Both operators, out of place and in place, and on a field that starts
    at an odd multiple of 8 bytes (complex numbers need no more); the last
    lattice is above the sizes whose 18-real sweeps read canonical input."""
    import ctypes
    import torch
    V = li.volume(dims)
    U = li.random_su3_field(dims, 0.4, seed=52)
    lat = wd.Lattice(dims)
    lat.gauge_load(dev(U), recon=recon)
    for eo, n in ((1, V // 2), (0, V)):
        psi = li.gaussian_spinor(n, seed=71 + eo)
        out, same = empty_like_dev(psi), dev(psi)
        lat.mdagm(out, dev(psi), 0.14, eo=eo)
        lat.mdagm(same, same, 0.14, eo=eo)
        assert np.array_equal(bits(out), bits(same))
        ref = oracle.mhatdag_mhat(dims, U, 0.14, psi) if eo else oracle.mdagm(dims, U, 0.14, psi)
        assert rel_err(host(out), ref) <= 1e-12
        buf = torch.zeros(2 * psi.size + 1, dtype=torch.float64, device="cuda")
        buf[1:] = torch.view_as_real(dev(psi)).reshape(-1)
        odd = torch.zeros(2 * psi.size + 1, dtype=torch.float64, device="cuda")
        wd._check(wd.lib().wd_mdagm(lat.ctx, ctypes.c_void_p(odd.data_ptr() + 8), ctypes.c_void_p(buf.data_ptr() + 8), 0.14, eo))
        assert np.array_equal(host(odd[1:]), torch.view_as_real(out).reshape(-1).cpu().numpy())
    lat.close()


@pytest.mark.parametrize("dims", [(2, 6, 4, 10), (4, 4, 4, 4)])
@pytest.mark.parametrize("src", [(0, 2, 1, 3), (1, 2, 1, 3)])
def test_propagator_columns_solve_the_full_operator(dims, src):
    """M psi_j = point_j for the twelve columns put together from their parity
    halves, both source parities, a site count that leaves the last work-group
    of the merge part empty.  |1 - Mhat| <= (8 kappa)^2 = 0.77, so the solve's
    1e-12 is a residual below 1.5e-11 here."""
    import torch
    from paper_1207_2223_amd import wd
    V, kappa = li.volume(dims), 0.11
    lat = wd.Lattice(dims)
    lat.gauge_load(dev(li.random_su3_field(dims, 0.5, seed=71)), recon=18)
    psi = torch.empty((12, V, 4, 3), dtype=torch.complex128, device="cuda")
    st, _ = lat.point_propagator(psi, src, kappa, wd.solver_params(prec=wd.WD_F64, tol=1e-12))
    assert st == wd.WD_OK
    x0 = src[0] + dims[0] * (src[1] + dims[1] * (src[2] + dims[2] * src[3]))
    hop = torch.empty_like(psi[0])
    for j in range(12):
        lat.dslash(hop, psi[j], 0, 0, 0)
        r = psi[j] - kappa * hop
        r.view(V, 12)[x0, j] -= 1.0
        note(f"propagator {dims} {src} column {j}")
        assert float(torch.linalg.vector_norm(r)) <= 1e-10
    lat.close()
