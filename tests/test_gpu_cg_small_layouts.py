"""FP64 solves in one launch where a wave is special: half idle (even-odd, an odd
number of 16-site groups) and, on the full lattice, holding sites of both
parities.  The bits and statistics of the launched kernels, and the solution by
the oracle's operator."""
import numpy as np
import pytest

import lattice_inputs as li
from gpu_util import dev, empty_like_dev, host, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eo,dims", [(1, (2, 2, 2, 4)),    # 16 even sites: half a wave
                                     (1, (2, 2, 4, 6)),    # 48: a wave and a half
                                     (1, (4, 4, 6, 4)),    # 192: whole waves, not a power of two
                                     (1, (2, 10, 4, 6)),   # 240
                                     (0, (2, 2, 2, 4)),    # 16 + 16: one wave of both parities
                                     (0, (2, 4, 2, 6)),    # 48 + 48: the second of three waves
                                     (0, (2, 4, 4, 6)),    # 96 + 96
                                     (0, (2, 4, 2, 14))])  # 112 + 112: the fourth of seven
@pytest.mark.parametrize("recon", [18, 12])
def test_waves_that_are_half_idle_or_mixed(oracle, recon, eo, dims):
    from paper_1207_2223_amd import wd
    V, nrhs = li.volume(dims), 3
    n = V // 2 if eo else V
    assert (V // 2) % 16 == 0 and n <= 256  # one launch takes it
    lat = wd.Lattice(dims)
    U = li.random_su3_field(dims, 0.3, seed=111)
    lat.gauge_load(dev(U), recon=recon)
    B = li.gaussian_spinor(n, seed=112, nrhs=nrhs)
    kap = np.array([0.11, 0.13, 0.145])
    X0 = 0.1 * li.gaussian_spinor(n, seed=113, nrhs=nrhs)
    for guess, kw in ((0, dict(tol=1e-12)), (0, dict(tol=1e-12, poll=5, maxiter=12)), (1, dict(tol=1e-10))):
        got = []
        for graphs in (1, 0):
            x = dev(X0) if guess else empty_like_dev(B)
            st, stats = lat.cg_solve(x, dev(B), kap, wd.solver_params(eo=eo, graphs=graphs, initial_guess=guess, **kw))
            got.append((st, [(s["iters"], s["reliable_updates"], s["status"], s["true_resid"]) for s in stats], host(x)))
        note(f"small cg {dims} eo {eo} recon {recon} {kw}: {got[0][:2]}")
        assert got[0][:2] == got[1][:2]
        assert np.array_equal(got[0][2].view(np.uint64), got[1][2].view(np.uint64))
        if not guess and "maxiter" not in kw:
            for j in range(nrhs):
                a = oracle.mhatdag_mhat if eo else oracle.mdagm
                assert np.linalg.norm(B[j] - a(dims, U, kap[j], got[0][2][j])) <= 1.1e-12 * np.linalg.norm(B[j])
    lat.close()
