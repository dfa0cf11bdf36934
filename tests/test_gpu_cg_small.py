"""FP64 solves of lattices that fit one work-group run whole steps in one launch
(graphs = 1); with graphs = 0 each iteration's kernels are launched.  Both give
the same bits and statistics: even-odd and full lattice, 18- and 12-real links,
more right-hand sides than one launch takes, a residual check interval that
does not divide the iteration cap, a starting guess, a zero and a non-finite
source, and a session.  The largest lattices are at the limit of 256 sites of a
vector; the last ones are past it, or have sites that do not fill
groups of 16 (both sides launch)."""
import numpy as np
import pytest

import lattice_inputs as li
from gpu_util import dev, empty_like_dev, host, note

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def wd():
    from paper_1207_2223_amd import wd
    wd.lib()
    return wd


def solve(wd, lat, B, kap, eo, graphs, x0=None, **kw):
    x = dev(x0) if x0 is not None else empty_like_dev(B)
    p = wd.solver_params(prec=wd.WD_F64, eo=eo, graphs=graphs, initial_guess=0 if x0 is None else 1, **kw)
    st, stats = lat.cg_solve(x, dev(B), kap, p)
    return st, [(s["iters"], s["iters_fp64"], s["reliable_updates"], s["status"], np.float64(s["true_resid"]).tobytes())
                for s in stats], host(x).view(np.uint64)


@pytest.mark.parametrize("eo,dims", [(1, (2, 2, 4, 4)), (1, (4, 4, 4, 4)), (1, (4, 4, 4, 8)), (0, (2, 4, 4, 4)), (0, (4, 4, 4, 4)),
                                     (1, (6, 4, 4, 6)), (0, (2, 2, 2, 2)), (0, (6, 2, 2, 6))])
@pytest.mark.parametrize("recon", [18, 12])
def test_one_launch_steps_equal_the_launches(wd, oracle, recon, eo, dims):
    V = li.volume(dims)
    n = V // 2 if eo else V
    lat = wd.Lattice(dims)
    U = li.random_su3_field(dims, 0.3, seed=81)
    lat.gauge_load(dev(U), recon=recon)
    B = li.gaussian_spinor(n, seed=82, nrhs=35)
    B[3] = 0.0
    kap = np.linspace(0.11, 0.15, 35)
    for kw in (dict(tol=1e-10), dict(tol=1e-12, poll=5), dict(tol=1e-10, maxiter=13, poll=5)):
        a, b = solve(wd, lat, B, kap, eo, 1, **kw), solve(wd, lat, B, kap, eo, 0, **kw)
        note(f"small cg {dims} eo {eo} recon {recon} {kw}: iters {[s[0] for s in a[1]][:6]}")
        assert a[0] == b[0] and a[1] == b[1]
        assert np.array_equal(a[2], b[2])
    x = solve(wd, lat, B[:1], kap[:1], eo, 1, tol=1e-12)[2].view(np.complex128)[0]
    r = B[0] - (oracle.mhatdag_mhat(dims, U, kap[0], x) if eo else oracle.mdagm(dims, U, kap[0], x))
    assert np.linalg.norm(r) <= 1.1e-12 * np.linalg.norm(B[0])
    X0 = 0.1 * li.gaussian_spinor(n, seed=83, nrhs=2)
    a, b = (solve(wd, lat, B[:2], kap[:2], eo, gr, x0=X0, tol=1e-10) for gr in (1, 0))
    assert a[:2] == b[:2] and np.array_equal(a[2], b[2])
    B[1, 0, 0, 0] = np.nan
    a, b = (solve(wd, lat, B[:3], kap[:3], eo, gr, tol=1e-10) for gr in (1, 0))
    assert a[0] == b[0] == wd.WD_ERR_NAN and a[1] == b[1] and np.array_equal(a[2][[0, 2]], b[2][[0, 2]])
    lat.close()


def test_session_steps_in_one_launch(wd):
    dims = (4, 4, 4, 4)
    lat = wd.Lattice(dims)
    lat.gauge_load(dev(li.random_su3_field(dims, 0.3, seed=84)))
    B = dev(li.gaussian_spinor(128, seed=85, nrhs=3))
    got = []
    for graphs in (1, 0):
        s = wd.wd_session_create(lat.ctx, 4, wd.solver_params(prec=wd.WD_F64, graphs=graphs))
        first = wd.wd_session_add(s, B[:2], [0.14, 0.13])
        wd.wd_session_step(s, 8)
        second = wd.wd_session_add(s, B[2:], [0.12])
        n = 0
        while any(v == 1 for v in wd.wd_session_poll(s)[0]):
            wd.wd_session_step(s, 8)
            n += 1
        stats = wd.wd_session_poll(s)[1]
        x = empty_like_dev(B.cpu().numpy())
        for k, slot in enumerate(first + second):
            wd.wd_session_take(s, slot, x[k])
        got.append((n, [(q["iters"], q["reliable_updates"], q["true_resid"]) for q in stats[:3]], host(x).view(np.uint64)))
        wd.wd_session_destroy(s)
    assert got[0][:2] == got[1][:2] and np.array_equal(got[0][2], got[1][2])
    lat.close()
