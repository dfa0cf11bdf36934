"""What a call promises beyond its numbers: a refused call leaves its output as
it was, the two ways a step of iterations can run (graphs = 1 and 0) agree in
everything a caller sees, a launch stays short, and the device memory held is
the memory needed."""
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


@pytest.mark.parametrize("src", [(0, 2, 1, 3), (1, 2, 1, 3)])
def test_refused_propagator_leaves_its_output(wd, src):
    """Every parameter the solver checks, both source parities."""
    import torch
    dims = (4, 4, 4, 4)
    lat = wd.Lattice(dims)
    lat.gauge_load(dev(li.random_su3_field(dims, 0.3, seed=101)))
    psi = torch.full((12, li.volume(dims), 4, 3), 7.0 - 3.0j, dtype=torch.complex128, device="cuda")
    for bad in (dict(tol=0.0), dict(tol=-1.0), dict(maxiter=-1), dict(poll=0), dict(delta=0.0), dict(delta=1.0),
                dict(prec=0x99), dict(prec=wd.WD_F64 | wd.WD_LINKS_F16), dict(eo=0)):
        note(f"propagator {src} {bad}")
        status, _ = wd.wd_point_propagator(lat.ctx, psi, src, 0.11, wd.solver_params(**bad), check=False)
        assert status == wd.WD_ERR_ARG
        assert torch.count_nonzero(psi - (7.0 - 3.0j)).item() == 0
    lat.close()


def test_propagator_without_memory_for_its_solve_leaves_its_output(wd):
    """24^3 x 48 with 12 columns: the solver's state (7 GB in FP16) does not fit
    the 5 GB that are left, the propagator's own two fields do."""
    import torch
    dims = (24, 24, 24, 48)
    V = li.volume(dims)
    lat = wd.Lattice(dims)
    U = torch.zeros((V, 4, 3, 3), dtype=torch.complex128, device="cuda")
    U[..., 0, 0] = U[..., 1, 1] = U[..., 2, 2] = 1.0
    lat.gauge_load(U, recon=12)
    psi = torch.full((12, V, 4, 3), 7.0 - 3.0j, dtype=torch.complex128, device="cuda")
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    ballast = torch.empty(torch.cuda.mem_get_info()[0] - 5 * 2 ** 30, dtype=torch.uint8, device="cuda")
    for src in ((0, 0, 0, 0), (1, 0, 0, 0)):
        status, _ = wd.wd_point_propagator(lat.ctx, psi, src, 0.11, wd.solver_params(prec=wd.WD_F16), check=False)
        assert status == wd.WD_ERR_OOM
        assert all(bool((p == 7.0 - 3.0j).all()) for p in psi)
    del ballast
    lat.close()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("eo", [1, 0])
@pytest.mark.parametrize("maxiter", [13, 16, 3, 0])
def test_session_at_the_iteration_cap(wd, eo, maxiter):
    """A step runs all its iterations of every running slot, also where the cap
    lies inside it; two right-hand sides of different ages."""
    dims = (4, 4, 4, 4)
    n = 128 if eo else 256
    lat = wd.Lattice(dims)
    lat.gauge_load(dev(li.random_su3_field(dims, 0.3, seed=84)))
    B = dev(li.gaussian_spinor(n, seed=85, nrhs=2))
    got = []
    for graphs in (1, 0):
        s = wd.wd_session_create(lat.ctx, 2, wd.solver_params(prec=wd.WD_F64, graphs=graphs, maxiter=maxiter, eo=eo, tol=1e-12))
        slots = wd.wd_session_add(s, B[:1], [0.14])
        wd.wd_session_step(s, 8)
        slots += wd.wd_session_add(s, B[1:], [0.12])
        steps = 1
        while any(v == 1 for v in wd.wd_session_poll(s)[0]):
            wd.wd_session_step(s, 8)
            steps += 1
        st = wd.wd_session_poll(s)[1]
        x = empty_like_dev(B.cpu().numpy())
        for k, j in enumerate(slots):
            wd.wd_session_take(s, j, x[k])
        got.append((steps, [(q["iters"], q["iters_fp64"], q["reliable_updates"], q["status"], q["true_resid"]) for q in st],
                    host(x).view(np.uint64).tolist()))
        wd.wd_session_destroy(s)
    note(f"session cap {maxiter} eo {eo}: {got[0][:2]}")
    assert got[0][:2] == got[1][:2]
    assert got[0][2] == got[1][2]
    assert got[1][1][0][0] == 8 * -(-max(maxiter, 1) // 8)  # whole steps
    lat.close()


def test_trace_prints_every_poll(wd, monkeypatch, capfd):
    dims = (4, 4, 4, 4)
    lat = wd.Lattice(dims)
    lat.gauge_load(dev(li.random_su3_field(dims, 0.3, seed=84)))
    B = dev(li.gaussian_spinor(128, seed=85, nrhs=2))
    monkeypatch.setenv("WD_SOLVER_TRACE", "1")
    lines = []
    for graphs in (1, 0):
        capfd.readouterr()
        lat.cg_solve(empty_like_dev(B.cpu().numpy()), B, [0.14, 0.12], wd.solver_params(tol=1e-10, graphs=graphs))
        lines.append([q for q in capfd.readouterr().err.splitlines() if q.startswith("[wd cg]")])
    assert len(lines[1]) > 8
    assert lines[0] == lines[1]
    lat.close()


def singular(wd, dims, eo):
    """U = 1 at kappa = 1/8: a zero mode, so that a source with a constant part
    has no solution and CG runs to its cap."""
    V = li.volume(dims)
    U = np.zeros((V, 4, 3, 3), complex)
    U[..., range(3), range(3)] = 1.0
    lat = wd.Lattice(dims)
    lat.gauge_load(dev(U))
    return lat, li.gaussian_spinor(V // 2 if eo else V, seed=86) + 1.0


@pytest.mark.parametrize("eo", [1, 0])
def test_one_launch_runs_a_bounded_number_of_iterations(wd, eo):
    """The host is back after some thousand iterations whatever the cap: the
    launches of a solve that does not converge, and the same result as a launch
    a kernel gives."""
    from torch.profiler import ProfilerActivity, profile
    import torch
    lat, b = singular(wd, (4, 4, 4, 4), eo)
    B = dev(b[None])
    x = empty_like_dev(b[None])
    res = []
    for graphs, cap in ((1, 20000), (1, 4500), (0, 4500)):
        p = wd.solver_params(tol=1e-10, maxiter=cap, graphs=graphs, eo=eo)
        if graphs and cap == 20000:
            with profile(activities=[ProfilerActivity.CUDA]) as prof:
                st, stats = lat.cg_solve(x, B, [0.125], p)
                torch.cuda.synchronize()
            launches = sum(e.count for e in prof.key_averages() if "k_cg_small" in e.key)
            note(f"eo {eo}: {stats[0]['iters']} iterations in {launches} launches, status {st}")
            assert stats[0]["iters"] == cap and launches >= 4
        else:
            st, stats = lat.cg_solve(x, B, [0.125], p)
            res.append((st, stats[0]["iters"], stats[0]["reliable_updates"], host(x).view(np.uint64).tolist()))
    assert res[0] == res[1]
    lat.close()


def held(f):
    """Device bytes that f() leaves allocated outside torch's pool."""
    import torch
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    before = torch.cuda.mem_get_info()[0]
    keep = f()
    torch.cuda.synchronize()
    return before - torch.cuda.mem_get_info()[0], keep


@pytest.mark.parametrize("eo,prec,vectors", [(1, "f64", 6), (0, "f64", 13), (1, "f16", 6)])
def test_session_holds_the_vectors_it_uses(wd, eo, prec, vectors):
    """FP64 vectors of a parity per slot: b, x, r, p and two temporaries (the
    full lattice, two parities each: A p too, one temporary of one parity), and
    in FP16 twelve vectors of 52 bytes and the increment of 96.  The charge is
    what the session holds."""
    dims = (16, 16, 16, 16)
    code = {"f64": wd.WD_F64, "f16": wd.WD_F16}[prec]
    lat = wd.Lattice(dims)
    lat.gauge_load(dev(li.unit_field(dims)))
    p = wd.solver_params(prec=code, eo=eo)
    n, stride = 64, (li.volume(dims) // 2 + 63) // 64 * 64 + 592
    need = n * stride * (192 * vectors + (11 * 52 + 96 if prec == "f16" else 0))
    got, s = held(lambda: wd.wd_session_create(lat.ctx, n, p))
    charge = wd.wd_session_bytes(dims, n, p)
    note(f"session eo {eo} {prec}: holds {got / 2 ** 20:.1f} MiB, needs {need / 2 ** 20:.1f}, charged {charge / 2 ** 20:.1f}")
    # norm partials and scalars: about 1 % of a vector a slot; allocations are whole pages of 2 MiB
    slack = 0.02 * need + 40 * 2 ** 21
    assert abs(charge - need) <= 0.02 * need
    assert got <= need + slack
    wd.wd_session_destroy(s)
    lat.close()


@pytest.mark.parametrize("eo,fields", [(0, 2), (1, 2)])
def test_normal_operator_holds_the_temporaries_it_uses(wd, eo, fields):
    """Even-odd: T and B of one parity; the full lattice: T of two."""
    import torch
    dims = (32, 32, 32, 16)
    V = li.volume(dims)
    lat = wd.Lattice(dims)
    U = torch.zeros((V, 4, 3, 3), dtype=torch.complex128, device="cuda")
    U[..., 0, 0] = U[..., 1, 1] = U[..., 2, 2] = 1.0
    lat.gauge_load(U, recon=12)
    b = torch.ones((V // 2 if eo else V, 4, 3), dtype=torch.complex128, device="cuda")
    out = torch.empty_like(b)
    got, _ = held(lambda: lat.mdagm(out, b, 0.1, eo=eo))
    note(f"normal operator eo {eo}: holds {got / 2 ** 20:.1f} MiB")
    assert got <= 1.02 * fields * (V // 2) * 192 + 8 * 2 ** 21
    lat.close()


def test_timing_names_the_instance_that_ran(wd):
    """Operator sweeps over links beyond the last-level cache run the instance
    that reads them non-temporally: link format 6 instead of 2 (FP32 12-real),
    9 instead of 0 (FP64 18-real)."""
    import torch
    for dims, lk32, lk64 in (((32, 32, 32, 32), 6, 9), ((8, 8, 8, 8), 2, 0)):
        V = li.volume(dims)
        lat = wd.Lattice(dims)
        U = torch.zeros((V, 4, 3, 3), dtype=torch.complex128, device="cuda")
        U[..., 0, 0] = U[..., 1, 1] = U[..., 2, 2] = 1.0
        lat.gauge_load(U, recon=18)
        b = torch.ones((V // 2, 4, 3), dtype=torch.complex128, device="cuda")
        out = torch.empty_like(b)
        wd.wd_timing_enable(lat.ctx, True)
        lat.dslash(out, b, wd.WD_EVEN, 0, wd.WD_F32)
        lat.dslash(out, b, wd.WD_EVEN, 1, wd.WD_F64)
        names = sorted(wd.wd_timing_report(lat.ctx))
        note(f"timing {dims}: {names}")
        canon = "false" if dims[0] == 32 else "true"
        assert names == [f"dslash_op_kernel<0, {lk64}, true, true>", f"dslash_op_kernel<1, {lk32}, false, {canon}>"]
        lat.close()


@pytest.mark.parametrize("eo,dims", [(1, (2, 2, 2, 4)), (1, (4, 4, 4, 8)), (0, (4, 4, 4, 4))])
def test_many_right_hand_sides_on_a_small_lattice(wd, eo, dims):
    """More right-hand sides than a launch holds, in steps of one launch per 256:
    the bits of the launched kernels, and not slower than those (best of six)."""
    import time
    import torch
    V, n = li.volume(dims), 600
    lat = wd.Lattice(dims)
    lat.gauge_load(dev(li.random_su3_field(dims, 0.4, seed=88)))
    B = li.gaussian_spinor(V // 2 if eo else V, seed=89, nrhs=n)
    b, x = dev(B), empty_like_dev(B)
    kap = np.linspace(0.11, 0.13, n)
    got, best = [], []
    for graphs in (1, 0):
        p = wd.solver_params(tol=1e-11, graphs=graphs, eo=eo)
        ts = []
        for _ in range(7):
            torch.cuda.synchronize()
            t = time.perf_counter()
            st, stats = lat.cg_solve(x, b, kap, p)
            ts.append(time.perf_counter() - t)
        got.append((st, [(s["iters"], s["reliable_updates"], s["true_resid"]) for s in stats], host(x).view(np.uint64)))
        best.append(min(ts[1:]))
    note(f"{n} RHS {dims} eo {eo}: one launch {best[0] * 1e3:.2f} ms, launches {best[1] * 1e3:.2f} ms")
    assert got[0][:2] == got[1][:2] and np.array_equal(got[0][2], got[1][2])
    assert best[0] <= 1.1 * best[1]
    lat.close()
