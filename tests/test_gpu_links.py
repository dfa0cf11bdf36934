"""Kernels that take 21 links a wave (plaquette, Polyakov loop, gauge force)
where the last wave and work-group are partial, a t range is shorter than the
waves that share it, and extents are 2 (both neighbours are one site): against
the oracle.  FP64 sums of at most a few thousand terms of order 1: 1e-13 on
the averages; the force of a solve to 1e-13 to 1e-10 relative."""
import numpy as np
import pytest

import lattice_inputs as li
from gpu_util import dev, empty_like_dev, host, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 4, 10, 2), (4, 6, 2, 18), (10, 6, 4, 10)])
def test_links_in_partial_waves(oracle, dims):
    from paper_1207_2223_amd import wd
    V = li.volume(dims)
    U = li.random_su3_field(dims, 0.4, seed=91)
    lat = wd.Lattice(dims)
    lat.gauge_load(dev(U), recon=12)
    assert abs(lat.plaquette(dev(U)) - oracle.plaquette(dims, U)) <= 1e-13
    assert abs(lat.polyakov(dev(U)) - oracle.polyakov(dims, U)) <= 1e-13
    phi = li.gaussian_spinor(V // 2, seed=92)
    F = empty_like_dev(U)
    wd.wd_md_force(lat.ctx, F, dev(U), dev(phi), 0.12, 5.6, wd.solver_params(tol=1e-13))
    ref = oracle.md_force(dims, U, 5.6, 0.12, phi)
    ref = ref[0] if isinstance(ref, tuple) else ref
    assert rel_err(host(F), ref) <= 1e-10
    lat.close()
