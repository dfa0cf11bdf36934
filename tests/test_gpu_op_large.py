"""Operator calls on a lattice whose links exceed the last-level cache: the
instances that read them non-temporally, and the packed copy that FP32, FP16
and int16 calls take by size, against the launch-shape entry point (packed
copy, ordinary loads, another kernel): the same bits in every storage format."""
import pytest

import lattice_inputs as li
from gpu_util import note, random_links

pytestmark = pytest.mark.gpu

DIMS = (32, 32, 32, 32)
# 8-real links exceed the cache in calls on both parities only, FP32 12-real ones
# in calls on one too; FP32 18-real and FP16 links have no non-temporal instance
CODES = {"f64": 0, "f32": 1, "f32l16": 1 | 0x10, "f32r18": 1 | 0x20, "f32r8": 1 | 0x40, "f16": 2, "f16l16": 2 | 0x10,
         "f16r18": 2 | 0x20, "f16r8": 2 | 0x40, "i16": 3, "i16l16": 3 | 0x10}


@pytest.mark.parametrize("recon", [12, 18])
def test_large_operator_calls_give_the_bits_of_the_shaped_sweeps(recon):
    import torch
    from paper_1207_2223_amd import wd
    V = li.volume(DIMS)
    lat = wd.Lattice(DIMS)
    lat.gauge_load(random_links(V, 11), recon=recon)
    g = torch.Generator(device="cuda")
    g.manual_seed(12)
    full = torch.randn((V, 4, 3), dtype=torch.complex128, device="cuda", generator=g)
    x = [torch.arange(n, device="cuda").view([-1 if q == k else 1 for q in range(4)]) for k, n in enumerate(reversed(DIMS))]
    odd = (sum(x) % 2).reshape(-1).bool()
    parts = {wd.WD_ODD: full[~odd].contiguous(), wd.WD_EVEN: full[odd].contiguous()}  # by output parity: the other one's field
    for prec in (sorted(CODES) if recon == 12 else ["f64"]):
        for dag in (0, 1):
            note(f"{prec} recon {recon} dag {dag}")
            whole = torch.empty_like(full)
            lat.dslash(whole, full, wd.WD_FULL, dag, CODES[prec])
            for par, sel in ((wd.WD_EVEN, ~odd), (wd.WD_ODD, odd)):
                out, ref = torch.empty_like(parts[par]), torch.empty_like(parts[par])
                lat.dslash(out, parts[par], par, dag, CODES[prec])
                wd.wd_dslash_shaped(lat.ctx, ref, parts[par], par, dag, CODES[prec])
                want = torch.view_as_real(ref).view(torch.int64)
                assert torch.equal(torch.view_as_real(out).view(torch.int64), want)
                assert torch.equal(torch.view_as_real(whole[sel]).view(torch.int64), want)
    lat.close()
