"""Decode parity where the workgroups have eight waves: in the many-split form
(capacity of six or more tiles per split; four waves below that) and with one
split per unit, at lengths that leave waves and whole splits without a tile."""
import math

import pytest
import torch

from paper_2608_04771_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("units,cap", [(4, 16640), (4, 12000), (16, 4000), (150, 700), (224, 4900)])
def test_lengths_around_tile_and_split_edges(dtype, D, units, cap):
    G = 5
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    splits = min(cus // units, ((cap + 32) // 32) // 4, 128)
    edge = 32 * splits * 4                                   # four tiles per split, then a fifth
    for lens in ([0, 31, 32, 33], [edge - 1, edge, min(edge + 1, cap), cap - 1]):
        lens = [min(x, cap) for x in (lens * units)[:units]]
        g = torch.Generator(device="cuda").manual_seed(cap + D)
        td = torch.float32 if dtype == "f32" else torch.bfloat16
        k = torch.randn((1, 1, units, cap, D), generator=g, device="cuda").to(td)
        v = torch.randn((1, 1, units, cap, D), generator=g, device="cuda").to(td)
        q = torch.randn((1, 1, units * G, D), generator=g, device="cuda").to(td)
        kn, vn = (torch.randn((1, 1, units, D), generator=g, device="cuda").to(td) for _ in range(2))
        cache = B.KVCache(k, v, torch.tensor(lens, dtype=torch.int32, device="cuda").reshape(1, 1, units))
        out, lse = B.reco_decode_attn(cache, q, kn, vn)
        for u, n in enumerate(lens):
            kk = torch.cat([k[0, 0, u, :n], kn[0, 0, u][None]]).double()
            vv = torch.cat([v[0, 0, u, :n], vn[0, 0, u][None]]).double()
            x = (q[0, 0, u * G:(u + 1) * G].double() @ kk.T.contiguous()) / math.sqrt(D)
            ref = torch.softmax(x, -1) @ vv
            err = (out[0, 0, u * G:(u + 1) * G].double() - ref).abs()
            # fp32: sums in another order; bf16: probabilities and results rounded to 8 bits
            lim = 1e-5 * ref.abs().amax() if dtype == "f32" else 2e-2
            assert float(err.max()) <= float(lim), (u, n)
            assert float((lse[0, 0, u * G:(u + 1) * G].double() - torch.logsumexp(x, -1)).abs().max()) <= 1e-4
            if n < cap:
                assert torch.equal(cache.k[0, 0, u, n], kn[0, 0, u]) and int(cache.length[0, 0, u]) == n + 1
