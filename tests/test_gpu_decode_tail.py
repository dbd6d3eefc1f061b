"""Decode where the rows past a unit's end hold NaN, at tile counts that leave
a wave with none, one, two or three tiles and a last tile of any filling."""
import math

import pytest
import torch

from paper_2608_04771_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("units,lens,cap", [(512, (1, 31, 32, 33, 127, 128, 129, 255, 256, 257, 384, 385, 500), 600),
                                            (4, (9000, 12289, 16383, 2049), 16400)])
@pytest.mark.parametrize("append", [False, True])
def test_rows_past_the_end_do_not_matter(dtype, D, units, lens, cap, append):
    G = 4
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(D + units)
    k, v = (torch.randn((1, 1, units, cap, D), generator=g, device="cuda").to(td) for _ in range(2))
    n = torch.tensor([lens[u % len(lens)] for u in range(units)], dtype=torch.int32, device="cuda")
    past = torch.arange(cap, device="cuda")[None, :] >= n[:, None]
    k[0, 0][past] = float("nan")
    v[0, 0][past] = float("nan")
    q = torch.randn((1, 1, units * G, D), generator=g, device="cuda").to(td)
    kn, vn = (torch.randn((1, 1, units, D), generator=g, device="cuda").to(td) for _ in range(2))
    cache = B.KVCache(k, v, n.reshape(1, 1, units).clone())
    out, lse = B.reco_decode_attn(cache, q, kn if append else None, vn if append else None)
    for u in list(range(min(units, 26))) + [units - 1]:
        m = int(n[u])
        kk, vv = k[0, 0, u, :m], v[0, 0, u, :m]
        if append:
            kk, vv = torch.cat([kk, kn[0, 0, u][None]]), torch.cat([vv, vn[0, 0, u][None]])
        x = (q[0, 0, u * G:(u + 1) * G].double() @ kk.double().T.contiguous()) / math.sqrt(D)
        ref = torch.softmax(x, -1) @ vv.double()
        err = float((out[0, 0, u * G:(u + 1) * G].double() - ref).abs().max())
        # fp32: sums in another order; bf16: probabilities and results rounded to 8 bits
        assert err <= (1e-5 * float(ref.abs().max()) if dtype == "f32" else 2e-2), (u, m)
        assert float((lse[0, 0, u * G:(u + 1) * G].double() - torch.logsumexp(x, -1)).abs().max()) <= 1e-4
