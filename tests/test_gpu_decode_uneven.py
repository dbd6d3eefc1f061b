"""Decode in calls whose units may take two splits or all that are launched, by
the lengths on the device: against fp64 where the units are uneven, short, empty
or even, bit for bit against the same rows in a capacity that launches two
splits where they are long and even, and bit for bit between the two entry
points (the partials of all launched splits lie in the static array)."""
import math

import pytest
import torch

from paper_2608_04771_amd import binding as B

pytestmark = pytest.mark.gpu

CAP = 10400                                             # 325 tiles: from 320 on more than two splits are launched


def _lengths(kind, units):
    g = torch.Generator().manual_seed(units)
    if kind == "even":
        return [3600] * units
    if kind == "short":                                 # the longest just below what counts as long
        return [3199] * (units - 1) + [0]
    if kind == "one long":                              # all but one empty or nearly so
        return [u % 3 for u in range(units - 1)] + [CAP - 1]
    return torch.randint(0, CAP, (units,), generator=g).tolist()


def _inputs(units, G, dtype, D, lens, cap):
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(D + units)
    k, v = (torch.randn((1, units, 1, CAP, D), generator=g, device="cuda").to(td)[:, :, :, :cap].contiguous()
            for _ in range(2))
    q = torch.randn((1, units, G, D), generator=g, device="cuda").to(td)
    kn, vn = (torch.randn((1, units, 1, D), generator=g, device="cuda").to(td) for _ in range(2))
    n = torch.tensor(lens, dtype=torch.int32, device="cuda").reshape(1, units, 1)
    return B.KVCache(k, v, n), q, kn, vn


def _nans(cache, G):
    """A workspace of NaNs: what a call reads of it has to come from the call."""
    return B.decode_workspace(cache, G).fill_(0xff)


@pytest.mark.parametrize("kind", ["even", "short", "one long", "ragged"])
@pytest.mark.parametrize("units,G,dtype,D", [(128, 7, "bf16", 128), (96, 4, "bf16", 128), (97, 4, "f32", 64),
                                             (96, 3, "bf16", 64), (100, 2, "f32", 128)])
def test_units_of_any_lengths(units, G, dtype, D, kind):
    lens = _lengths(kind, units)
    cache, q, kn, vn = _inputs(units, G, dtype, D, lens, CAP)
    other, _, _, _ = _inputs(units, G, dtype, D, lens, CAP)
    stats = torch.empty((1, units, G, 2), dtype=torch.float32, device="cuda")
    out, lse = B.reco_decode_attn(cache, q, kn, vn, ws=_nans(cache, G), row_stats=stats)
    for u, n in enumerate(lens):
        kk = torch.cat([other.k[0, u, 0, :n], kn[0, u]]).double()
        vv = torch.cat([other.v[0, u, 0, :n], vn[0, u]]).double()
        x = q[0, u].double() @ kk.T.contiguous() / math.sqrt(D)
        ref = torch.softmax(x, -1) @ vv
        err = float((out[0, u].double() - ref).abs().max())
        # fp32: sums in another order; bf16: probabilities and results rounded to 8 bits
        assert err <= (1e-5 * float(ref.abs().max()) if dtype == "f32" else 2e-2), (u, n)
        assert float((lse[0, u].double() - torch.logsumexp(x, -1)).abs().max()) <= 1e-4, (u, n)
        assert torch.equal(cache.k[0, u, 0, n], kn[0, u, 0]) and torch.equal(cache.v[0, u, 0, n], vn[0, u, 0])
    assert torch.equal(cache.length, other.length + 1)
    o2, l2, s2 = torch.empty_like(out), torch.empty_like(lse), torch.empty_like(stats)
    B.reco_decode_attn_noalloc(other, q, o2, l2, kn, vn, row_stats=s2)
    assert torch.equal(out, o2) and torch.equal(lse, l2) and torch.equal(stats, s2)
    assert torch.equal(cache.k, other.k) and torch.equal(cache.v, other.v) and torch.equal(cache.length, other.length)


@pytest.mark.parametrize("units,G,dtype,D", [(128, 7, "bf16", 128), (96, 4, "f32", 64)])
def test_long_even_units_take_two_splits(units, G, dtype, D):
    lens = [9000 + 100 * (u % 9) for u in range(units)]
    cache, q, kn, vn = _inputs(units, G, dtype, D, lens, CAP)
    less, _, _, _ = _inputs(units, G, dtype, D, lens, CAP - 300)
    out, lse = B.reco_decode_attn(cache, q, kn, vn, ws=_nans(cache, G))
    ref, ref_lse = B.reco_decode_attn(less, q, kn, vn)
    assert torch.equal(out, ref) and torch.equal(lse, ref_lse)
