"""GPU parity of reco_score where its plan changes form: several row blocks
(sums carried across them) over segments that are cut, short units kept whole,
the least workspace a call takes, and a logit that overflows a row's reference.
The reference is a plain fp64 softmax of the same inputs."""
import math

import pytest
import torch

from gpu_helpers import SCORE_RTOL
from paper_2608_04771_amd import binding as B

pytestmark = pytest.mark.gpu


def _make(dtype, D, G, w, lens, cap, seed=11):
    NL, Bsz, H = lens.shape
    g = torch.Generator(device="cuda").manual_seed(seed)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    k = torch.randn((NL, Bsz, H, cap, D), generator=g, device="cuda").to(td)
    q = torch.randn((NL, Bsz, H * G, w, D), generator=g, device="cuda").to(td)
    return B.KVCache(k, torch.zeros_like(k), lens.cuda()), q


def _check(cache, q, w, scores, far=False):
    NL, Bsz, H, Cap, D = cache.shape
    G = q.shape[2] // H
    lens = cache.length.cpu()
    worst = x_max = 0.0
    for l in range(NL):
        for b in range(Bsz):
            for h in range(H):
                n = int(lens[l, b, h])
                if n == 0:
                    continue
                t = min(w, n)
                qq = q[l, b, h * G:(h + 1) * G, w - t:].double().reshape(G * t, D)
                x = (qq @ cache.k[l, b, h, :n].double().T.contiguous()).reshape(G, t, n) / math.sqrt(D)
                pos = torch.arange(n - t, n, device="cuda")
                x_max = max(x_max, float(x.abs().max()) / math.log(2.0))
                x = x.masked_fill(torch.arange(n, device="cuda")[None, None] > pos[None, :, None], -math.inf)
                ref = torch.softmax(x, -1).sum((0, 1))
                got = scores[l, b, h, :n].double()
                big = ref > 1e-20
                worst = max(worst, float(((got - ref).abs() / ref)[big].max()))
                assert abs(float(got.sum()) - G * t) <= 1e-4 * G * t
    # far logits: an exponent of size x is rounded to x * 2^-24 (log2) twice, as a product and as a difference
    assert worst <= SCORE_RTOL + (2 * math.log(2.0) * x_max * 2.0 ** -24 if far else 0.0), f"score rel err {worst:.3e}"


@pytest.mark.parametrize("dtype,D,G,w,cap", [("f32", 128, 4, 80, 9000),     # 2 row blocks, segments cut at 4,096 keys
                                             ("bf16", 128, 9, 60, 9000), ("bf16", 64, 16, 60, 9000)])
def test_row_blocks_over_long_units(dtype, D, G, w, cap):
    cache, q = _make(dtype, D, G, w, torch.tensor([[[9000, 8191]]], dtype=torch.int32), cap)
    # one workgroup walks whole units with the least workspace a call takes: 2 units, ceil(cap / 512) + 1 slots each
    rows = (G * w + 15) // 16 * 16
    least = 2 * rows * ((cap + 511) // 512 + 1) * 8
    for ws in (None, torch.empty(least, dtype=torch.uint8, device="cuda")):
        _check(cache, q, w, B.reco_score(cache, q, w, ws=ws))
    with pytest.raises(RuntimeError, match="workspace"):
        B.reco_score(cache, q, w, ws=torch.empty(least - 1, dtype=torch.uint8, device="cuda"))


@pytest.mark.parametrize("cap,w", [(300, 128), (512, 31), (513, 31)])
def test_short_units(cap, w):
    gen = torch.Generator().manual_seed(cap)
    lens = torch.randint(0, cap + 1, (4, 8, 8), generator=gen, dtype=torch.int32)
    lens[0, 0, :4] = torch.tensor([0, 1, cap, w], dtype=torch.int32)
    cache, q = _make("bf16", 128, 4, w, lens, cap)
    _check(cache, q, w, B.reco_score(cache, q, w))


def test_logit_far_above_the_reference():
    """A key whose logit lies far above everything among a segment's first keys
    overflows the row sums against that reference; the exact maxima are used then."""
    cache, q = _make("bf16", 128, 4, 32, torch.tensor([[[3000, 777]]], dtype=torch.int32), 3000)
    cache.k[0, 0, :, 700] *= 60.0
    _check(cache, q, 32, B.reco_score(cache, q, 32), far=True)
