"""GPU parity of reco_score where a few keys lie far above everything among a
segment's first keys, as the peaked rows of trained models have them: the row
sums are taken against a reference from those first keys, and neither their
range (sums of several waves, near the end of fp32's) nor the precision of the
heavy keys' exponents may depend on how far above it the heavy keys lie.  The
reference is a plain fp64 softmax of the same inputs."""
import math

import pytest
import torch

from gpu_helpers import SCORE_RTOL
from paper_2608_04771_amd import binding as B

pytestmark = pytest.mark.gpu

N, W, G = 3000, 1, 2
# Heavy keys (position, log2 below the highest): the first two are equal and, with
# the least workspace (7 workgroups of 6 or 7 chunks of 64 keys), in two waves of
# the segment that begins at key 384; the others in this and in other segments.
HEAVY = [(460, 0.0), (600, 0.0), (470, 1.37), (700, 0.61), (810, 2.9), (1500, 0.23), (2222, 1.05), (2223, 3.3)]

# Exponents of the heavy keys are at most 20 in a row's sum and 9 in the weight, so they are rounded by at most
# 2^-20 and 2^-21; each exponential is right to 2^-23.
HEAVY_RTOL = math.log(2.0) * (2.0 ** -20 + 2.0 ** -21) + 2 * 2.0 ** -23


def _inputs(dtype, D, above):
    """Light keys with N(0, 1) logits; the heavy keys' logits are the same for every window row and `above`
    (log2) higher than 0, their values a sum of two parts that bf16 holds exactly."""
    g = torch.Generator(device="cuda").manual_seed(D + int(above))
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    k = torch.randn((1, 1, 1, N, D), generator=g, device="cuda")
    q = torch.randn((1, 1, G, W, D), generator=g, device="cuda")
    k[..., :2] = 0.0
    q[..., :2] = 1.0
    for pos, below in HEAVY:
        k[0, 0, 0, pos] = 0.0
        x = (above - below) * math.log(2.0) * math.sqrt(D)
        hi = torch.tensor(x).bfloat16().float()
        k[0, 0, 0, pos, 0] = hi
        k[0, 0, 0, pos, 1] = (x - hi).bfloat16().float()
    length = torch.full((1, 1, 1), N, dtype=torch.int32, device="cuda")
    k = k.to(td)
    return B.KVCache(k, torch.zeros_like(k), length), q.to(td)


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("above", [12.0, 19.5, 21.0, 30.0, 40.0, 61.0, 99.0, 101.0, 126.5, 127.3, 127.9, 140.0, 300.0])
def test_heavy_keys_far_above_the_first_ones(dtype, D, above):
    cache, q = _inputs(dtype, D, above)
    x = q.double().reshape(G * W, D) @ cache.k[0, 0, 0].double().T.contiguous() / math.sqrt(D)
    pos = torch.arange(N - W, N, device="cuda").repeat(G)
    x = x.masked_fill(torch.arange(N, device="cuda")[None] > pos[:, None], -math.inf)
    ref = torch.softmax(x, -1).sum(0)
    heavy = torch.tensor([p for p, _ in HEAVY], device="cuda")
    light = torch.ones(N, dtype=torch.bool, device="cuda")
    light[heavy] = False
    light &= ref > 1e-30
    rows = (G * W + 15) // 16 * 16
    least = rows * ((N + 511) // 512 + 1) * 8
    for ws in (torch.empty(least, dtype=torch.uint8, device="cuda"), None):
        got = B.reco_score(cache, q, W, ws=ws)[0, 0, 0].double()
        err = (got - ref).abs() / ref
        assert abs(float(got.sum()) - G * W) <= 1e-6 * G * W
        assert float(err[heavy].max()) <= HEAVY_RTOL, f"heavy keys: {float(err[heavy].max()):.3e}"
        # the others' exponents are as large as they lie below the heavy ones (product and difference rounded)
        if bool(light.any()):
            worst = float(err[light].max())
            assert worst <= SCORE_RTOL + 2 * math.log(2.0) * (above + 8) * 2.0 ** -24, f"light keys: {worst:.3e}"
