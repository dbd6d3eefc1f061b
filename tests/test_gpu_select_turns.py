"""Selection at prefix lengths around the turns of a workgroup (1,024 positions
a turn) and around the longest prefix whose scores stay in registers (16
turns), with ties, crowded bins, zeros of either sign and infinities."""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_04771_amd import binding as B

pytestmark = pytest.mark.gpu


def _scores(kind, n, rng):
    if kind == "lognormal":
        return np.exp(rng.standard_normal(n))
    if kind == "two_levels":
        return rng.integers(0, 2, n).astype(np.float64)
    if kind == "last_bits":                                  # one bin in both first passes
        return 1.0 + rng.integers(0, 900, n) * 2.0 ** -23
    s = rng.random(n)                                         # zeros of both signs and infinities
    s[rng.random(n) < 0.4] = 0.0
    s[rng.random(n) < 0.2] = -0.0
    s[rng.random(n) < 0.1] = np.inf
    return s


@pytest.mark.parametrize("kind", ["lognormal", "two_levels", "last_bits", "edges"])
@pytest.mark.parametrize("r", [0.05, 0.6, 0.97])
def test_kept_positions_equal_the_oracles(kind, r):
    w = 16
    lens = [w, w + 1, w + 64, w + 1023, w + 1024, w + 1025, w + 16383, w + 16384, w + 16385, 40001]
    cap, units = max(lens) + 5, len(lens)
    rng = np.random.default_rng(int(r * 100))
    sc = np.full((1, units, 1, cap), np.nan, dtype=np.float32)      # nothing past the prefix is looked at
    for u, n in enumerate(lens):
        sc[0, u, 0, :n - w] = _scores(kind, n - w, rng).astype(np.float32)
    k = torch.zeros((1, units, 1, cap, 64), dtype=torch.bfloat16, device="cuda")
    cache = B.KVCache(k, torch.zeros_like(k), torch.tensor(lens, dtype=torch.int32, device="cuda").reshape(1, units, 1))
    kept = torch.full((1, units, 1, cap), -1, dtype=torch.int32, device="cuda")
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    B.reco_select_compact(cache, torch.from_numpy(sc).cuda(), torch.full((units,), r, dtype=torch.float64, device="cuda"),
                          w, kept_idx=kept, dev_err=err)
    assert int(err.item()) == 0
    kk = kept.cpu().numpy()
    for u, n in enumerate(lens):
        s = np.concatenate([sc[0, u, 0, :n - w], np.zeros(w, dtype=np.float32)]).astype(np.float64)
        ref = oracle.select_unit(s, n, w, r)
        assert int(cache.length[0, u, 0]) == len(ref)
        np.testing.assert_array_equal(kk[0, u, 0, :len(ref)], ref, err_msg=f"{kind} r={r} L={n}")
        assert (kk[0, u, 0, len(ref):] == -1).all()
