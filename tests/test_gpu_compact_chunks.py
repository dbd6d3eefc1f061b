"""Compaction at kept counts around its chunks of 256 rows (one chunk, an odd
and an even number of them, a last chunk of one row), with rows that move far,
by one row, or not at all, and at every row size."""
import pytest
import torch

from paper_2608_04771_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,D", [("bf16", 64), ("bf16", 128), ("f32", 128)])
@pytest.mark.parametrize("L", [1, 300, 1030, 2600])
def test_rows_move_to_their_places(dtype, D, L):
    units, w, cap = 12, 1, L + 3
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(L + D)
    k, v = (torch.randn((1, units, 1, cap, D), generator=g, device="cuda").to(td) for _ in range(2))
    sc = torch.rand((1, units, 1, cap), generator=g, device="cuda")
    sc[0, 1] = torch.arange(cap, device="cuda")              # keep the last rows
    sc[0, 2] = -torch.arange(cap, device="cuda") + cap        # keep the first rows
    sc[0, 3] = 1.0
    sc[0, 3, :, 0] = 0.0                                      # every row moves by one
    want = [min(L, max(1, x)) for x in (1, 255, 256, L - 1, 257, 511, 512, 513, 768, 769, 1024, L)]
    r = torch.tensor([(x - 0.5) / L for x in want], dtype=torch.float64, device="cuda")
    cache = B.KVCache(k.clone(), v.clone(), torch.full((1, units, 1), L, dtype=torch.int32, device="cuda"))
    kept = torch.zeros((1, units, 1, cap), dtype=torch.int32, device="cuda")
    B.reco_select_compact(cache, sc, r, w, kept_idx=kept)
    for u, m in enumerate(want):
        assert int(cache.length[0, u, 0]) == m
        idx = kept[0, u, 0, :m].long()
        assert bool((idx[1:] > idx[:-1]).all()) and int(idx[-1]) == L - 1
        for new, old in ((cache.k, k), (cache.v, v)):
            assert torch.equal(new[0, u, 0, :m], old[0, u, 0][idx])
            assert torch.equal(new[0, u, 0, m:], old[0, u, 0, m:])      # nothing is written past the kept rows
