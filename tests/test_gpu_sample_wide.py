"""The sampler in calls of many chunks, where each workgroup bounds its values
first and computes the exact ones only where they can win: the draws and the
penalised logits have to be those of the calls of few chunks (same row index,
seed and offset), bit for bit, whatever the logits hold."""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_04771_amd import binding as B
from paper_2608_04771_amd import inputs as I

pytestmark = pytest.mark.gpu


def _draw(z, vocab, ids, reward, T):
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    tok = B.reco_penalty_sample(z[:, :vocab], ids, reward, 0.4, 0.8, 0.0, 1.0, 3.0, T, 77, 5, dev_err=err)
    return tok, int(err.item())


@pytest.mark.parametrize("vocab,ld,T", [(4096, 4096, 1.0), (4095, 4096, 0.6), (4097, 4099, 1.0), (8191, 8196, 2.5),
                                        (12288, 12289, 1.0), (5000, 5000, 0.0), (4096, 4096, 1e-31),
                                        (9001, 9004, 1e-29), (4100, 4100, 3e30), (4100, 4100, 9e29)])
@pytest.mark.parametrize("base", [0, 1])
def test_draws_equal_those_of_small_calls(vocab, ld, T, base):
    rows = 2112
    flat = torch.empty(base + rows * ld, dtype=torch.float32, device="cuda")
    z = flat[base:].view(rows, ld)                       # base 1: rows that start 4 bytes past 16
    z.copy_(I.make_logits(rows, ld, 9, device="cuda"))
    z[1] = -float("inf")                                 # masked row
    z[2] = -float("inf")
    z[2, vocab // 2:vocab // 2 + 3] = 1.0                # all but three masked
    z[3, ::3] = float("nan")
    z[4] = float("nan")
    z[5, 17] = float("inf")
    z[6] = 0.0                                           # ties before the noise
    z[7] *= 1e30
    z[8] = -3e38
    z[9, vocab - 1] = 60.0
    z[10] *= 1e-30
    ids = torch.from_numpy(I.make_reflection_ids(64, vocab, 3)).cuda()
    reward = torch.rand(rows, generator=torch.Generator().manual_seed(1)).cuda()
    z0 = z.clone()
    tok, err = _draw(z, vocab, ids, reward, T)
    assert err == 6                                      # the row of NaN
    few = 16                                             # at most 16 x 12 chunks: the form of small calls
    zs = z0[:few].clone()
    ref, _ = _draw(zs, vocab, ids, reward[:few], T)
    assert tok[:few].tolist() == ref.tolist()
    assert z[:few].cpu().numpy().tobytes() == zs.cpu().numpy().tobytes()
    # every other row: the penalty touches its ids alone, and the token is in range (and below, the oracle's)
    beta = torch.where(reward <= 0.4, 0.0, torch.where(reward >= 0.8, 3.0, 1.0))[:, None]
    want = z0.clone()
    want[:, ids.long()] = want[:, ids.long()] - beta
    assert z.cpu().numpy().tobytes() == want.cpu().numpy().tobytes()
    assert bool(((tok[few:] >= 0) & (tok[few:] < vocab)).all())
    if T == 0.0:
        finite = torch.nan_to_num(z[few:, :vocab], nan=-float("inf"))
        assert torch.equal(tok[few:].long(), finite.argmax(1))


@pytest.mark.parametrize("rows,vocab,T", [(2112, 4096, 1.0), (683, 8191, 0.6), (300, 32000, 2.5)])
def test_every_row_draws_the_oracles_token(rows, vocab, T):
    """Every row of a call of many chunks (the rows above compare 16): the oracle's token, or one whose value is
    within what two float32 logarithms of another library's rounding can move it."""
    z = I.make_logits(rows, vocab, 21, device="cuda")
    ids = torch.from_numpy(I.make_reflection_ids(64, vocab, 3)).cuda()
    reward = torch.rand(rows, generator=torch.Generator().manual_seed(2)).cuda()
    z0 = z.cpu().numpy()
    tok, err = _draw(z, vocab, ids, reward, T)
    assert err == 0
    zp, ref, vals = oracle.penalty_sample(z0, ids.cpu().numpy(), reward.cpu().numpy(), 0.4, 0.8, 0.0, 1.0, 3.0, T,
                                          77, 5)
    assert z.cpu().numpy().tobytes() == zp.astype(np.float32).tobytes()
    got = tok.cpu().numpy().astype(np.int64)
    top, mine = vals[np.arange(rows), ref], vals[np.arange(rows), got]
    assert np.all(mine >= top - 1e-5 * np.maximum(1.0, np.abs(top)))
    assert np.mean(got == ref) > 0.99
