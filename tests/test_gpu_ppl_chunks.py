"""Answer perplexity with either chunk size (chosen by the workspace that the
caller gives) and at lengths around the waves of the last kernel."""
import ctypes

import pytest
import torch

from paper_2608_04771_amd import binding as B
from paper_2608_04771_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,n,vocab", [(1, 1, 1), (1, 15, 4095), (2, 16, 4096), (3, 17, 4097), (1, 33, 16385),
                                           (2, 4, 151931), (1, 3, 16384 * 65 + 1)])
@pytest.mark.parametrize("coarse", [False, True])
def test_matches_fp64(batch, n, vocab, coarse):
    z = I.make_logits(0, 0, 5, device="cuda", shape=(batch, n, vocab))
    z[0, 0, vocab // 2:] = -float("inf")                     # whole chunks without a finite logit
    tok = torch.randint(0, (vocab + 1) // 2, (batch, n), dtype=torch.int32, device="cuda")
    if vocab == 1:
        z[:] = 0.5
    size = B.answer_ppl_workspace_size(batch, n, vocab)
    if coarse:                                               # 16,384 logits a chunk, 8 bytes a partial
        size = batch * n * ((vocab + 16383) // 16384) * 8
    ws = torch.empty(size + 4, dtype=torch.uint8, device="cuda")[4:]     # aligned to 4 bytes only
    ppl = torch.empty(batch, device="cuda")
    lib = B.load_library()
    st = lib.reco_answer_ppl(*(ctypes.c_void_p(x.data_ptr()) for x in (z, tok)), batch, n, vocab, 1.1,
                             ctypes.c_void_p(ppl.data_ptr()), None, ctypes.c_void_p(ws.data_ptr()), size, None,
                             ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == B.RECO_OK
    zd = z.double()
    nll = torch.logsumexp(zd, -1) - zd.gather(2, tok.long()[:, :, None])[:, :, 0]
    # an fp32 sum of at most 64 terms a thread and 8 levels above it, and the fp32 result
    assert float((torch.log(ppl.double()) - nll.mean(-1)).abs().max()) <= 1e-5
    assert lib.reco_answer_ppl(None, None, batch, n, vocab, 1.1, None, None, None, 0, None, None) != B.RECO_OK
