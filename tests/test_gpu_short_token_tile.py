"""Forward-only calls whose last token tile holds few rows, on both sides of the lines between a shortened and a whole one (four and five
token tiles in the last panel, contractions of 3072, eight rounds of tiles): against plain fp64 arithmetic on the same bf16 operands."""
import pytest
import torch

from paper_2602_05885_amd import binding as B
from paper_2602_05885_amd import synth

pytestmark = pytest.mark.gpu


# (V: 2 vocab tiles, or as many as make eight rounds of tiles on 256 compute units)
@pytest.mark.parametrize("d,V", [(3008, 300), (3072, 300), (3008, 256 * 410), (3072, 256 * 410)])
@pytest.mark.parametrize("T", [769, 1025, 1152, 1153, 2048 - 128, 2049, 3073])
def test_forward_with_a_short_last_tile(T, d, V):
    dev = torch.device("cuda:0")
    H, W, y = synth.make_head(T, d, V, "bf16", T, dev)
    p = B.Params()
    ws = B.alloc_workspace(T, d, V, 0, p, B.CALL_LOGPROB_FWD, dev)
    ws.fill_(255)                                   # NaN patterns
    logp, ent, lse = B.pg_logprob_fwd(H, W, y, None, p, ws)
    z = H.double() @ W.double().T
    want = torch.logsumexp(z, 1)
    q = torch.softmax(z, 1)
    # fp32 sums of d products of bf16 values (|z| is a few units: d * 2^-24 of it at most) and of 300 exponentials
    tol = d * 2.0 ** -24 * z.abs().max().item()
    assert (lse.double() - want).abs().max() <= tol
    assert (logp.double() - (z.gather(1, y.long()[:, None])[:, 0] - want)).abs().max() <= 2 * tol
    assert (ent.double() - (want - (q * z).sum(1))).abs().max() <= 4 * tol
