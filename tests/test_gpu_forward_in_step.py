"""A forward of so many rounds of tiles that the workgroups of an XCD keep each other's step: repeated on a workspace whose counters the
call before left behind, on two streams at a time (whose workgroups cannot all have a compute unit at once), and against plain fp64 arithmetic."""
import pytest
import torch

from paper_2602_05885_amd import binding as B
from paper_2602_05885_amd import synth

pytestmark = pytest.mark.gpu


# rounds of 256 tiles: 64.2 and 63.9, either side of the line, and 71 with a contraction of one stage
@pytest.mark.parametrize("T,d,V", [(14 * 256, 320, 256 * 1174), (14 * 256 - 100, 320, 256 * 1168), (20000, 64, 256 * 230)])
def test_many_rounds_of_tiles(T, d, V):
    dev = torch.device("cuda:0")
    H, W, y = synth.make_head(T, d, V, "bf16", T, dev)
    p = B.Params()
    streams = [torch.cuda.Stream() for _ in range(2)]
    spaces = [B.alloc_workspace(T, d, V, 0, p, B.CALL_LOGPROB_FWD, dev).fill_(255) for _ in streams]
    first = [t.clone() for t in B.pg_logprob_fwd(H, W, y, None, p, spaces[0])]
    torch.cuda.synchronize()
    outs = []
    for _ in range(2):
        for s, ws in zip(streams, spaces):
            with torch.cuda.stream(s):
                outs.append(B.pg_logprob_fwd(H, W, y, None, p, ws))
    torch.cuda.synchronize()
    for out in outs:
        assert all(torch.equal(a, b) for a, b in zip(out, first))
    logp, ent, lse = first
    rows = torch.arange(0, T, max(1, T // 150), device=dev)
    z = H[rows].double() @ W.double().T
    want = torch.logsumexp(z, 1)
    q = torch.softmax(z, 1)
    # fp32 sums of d products of bf16 values (|z| is a few units: d * 2^-24 of it at most) and of V exponentials in tiles of 256
    tol = (d + 256) * 2.0 ** -24 * z.abs().max().item()
    assert (lse[rows].double() - want).abs().max() <= tol
    assert (logp[rows].double() - (z.gather(1, y[rows].long()[:, None])[:, 0] - want)).abs().max() <= 2 * tol
    assert (ent[rows].double() - (want - (q * z).sum(1))).abs().max() <= 4 * tol
