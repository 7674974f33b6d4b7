"""pg_head_shard_fwd on every row (no mask): the rows are read where they lie and the pre-pass writes the token ids, counted from the
shard's first vocab row and -1 outside it."""
import pytest
import torch

from paper_2602_05885_amd import binding as B
from paper_2602_05885_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,V,v0,v1", [(1, 64, 300, 100, 101), (70, 128, 700, 0, 257), (257, 64, 700, 257, 700), (600, 192, 1000, 512, 777)])
def test_shard_states_without_a_mask(T, d, V, v0, v1):
    dev = torch.device("cuda:0")
    H, W, y = synth.make_head(T, d, V, "bf16", T, dev)
    y[: T // 8 + 1] = torch.tensor([v0, v1 - 1, v0 - 1, v1, 0, V - 1], device=dev, dtype=torch.int32).repeat(T)[: T // 8 + 1].clamp(0, V - 1)
    Ws = W[v0:v1].contiguous()
    p = B.Params(temperature=0.8)
    ws = B.alloc_workspace(T, d, v1 - v0, 0, p, B.CALL_LOGPROB_FWD, dev)
    ws.fill_(255)                                   # NaN patterns
    every = B.pg_head_shard_fwd(H, Ws, y, None, v0, p, ws)
    ws.fill_(255)
    masked = B.pg_head_shard_fwd(H, Ws, y, torch.ones(T, dtype=torch.uint8, device=dev), v0, p, ws)
    assert torch.equal(every, masked)               # the same contraction on the same rows
    z = H.double() @ Ws.double().T / p.temperature
    m = z.max(1).values
    e = torch.exp(z - m[:, None])
    mine = (y >= v0) & (y < v1)
    zy = torch.where(mine, z.gather(1, (y.long() - v0).clamp(0, v1 - v0 - 1)[:, None])[:, 0], 0.0)
    # fp32 sums of d products of bf16 values: a logit is off by `tol` at most, a term e^x by tol of itself, x e^x (x in [-20, 0])
    # by tol (1 + |x|) of e^x, and the sums of up to 443 such terms by as much again
    tol = d * 2.0 ** -23 * max(1.0, z.abs().max().item())
    got, s, x = every.double(), e.sum(1), z - m[:, None]
    assert (got[:, 0] - m).abs().max() <= tol and (got[:, 3] - zy).abs().max() <= tol
    assert ((got[:, 1] - s).abs() <= 4 * tol * s).all()
    assert ((got[:, 2] - (e * x).sum(1)).abs() <= 4 * tol * (e * (1 + x.abs())).sum(1)).all()
    assert (got[~mine, 3] == 0).all()
