"""The merge of the vocab tiles' softmax states by workgroups of 16 rows (up to 3072 padded rows) and of 64: fewer tiles than parts, one or several turns of
them, ragged last tiles and rows.  Against plain fp64 arithmetic."""
import pytest
import torch

from paper_2602_05885_amd import binding as B
from paper_2602_05885_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 700, 3072, 3073])
@pytest.mark.parametrize("V", [200, 256 * 16 + 1, 256 * 64, 256 * 64 + 1, 256 * 300 + 5])
def test_states_of_few_rows(T, V):
    dev, d = torch.device("cuda:0"), 64
    H, W, y = synth.make_head(T, d, V, "bf16", T, dev)
    W[V - 1] = W[0] * 40                                   # a last tile that outweighs the others, for some of the rows
    mask = torch.ones(T, dtype=torch.uint8, device=dev)
    if T > 1:
        mask[::7] = 0
    prm = B.Params(temperature=0.8)
    ws = torch.full((B.pg_workspace_bytes(T, d, V, 0, prm, B.CALL_LOGPROB_FWD),), 0xFF, dtype=torch.uint8, device=dev)
    logp, ent, lse = B.pg_logprob_fwd(H, W, y, mask, prm, ws)
    on = mask.bool()
    assert not logp[~on].any() and not ent[~on].any()
    z = H[on].double() @ W.double().T / prm.temperature
    p = torch.log_softmax(z, 1)
    big = z.abs().max().item()
    # fp32: 64 products of a logit, exponent and logarithm in base 2 (a few 2^-24 of the largest logit), 1024 merges at most
    bound = 64 * 2.0 ** -24 * max(big, 1.0)
    for got, want in ((logp, p[torch.arange(int(on.sum()), device=dev), y[on].long()]), (lse, torch.logsumexp(z, 1)), (ent, -(p.exp() * p).sum(1))):
        err = (got[on].double() - want).abs().max().item()
        assert err <= (bound if got is not ent else 4 * bound), (err, bound)      # (entropy: lse less a mean of logits, whose weights carry the error too)
