"""Active row counts around every line at which the kernels cut the last token tile short (64 rows of a contraction over
the tokens, 128 and 192 columns of a token tile): against the oracle, from a workspace full of NaN patterns, with all logits
kept and with none."""
import pytest
import torch

from oracle import pg_oracle as O
from paper_2602_05885_amd import binding as B
from paper_2602_05885_amd import synth
from tests._cases import block_rel_fro, np64

pytestmark = pytest.mark.gpu
T = 700


@pytest.mark.parametrize("dtype,d,V", [("bf16", 128, 700), ("f32", 64, 300), ("bf16", 320, 257)])
@pytest.mark.parametrize("active", [1, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256, 257, 320, 385, 449, 513, 700])
def test_sft_row_counts(dtype, d, V, active):
    dev = torch.device("cuda:0")
    H, W, y = synth.make_head(T, d, V, dtype, 21, dev)
    m = torch.zeros(T, dtype=torch.uint8)
    m[torch.randperm(T, generator=torch.Generator().manual_seed(active))[:active]] = 1
    prm = B.Params(dtype=int(dtype == "f32"))
    full = B.pg_workspace_bytes(T, d, V, 0, prm, B.CALL_LOSS_FWD_BWD)
    least = B.pg_workspace_min_bytes(T, d, V, 0, prm, B.CALL_LOSS_FWD_BWD)
    outs = []
    for n in (full, least):
        ws = torch.full((n,), 0xFF, dtype=torch.uint8, device=dev)
        outs.append(B.pg_sft_fwd_bwd(H, W, y, m.to(dev), prm, ws, dW=torch.full((V, d), float("nan"), device=dev)))
    logp, ent, _ = B.pg_logprob_fwd(H, W, y, m.to(dev), prm, torch.full((full,), 0xFF, dtype=torch.uint8, device=dev))
    torch.cuda.synchronize()
    ref = O.sft_ce_fwd_bwd(np64(H), np64(W), y.cpu().numpy(), m.numpy())
    for q in ("dH", "dW"):                     # bf16 dS: 2^-9 per element; fp32 heads carry about 16 mantissa bits
        assert block_rel_fro(np64(outs[0][q]), ref[q], 64) <= (5e-5 if dtype == "f32" else 1e-2), q
    for q in outs[0]:                          # kept logits are the very values that a recompute gives
        assert torch.equal(outs[0][q], outs[1][q]), q
    want = O.lm_head_logprob(np64(H), np64(W), y.cpu().numpy(), 1.0)
    on = m.bool()
    for got, w in ((logp, want[0]), (ent, want[1]), (outs[0]["logp"], want[0]), (outs[0]["entropy"], want[1])):
        assert (got.cpu().double()[on] - torch.from_numpy(w)[on]).abs().max() <= 2e-4       # fp32 sums of exact products
        assert not got.cpu()[~on].any()
