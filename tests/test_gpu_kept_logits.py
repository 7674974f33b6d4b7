"""The loss calls park logits tiles in the last part of the workspace and recompute those that do not fit: the results
must not depend on how many fit (bit for bit), from none to all of them, and agree with the oracle."""
import pytest
import torch

from oracle import pg_oracle as O
from paper_2602_05885_amd import binding as B
from paper_2602_05885_amd import synth
from tests._cases import build_loss_case, rel_fro

pytestmark = pytest.mark.gpu
TILE = 256 * 256 * 4


def _oracle_logp(H, W, y, tau):
    return O.lm_head_logprob(H, W, y, tau)[0]


# (d, V, dtype, share of the rows, dS budget, mismatch mode): single tiles, a ragged last vocab tile, several chunks, few rows of several chunks
@pytest.mark.parametrize("d,V,dtype,scale,budget,mode", [
    (64, 200, "bf16", 0.2, None, 0), (128, 2500, "bf16", 1.0, None, 2), (128, 2500, "f32", 1.0, None, 2),
    (192, 2561, "bf16", 1.0, 1 << 20, 2), (128, 1537, "f32", 1.0, 1 << 20, 0), (64, 3000, "bf16", 1.0, 1 << 20, 1)])
def test_results_do_not_depend_on_the_kept_tiles(d, V, dtype, scale, budget, mode, monkeypatch):
    dev = torch.device("cuda:0")
    if budget:
        monkeypatch.setenv("PG_HEAD_DS_BUDGET_BYTES", str(budget))
    spec = synth.small_spec(d=d, V=V, dtype=dtype, seed=4321, pack_rows=1500 if scale == 1.0 else 900)
    batch, t, n = build_loss_case(spec, dev, _oracle_logp, "window" if mode == 1 else "token" if mode == 2 else "none", scale_rows=scale)
    T, S = batch.T, batch.S
    prm = B.Params(dtype=int(dtype == "f32"), mismatch_mode=mode)
    adv, _, _ = B.trloo_advantage(t["rewards"], t["valid"], 1.0)
    full = B.pg_workspace_bytes(T, d, V, S, prm, B.CALL_LOSS_FWD_BWD)
    tiles = (T + 255) // 256 * ((V + 255) // 256)
    kept = min(tiles, (budget or 2 << 30) // 8 * 39 // TILE)
    ref = None
    for k in sorted({0, 1, kept // 3, kept // 2 + 1, kept - 1, kept} & set(range(kept + 1))):
        ws = torch.full((full - (kept - k) * TILE,), 0xFF, dtype=torch.uint8, device=dev)      # NaN patterns
        out = B.pg_loss_fwd_bwd(t["H"], t["W"], t["y"], t["loss_mask"], t["cu"], adv.reshape(-1), t["seg_sample"], t["old"],
                                t["rollout"], prm, ws)
        torch.cuda.synchronize()
        out = {q: v.cpu() for q, v in out.items()}
        if ref is None:
            ref = out
            A = adv.cpu().numpy().reshape(-1)[batch.seg_sample]
            want = O.pg_loss_fwd_bwd(n["H"], n["W"], n["y"], n["loss_mask"], n["cu"], A, n["old"], n["rollout"], O.Params(mismatch_mode=mode))
            for q in ("dH", "dW"):      # bf16 dS: 2^-9 per element; fp32 heads carry about 16 mantissa bits
                assert rel_fro(out[q].double().numpy(), want[q]) <= (5e-5 if dtype == "f32" else 1e-2), q
        for q in ref:
            assert torch.equal(out[q], ref[q]), (q, k, kept)
    with pytest.raises(B.PgError, match="needed"):      # shorter than everything but the kept tiles
        B.pg_loss_fwd_bwd(t["H"], t["W"], t["y"], t["loss_mask"], t["cu"], adv.reshape(-1), t["seg_sample"], t["old"], t["rollout"], prm,
                          torch.empty(full - kept * TILE - 1, dtype=torch.uint8, device=dev))
