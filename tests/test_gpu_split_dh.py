"""The dH contraction: split with every row active (eight parts per chunk, of which a short last chunk leaves some without a
single stage; the accumulator holds more rows than the call has tokens), and the form that reads W as it lies."""
import pytest
import torch

from oracle import pg_oracle as O
from paper_2602_05885_amd import binding as B
from paper_2602_05885_amd import synth
from tests._cases import block_rel_fro, np64, recompute_covers_vocabulary

pytestmark = pytest.mark.gpu


# (T, d, vocab tiles of the first chunk, V): one row tile and two, one column tile and a ragged second one, a last chunk
# of 4 stages (fewer than parts) and of one ragged vocab tile, a single chunk, a head of too many dW tiles to split dW
@pytest.mark.parametrize("T,d,chunk_tiles,V", [(1, 64, 16, 256 * 17), (300, 320, 16, 256 * 16 + 3), (256, 128, 32, 256 * 33 + 100),
                                               (513, 64, None, 256 * 20), (300, 64, None, 33100)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_split_dh_all_rows_active(T, d, chunk_tiles, V, dtype, monkeypatch):
    dev = torch.device("cuda:0")
    if chunk_tiles:
        monkeypatch.setenv("PG_HEAD_DS_BUDGET_BYTES", str((T + 255) // 256 * 256 * 2 * 256 * chunk_tiles))
    H, W, y = synth.make_head(T, d, V, dtype, 99 + T, dev)
    mask = torch.ones(T, dtype=torch.uint8, device=dev)
    prm = B.Params(dtype=int(dtype == "f32"))
    ws = torch.full((B.pg_workspace_bytes(T, d, V, 0, prm, B.CALL_LOSS_FWD_BWD),), 0xFF, dtype=torch.uint8, device=dev)
    out = B.pg_sft_fwd_bwd(H, W, y, mask, prm, ws)
    torch.cuda.synchronize()
    ref = O.sft_ce_fwd_bwd(np64(H), np64(W), y.cpu().numpy(), mask.cpu().numpy())
    tol = 5e-5 if dtype == "f32" else 1e-2       # bf16 dS: 2^-9 per element; fp32 heads carry about 16 mantissa bits
    for q in ("dH", "dW"):
        assert block_rel_fro(np64(out[q]), ref[q]) <= tol, q


# more rows than the direct form of the dH contraction takes: the device chooses by the active ones; the W^T cache
# forces the other form, whose products and sums are the same
@pytest.mark.parametrize("active", [0, 1, 8192, 8193, 8700])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_direct_dh_is_chosen_by_the_active_rows(active, dtype):
    dev = torch.device("cuda:0")
    T, d, V = 8700, 192, 515
    H, W, y = synth.make_head(T, d, V, dtype, 7, dev)
    mask = torch.zeros(T, dtype=torch.uint8, device=dev)
    mask[torch.randperm(T, generator=torch.Generator().manual_seed(1))[:active].to(dev)] = 1
    outs = []
    for cache in (None, B.alloc_w_transposed(d, V, dev)):
        prm = B.Params(dtype=int(dtype == "f32"), w_transposed=cache)
        ws = torch.full((B.pg_workspace_bytes(T, d, V, 0, prm, B.CALL_LOSS_FWD_BWD),), 0xFF, dtype=torch.uint8, device=dev)
        outs.append(B.pg_sft_fwd_bwd(H, W, y, mask, prm, ws))
    torch.cuda.synchronize()
    for q in outs[0]:
        assert torch.equal(outs[0][q], outs[1][q]), q
    if active:
        rows = mask.nonzero()[:40, 0].cpu().numpy()
        ref = O.sft_ce_fwd_bwd(np64(H)[rows], np64(W), y.cpu().numpy()[rows], [1] * len(rows), norm_override=float(active))
        assert block_rel_fro(np64(outs[0]["dH"])[rows], ref["dH"]) <= (5e-5 if dtype == "f32" else 1e-2)


# a small head's dW: one part (written to dW itself; no active row at all among them), two and more, over one vocab chunk
# and several, added to what is there or not
@pytest.mark.parametrize("T,active", [(1100, 0), (1100, 1), (1100, 256), (1100, 257), (1100, 1100), (200, 200)])
@pytest.mark.parametrize("dtype,dw16,acc,budget", [("bf16", 1, 1, None), ("bf16", 0, 1, 2), ("bf16", 1, 0, 2), ("f32", 0, 1, None)])
def test_split_dw_of_small_heads(T, active, dtype, dw16, acc, budget, monkeypatch):
    dev = torch.device("cuda:0")
    d, V = 320, 1500
    if budget:
        monkeypatch.setenv("PG_HEAD_DS_BUDGET_BYTES", str((T + 255) // 256 * 256 * 2 * 256 * budget))
    H, W, y = synth.make_head(T, d, V, dtype, 17, dev)
    mask = torch.zeros(T, dtype=torch.uint8, device=dev)
    mask[torch.randperm(T, generator=torch.Generator().manual_seed(4))[:active].to(dev)] = 1
    prm = B.Params(dtype=int(dtype == "f32"), dW_dtype=dw16, accumulate_dW=acc)
    start = (torch.randn((V, d), generator=torch.Generator().manual_seed(5)) * 1e-3).to(torch.bfloat16 if dw16 else torch.float32).to(dev)
    dW = start.clone() if acc else torch.full_like(start, float("nan"))
    ws = torch.full((B.pg_workspace_bytes(T, d, V, 0, prm, B.CALL_LOSS_FWD_BWD),), 0xFF, dtype=torch.uint8, device=dev)
    out = B.pg_sft_fwd_bwd(H, W, y, mask, prm, ws, dW=dW)
    torch.cuda.synchronize()
    ref = O.sft_ce_fwd_bwd(np64(H), np64(W), y.cpu().numpy(), mask.cpu().numpy(), dW_prev=np64(start) if acc else None)
    tol = 1e-2 if dtype == "bf16" else 5e-5      # bf16 dS and dW: 2^-9 per element each; fp32 heads carry about 16 mantissa bits
    for q in ("dH", "dW"):
        assert block_rel_fro(np64(out[q]), ref[q]) <= tol, q
    if acc and active == 0:
        assert torch.equal(out["dW"], start)


# the same choice where the rows are few enough that dS spans the vocabulary (planned in two chunks): up to 8192 rows dH is
# one launch that reads W as it lies, beyond it keeps its chunks, with their W^T and their columns of the wide dS.  Kept
# logits (201 tiles, at most 256) and recomputed ones (335).
@pytest.mark.parametrize("V,chunk_tiles", [(515, 2), (1027, 3)])
@pytest.mark.parametrize("active", [8192, 8193, 8700])
def test_wide_ds_with_chunked_and_whole_dh(active, V, chunk_tiles, monkeypatch):
    dev = torch.device("cuda:0")
    T, d = 17000, 192
    monkeypatch.setenv("PG_HEAD_DS_BUDGET_BYTES", str((T + 255) // 256 * 256 * 2 * 256 * chunk_tiles))
    n_pad = (active + 255) // 256 * 256
    assert B.pg_backward_chunk_rows(T, d, V, 0, B.Params()) == 256 * chunk_tiles
    assert recompute_covers_vocabulary(T, V, n_pad, 256 * chunk_tiles)
    H, W, y = synth.make_head(T, d, V, "bf16", 8, dev)
    mask = torch.zeros(T, dtype=torch.uint8, device=dev)
    mask[torch.randperm(T, generator=torch.Generator().manual_seed(2))[:active].to(dev)] = 1
    outs = []
    for cache in (None, B.alloc_w_transposed(d, V, dev)):
        prm = B.Params(w_transposed=cache)
        ws = torch.full((B.pg_workspace_bytes(T, d, V, 0, prm, B.CALL_LOSS_FWD_BWD),), 0xFF, dtype=torch.uint8, device=dev)
        outs.append(B.pg_sft_fwd_bwd(H, W, y, mask, prm, ws))
    torch.cuda.synchronize()
    for q in outs[0]:
        assert torch.equal(outs[0][q], outs[1][q]), q
    ref = O.sft_ce_fwd_bwd(np64(H), np64(W), y.cpu().numpy(), mask.cpu().numpy())
    for q in ("dH", "dW"):                  # bf16 dS: 2^-9 per element
        assert block_rel_fro(np64(outs[0][q]), ref[q]) <= 1e-2, q
