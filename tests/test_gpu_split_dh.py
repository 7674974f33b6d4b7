"""The split dH contraction with every row active: eight parts per chunk, of which a short last chunk leaves some without
a single stage; the accumulator holds more rows than the call has tokens."""
import pytest
import torch

from oracle import pg_oracle as O
from paper_2602_05885_amd import binding as B
from paper_2602_05885_amd import synth
from tests._cases import block_rel_fro, np64

pytestmark = pytest.mark.gpu


# (T, d, vocab tiles of the first chunk, V): one row tile and two, one column tile and a ragged second one, a last chunk
# of 4 stages (fewer than parts) and of one ragged vocab tile, a single chunk
@pytest.mark.parametrize("T,d,chunk_tiles,V", [(1, 64, 16, 256 * 17), (300, 320, 16, 256 * 16 + 3), (256, 128, 32, 256 * 33 + 100),
                                               (513, 64, None, 256 * 20)])
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
