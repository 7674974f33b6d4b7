"""dW and dH in tiles of 320 output columns: both readers of W, widths that end in the middle of a tile (with and without a part of its
last 64 columns), split and whole contractions, every store of dW.  Against plain fp64 arithmetic on the same bf16 operands."""
import pytest
import torch

from paper_2602_05885_amd import binding as B
from paper_2602_05885_amd import synth
from tests._cases import block_rel_fro, dh_acc_rows, dh_form, np64, wide_pays

pytestmark = pytest.mark.gpu


# T, d, V, which of dW / dH are wide.  d = 320: one tile; 576: the second has its first four MFMA rows per wavefront and not the fifth;
# 832, 1472: the last has some wavefronts only; 1536: the fifth rows of three wavefronts; 1600: whole tiles.  20000 rows read W^T, the others W as it lies.
CASES = [(70, 320, 17000, "dW"), (300, 576, 23552, "dW"), (130, 832, 37000, "dW"), (20000, 320, 700, "dH"), (1500, 1600, 25600, "dW dH"),
         (8000, 576, 5000, "dH"), (4000, 1472, 13000, "dW dH"), (4000, 1536, 13000, "dW dH"), (2500, 832, 26000, "dH")]


@pytest.mark.parametrize("T,d,V,wide", CASES)
@pytest.mark.parametrize("dw16,acc", [(0, 0), (0, 1), (1, 1)])
def test_wide_tiles(T, d, V, wide, dw16, acc):
    dev = torch.device("cuda:0")
    tiles_v, t_pad = -(-V // 256), -(-T // 256) * 256
    whole_dW = 2 * tiles_v * -(-d // 256) > 256            # (a smaller head's dW is split into slabs)
    whole = (1, -(-T // 64))
    assert (whole_dW and wide_pays(tiles_v, d, whole, whole)) == ("dW" in wide)
    assert dh_form(t_pad, dh_acc_rows(T, d, V), d, 4 * tiles_v)[2] == ("dH" in wide)
    H, W, y = synth.make_head(T, d, V, "bf16", T, dev)
    mask = torch.ones(T, dtype=torch.uint8, device=dev)
    mask[T // 2] = 0                                       # the compacted rows are not the rows
    prm = B.Params(dW_dtype=dw16, accumulate_dW=acc)
    g = torch.Generator(device=dev).manual_seed(5)
    start = (torch.randn((V, d), generator=g, device=dev) * 1e-5).to(torch.bfloat16 if dw16 else torch.float32)
    dW = start.clone() if acc else torch.full_like(start, float("nan"))
    ws = torch.full((B.pg_workspace_bytes(T, d, V, 0, prm, B.CALL_LOSS_FWD_BWD),), 0xFF, dtype=torch.uint8, device=dev)
    out = B.pg_sft_fwd_bwd(H, W, y, mask, prm, ws, dW=dW)
    Hd, Wd, on = H.double(), W.double(), mask.bool()
    want_dW = start.double() if acc else torch.zeros((V, d), dtype=torch.float64, device=dev)
    want_dH = torch.zeros((T, d), dtype=torch.float64, device=dev)
    for a in range(0, T, 2000):
        rows = torch.arange(a, min(a + 2000, T), device=dev)
        rows = rows[on[rows]]
        dS = torch.softmax(Hd[rows] @ Wd.T, 1)
        dS[torch.arange(len(rows), device=dev), y[rows].long()] -= 1
        dS /= T - 1
        want_dH[rows] = dS @ Wd
        want_dW += dS.T @ Hd[rows]
    assert block_rel_fro(np64(out["dH"]), np64(want_dH)) <= 1e-2        # bf16 dS and dH (and dW): 2^-9 per element each
    assert block_rel_fro(np64(out["dW"]), np64(want_dW)) <= 1e-2
