"""dS from parked logits in items of 32 tokens (up to 96 half tiles of a launch) and of 128: last token tiles that end inside an item, one row,
several token tiles, fp32 remainders.  Against the recomputing kernel (the same bits) and against plain fp64 arithmetic."""
import pytest
import torch

from paper_2602_05885_amd import binding as B
from paper_2602_05885_amd import synth
from tests._cases import block_rel_fro, np64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,V,dtype", [(1, 256, "bf16"), (33, 12288, "bf16"), (33, 12289, "bf16"), (545, 4096, "bf16"), (545, 4097, "bf16"), (225, 300, "f32"),
                                       (300, 3072, "f32"), (300, 3073, "f32")])
def test_small_items(T, V, dtype):
    dev, d = torch.device("cuda:0"), 64
    H, W, y = synth.make_head(T, d, V, dtype, T, dev)
    mask = torch.ones(T, dtype=torch.uint8, device=dev)
    if T > 1:
        mask[T // 2] = 0                               # the compacted rows are not the rows
    prm = B.Params(dtype=int(dtype == "f32"))
    size = B.pg_workspace_bytes(T, d, V, 0, prm, B.CALL_LOSS_FWD_BWD)
    tiles = -(-T // 256) * -(-V // 256)
    out = [B.pg_sft_fwd_bwd(H, W, y, mask, prm, torch.full((size - short * 256 * 256 * 4,), 0xFF, dtype=torch.uint8, device=dev)) for short in (0, tiles)]
    for q in out[0]:
        assert torch.equal(out[0][q], out[1][q]), q
    Hd, Wd, on = H.double(), W.double(), mask.bool()
    dS = torch.softmax(Hd @ Wd.T, 1)
    dS[torch.arange(T, device=dev), y.long()] -= 1
    dS *= on[:, None] / int(on.sum())
    bound = 5e-5 if dtype == "f32" else 1e-2           # bf16 dS: 2^-9 per element; fp32 heads carry about 16 mantissa bits
    assert block_rel_fro(np64(out[0]["dH"]), np64(dS @ Wd)) <= bound
    assert block_rel_fro(np64(out[0]["dW"]), np64(dS.T @ Hd)) <= bound
