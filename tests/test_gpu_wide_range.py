"""dH where 320 rows of W^T reach beyond 4 GiB, the range of a tile's 32-bit operand offsets, and 256 rows do not: the launch stays with tiles of 256
columns.  At the far end of the vocabularies that a W^T cache is accepted for; every column of sampled rows against plain fp64 arithmetic."""
import pytest
import torch

from paper_2602_05885_amd import binding as B
from paper_2602_05885_amd import synth
from tests._cases import pad_ld

pytestmark = pytest.mark.gpu


def test_dh_of_a_vocabulary_that_wide_tiles_do_not_reach():
    dev = torch.device("cuda:0")
    T, d, V = 8192, 320, 7_000_000
    ld = pad_ld(-(-V // 256) * 256)
    assert ld * 2 * 256 < 1 << 32 <= ld * 2 * 320 and B.lib().pg_w_transposed_bytes(d, V) > 0
    H, W, y = synth.make_head(T, d, V, "bf16", 3, dev)
    mask = torch.ones(T, dtype=torch.uint8, device=dev)
    prm = B.Params(dW_dtype=1, w_transposed=B.alloc_w_transposed(d, V, dev))
    ws = torch.empty(B.pg_workspace_bytes(T, d, V, 0, prm, B.CALL_LOSS_FWD_BWD), dtype=torch.uint8, device=dev)
    out = B.pg_sft_fwd_bwd(H, W, y, mask, prm, ws)
    rows = torch.arange(0, T, T // 16, device=dev)
    step = 500_000
    z = torch.cat([H[rows].double() @ W[a:a + step].double().T for a in range(0, V, step)], 1)
    dS = torch.softmax(z, 1)
    dS[torch.arange(len(rows), device=dev), y[rows].long()] -= 1
    want = sum((dS[:, a:a + step] @ W[a:a + step].double()) for a in range(0, V, step)) / T
    got = out["dH"][rows].double()
    for c in range(0, d, 16):           # the columns of one MFMA row at a time: bf16 dS and dH, 2^-9 per element each
        err = float((got[:, c:c + 16] - want[:, c:c + 16]).norm() / want[:, c:c + 16].norm())
        assert err <= 1e-2, (c, err)
