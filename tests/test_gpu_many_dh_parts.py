"""dH of few tiles in more than eight parts, whose slabs lie over the dS^T that dW has read: the most parts, as many as the room or the stages allow,
wide tiles, fp32 products, few active rows of several vocab chunks; and the scatter of a row by one workgroup and by several.
Against plain fp64 arithmetic on the same operands; W as it lies and a W^T cache must give the same bits."""
import pytest
import torch

from paper_2602_05885_amd import binding as B
from paper_2602_05885_amd import synth
from tests._cases import block_rel_fro, dh_acc_rows, dh_form, dh_slabs, np64

pytestmark = pytest.mark.gpu


# T, active rows, d, V, dtype, vocab tiles of a chunk; parts, products and whether the tiles are wide.  64 parts of 4 stages; all that the room takes; all
# that the stages do; of two row tiles and three; three products; few active rows of several vocab chunks, their columns in one launch; wide tiles: one
# a row tile, a last one without its fifth MFMA rows, whole ones; few active of more rows than the scatter's form for few
@pytest.mark.parametrize("T,active,d,V,dtype,chunk,form", [
    (100, 100, 64, 16384, "bf16", None, (64, 1, False)), (1, 1, 1088, 65536, "bf16", None, (45, 1, False)), (200, 199, 1024, 2100, "bf16", None, (9, 1, False)),
    (512, 500, 1088, 2600, "bf16", None, (9, 1, False)), (513, 513, 1088, 2600, "bf16", None, (9, 1, False)), (100, 90, 192, 2900, "f32", None, (8, 3, False)),
    (300, 257, 320, 9000, "f32", None, (12, 3, False)), (2000, 150, 320, 9000, "bf16", 18, (36, 1, False)), (2000, 0, 320, 9000, "bf16", None, (1, 1, False)),
    (500, 490, 320, 32000, "bf16", None, (63, 1, True)), (1250, 1250, 576, 24000, "bf16", None, (24, 1, True)), (1000, 999, 1600, 24000, "bf16", None, (12, 1, True)),
    (2500, 90, 320, 16000, "bf16", None, (42, 1, False)), (4000, 64, 1088, 20000, "bf16", None, (32, 1, False)), (2600, 100, 192, 9000, "f32", None, (29, 3, False))])
@pytest.mark.parametrize("acc", [0, 1])
def test_many_parts(T, active, d, V, dtype, chunk, form, acc, monkeypatch):
    dev = torch.device("cuda:0")
    tiles_v, f32 = -(-V // 256), dtype == "f32"
    if active:
        assert dh_form(-(-active // 256) * 256, dh_acc_rows(T, d, V, f32, 2 if chunk else 1), d, 4 * tiles_v, f32) == form
    if chunk:
        monkeypatch.setenv("PG_HEAD_DS_BUDGET_BYTES", str((T + 255) // 256 * 256 * 2 * 256 * chunk))
    H, W, y = synth.make_head(T, d, V, dtype, T, dev)
    mask = torch.zeros(T, dtype=torch.uint8, device=dev)
    mask[torch.randperm(T, generator=torch.Generator().manual_seed(2))[:active].to(dev)] = 1
    start = torch.randn((V, d), generator=torch.Generator(device=dev).manual_seed(5), device=dev) * 1e-5
    outs = []
    for cache in (None, B.alloc_w_transposed(d, V, dev)):
        prm = B.Params(dtype=int(dtype == "f32"), accumulate_dW=acc, w_transposed=cache)
        ws = torch.full((B.pg_workspace_bytes(T, d, V, 0, prm, B.CALL_LOSS_FWD_BWD),), 0xFF, dtype=torch.uint8, device=dev)
        outs.append(B.pg_sft_fwd_bwd(H, W, y, mask, prm, ws, dW=start.clone() if acc else torch.full_like(start, float("nan"))))
        assert dh_slabs(ws) == form[0] * form[1]
    out = outs[0]
    for q in out:
        assert torch.equal(out[q], outs[1][q]), q
    on = mask.bool()
    assert not out["dH"][~on].any()
    Hd, Wd = H[on].double(), W.double()
    dS = torch.softmax(Hd @ Wd.T, 1)
    dS[torch.arange(active, device=dev), y[on].long()] -= 1
    dS /= max(active, 1)
    bound = 5e-5 if dtype == "f32" else 1e-2           # bf16 dS: 2^-9 per element; fp32 heads carry about 16 mantissa bits
    if active:
        assert block_rel_fro(np64(out["dH"][on]), np64(dS @ Wd)) <= bound
    assert block_rel_fro(np64(out["dW"]), np64(dS.T @ Hd + (start.double() if acc else 0))) <= bound


@pytest.mark.parametrize("T,active", [(300, 290), (2200, 130)])
def test_many_parts_of_a_shard(T, active):
    """The backward from the rows' states, fp32 dH out, against the same call on the whole head."""
    dev = torch.device("cuda:0")
    d, V = 320, 16000
    H, W, y = synth.make_head(T, d, V, "bf16", T, dev)
    mask = torch.zeros(T, dtype=torch.uint8, device=dev)
    mask[torch.randperm(T, generator=torch.Generator().manual_seed(3))[:active].to(dev)] = 1
    cu, adv = torch.tensor([0, T], dtype=torch.int32, device=dev), torch.tensor([-0.7], dtype=torch.float64, device=dev)
    prm = B.Params()
    ws = torch.full((B.pg_workspace_bytes(T, d, V, 1, prm, B.CALL_LOSS_FWD_BWD),), 0xFF, dtype=torch.uint8, device=dev)
    states = B.pg_head_shard_fwd(H, W, y, mask, 0, prm, ws)
    out = B.pg_loss_shard_bwd(H, W, y, mask, cu, adv, None, None, None, states, 0, prm, ws)
    assert dh_slabs(ws) == dh_form(-(-active // 256) * 256, dh_acc_rows(T, d, V), d, 4 * -(-V // 256))[0] > 8
    on = mask.bool()
    Hd, Wd = H[on].double(), W.double()
    dS = torch.softmax(Hd @ Wd.T, 1)
    dS[torch.arange(active, device=dev), y[on].long()] -= 1
    dS *= -0.7 / active                            # loss = -A log p / n: dz = A (p - onehot) / n
    assert not out["dH"][~on].any()
    assert block_rel_fro(np64(out["dH"][on]), np64(dS @ Wd)) <= 1e-2           # bf16 dS: 2^-9 per element
    assert block_rel_fro(np64(out["dW"]), np64(dS.T @ Hd)) <= 1e-2


# one to four column groups a thread; rows that fit the strips and rows that do not; an odd number of slabs and an even one
@pytest.mark.parametrize("T,active,d,V,dtype,slabs", [
    (90, 90, 256, 12000, "bf16", 32), (2300, 300, 256, 12000, "bf16", 38), (2300, 200, 2112, 10000, "bf16", 16), (1100, 200, 4160, 20000, "bf16", 14),
    (1100, 40, 6208, 20000, "bf16", 10), (1100, 300, 192, 9000, "f32", 54), (1100, 100, 2112, 9000, "f32", 27), (1100, 100, 4160, 6000, "f32", 15), (1100, 100, 6208, 6000, "f32", 9)])
def test_many_parts_behind_a_normalisation(T, active, d, V, dtype, slabs):
    dev = torch.device("cuda:0")
    X, W, y = synth.make_head(T, d, V, dtype, T, dev)
    gamma = 1 + 0.2 * torch.randn(d, generator=torch.Generator(device=dev).manual_seed(7), device=dev)
    gamma = gamma.to(X.dtype)
    mask = torch.zeros(T, dtype=torch.uint8, device=dev)
    mask[torch.randperm(T, generator=torch.Generator().manual_seed(3))[:active].to(dev)] = 1
    cu, adv = torch.tensor([0, T], dtype=torch.int32, device=dev), torch.tensor([-0.7], dtype=torch.float64, device=dev)
    prm = B.Params(dtype=int(dtype == "f32"))
    ws = torch.full((B.pg_workspace_bytes(T, d, V, 1, prm, B.CALL_LOSS_FWD_BWD_NORMED),), 0xFF, dtype=torch.uint8, device=dev)
    out = B.pg_loss_fwd_bwd_normed(X, gamma, 1e-5, W, y, mask, cu, adv, None, None, None, prm, ws)
    assert dh_slabs(ws) == slabs
    on = mask.bool()
    Xd, gd, Wd = X[on].double(), gamma.double(), W.double()
    rstd = (Xd.pow(2).mean(1, keepdim=True) + 1e-5).rsqrt()
    xhat = Xd * rstd
    H = (xhat * gd).to(X.dtype).double()           # the head sees it in the storage type
    dS = torch.softmax(H @ Wd.T, 1)
    dS[torch.arange(active, device=dev), y[on].long()] -= 1
    dH = (dS * (-0.7 / active)) @ Wd
    want = rstd * (gd * dH - xhat * (gd * dH * xhat).mean(1, keepdim=True))
    bound = 5e-5 if dtype == "f32" else 1e-2           # bf16 dS and dX: 2^-9 per element each; fp32 heads carry about 16 mantissa bits
    assert not out["dX"][~on].any()
    assert block_rel_fro(np64(out["dX"][on]), np64(want)) <= bound
    assert block_rel_fro(np64(out["dgamma"][:, None]), np64((dH * xhat).sum(0)[:, None])) <= bound
