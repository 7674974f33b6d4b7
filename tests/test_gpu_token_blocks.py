"""Loss calls whose kept logits do not fit at once work their rows off in token blocks: results against the oracle and
against the one-block plan (which a shorter workspace gets), for every number of live blocks from none to all."""
import pytest
import torch

from oracle import pg_oracle as O
from paper_2602_05885_amd import binding as B
from paper_2602_05885_amd import synth
from tests._cases import block_rel_fro, np64

pytestmark = pytest.mark.gpu
# three vocab tiles; 48 kept tiles: blocks of 16 token tiles, three of them; d: 512 dH tiles per block, the two rounds over
# 256 compute units from which a call is planned in blocks
T, V, BLOCK, D = 9000, 515, 4096, 8192


@pytest.fixture()
def budget(monkeypatch):
    monkeypatch.setenv("PG_HEAD_DS_BUDGET_BYTES", "2600000")      # 39/8 of it: 48 tiles of 256 KiB; a vocab chunk is one tile


def _mask(active, dev):
    m = torch.zeros(T, dtype=torch.uint8)
    m[torch.randperm(T, generator=torch.Generator().manual_seed(3))[:active]] = 1
    return m.to(dev)


@pytest.mark.parametrize("active", [0, 1, BLOCK, BLOCK + 1, 2 * BLOCK, 2 * BLOCK + 1, T])
@pytest.mark.parametrize("accumulate,cache", [(0, False), (1, True)])
def test_sft_in_token_blocks(budget, active, accumulate, cache):
    dev, d = torch.device("cuda:0"), D
    H, W, y = synth.make_head(T, d, V, "bf16", 11, dev)
    mask = _mask(active, dev)
    prm = B.Params(accumulate_dW=accumulate, w_transposed=B.alloc_w_transposed(d, V, dev) if cache else None)
    need = B.pg_workspace_bytes(T, d, V, 0, prm, B.CALL_LOSS_FWD_BWD)
    start = torch.randn((V, d), generator=torch.Generator().manual_seed(5)).mul_(1e-3).to(dev)
    outs = []
    for n in (need, need - 1):                 # token blocks; one block
        dW = start.clone() if accumulate else torch.full((V, d), float("nan"), device=dev)
        outs.append(B.pg_sft_fwd_bwd(H, W, y, mask, prm, torch.full((n,), 0xFF, dtype=torch.uint8, device=dev), dW=dW))
    torch.cuda.synchronize()
    ref = O.sft_ce_fwd_bwd(np64(H), np64(W), y.cpu().numpy(), mask.cpu().numpy(), dW_prev=np64(start) if accumulate else None)
    for o in outs:
        for q in ("dH", "dW"):                 # bf16 dS: 2^-9 per element
            assert block_rel_fro(np64(o[q]), ref[q]) <= 1e-2, q
    for q in ("loss", "logp", "entropy", "counters"):
        assert torch.equal(outs[0][q], outs[1][q]), q


def test_normed_loss_in_token_blocks_repeats_and_replays(budget):
    """Fused normalisation, off-policy surrogate with weights, three live blocks: against the one-block plan (fp32 sums in
    another order), bit for bit on a second call with a scrambled workspace and on replays of a captured graph."""
    dev, d, S = torch.device("cuda:0"), D, 3
    H, W, y = synth.make_head(T, d, V, "bf16", 12, dev)
    g = torch.Generator(device=dev).manual_seed(1)
    gamma = (1 + 0.1 * torch.randn(d, generator=g, device=dev)).to(torch.bfloat16)
    mask, cu = _mask(8900, dev), torch.tensor([0, 3000, 6100, T], dtype=torch.int32, device=dev)
    adv = torch.tensor([0.7, -0.4, 1.1], dtype=torch.float64, device=dev)
    old = -6.3 + 0.05 * torch.randn(T, generator=g, device=dev)
    rollout = old + 0.1 * torch.randn(T, generator=g, device=dev)
    prm = B.Params(mismatch_mode=2, clip_eps_lo=10.0, clip_eps_hi=10.0)
    need = B.pg_workspace_bytes(T, d, V, S, prm, B.CALL_LOSS_FWD_BWD_NORMED)
    call = lambda ws: B.pg_loss_fwd_bwd_normed(H, gamma, 1e-6, W, y, mask, cu, adv, None, old, rollout, prm, ws)      # noqa: E731
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device=dev)
    a = {q: v.clone() for q, v in call(ws).items()}
    one = call(torch.empty(need - 1, dtype=torch.uint8, device=dev))
    ws.random_(0, 255)
    b = call(ws)
    torch.cuda.synchronize()
    for q in a:
        assert torch.equal(a[q], b[q]), q
        if a[q].is_floating_point():
            e = ((a[q].double() - one[q].double()).norm() / one[q].double().norm()).item()
            assert e <= (1e-3 if q == "dX" else 1e-5), (q, e)     # dX is rounded to bf16, the others are fp32 sums
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        c = call(ws)
    for _ in range(3):
        ws.random_(0, 255)
        graph.replay()
        torch.cuda.synchronize()
        for q in a:
            assert torch.equal(a[q], c[q]), q


def test_shorter_workspaces_down_to_the_least(monkeypatch):
    """Token blocks; one block with part of the logits; with none; with half of the dS scratch (one vocab tile per chunk
    instead of two), at the least workspace the call takes."""
    dev, d, V2 = torch.device("cuda:0"), D, 2600
    monkeypatch.setenv("PG_HEAD_DS_BUDGET_BYTES", "9500000")      # 176 kept tiles, of 11 vocab tiles: again 16 token tiles
    H, W, y = synth.make_head(T, d, V2, "bf16", 13, dev)
    prm, mask = B.Params(), _mask(8800, dev)
    full, least = (f(T, d, V2, 0, prm, B.CALL_LOSS_FWD_BWD) for f in (B.pg_workspace_bytes, B.pg_workspace_min_bytes))
    row_tile = 9216 * 2 * 256 * 2                                 # a vocab tile of both orientations of dS
    outs = []
    for n in (full, full - 1, least + row_tile // 2, least):
        outs.append(B.pg_sft_fwd_bwd(H, W, y, mask, prm, torch.full((n,), 0xFF, dtype=torch.uint8, device=dev)))
    torch.cuda.synchronize()
    for o in outs[1:]:
        for q in ("loss", "logp", "entropy", "counters"):
            assert torch.equal(o[q], outs[0][q]), q
        for q in ("dH", "dW"):
            e = ((o[q].double() - outs[0][q].double()).norm() / outs[0][q].double().norm()).item()
            assert e <= (1e-3 if q == "dH" else 1e-5), (q, e)     # dH is rounded to bf16, dW is fp32 sums in another order
    with pytest.raises(B.PgError, match="needed"):
        B.pg_sft_fwd_bwd(H, W, y, mask, prm, torch.empty(least - 1, dtype=torch.uint8, device=dev))
