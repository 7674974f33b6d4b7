"""The pre-pass's flags and counts: rows in no segment (before, behind and between what the offsets span), empty segments and segments without a loss row,
samples filtered, vetoed, outside the window and outside the table, truncated rows, row counts around a wavefront's 256 and a workgroup's turn."""
import numpy as np
import pytest
import torch

from paper_2602_05885_amd import binding as B
from paper_2602_05885_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,lo,hi", [(1, 0, 1), (5, 1, 4), (255, 0, 255), (1000, 3, 997), (4097, 256, 4096), (9000, 0, 9000), (700, 0, 0)])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_counts(T, lo, hi, mode):
    dev, rng = torch.device("cuda:0"), np.random.default_rng(T + mode)
    d, V = 64, 300
    S = max(1, (hi - lo) // 37)
    cu = np.sort(np.concatenate([[lo, hi], rng.integers(lo, hi + 1, S - 1)])).astype(np.int32)      # (repeated offsets: empty segments)
    mask = (rng.random(T) < 0.7).astype(np.uint8)
    if S > 3:
        mask[cu[2]:cu[3]] = 0
    n_samples = S + 2
    idx = rng.permutation(n_samples)[:S].astype(np.int32)
    if S > 4:
        idx[1], idx[4] = n_samples, -1                    # outside the table
    keep = (rng.random(n_samples) < 0.8).astype(np.uint8)
    old = rng.normal(-3, 0.5, T).astype(np.float32)
    delta = rng.normal(0, 1e-4 if mode == 1 else 0.4, T)
    for s in range(0, S, 3):
        delta[cu[s]:cu[s + 1]] += 0.5                     # outside the window
    for s in range(1, S, 5):
        if cu[s + 1] > cu[s]:
            delta[cu[s]] = -12.0                          # vetoed, if that row carries loss
    rollout = (old.astype(np.float64) - delta).astype(np.float32)
    prm = B.Params(mismatch_mode=mode)
    want, active = np.zeros(8, np.int64), np.zeros(T, bool)
    for s in range(S):
        rows = np.arange(cu[s], cu[s + 1])[mask[cu[s]:cu[s + 1]] != 0]
        if not len(rows):
            continue
        if not 0 <= idx[s] < n_samples or not keep[idx[s]]:
            want[7] += 1
            continue
        want[6] += len(rows)
        dl = old[rows].astype(np.float64) - rollout[rows].astype(np.float64)
        out = False
        if mode:
            veto = prm.veto_ratio > 0 and np.exp(dl.min()) < prm.veto_ratio
            window = mode == 1 and not prm.geo_lo <= np.exp(dl.mean()) <= prm.geo_hi
            want[4] += veto
            want[3] += window
            out = veto or window
        if not out:
            active[rows] = True
            want[0] += len(rows)
            if mode == 2:
                want[5] += int((np.exp(dl) > prm.trunc_c).sum())
    H, W, y = synth.make_head(T, d, V, "bf16", T, dev)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    ws = torch.full((B.pg_workspace_bytes(T, d, V, S, prm, B.CALL_LOSS_FWD_BWD),), 0xFF, dtype=torch.uint8, device=dev)
    adv = t(rng.normal(0, 1, n_samples))
    for _ in range(2):                                    # (again on what the first call left behind)
        out = B.pg_loss_fwd_bwd(H, W, y, t(mask), t(cu), adv, t(idx), t(old), t(rollout), prm, ws, sample_keep=t(keep))
        got = out["counters"].cpu().numpy()
        assert (got[[0, 3, 4, 5, 6, 7]] == want[[0, 3, 4, 5, 6, 7]]).all(), (got, want)
        logp = out["logp"].cpu().numpy()
        assert ((logp != 0) == active).all() and not out["dH"].cpu().float().numpy()[~active].any()


@pytest.mark.parametrize("cu", [[0, 100, 50], [90, 120, 40, 70], [0, 0, 0], [200, 300, 200]])
def test_offsets_that_go_back(cu):
    """A segment whose end lies before its start is empty; the rows of the others stay theirs, and rows of none are not active."""
    dev, T, d, V = torch.device("cuda:0"), 600, 64, 300
    H, W, y = synth.make_head(T, d, V, "bf16", 3, dev)
    S, prm = len(cu) - 1, B.Params()
    active = np.zeros(T, bool)
    for a, b in zip(cu, cu[1:]):
        active[a:b] = True
    z = torch.zeros(T, device=dev)
    ws = torch.full((B.pg_workspace_bytes(T, d, V, S, prm, B.CALL_LOSS_FWD_BWD),), 0xFF, dtype=torch.uint8, device=dev)
    out = B.pg_loss_fwd_bwd(H, W, y, torch.ones(T, dtype=torch.uint8, device=dev), torch.tensor(cu, dtype=torch.int32, device=dev),
                            torch.ones(S, dtype=torch.float64, device=dev), torch.arange(S, dtype=torch.int32, device=dev), z, z, prm, ws)
    assert out["counters"][0].item() == out["counters"][6].item() == active.sum()
    assert ((out["logp"].cpu().numpy() != 0) == active).all()
