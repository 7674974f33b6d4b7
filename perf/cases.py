"""Workloads that the speed of this library is judged by: calls of its public entry points over the range that
a trainer of a multi-turn RL policy makes them.

Kinds of case (key "kind"):
  advantages   the rollout batch's small stages in a row: rewards, rejection sampling, TRLOO advantages
  logprob      old-policy recompute: log-prob, entropy and logsumexp of every row, no gradient
  loss         one packed microbatch: mismatch correction, clipped surrogate, backward to dH and dW
               ("normed": with the RMS normalisation fused around the head)
  sft          token-mean cross-entropy of the same head, forward and backward
  shard        one device's share of the head when its vocabulary rows are split: forward, merge, backward
  rmsnorm      the normalisation in front of the head and its backward, as separate calls
  monitors     the step's training-dynamics monitors

Hidden states and weights are drawn as in the repository's synthetic workloads: rows of unit RMS, W ~ N(0, 0.02),
uniform token ids, one third of the packed rows masked context, responses of 256 to 1024 tokens.
"""
import math

import numpy as np
import torch

from paper_2602_05885_amd import binding as B

DEV = "cuda:0"
W_STD = 0.02
V_FULL = 151936          # vocabulary of the 8B and 14B heads that the benchmark names
GEO_SHIFT = 0.05         # mean log-ratio of a sample that the geometric window rejects


def _loss(name, d, V, rows, **kw):
    c = {"kind": "loss", "d": d, "V": V, "rows": rows, "ctx": 1 / 3, "len_lo": 256, "len_hi": 1024, "mode": 2, "kept": 1.0,
         "f32": False, "tau": 1.0, "dW_bf16": False, "accumulate": False, "normed": False}
    c.update(kw)
    return dict(c, name=name) if name else c


def listed():
    return [
        # once per rollout batch, before any gradient: 384 samples, launch latency is all there is
        {"name": "advantages 16x8x3", "kind": "advantages", "P": 16, "K": 8, "Tmax": 3},
        # the smallest configuration of the benchmark: fp32 head, used to check a trainer's numerics
        _loss("loss f32 h64", 64, 1000, 1024, f32=True, ctx=0.0, len_lo=32, len_hi=32),
        # old-policy recompute of a single short sample (one turn of one rollout) at the 8B head
        {"name": "logprob 8B one sample", "kind": "logprob", "d": 4096, "V": V_FULL, "rows": 677, "tau": 1.0},
        # a microbatch of one sample at the 14B head, as a trainer with long contexts runs it
        _loss("loss 14B one sample", 5120, V_FULL, 1013),
        # cold-start fine-tuning at the 8B head: gradients accumulate over microbatches, W^T is kept between them
        {"name": "sft 8B accumulate", "kind": "sft", "d": 4096, "V": V_FULL, "rows": 4099, "loss_share": 0.7, "tau": 1.0,
         "accumulate": True, "wt_cache": True},
        # normalisation fused around the head, on-policy update (first gradient step on a rollout batch), bf16 dW
        _loss("loss 8B normed", 4096, V_FULL, 6151, normed=True, mode=0, dW_bf16=True),
        # the paper's geometric rejection on a 16k-row microbatch of the 8B head; a quarter of the samples survive
        _loss("loss 8B geometric", 4096, V_FULL, 16082, mode=1, kept=0.25),
        # the benchmark's headline: 14B head, 32k loss tokens, truncated importance weights
        _loss("loss 14B 32k tokens", 5120, V_FULL, 43697, ctx=0.25),
        # one of eight vocabulary shards of the 14B head on a 16k-row microbatch
        {"name": "shard 14B 1/8", "kind": "shard", "d": 5120, "V": V_FULL, "shards": 8, "shard": 3, "rows": 16411, "ctx": 1 / 3},
        # old-policy recompute of a whole rollout batch at the 14B head, sampling temperature 0.7
        {"name": "logprob 14B 128k rows", "kind": "logprob", "d": 5120, "V": V_FULL, "rows": 131072, "tau": 0.7},
        # the normalisation as separate calls over the headline microbatch
        {"name": "rmsnorm 14B", "kind": "rmsnorm", "d": 5120, "rows": 43697, "f32": False},
        # monitors of a 14B step: every gradient is read once
        {"name": "monitors 14B", "kind": "monitors", "d": 5120, "V": V_FULL, "rows": 43697},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["advantages", "logprob", "logprob", "loss", "loss", "loss", "loss", "sft", "shard", "rmsnorm", "monitors"])
    if kind == "advantages":
        return {"kind": kind, "P": rng.randint(1, 64), "K": rng.randint(2, 100), "Tmax": rng.randint(1, 6)}
    if kind == "rmsnorm":
        return {"kind": kind, "d": 64 * rng.randint(8, 112), "rows": _log_int(rng, 100, 40000), "f32": rng.random() < 0.25}
    if kind == "monitors":
        return {"kind": kind, "d": 64 * rng.randint(16, 80), "V": _log_int(rng, 20000, V_FULL), "rows": _log_int(rng, 200, 40000)}
    # heads: the two of the benchmark, or a generic one with a ragged vocabulary
    d, V = rng.choice([(4096, V_FULL), (5120, V_FULL), (64 * rng.randint(16, 80), _log_int(rng, 20000, V_FULL))])
    if kind == "logprob":
        return {"kind": kind, "d": d, "V": V, "rows": _log_int(rng, 100, 100000), "tau": rng.choice([1.0, 1.0, 0.7, 0.9])}
    if kind == "sft":
        return {"kind": kind, "d": d, "V": V, "rows": _log_int(rng, 200, 40000), "loss_share": round(rng.uniform(0.4, 1.0), 3), "tau": 1.0,
                "accumulate": rng.random() < 0.5, "wt_cache": rng.random() < 0.5}
    if kind == "shard":
        g = rng.choice([2, 4, 8])
        return {"kind": kind, "d": d, "V": V, "shards": g, "shard": rng.randrange(g), "rows": _log_int(rng, 500, 40000), "ctx": round(rng.uniform(0.1, 0.5), 3)}
    if rng.random() < 0.2:      # fp32 heads serve checks: small ones
        return _loss(None, 64 * rng.randint(1, 16), _log_int(rng, 1000, 32000), _log_int(rng, 200, 8000), f32=True, ctx=round(rng.uniform(0.0, 0.5), 3),
                     len_lo=32, len_hi=256, mode=rng.choice([0, 2]))
    mode = rng.choice([0, 1, 2, 2])
    return _loss(None, d, V, _log_int(rng, 200, 40000), mode=mode, kept=round(rng.uniform(0.05, 0.6), 3) if mode == 1 else 1.0, ctx=round(rng.uniform(0.1, 0.6), 3),
                 tau=rng.choice([1.0, 1.0, 0.8]), dW_bf16=rng.random() < 0.25, accumulate=rng.random() < 0.25, normed=rng.random() < 0.25)


# ---------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _rows(T, d, dtype, g, unit=True):
    out = torch.empty((T, d), dtype=dtype, device=DEV)
    step = max(1, (1 << 27) // d)
    for a in range(0, T, step):
        h = torch.randn((min(step, T - a), d), generator=g, device=DEV)
        if unit:
            h *= torch.rsqrt((h * h).mean(dim=1, keepdim=True))
        out[a:a + h.shape[0]] = h
    return out


def _head(c, V, seed):
    """H, W, y of a head with V rows (or a shard of it: y still ranges over c["V"])."""
    g = _gen(seed)
    dt = torch.float32 if c.get("f32") else torch.bfloat16
    H = _rows(c["rows"], c["d"], dt, g)
    W = torch.empty((V, c["d"]), dtype=dt, device=DEV)
    step = max(1, (1 << 27) // c["d"])
    for a in range(0, V, step):
        W[a:a + step] = torch.randn((min(step, V - a), c["d"]), generator=g, device=DEV) * W_STD
    y = torch.randint(0, c["V"], (c["rows"],), generator=g, device=DEV, dtype=torch.int32)
    return H, W, y, g


def _packing(c, seed):
    """Segments (context prefix + response) that fill exactly c["rows"] rows: cu_seqlens, loss_mask."""
    rng = np.random.Generator(np.random.Philox(key=seed))
    lo, hi, T = c.get("len_lo", 256), c.get("len_hi", 1024), c["rows"]
    cu, mask = [0], np.zeros(T, np.uint8)
    while cu[-1] < T:
        resp = int(rng.integers(lo, hi + 1))
        n_ctx = int(round(resp * c["ctx"] / (1 - c["ctx"])))
        a, b = cu[-1], min(T, cu[-1] + n_ctx + resp)
        if T - b < lo // 2:      # no stub at the end
            b = T
        mask[min(a + n_ctx, b - 1):b] = 1
        cu.append(b)
    return np.asarray(cu, np.int32), mask


def _old_logp(c, H, W, y, g, v_rows=None):
    """Log-probs of the policy that the update starts from: those of this head but for a small drift (the logits of a
    row are normal with variance |h|^2 W_STD^2, which gives the logsumexp closely), with 3 % of the tokens moved
    far enough to be clipped."""
    T, tau = c["rows"], c.get("tau", 1.0)
    hf = H.float()
    var = (hf * hf).sum(dim=1) * (W_STD / tau) ** 2
    zy = (hf * W[y.long()].float()).sum(dim=1) / tau if v_rows is None else v_rows
    u = torch.rand((T, 2), generator=g, device=DEV)
    drift = (u[:, 0] - 0.5) * 0.2 + torch.where(u[:, 1] < 0.03, torch.where(u[:, 0] < 0.5, -0.4, 0.4), 0.0)
    return (zy - math.log(c["V"]) - var / 2 + drift).float()


def _rollout_logp(c, old, cu, mask, g, seed):
    """What the rollout engine reported: noise N(0, 0.1), 1 % outliers of +-3 (mode 2); under the geometric rule (mode 1)
    the noise of the share `kept` of the samples averages to nothing and that of the others to GEO_SHIFT."""
    T = c["rows"]
    delta = 0.1 * torch.randn(T, generator=g, device=DEV, dtype=torch.float64)
    if c["mode"] == 2:
        u = torch.rand((T, 2), generator=g, device=DEV)
        delta += torch.where(u[:, 0] < 0.01, torch.where(u[:, 1] < 0.5, -3.0, 3.0), 0.0)
    else:
        S = len(cu) - 1
        seg = torch.from_numpy(np.repeat(np.arange(S), np.diff(cu))).to(DEV)
        m = torch.from_numpy(mask).to(DEV).double()
        n = torch.zeros(S, dtype=torch.float64, device=DEV).index_add_(0, seg, m)
        mean = torch.zeros(S, dtype=torch.float64, device=DEV).index_add_(0, seg, m * delta) / n.clamp(min=1)
        shift = torch.full((S,), GEO_SHIFT, dtype=torch.float64, device=DEV)
        kept = np.random.Generator(np.random.Philox(key=seed + 1)).permutation(S)[:max(1, int(round(c["kept"] * S)))]
        shift[torch.from_numpy(kept).to(DEV)] = 0.0
        delta += (shift - mean)[seg]
    return (old.double() - delta).float()


def _advantages(S, seed):
    """fp64 advantage table of a rollout batch of which the microbatch packs S samples, and the sample of each segment."""
    rng = np.random.Generator(np.random.Philox(key=seed + 2))
    n = max(384, 2 * S)
    R = np.where(rng.random((n // 8, 8)) < 0.5, 1 + np.minimum(rng.lognormal(0.0, 0.5, (n // 8, 8)), 3.0), 0.0)
    A = (R - (R.sum(1, keepdims=True) - R) / 7).reshape(-1)
    return torch.from_numpy(A).to(DEV), torch.from_numpy(np.sort(rng.permutation(A.size)[:S]).astype(np.int32)).to(DEV)


def _out(T, d, dtype):
    return (torch.empty(1, device=DEV), torch.empty((T, d), dtype=dtype, device=DEV), torch.empty(T, device=DEV), torch.empty(T, device=DEV),
            torch.empty(8, dtype=torch.int64, device=DEV))


def _params(c, **kw):
    return B.Params(dtype=int(bool(c.get("f32"))), temperature=c.get("tau", 1.0), mismatch_mode=c.get("mode", 0), dW_dtype=int(bool(c.get("dW_bf16"))),
                    accumulate_dW=int(bool(c.get("accumulate"))), **kw)


def _dW(c, V, g):
    dt = torch.bfloat16 if c.get("dW_bf16") else torch.float32
    if not c.get("accumulate"):
        return torch.empty((V, c["d"]), dtype=dt, device=DEV)
    dW = torch.empty((V, c["d"]), dtype=dt, device=DEV)         # the gradient of the microbatches before this one
    step = max(1, (1 << 27) // c["d"])
    for a in range(0, V, step):
        dW[a:a + step] = torch.randn((min(step, V - a), c["d"]), generator=g, device=DEV) * (0.5 / math.sqrt(c["rows"] * V))
    return dW


def _shard_range(c):
    n = -(-c["V"] // c["shards"])
    return min(c["shard"] * n, c["V"] - 1), min((c["shard"] + 1) * n, c["V"])


def _loss_inputs(c, seed):
    a, b = _shard_range(c) if c["kind"] == "shard" else (0, c["V"])
    H, W, y, g = _head(c, b - a, seed)
    s = {"kind": c["kind"], "H": H, "W": W, "y": y, "v0": a}
    cu, mask = _packing(c, seed)
    s["cu"], s["mask"] = torch.from_numpy(cu).to(DEV), torch.from_numpy(mask).to(DEV)
    s["adv"], s["seg"] = _advantages(len(cu) - 1, seed)
    s["S"] = len(cu) - 1
    mode = c.get("mode", 2)
    if c["kind"] == "shard":
        # the states that the other shards' devices send: those of logits of this spread
        sd = W_STD * math.sqrt(c["d"])
        n, m = c["V"] - (b - a), torch.full((c["rows"],), 4.5 * sd, device=DEV)
        e = n * torch.exp(sd * sd / 2 - m) * (1 + 0.005 * torch.randn(c["rows"], generator=g, device=DEV))
        mine = (y >= a) & (y < b)
        zo = torch.where(mine, 0.0, sd * torch.randn(c["rows"], generator=g, device=DEV))
        s["others"] = torch.stack([m, e, e * (sd * sd - m), zo], dim=1).contiguous()
        zy = torch.where(mine, (H.float() * W[(y - a).clamp(0, b - a - 1).long()].float()).sum(dim=1), zo)
        s["old"] = _old_logp(c, H, W, y, g, zy)
        s["rollout"] = _rollout_logp(dict(c, mode=2), s["old"], cu, mask, g, seed)
    elif c.get("normed"):
        H *= (0.5 + torch.rand((c["rows"], 1), generator=g, device=DEV)).to(H.dtype)
        s["gamma"] = (1 + 0.1 * torch.randn(c["d"], generator=g, device=DEV)).to(H.dtype)
        s["eps"] = 1e-6
        if mode:
            hn = (H.float() * torch.rsqrt((H.float() ** 2).mean(dim=1, keepdim=True) + s["eps"]) * s["gamma"].float()).to(H.dtype)
            s["old"] = _old_logp(c, hn, W, y, g)
            s["rollout"] = _rollout_logp(c, s["old"], cu, mask, g, seed)
    elif mode:
        s["old"] = _old_logp(c, H, W, y, g)
        s["rollout"] = _rollout_logp(c, s["old"], cu, mask, g, seed)
    s.setdefault("old", None)
    s.setdefault("rollout", None)
    s["g"] = g
    return s


def _advantage_inputs(c, seed):
    g = torch.Generator().manual_seed(seed)
    n = c["P"] * c["K"] * c["Tmax"]
    stop = (torch.rand(c["P"], c["K"], c["Tmax"], generator=g) < 0.15).int()      # a rollout ends after such a turn
    valid = (torch.cumsum(stop, dim=2) - stop == 0).to(torch.uint8)
    s = {"kind": c["kind"], "shape": (c["P"], c["K"], c["Tmax"]), "valid": valid.to(DEV), "vflat": valid.reshape(-1).to(DEV),
         "correct": (torch.rand(n, generator=g) < 0.5).to(torch.uint8).mul(valid.reshape(-1)).to(DEV), "seed": seed}
    ref = torch.rand(n, generator=g) + 0.5
    s["t_ref"], s["t_ker"] = ref.to(DEV), (ref / torch.exp(0.5 * torch.randn(n, generator=g))).to(DEV)
    tot = torch.rand(n, generator=g) + 0.5
    s["t_tot"], s["t_gen"] = tot.to(DEV), (tot * torch.rand(n, generator=g)).to(DEV)
    return s


def prepare(case, seed):
    c, k = case, case["kind"]
    if k == "advantages":
        return _advantage_inputs(c, seed)
    if k == "rmsnorm":
        g = _gen(seed)
        dt = torch.float32 if c["f32"] else torch.bfloat16
        s = {"kind": k, "X": _rows(c["rows"], c["d"], dt, g, False), "dH": _rows(c["rows"], c["d"], dt, g, False) * 0.01}
        s["gamma"] = (1 + 0.1 * torch.randn(c["d"], generator=g, device=DEV)).to(dt)
        s["h"], s["dX"] = torch.empty_like(s["X"]), torch.empty_like(s["X"])
        return s
    if k == "monitors":
        g = _gen(seed)
        T = c["rows"]
        dW = torch.empty((c["V"], c["d"]), device=DEV).normal_(0, 1e-6, generator=g)
        return {"kind": k, "logp": -11 - torch.randn(T, generator=g, device=DEV), "rollout": -11 - torch.randn(T, generator=g, device=DEV),
                "entropy": 10 + torch.rand(T, generator=g, device=DEV), "mask": (torch.rand(T, generator=g, device=DEV) < 0.75).to(torch.uint8),
                "dH": (_rows(T, c["d"], torch.float32, g, False) * 1e-5).to(torch.bfloat16), "dW": dW}
    if k == "logprob":
        H, W, y, _ = _head(c, c["V"], seed)
        p = _params(c)
        return {"kind": k, "H": H, "W": W, "y": y, "p": p, "ws": B.alloc_workspace(c["rows"], c["d"], c["V"], 0, p, B.CALL_LOGPROB_FWD, DEV),
                "out": tuple(torch.empty(c["rows"], device=DEV) for _ in range(3))}
    if k == "sft":
        H, W, y, g = _head(c, c["V"], seed)
        s = {"kind": k, "H": H, "W": W, "y": y, "mask": (torch.rand(c["rows"], generator=g, device=DEV) < c["loss_share"]).to(torch.uint8), "dW": _dW(c, c["V"], g)}
        s["p"] = _params(c)
        s["ws"] = B.alloc_workspace(c["rows"], c["d"], c["V"], 0, s["p"], B.CALL_LOSS_FWD_BWD, DEV)
        s["out"] = _out(c["rows"], c["d"], H.dtype)
        if c["wt_cache"]:        # filled by the first microbatch of the optimizer step, valid until W changes
            wt = B.alloc_w_transposed(c["d"], c["V"], DEV)
            first = B.Params(dtype=s["p"].dtype, w_transposed=wt)
            B.pg_sft_fwd_bwd(H, W, y, s["mask"], first, s["ws"], dW=torch.empty_like(s["dW"]), out=s["out"])
            s["p"].w_transposed, s["p"].w_transposed_valid = wt, 1
        return s
    s = _loss_inputs(c, seed)
    V, d = s["W"].shape
    s["dW"] = _dW(c, V, s.pop("g"))
    s["p"] = _params(dict(c, mode=2) if k == "shard" else c)
    which = B.CALL_LOSS_FWD_BWD_NORMED if c.get("normed") else B.CALL_LOSS_FWD_BWD
    s["ws"] = B.alloc_workspace(c["rows"], d, V, s["S"], s["p"], which, DEV)
    s["out"] = _out(c["rows"], d, torch.float32 if k == "shard" else s["H"].dtype)
    if k == "shard":
        s["ws_fwd"] = B.alloc_workspace(c["rows"], d, V, 0, s["p"], B.CALL_LOGPROB_FWD, DEV)
        s["parts"] = torch.empty((c["rows"], 4), device=DEV)
        s["merged"] = torch.empty((c["rows"], 4), device=DEV)
    return s


def run(s):
    k = s["kind"]
    if k == "advantages":
        R, pr = B.turn_reward(s["correct"], s["t_ref"], s["t_ker"], s["t_gen"], s["t_tot"])
        keep, _ = B.prs_retain(pr, s["vflat"], s["seed"])
        adv, ret, n = B.trloo_advantage(R.view(s["shape"]), s["valid"], 1.0)
        return {"rewards": R, "keep": keep, "adv": adv, "returns": ret, "n": n}
    if k == "rmsnorm":
        h, rstd = B.pg_rmsnorm_fwd(s["X"], s["gamma"], 1e-6, out=s["h"])
        dX, dgamma = B.pg_rmsnorm_bwd(s["X"], s["gamma"], s["dH"], 1e-6, out=s["dX"])
        return {"h": h, "rstd": rstd, "dX": dX, "dgamma": dgamma}
    if k == "monitors":
        return B.pg_monitors(s["logp"], s["rollout"], s["entropy"], s["mask"], s["dH"], s["dW"])
    if k == "logprob":
        logp, ent, lse = B.pg_logprob_fwd(s["H"], s["W"], s["y"], None, s["p"], s["ws"], out=s["out"])
        return {"logp": logp, "entropy": ent, "lse": lse}
    if k == "sft":
        return B.pg_sft_fwd_bwd(s["H"], s["W"], s["y"], s["mask"], s["p"], s["ws"], dW=s["dW"], out=s["out"])
    if k == "shard":
        B.pg_head_shard_fwd(s["H"], s["W"], s["y"], s["mask"], s["v0"], s["p"], s["ws_fwd"], out=s["parts"])
        B.pg_head_partials_merge(s["parts"], s["others"], out=s["merged"])
        r = B.pg_loss_shard_bwd(s["H"], s["W"], s["y"], s["mask"], s["cu"], s["adv"], s["seg"], s["old"], s["rollout"], s["merged"], s["v0"], s["p"], s["ws"],
                                dH_f32=True, dW=s["dW"], out=s["out"])
        return dict(r, states=s["merged"])
    if "gamma" in s:
        return B.pg_loss_fwd_bwd_normed(s["H"], s["gamma"], s["eps"], s["W"], s["y"], s["mask"], s["cu"], s["adv"], s["seg"], s["old"], s["rollout"], s["p"], s["ws"],
                                        dW=s["dW"], out=s["out"])
    return B.pg_loss_fwd_bwd(s["H"], s["W"], s["y"], s["mask"], s["cu"], s["adv"], s["seg"], s["old"], s["rollout"], s["p"], s["ws"], dW=s["dW"], out=s["out"])


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    c, k = case, case["kind"]
    if k == "advantages":
        n = c["P"] * c["K"] * c["Tmax"]
        return {"bytes": n * (1 + 16 + 4 + 1 + 1 + 16) + 4 * c["P"] * c["Tmax"], "flops": 20 * n}
    T, d = c["rows"], c["d"]
    e = 4 if c.get("f32") else 2
    if k == "rmsnorm":
        return {"bytes": 5 * T * d * e + 4 * T + 4 * d, "flops": 12 * T * d}
    if k == "monitors":
        return {"bytes": 4 * c["V"] * d + 2 * T * d + 13 * T, "flops": 2 * (c["V"] + T) * d}
    V = _shard_range(c)[1] - _shard_range(c)[0] if k == "shard" else c["V"]
    if k == "logprob":
        return {"bytes": 2 * (T + V) * d + 16 * T, "flops": 2 * T * d * V}
    active = T * c["loss_share"] if k == "sft" else T * (1 - c["ctx"]) * c.get("kept", 1.0)
    dw = (2 if c.get("dW_bf16") else 4) * (2 if c.get("accumulate") else 1)
    return {"bytes": int(V * d * (e + dw) + active * d * e + T * d * (4 if k == "shard" else e) + 32 * T), "flops": int(6 * active * d * V)}


def tolerance(case):
    k = case["kind"]
    # (in brackets: the largest relative error against exact() that the library showed over the listed cases and draws)
    if k == "advantages":
        return {"rel": 1e-7, "max": 1e-6, "differ": 0.0}      # rewards are rounded to float32 (2.5e-8), the sums are fp64
    if k == "monitors":
        return {"rel": 1e-12, "max": 1e-11}                   # fp64 sums in another order
    if k == "logprob":
        return {"rel": 1e-6, "max": 2e-5}                     # fp32 sums over d and V of exact bf16 products (8e-8)
    if k == "rmsnorm":
        return {"rel": 1e-6, "max": 1e-4} if case["f32"] else {"rel": 7e-3, "max": 3e-2}   # one rounding to bf16 (1.7e-3)
    if case.get("f32"):
        return {"rel": 3e-5, "max": 2e-3}                     # operands of about 16 mantissa bits (4.4e-6)
    return {"rel": 1.2e-2, "max": 0.2}                        # dS and dH are rounded to bf16 (3.2e-3)


# ---------------------------------------------------------------- the same in 64 bits, by plain torch
def _softmax_rows(h, W, y, v0, tau, state=None):
    """fp64 logits of a block of rows, its logsumexp, entropy and log-prob (over all shards where `state` gives the others')."""
    z = (h @ W.t()) / tau
    mine = (y >= v0) & (y < v0 + W.shape[0])
    zy = torch.where(mine, z.gather(1, (y - v0).clamp(0, W.shape[0] - 1)[:, None])[:, 0], 0.0)
    m = z.max(dim=1).values
    p = torch.exp(z - m[:, None])
    s = p.sum(dim=1)
    u = (p * (z - m[:, None])).sum(dim=1)
    del p
    if state is not None:
        mo, so, uo, zo = state.unbind(1)
        mm = torch.maximum(m, mo)
        a, b = torch.exp(m - mm), torch.exp(mo - mm)
        m, s, u, zy = mm, a * s + b * so, a * (u + (m - mm) * s) + b * (uo + (mo - mm) * so), zy + zo
    lse = m + torch.log(s)
    return z, mine, lse, zy - lse, torch.log(s) - u / s, torch.stack([m, s, u, zy], dim=1)


def _exact_head(c, s):
    """loss, dH (dX), dW, logp, entropy and counters of the loss calls."""
    T, d = s["H"].shape
    V, tau = s["W"].shape[0], c.get("tau", 1.0)
    sft = c["kind"] == "sft"
    mode = 0 if sft else 2 if c["kind"] == "shard" else c["mode"]
    mask = s["mask"].bool()
    cnt = [0] * 8
    act, w = mask.clone(), torch.ones(T, dtype=torch.float64, device=DEV)
    cnt[6] = int(mask.sum())
    if not sft:
        seg = torch.repeat_interleave(torch.arange(s["S"], device=DEV), (s["cu"][1:] - s["cu"][:-1]).long())
        A = s["adv"][s["seg"].long()].float().double()[seg]
        if mode:
            delta = s["old"].double() - s["rollout"].double()
            low = torch.full((s["S"],), 1e300, dtype=torch.float64, device=DEV).scatter_reduce(0, seg[mask], delta[mask], "amin")
            veto = torch.exp(low) < np.float64(np.float32(1e-4))
            rejected = veto.clone()
            cnt[4] = int(veto.sum())
            if mode == 1:
                n = torch.zeros(s["S"], dtype=torch.float64, device=DEV).index_add_(0, seg, mask.double())
                mean = torch.zeros(s["S"], dtype=torch.float64, device=DEV).index_add_(0, seg, torch.where(mask, delta, 0.0)) / n
                out = ~((torch.exp(mean) >= np.float64(np.float32(0.999))) & (torch.exp(mean) <= np.float64(np.float32(1.001)))) & (n > 0)
                cnt[3] = int(out.sum())
                rejected |= out
            act &= ~rejected[seg]
            if mode == 2:
                ratio = torch.exp(delta)
                cnt[5] = int(((ratio > 2.0) & act).sum())
                w = ratio.clamp(max=2.0)
    rows = act.nonzero()[:, 0]
    n = rows.numel()
    cnt[0] = n
    norm = float(max(n, 1))
    W = s["W"].double()
    x = s["H"][rows].double()
    if "gamma" in s:
        rstd = torch.rsqrt((x * x).mean(dim=1, keepdim=True) + s["eps"])
        gam = s["gamma"].double()
        h = x * rstd * gam
    else:
        h = x
    # the call adds to the gradient that was there (an accumulating case has run once when its first outputs are read)
    dW = s["dW0"].double() if s.get("dW0") is not None else torch.zeros((V, d), dtype=torch.float64, device=DEV)
    dHr = torch.empty_like(h)
    logp, ent = torch.zeros(T, dtype=torch.float64, device=DEV), torch.zeros(T, dtype=torch.float64, device=DEV)
    loss = torch.zeros((), dtype=torch.float64, device=DEV)
    step = max(64, (1 << 29) // V)
    for a in range(0, n, step):
        r, hb = rows[a:a + step], h[a:a + step]
        yb = s["y"][r].long()
        z, mine, lse, lp, en, _ = _softmax_rows(hb, W, yb, s.get("v0", 0), tau, s["others"][r].double() if "others" in s else None)
        logp[r], ent[r] = lp, en
        if sft:
            l, g, wb = -lp, -torch.ones_like(lp), torch.ones_like(lp)
        else:
            Ab, wb = A[r], w[r]
            q = torch.exp(lp - s["old"][r].double()) if s["old"] is not None else torch.ones_like(lp)
            lo, hi = np.float64(np.float32(1) - np.float32(0.2)), np.float64(np.float32(1) + np.float32(0.2))
            l = -torch.minimum(q * Ab, q.clamp(lo, hi) * Ab)
            up, down = (Ab >= 0) & (q > hi), (Ab < 0) & (q < lo)
            cnt[1] += int(up.sum())
            cnt[2] += int(down.sum())
            g = torch.where(up | down, 0.0, -Ab * q)
        loss += (wb * l).sum() / norm
        coef = wb * g / norm / tau
        z.sub_(lse[:, None]).exp_().mul_(-coef[:, None])
        z.scatter_add_(1, (yb - s.get("v0", 0)).clamp(0, V - 1)[:, None], torch.where(mine, coef, 0.0)[:, None])
        dHr[a:a + step] = z @ W
        dW.addmm_(z.t(), hb)
        del z
    out = {"loss": loss.reshape(1), "dW": dW, "logp": logp, "entropy": ent, "counters": torch.tensor(cnt, device=DEV)}
    if "gamma" in s:
        xh = x * rstd
        gg = dHr * gam
        out["dgamma"] = (dHr * xh).sum(dim=0)
        dHr = rstd * (gg - xh * (gg * xh).mean(dim=1, keepdim=True))
    dH = torch.zeros((T, d), dtype=torch.float64, device=DEV)
    dH[rows] = dHr
    out["dX" if "gamma" in s else "dH"] = dH
    return out


def exact(case, seed):
    c, k = case, case["kind"]
    if k == "advantages":
        s = _advantage_inputs(c, seed)
        ok = s["correct"].bool()
        R = torch.where(ok, 1 + (s["t_ref"].double() / s["t_ker"].double()).clamp(max=3.0) + s["t_gen"].double() / s["t_tot"].double(), 0.0)
        v = s["valid"].double()
        G = R.float().double().view(s["shape"]).flip(2).cumsum(2).flip(2)
        n = v.sum(dim=1, keepdim=True)
        A = torch.where((v > 0) & (n > 1), G - ((v * G).sum(dim=1, keepdim=True) - G) / (n - 1).clamp(min=1), 0.0)
        return {"rewards": R, "keep": None, "adv": A, "returns": G, "n": n[:, 0].int()}
    if k == "rmsnorm":
        s = prepare(c, seed)
        X, g, gam = s["X"].double(), s["dH"].double(), s["gamma"].double()
        rstd = torch.rsqrt((X * X).mean(dim=1, keepdim=True) + float(np.float32(1e-6)))
        xh = X * rstd
        gg = g * gam
        return {"h": xh * gam, "rstd": rstd[:, 0], "dX": rstd * (gg - xh * (gg * xh).mean(dim=1, keepdim=True)), "dgamma": (g * xh).sum(dim=0)}
    if k == "monitors":
        s = prepare(c, seed)
        m = s["mask"].bool()
        n = m.sum().double()
        out = torch.zeros(8, dtype=torch.float64, device=DEV)
        out[0] = s["entropy"].double()[m].sum() / n
        out[1], out[2] = torch.exp(-s["logp"].double()[m].sum() / n), torch.exp(-s["rollout"].double()[m].sum() / n)
        out[3], out[4], out[5] = s["dH"].double().square().sum().sqrt(), sum(x.double().square().sum() for x in s["dW"].split(8192)).sqrt(), n
        return out
    if k == "logprob":
        H, W, y, _ = _head(c, c["V"], seed)
        W, T = W.double(), c["rows"]
        out = torch.empty((3, T), dtype=torch.float64, device=DEV)
        step = max(64, (1 << 29) // c["V"])
        for a in range(0, T, step):
            _, _, lse, lp, en, _ = _softmax_rows(H[a:a + step].double(), W, y[a:a + step].long(), 0, c["tau"])
            out[0, a:a + step], out[1, a:a + step], out[2, a:a + step] = lp, en, lse
        return {"logp": out[0], "entropy": out[1], "lse": out[2]}
    if k == "sft":
        H, W, y, g = _head(c, c["V"], seed)
        s = {"H": H, "W": W, "y": y, "mask": (torch.rand(c["rows"], generator=g, device=DEV) < c["loss_share"]).to(torch.uint8)}
        s["dW0"] = _dW(c, c["V"], g) if c["accumulate"] else None
        return _exact_head(c, s)
    s = _loss_inputs(c, seed)
    s["dW0"] = _dW(c, s["W"].shape[0], s["g"]) if c.get("accumulate") else None
    out = _exact_head(c, s)
    if k == "shard":
        T = c["rows"]
        W = s["W"].double()
        st = s["others"].double().clone()
        rows = s["mask"].bool().nonzero()[:, 0]
        for r in rows.split(max(64, (1 << 29) // W.shape[0])):
            st[r] = _softmax_rows(s["H"][r].double(), W, s["y"][r].long(), s["v0"], 1.0, s["others"][r].double())[5]
        out["states"] = st
    return out
