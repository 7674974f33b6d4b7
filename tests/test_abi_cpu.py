"""The C-ABI library loads, exports what the header declares, and validates arguments on the host.
No kernel is launched here (no GPU needed): every call below fails validation before any HIP call."""
import ctypes as C
import os
import re

import pytest

from paper_2602_05885_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_functions():
    src = open(os.path.join(ROOT, "include", "pg_head.h")).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(\w+)\s*\([^;{]*\)\s*;", src)))


def test_header_symbols_are_exported():
    names = _declared_functions()
    assert set(names) == set(B.EXPORTS), names
    lib = C.CDLL(B.LIB_PATH)
    for n in names:
        assert getattr(lib, n) is not None


def test_params_struct_layout_matches_header():
    src = open(os.path.join(ROOT, "include", "pg_head.h")).read()
    body = re.search(r"typedef struct pg_params \{(.*?)\} pg_params;", src, flags=re.S).group(1)
    body = re.sub(r"/\*.*?\*/", "", body, flags=re.S)
    fields = re.findall(r"(int32_t|float|void\*)\s+(\w+)\s*;", body)
    ctype = {"int32_t": C.c_int32, "float": C.c_float, "void*": C.c_void_p}
    assert [(n, ctype[t]) for t, n in fields] == list(B.PgParams._fields_)


def test_workspace_query_and_shape_errors():
    P = B.Params()
    small = B.pg_workspace_bytes(1024, 64, 1000, 32, P, B.CALL_LOSS_FWD_BWD)
    fwd = B.pg_workspace_bytes(1024, 64, 1000, 0, P, B.CALL_LOGPROB_FWD)
    assert 0 < fwd < small
    big = B.pg_workspace_bytes(43776, 5120, 151936, 60, P, B.CALL_LOSS_FWD_BWD)
    assert 2 << 30 < big < 16 << 30
    assert B.pg_workspace_bytes(1024, 100, 1000, 1, P, 1) == 0 and "multiple of 64" in B.pg_last_error()
    assert B.pg_workspace_bytes(-1, 64, 1000, 1, P, 1) == 0
    assert B.pg_workspace_bytes(1024, 64, 1000, 1, B.Params(temperature=0.0), 1) == 0
    assert B.pg_workspace_bytes(1024, 64, 1000, 1, B.Params(mismatch_mode=7), 1) == 0
    assert B.pg_workspace_bytes(1 << 20, 5120, 151936, 1, P, 0) > 8 << 30      # operands beyond 4 GiB are fine
    assert B.pg_workspace_bytes(2048, 5120, 151936, 0, B.Params(dtype=1), 1) > 4 << 30  # fp32 head: 4.7 GB split operand
    assert B.pg_workspace_bytes(1 << 23, 64, 1000, 1, P, 0) == 0 and "4 GiB" in B.pg_last_error()
    assert B.pg_workspace_bytes(8, 1 << 23, 1000, 0, P, 1) == 0 and "4 GiB" in B.pg_last_error()
    assert B.pg_workspace_bytes(1 << 22, 64, 1 << 26, 0, P, 0) == 0 and "logits tiles" in B.pg_last_error()
    assert B.pg_workspace_bytes(1024, 64, 1000, 1, P, 5) == 0
    assert B.pg_workspace_bytes(0, 64, 1000, 0, P, 1) > 0          # empty microbatch is legal


def test_w_transposed_cache_size_and_validation():
    lib = B.lib()
    n = int(lib.pg_w_transposed_bytes(5120, 151936))
    assert 5120 * 151936 * 2 <= n <= 5120 * (151936 + 512) * 2 + 256
    assert int(lib.pg_w_transposed_bytes(100, 1000)) == 0 and int(lib.pg_w_transposed_bytes(64, 0)) == 0
    one = C.c_void_p(16)
    p = B.Params().c_struct()
    p.w_transposed = 8                       # misaligned cache pointer
    rc = lib.pg_loss_fwd_bwd(one, one, one, one, one, 1, one, None, None, None, None, 8, 64, 100, C.byref(p), one, one, one,
                             None, None, None, one, 1 << 30, None)
    assert rc == -1 and "w_transposed" in B.pg_last_error()
    p = B.Params().c_struct()
    p.w_transposed_valid = 3
    assert lib.pg_workspace_bytes(8, 64, 100, 1, C.byref(p), 1) == 0


def test_invalid_arguments_return_error_codes():
    lib = B.lib()
    p = B.Params().c_struct()
    one = C.c_void_p(16)      # never dereferenced: validation fails first
    rc = lib.trloo_advantage(None, one, 1, 1, 1, 1.0, None, one, None, None)
    assert rc == -1 and "NULL" in B.pg_last_error()
    rc = lib.trloo_advantage(one, one, 0, 1, 1, 1.0, None, one, None, None)
    assert rc == -1
    rc = lib.pg_logprob_fwd(None, one, one, None, 8, 64, 100, C.byref(p), one, None, None, one, 1 << 30, None)
    assert rc == -1
    rc = lib.pg_logprob_fwd(one, one, one, None, 8, 64, 100, C.byref(p), one, None, None, one, 16, None)
    assert rc == -3 and "needed" in B.pg_last_error()
    rc = lib.pg_logprob_fwd(C.c_void_p(8), one, one, None, 8, 64, 100, C.byref(p), one, None, None, one, 1 << 30, None)
    assert rc == -1 and "aligned" in B.pg_last_error()
    rc = lib.pg_logprob_fwd(one, one, one, None, 8, 72, 100, C.byref(p), one, None, None, one, 1 << 30, None)
    assert rc == -2
    pm = B.Params(mismatch_mode=1).c_struct()
    rc = lib.pg_loss_fwd_bwd(one, one, one, one, one, 1, one, None, None, one, None, 8, 64, 100, C.byref(pm), one, one, one,
                             None, None, None, one, 1 << 30, None)
    assert rc == -1 and "rollout_logp" in B.pg_last_error()
    rc = lib.pg_loss_fwd_bwd(one, one, one, one, one, 0, one, None, None, None, None, 8, 64, 100, C.byref(p), one, one, one,
                             None, None, None, one, 1 << 30, None)
    assert rc == -1
    rc = lib.pg_loss_fwd_bwd(one, one, one, one, one, 1, one, None, None, None, None, 8, 64, 100, None, one, one, one,
                             None, None, None, one, 1 << 30, None)
    assert rc == -1 and "params" in B.pg_last_error()


def test_stage_entry_points_validate_arguments():
    lib = B.lib()
    one = C.c_void_p(16)      # never dereferenced: validation fails first
    assert lib.grpo_advantage(None, one, 1, 1, 1, 1.0, None, one, None, None) == -1
    assert lib.turn_reward(None, one, one, None, None, 4, 3.0, one, None, None) == -1
    assert lib.turn_reward(one, one, one, one, None, 4, 3.0, one, None, None) == -1 and "together" in B.pg_last_error()
    assert lib.turn_reward(one, one, one, None, None, 4, 0.0, one, None, None) == -1
    assert lib.turn_reward(one, one, one, None, None, -1, 3.0, one, None, None) == -1
    assert lib.turn_reward(None, None, None, None, None, 0, 3.0, None, None, None) == 0      # nothing to do
    assert lib.prs_retain(None, None, 4, 0.3, 0.1, 0, 1, one, None, None) == -1
    assert lib.prs_retain(one, None, 4, 0.3, 0.0, 0, 1, one, None, None) == -1 and "> 0" in B.pg_last_error()
    assert lib.prs_retain(None, None, 0, 0.3, 0.1, 0, 1, None, None, None) == 0
    ws = int(lib.pg_monitors_workspace_bytes())
    assert ws > 0
    assert lib.pg_monitors(one, None, None, one, 4, None, 0, 0, None, 0, 0, None, one, ws, None) == -1
    assert lib.pg_monitors(one, None, None, one, 4, None, 0, 0, None, 0, 0, one, one, ws - 1, None) == -3
    assert lib.pg_monitors(one, None, None, one, 4, one, 5, 8, None, 0, 0, one, one, ws, None) == -1
    p = B.Params().c_struct()
    rc = lib.pg_sft_fwd_bwd(one, one, one, None, 8, 64, 100, C.byref(p), one, one, one, None, None, None, one, 1 << 30, None)
    assert rc == -1 and "NULL" in B.pg_last_error()
    rc = lib.pg_sft_fwd_bwd(one, one, one, one, 8, 64, 100, C.byref(p), one, one, one, None, None, None, one, 16, None)
    assert rc == -3


def test_rmsnorm_entry_points_validate_arguments():
    lib = B.lib()
    one = C.c_void_p(16)
    assert lib.pg_rmsnorm_fwd(one, one, 4, 100, 1e-6, 0, one, None, None) == -2         # d not a multiple of 8
    assert lib.pg_rmsnorm_fwd(one, one, 4, 64, 1e-6, 7, one, None, None) == -1
    assert lib.pg_rmsnorm_fwd(one, one, 4, 8200, 1e-6, 0, one, None, None) == -2        # beyond the register-resident row
    assert lib.pg_rmsnorm_fwd(None, one, 4, 64, 1e-6, 0, one, None, None) == -1
    assert lib.pg_rmsnorm_fwd(None, None, 0, 64, 1e-6, 0, None, None, None) == 0
    assert int(lib.pg_rmsnorm_bwd_workspace_bytes(5120)) == 1024 * 5120 * 4
    assert int(lib.pg_rmsnorm_bwd_workspace_bytes(8200)) == 0
    assert lib.pg_rmsnorm_bwd(one, one, one, 4, 16384, 1e-6, 0, one, one, one, 1 << 30, None) == -2
    assert lib.pg_rmsnorm_bwd(one, one, one, 4, 64, 1e-6, 0, one, one, one, 16, None) == -3
    assert lib.pg_rmsnorm_bwd(one, one, one, 4, 64, -1.0, 0, one, one, one, 1 << 30, None) == -1


def test_fused_norm_entry_point_validates_arguments():
    lib = B.lib()
    one = C.c_void_p(16)
    p = B.Params().c_struct()
    big = 1 << 30
    call = lambda gamma, eps, dg, d, ws: lib.pg_loss_fwd_bwd_normed(one, gamma, eps, one, one, one, one, 1, one, None, None, None,
                                                                    None, 8, d, 100, C.byref(p), one, one, dg, one, None, None,
                                                                    None, one, ws, None)
    assert call(None, 1e-6, one, 64, big) == -1 and "gamma" in B.pg_last_error()
    assert call(one, 1e-6, None, 64, big) == -1
    assert call(one, -1.0, one, 64, big) == -1 and "norm_eps" in B.pg_last_error()
    assert call(one, 1e-6, one, 16384, big) == -2
    assert call(one, 1e-6, one, 64, 16) == -3
    n1 = B.pg_workspace_bytes(1024, 64, 1000, 4, B.Params(), B.CALL_LOSS_FWD_BWD)
    n2 = B.pg_workspace_bytes(1024, 64, 1000, 4, B.Params(), B.CALL_LOSS_FWD_BWD_NORMED)
    assert n2 > n1 > 0


def test_shard_entry_points_validate_arguments():
    lib = B.lib()
    one = C.c_void_p(16)      # never dereferenced: validation fails first
    p = B.Params().c_struct()
    big = 1 << 30
    assert lib.pg_head_shard_fwd(one, one, one, None, 8, 64, 100, 0, C.byref(p), None, one, big, None) == -1
    assert lib.pg_head_shard_fwd(one, one, one, None, 8, 64, 100, -1, C.byref(p), one, one, big, None) == -1
    assert "v_offset" in B.pg_last_error()
    assert lib.pg_head_shard_fwd(one, one, one, None, 8, 64, 100, 0, C.byref(p), C.c_void_p(8), one, big, None) == -1
    assert lib.pg_head_shard_fwd(one, one, one, None, 8, 64, 100, 0, C.byref(p), one, one, 16, None) == -3
    assert lib.pg_head_shard_fwd(one, one, one, None, 8, 72, 100, 0, C.byref(p), one, one, big, None) == -2
    assert lib.pg_head_shard_fwd(None, None, None, None, 0, 64, 100, 0, C.byref(p), None, None, 0, None) == 0   # T = 0
    assert lib.pg_head_partials_merge(one, None, one, 4, None) == -1
    assert lib.pg_head_partials_merge(one, C.c_void_p(4), one, 4, None) == -1 and "aligned" in B.pg_last_error()
    assert lib.pg_head_partials_merge(one, one, one, -1, None) == -1
    assert lib.pg_head_partials_merge(None, None, None, 0, None) == 0
    assert lib.pg_head_partials_finish(None, 4, one, None, None, None) == -1
    assert lib.pg_head_partials_finish(one, 4, None, None, None, None) == -1
    assert lib.pg_head_partials_finish(C.c_void_p(4), 4, one, None, None, None) == -1
    assert lib.pg_head_partials_finish(None, 0, None, None, None, None) == 0
    args = lambda partials, voff, f32, ws: (one, one, one, one, one, 1, one, None, None, None, None, partials, 8, 64, 100, voff,
                                            C.byref(p), one, one, f32, one, None, None, None, one, ws, None)
    assert lib.pg_loss_shard_bwd(*args(None, 0, 1, big)) == -1 and "partials" in B.pg_last_error()
    assert lib.pg_loss_shard_bwd(*args(one, -5, 1, big)) == -1
    assert lib.pg_loss_shard_bwd(*args(one, 0, 2, big)) == -1 and "dH_f32" in B.pg_last_error()
    assert lib.pg_loss_shard_bwd(*args(one, 0, 1, 16)) == -3


def test_static_monitors_and_init_validate_arguments():
    lib = B.lib()
    one = C.c_void_p(16)      # never dereferenced: validation fails first
    assert lib.pg_monitors_static(one, None, None, one, 4, None, 0, 0, None, 0, 0, None, None) == -1
    assert lib.pg_monitors_static(one, None, None, one, -1, None, 0, 0, None, 0, 0, one, None) == -1
    assert lib.pg_monitors_static(one, None, None, one, (1 << 31) + 1, None, 0, 0, None, 0, 0, one, None) == -2
    assert "at most" in B.pg_last_error()
    assert lib.pg_monitors_static(one, None, None, one, 4, one, 0, (1 << 40) + 1, None, 0, 0, one, None) == -2
    assert lib.pg_monitors_static(one, None, None, one, 4, C.c_void_p(8), 0, 8, None, 0, 0, one, None) == -1


def test_binding_rejects_wrong_dtypes_shapes_and_devices():
    """The C ABI sees raw pointers: the Python wrappers must refuse tensors whose dtype, shape or device is
    not what the library will assume, before any pointer is handed over (no GPU needed: every case fails
    in the wrapper)."""
    import torch
    T, d, V, S = 16, 64, 100, 2
    cpu = torch.device("cpu")
    H = torch.zeros((T, d), dtype=torch.bfloat16)
    W = torch.zeros((V, d), dtype=torch.bfloat16)
    y = torch.zeros(T, dtype=torch.int32)
    ws = torch.zeros(1024, dtype=torch.uint8)
    P = B.Params()
    with pytest.raises(ValueError, match="device pointers"):          # CPU tensors never reach the library
        B.pg_logprob_fwd(H, W, y, None, P, ws)
    with pytest.raises(ValueError, match="device pointers"):
        B.pg_sft_fwd_bwd(H, W, y, torch.ones(T, dtype=torch.uint8), P, ws)

    # the remaining checks are exercised through the helpers with the device check satisfied by a fake
    # device argument (the tensors live on the CPU here; with a GPU the same code sees cuda tensors)
    with pytest.raises(ValueError, match="dtype"):                    # torch's default int64 token ids
        B._want("y", y.long(), torch.int32, (T,), cpu)
    with pytest.raises(ValueError, match="dtype"):                    # bf16 H with params.dtype = fp32
        B._want("H", H, B._HEAD_DTYPES[1], (T, d))
    with pytest.raises(ValueError, match="shape"):
        B._want("W", torch.zeros((V, d + 64), dtype=torch.bfloat16), torch.bfloat16, (V, d), cpu)
    with pytest.raises(ValueError, match="shape"):
        B._want("y", y[:-1], torch.int32, (T,), cpu)
    with pytest.raises(ValueError, match="contiguous"):
        B._want("H", torch.zeros((d, T), dtype=torch.bfloat16).t(), torch.bfloat16, (T, d), cpu)
    with pytest.raises(ValueError, match="None"):
        B._want("y", None, torch.int32)
    B._want("mask", torch.ones(T, dtype=torch.bool), torch.uint8, (T,), cpu)          # bool is one byte per flag

    mask = torch.ones(T, dtype=torch.uint8)
    cu = torch.tensor([0, 8, 16], dtype=torch.int32)
    adv = torch.zeros(6, dtype=torch.float64)
    seg = torch.tensor([0, 5], dtype=torch.int32)
    lp = torch.zeros(T, dtype=torch.float32)
    ok = dict(T=T, dev=cpu, loss_mask=mask, cu_seqlens=cu, adv=adv, seg_sample=seg, sample_keep=None, old_logp=lp,
              rollout_logp=lp)
    assert B._want_loss_args(**ok) == S
    for key, bad, pat in (("adv", adv.float(), "dtype"), ("cu_seqlens", cu.long(), "dtype"), ("seg_sample", seg.long(), "dtype"),
                          ("seg_sample", seg[:1], "shape"), ("old_logp", lp.bfloat16(), "dtype"), ("old_logp", lp[:-1], "shape"),
                          ("rollout_logp", lp.double(), "dtype"), ("loss_mask", mask.int(), "dtype"),
                          ("sample_keep", torch.ones(5, dtype=torch.uint8), "shape"), ("adv", adv.reshape(2, 3), "1-d")):
        with pytest.raises(ValueError, match=pat):
            B._want_loss_args(**{**ok, key: bad})
    with pytest.raises(ValueError, match="no seg_sample"):
        B._want_loss_args(**{**ok, "adv": adv[:1], "seg_sample": None})

    out = (torch.zeros(1), torch.zeros((T, d), dtype=torch.bfloat16), torch.zeros(T), torch.zeros(T),
           torch.zeros(8, dtype=torch.int64))
    B._want_loss_out(out, T, d, V, cpu, torch.bfloat16, torch.zeros((V, d)), P)
    with pytest.raises(ValueError, match="dtype"):                    # fp32 dW buffer with params.dW_dtype = bf16
        B._want_loss_out(out, T, d, V, cpu, torch.bfloat16, torch.zeros((V, d)), B.Params(dW_dtype=1))
    with pytest.raises(ValueError, match="dtype"):
        B._want_loss_out(out[:4] + (torch.zeros(8, dtype=torch.int32),), T, d, V, cpu, torch.bfloat16, None, P)
    with pytest.raises(ValueError, match="shape"):
        B._want_loss_out(out, T, d, V, cpu, torch.bfloat16, torch.zeros((V + 1, d)), P)


def test_current_stream_without_the_private_short_cut(monkeypatch):
    import torch
    from types import SimpleNamespace
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: SimpleNamespace(cuda_stream=77))
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 1000 + device, raising=False)
    assert B._stream() == 1003
    assert B._stream(SimpleNamespace(cuda_stream=5)) == 5
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream")
    assert B._stream() == 77
