"""What the library plans for a call's sizes, seen through its workspace queries (host arithmetic, no GPU needed)."""
import ctypes as C

import pytest

from paper_2602_05885_amd import binding as B
from tests._cases import block_rows


def _in_blocks(T, d, V):
    """Token blocks need an fp32 dW; beside them the type of dW does not enter the plan."""
    sizes = [B.pg_workspace_bytes(T, d, V, 0, B.Params(dW_dtype=w), B.CALL_LOSS_FWD_BWD) for w in (0, 1)]
    assert all(sizes)
    return sizes[0] != sizes[1]


@pytest.mark.parametrize("T,d,V,blocks", [
    (16000, 1536, 512000, False), (20000, 1536, 256000, False), (43697, 1536, 151936, False), (20000, 3072, 256000, False),
    (16000, 5120, 512000, False), (50000, 1536, 100000, True), (43697, 2048, 151936, True), (43697, 5120, 151936, True),
    (16000, 8192, 512000, True), (16640, 5120, 151936, False), (50000, 1472, 100000, False)])
def test_blocks_only_where_their_dh_fills_the_chip_twice(T, d, V, blocks):
    """A block whose dH launch has less than two rounds of tiles made the call up to 1.6 times as long."""
    assert _in_blocks(T, d, V) == blocks == (block_rows(T, d, V) < (T + 255) // 256 * 256)


def _needed(T, d, V, which, nbytes, prm):
    """What a loss call says it needs when it is given `nbytes` (refused before any HIP call), None if it does not refuse."""
    lib, p, one = B.lib(), prm.c_struct(), C.c_void_p(16)
    if which == B.CALL_LOSS_SHARD_BWD:
        rc = lib.pg_loss_shard_bwd(one, one, one, one, one, 1, one, None, None, None, None, one, T, d, V, 0, C.byref(p), one, one, 1, one,
                                   None, None, None, one, nbytes, None)
    elif which == B.CALL_LOSS_FWD_BWD_NORMED:
        rc = lib.pg_loss_fwd_bwd_normed(one, one, 1e-6, one, one, one, one, 1, one, None, None, None, None, T, d, V, C.byref(p), one, one,
                                        one, one, None, None, None, one, nbytes, None)
    else:
        rc = lib.pg_loss_fwd_bwd(one, one, one, one, one, 1, one, None, None, None, None, T, d, V, C.byref(p), one, one, one, None, None,
                                 None, one, nbytes, None)
    assert rc == -3, rc
    return int(B.pg_last_error().split(",")[1].split()[0])


SHAPES = [(T, d, V) for d, V in ((5120, 151936), (4096, 151936), (2048, 151936), (1536, 100000), (1536, 50000), (8192, 512000), (512, 151936))
          for T in (1, 1000, 17152, 17408, 40000, 43697, 70000, 131072)]


@pytest.mark.parametrize("which", [B.CALL_LOSS_FWD_BWD, B.CALL_LOSS_FWD_BWD_NORMED])
def test_a_loss_call_takes_everything_from_the_documented_minimum_on(which):
    """The kept logits (39/8 of the dS scratch) may be missing in whole or in part, also where the call works in token
    blocks: beside them it takes about what one block without kept logits needs."""
    for T, d, V in SHAPES:
        full, least = (f(T, d, V, 1, B.Params(), which) for f in (B.pg_workspace_bytes, B.pg_workspace_min_bytes))
        assert 0 < least <= full, (T, d, V)
        for n in (least - 1, least // 2, 0):
            assert _needed(T, d, V, which, n, B.Params()) == least, (T, d, V, n)
        if _in_blocks(T, d, V):
            td, tiles_v = (d + 255) // 256, (V + 255) // 256
            kept = (39936 // tiles_v * td // 256 * 256 // td * tiles_v) << 18      # 39936 tiles of 256 KiB, in whole rounds of dH tiles
            assert least <= 1.2 * (full - kept), (T, d, V)


def test_the_minimum_of_the_other_calls_is_their_size():
    args = (5000, 5120, 151936, 0, B.Params(), B.CALL_LOGPROB_FWD)
    assert B.pg_workspace_min_bytes(*args) == B.pg_workspace_bytes(*args) > 0
    assert B.pg_workspace_min_bytes(1024, 100, 1000, 1, B.Params(), 1) == 0 and "multiple of 64" in B.pg_last_error()


def test_the_shard_backward_reserves_no_logits():
    """It starts from states of another call, so its size is what a loss call needs beside the kept logits, and the least it
    takes; the size of the loss call is enough for it as well."""
    for T, d, V in SHAPES:
        for dw in (0, 1):
            prm = B.Params(dW_dtype=dw)
            n = B.pg_workspace_bytes(T, d, V, 1, prm, B.CALL_LOSS_SHARD_BWD)
            assert 0 < n == B.pg_workspace_min_bytes(T, d, V, 1, prm, B.CALL_LOSS_SHARD_BWD)
            assert n <= B.pg_workspace_bytes(T, d, V, 1, prm, B.CALL_LOSS_FWD_BWD), (T, d, V)
            assert n >= B.pg_workspace_bytes(T, d, V, 1, prm, B.CALL_LOGPROB_FWD), (T, d, V)
            assert _needed(T, d, V, B.CALL_LOSS_SHARD_BWD, n - 1, prm) == n
    n = B.pg_workspace_bytes(16411, 5120, 18992, 30, B.Params(), B.CALL_LOSS_SHARD_BWD)      # one of eight shards of a 14B head
    assert n < 2.4 * (1 << 30) < 3.4 * (1 << 30) < B.pg_workspace_bytes(16411, 5120, 18992, 30, B.Params(), B.CALL_LOSS_FWD_BWD)


def test_no_second_w_transposed_beside_the_callers():
    """Token blocks hold the whole W^T, unless the caller keeps it."""
    for T, d, V in SHAPES:
        lib, sizes, least = B.lib(), [], []
        for cache in (None, 256):
            p = B.Params().c_struct()
            p.w_transposed = cache
            sizes.append(int(lib.pg_workspace_bytes(T, d, V, 1, C.byref(p), B.CALL_LOSS_FWD_BWD)))
            least.append(int(lib.pg_workspace_min_bytes(T, d, V, 1, C.byref(p), B.CALL_LOSS_FWD_BWD)))
        assert least[0] == least[1] <= sizes[1]          # a call without the cache takes the size asked for with it
        one = B.pg_workspace_bytes(T, d, V, 1, B.Params(), B.CALL_LOSS_SHARD_BWD)      # enough for that call, too
        saved = min(int(lib.pg_w_transposed_bytes(d, V)), sizes[0] - one) if _in_blocks(T, d, V) else 0
        assert sizes[0] - sizes[1] == saved, (T, d, V)
