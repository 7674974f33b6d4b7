"""What the library plans for a call's sizes, seen through its workspace queries (host arithmetic, no GPU needed)."""
import pytest

from paper_2602_05885_amd import binding as B


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
    assert _in_blocks(T, d, V) == blocks
