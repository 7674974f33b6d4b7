"""RMS normalisation on both sides of each size at which another kernel takes over (144 and 256 MiB of one bf16 matrix)."""
import pytest
import torch

from tests.test_gpu_row_streams import test_rmsnorm_variants as check_rmsnorm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,dtype", [(9216, 8192, torch.bfloat16), (9217, 8192, torch.bfloat16), (16384, 8192, torch.bfloat16), (16385, 8192, torch.bfloat16),
                                       (9217, 4096, torch.float32)])
def test_rmsnorm_around_the_cache_lines(T, d, dtype):
    check_rmsnorm(T, d, dtype)
