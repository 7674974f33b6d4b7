"""RMS normalisation on both sides of each size at which another kernel takes over (144 and 256 MiB of one bf16 matrix), and the fold of
its dgamma partials for full and short sets of strips."""
import pytest
import torch

from paper_2602_05885_amd import binding as B
from tests.test_gpu_row_streams import test_rmsnorm_variants as check_rmsnorm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,dtype", [(9216, 8192, torch.bfloat16), (9217, 8192, torch.bfloat16), (16384, 8192, torch.bfloat16), (16385, 8192, torch.bfloat16),
                                       (9217, 4096, torch.float32)])
def test_rmsnorm_around_the_cache_lines(T, d, dtype):
    check_rmsnorm(T, d, dtype)


@pytest.mark.parametrize("strips", [1, 33, 255, 256, 257, 1023, 1024])
@pytest.mark.parametrize("d", [8, 40, 4104])
def test_dgamma_fold_of_every_strip(strips, d):
    """One row per strip, and only one of them counts: dgamma is that row's, bit for bit, whichever it is."""
    dev = torch.device("cuda:0")
    X = torch.randn((strips, d), generator=torch.Generator(device=dev).manual_seed(d), device=dev)
    gamma = torch.ones(d, device=dev)
    for row in {0, strips // 2, strips - 1}:
        dH = torch.zeros((strips, d), device=dev)
        dH[row] = 2.0
        dgamma = B.pg_rmsnorm_bwd(X, gamma, dH, 1e-6)[1]
        alone = B.pg_rmsnorm_bwd(X[row:row + 1].contiguous(), gamma, dH[row:row + 1].contiguous(), 1e-6)[1]
        assert torch.equal(dgamma, alone) and alone.abs().max() > 0, row
