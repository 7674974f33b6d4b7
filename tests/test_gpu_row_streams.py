"""The bandwidth-bound row kernels at the edges of their variants: RMS normalisation with fewer rows than strips and beyond the
size from which rows are read past the caches, gradient norms of every remainder."""
import pytest
import torch

from paper_2602_05885_amd import binding as B

pytestmark = pytest.mark.gpu


# (rows, d, dtype): strips 1, 31, 1023, 1024, 1025; bf16 and fp32 matrices of more than 256 MiB
@pytest.mark.parametrize("T,d,dtype", [(1, 64, torch.bfloat16), (31, 2056, torch.float32), (1023, 520, torch.bfloat16), (1024, 8, torch.float32),
                                       (1025, 5120, torch.bfloat16), (26300, 5120, torch.bfloat16), (13150, 5120, torch.float32)])
def test_rmsnorm_variants(T, d, dtype):
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(T)
    X = torch.randn((T, d), generator=g, device=dev).to(dtype)
    dH = torch.randn((T, d), generator=g, device=dev).to(dtype)
    gamma = (1 + 0.1 * torch.randn(d, generator=g, device=dev)).to(dtype)
    h, rstd = B.pg_rmsnorm_fwd(X, gamma, 1e-6)
    dX, dgamma = B.pg_rmsnorm_bwd(X, gamma, dH, 1e-6)
    tol = 4e-3 if dtype is torch.bfloat16 else 1e-5       # one rounding to bf16 (2^-9 per element at most); fp32 sums over d
    want_g = torch.zeros(d, dtype=torch.float64, device=dev)
    for a in range(0, T, 4096):
        x, o, ga = X[a:a + 4096].double(), dH[a:a + 4096].double(), gamma.double()
        r = torch.rsqrt((x * x).mean(1, keepdim=True) + 1e-6)
        xh = x * r
        want = r * (ga * o - xh * (ga * o * xh).mean(1, keepdim=True))
        want_g += (o * xh).sum(0)
        assert (rstd[a:a + 4096].double() - r[:, 0]).abs().max() <= 1e-5 * r.max()
        for got, ref in ((h[a:a + 4096], xh * ga), (dX[a:a + 4096], want)):
            assert ((got.double() - ref).norm(dim=1) <= tol * ref.norm(dim=1) + 1e-12).all()
    assert (dgamma.double() - want_g).norm() <= 1e-5 * want_g.norm()


@pytest.mark.parametrize("n", [1, 7, 8, 9, 2047, 2048 * 1024 + 3, 4 * 2048 * 1024, 4 * 2048 * 1024 + 8 * 255 + 5, 5 * 2048 * 1024 + 2049])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_gradient_norms_of_every_remainder(n, dtype):
    dev = torch.device("cuda:0")
    g = torch.randn(n, generator=torch.Generator(device=dev).manual_seed(n), device=dev).to(dtype)
    one = torch.full((3,), -1.0, device=dev)
    out = B.pg_monitors(one, None, None, torch.ones(3, dtype=torch.uint8, device=dev), g, g)
    want = g.double().norm().item()
    assert abs(out[3].item() - want) <= 1e-12 * want and out[4].item() == out[3].item()      # fp64 sums
