"""dgamma_out need not be aligned to more than a float: at every offset into a flat gradient buffer it holds the same bits, and what
lies beside it stays."""
import ctypes as C

import pytest
import torch

from paper_2602_05885_amd import binding as B
from paper_2602_05885_amd import synth

pytestmark = pytest.mark.gpu


class _DgammaAt:
    """The library with another address in the place of one call's dgamma_out."""
    def __init__(self, lib, call, index, out):
        self._lib, self._call, self._index, self._out = lib, call, index, out

    def __getattr__(self, name):
        f = getattr(self._lib, name)
        if name != self._call:
            return f
        return lambda *a: f(*a[:self._index], C.c_void_p(self._out.data_ptr()), *a[self._index + 1:])


@pytest.mark.parametrize("dtype,d,fused", [("bf16", 8, False), ("bf16", 64, False), ("f32", 5832, False), ("bf16", 64, True), ("f32", 192, True)])
def test_dgamma_at_any_float(monkeypatch, dtype, d, fused):
    T, V, dev = 70, 300, torch.device("cuda:0")
    X, W, y = synth.make_head(T, d, V, dtype, 3, dev)
    gamma = torch.linspace(0.5, 1.5, d, device=dev).to(X.dtype)
    if fused:
        p = B.Params(dtype=int(dtype == "f32"))
        ws = B.alloc_workspace(T, d, V, 1, p, B.CALL_LOSS_FWD_BWD_NORMED, dev)
        m, cu = torch.ones(T, dtype=torch.uint8, device=dev), torch.tensor([0, T], dtype=torch.int32, device=dev)
        adv = torch.full((1,), -0.8, dtype=torch.float64, device=dev)
        call, index = "pg_loss_fwd_bwd_normed", 19
        run = lambda: B.pg_loss_fwd_bwd_normed(X, gamma, 1e-6, W, y, m, cu, adv, None, None, None, p, ws)["dgamma"]      # noqa: E731
    else:
        dH = torch.randn(T, d, device=dev).to(X.dtype)
        call, index = "pg_rmsnorm_bwd", 8
        run = lambda: B.pg_rmsnorm_bwd(X, gamma, dH, 1e-6)[1]      # noqa: E731
    want = run()
    assert want.abs().max() > 0
    lib = B.lib()
    for at in range(1, 5):
        flat = torch.full((d + 8,), 7.0, device=dev)
        monkeypatch.setattr(B, "_lib", _DgammaAt(lib, call, index, flat[at:at + d]))
        run()
        monkeypatch.setattr(B, "_lib", lib)
        torch.cuda.synchronize()
        assert torch.equal(flat[at:at + d], want), at
        assert (flat[:at] == 7).all() and (flat[at + d:] == 7).all(), at
