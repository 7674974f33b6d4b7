"""The native step of the small stages against the general path of the binding: same outputs, and whatever is not plainly
in order is left to the general path."""
import pytest
import torch

from paper_2602_05885_amd import binding as B


def _inputs(dev, P=5, K=7, Tm=3):
    g = torch.Generator().manual_seed(4)
    n = P * K * Tm
    f = lambda: (torch.rand(n, generator=g) + 0.2).to(dev)                      # noqa: E731
    u = lambda: (torch.rand(n, generator=g) < 0.6).to(torch.uint8).to(dev)      # noqa: E731
    return dict(correct=u(), ref=f(), ker=f(), gen=f(), tot=f() + 1, valid=u(), shape=(P, K, Tm))


def _calls(x):
    """name, function(gets the binding) for every option."""
    R, V = x["ref"].view(x["shape"]), x["valid"].view(x["shape"])
    yield "reward", lambda: B.turn_reward(x["correct"], x["ref"], x["ker"], x["gen"], x["tot"])
    yield "reward without ratio", lambda: B.turn_reward(x["correct"], x["ref"], x["ker"], speedup_cap=2, want_pr=False)
    for hard in (False, True):
        yield "retain", lambda: B.prs_retain(x["ref"], x["valid"], 12345678901234567890, hard=hard)
        yield "retain without flags", lambda: B.prs_retain(x["ref"], None, -1, tau=0.5, s=0.3, hard=hard, want_p=False)
    for f in (B.trloo_advantage, B.grpo_advantage):
        yield "advantage", lambda: f(R, V, 0.9)
        yield "advantage alone", lambda: f(R, V, 1, want_returns=False, want_group_n=False)


class _General:
    """Stands in for the native module and declines everything."""
    def __getattr__(self, name):
        return lambda *a: None


@pytest.mark.gpu
def test_native_step_equals_the_general_path(monkeypatch):
    x = _inputs("cuda:0")
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        native = [f() for _, f in _calls(x)]
    side.synchronize()
    monkeypatch.setattr(B, "_stage", _General())
    for (name, f), got in zip(_calls(x), native):
        want = f()
        torch.cuda.synchronize()
        assert len(got) == len(want), name
        for a, b in zip(got, want):
            assert (a is None) == (b is None), name
            if a is not None:
                assert a.dtype == b.dtype and a.device == b.device and torch.equal(a, b), name


@pytest.mark.gpu
def test_what_is_not_in_order_goes_the_general_way():
    x = _inputs("cuda:0")
    n = x["ref"].numel()
    with pytest.raises(AssertionError):
        B.turn_reward(x["correct"].bool(), x["ref"], x["ker"])
    with pytest.raises(AssertionError):
        B.turn_reward(x["correct"], x["ref"][:-1], x["ker"])
    with pytest.raises(ValueError, match="contiguous"):
        B.turn_reward(x["correct"], torch.ones(2 * n, device="cuda:0")[::2], x["ker"])
    with pytest.raises(B.PgError):
        B.turn_reward(x["correct"], None, x["ker"])
    with pytest.raises(B.PgError):
        B.prs_retain(x["ref"], None, 1, s=-1.0)
    with pytest.raises(ValueError):
        B.trloo_advantage(x["ref"], x["valid"])
    with pytest.raises(B.PgError):
        B.trloo_advantage(x["ref"].view(x["shape"]), x["valid"].view(x["shape"]), float("nan"))


def test_host_tensors_are_declined():
    x = _inputs("cpu")
    B.lib()
    assert B._stage.turn_reward(x["correct"], x["ref"], x["ker"], None, None, 3.0, True, None) is None
    assert B._stage.prs_retain(x["ref"], None, 1, 0.3, 0.1, False, True, None) is None
    assert B._stage.turn_advantage(x["ref"].view(x["shape"]), x["valid"].view(x["shape"]), 1.0, True, True, False, None) is None
    with pytest.raises(AssertionError):
        B.turn_reward(x["correct"], x["ref"][:-1], x["ker"])
