"""The native argument marshalling of the per-token entry points against the Python code it
stands in for: same outputs (values, shapes, dtypes) and same refusals."""
import pytest
import torch

import paper_2607_07508_amd as sao
from paper_2607_07508_amd import binding
from tests.gpu_common import say


def _calls(x, status=None):
    f, m, cu = x["f"], x["m"], x["cu"]
    return {
        "advantage": lambda: sao.advantage(f, x["r"], m, cu, alpha=1.5, status=status),
        "advantage_fixed": lambda: sao.advantage(f, x["r"], m, cu, 0.99, 0.95, want_count=False),
        "step": lambda: sao.step_advantage(f, x["r"], m, cu, alpha=1.5, status=status),
        "step_last": lambda: sao.step_advantage(f, x["r"], m, cu, step_value="last", want_last=False, want_count=0),
        "group": lambda: sao.group_advantage(x["r"], m, cu, 2, 1e-6, status=status),
        "clipped": lambda: sao.clipped_loss(f, x["r"], f, m, 0.2, 0.28),
        "clipped_n": lambda: sao.clipped_loss(f, x["r"], f, m, 0.2, 0.28, x["n"]),
        "ppo": lambda: sao.ppo_loss(f, x["r"], f, m, 0.2, 0.28, logp_behav=x["r"]),
        "ppo_n": lambda: sao.ppo_loss(f, x["r"], f, m, 0.2, 0.28, x["n"]),
        "ev": lambda: sao.explained_variance(f, x["r"], m),
    }


def _inputs(T, device):
    gen = torch.Generator().manual_seed(T)
    cu = torch.tensor([0, T // 3, T // 3, T // 2, T], dtype=torch.int32)
    x = dict(f=-torch.rand(T, generator=gen), r=-torch.rand(T, generator=gen), cu=cu,
             m=(torch.rand(T, generator=gen) < 0.7).to(torch.uint8), n=torch.tensor([T // 2 + 1]))
    return {k: v.to(device) for k, v in x.items()}


def _outcome(fn):
    try:
        return "ok", fn()
    except Exception as e:  # noqa: BLE001 (the type and text are what is compared)
        return type(e), str(e)


def _both(monkeypatch, calls):
    native = {k: _outcome(f) for k, f in calls.items()}
    with monkeypatch.context() as mp:
        mp.setattr(binding, "_fast", binding._Plain)
        python = {k: _outcome(f) for k, f in calls.items()}
    return native, python


def _same(a, b):
    """Equal in type, shape, device and every value, NaN in the same places."""
    return (a.dtype == b.dtype and a.shape == b.shape and a.device == b.device
            and bool(((a == b) | (a.isnan() & b.isnan())).all()))


def test_same_tells_values_apart():
    a, nan = torch.tensor([1.0, 2.0]), float("nan")
    assert _same(a, a.clone()) and _same(torch.tensor([nan, 2.0]), torch.tensor([nan, 2.0]))
    assert _same(torch.empty(0), torch.empty(0))
    assert not _same(a, torch.tensor([1.0, 9.0])) and not _same(torch.tensor([1, 2]), torch.tensor([5, 9]))
    assert not _same(torch.tensor([nan, 2.0]), a) and not _same(a, torch.tensor([1.0, nan]))
    assert not _same(a, a.double()) and not _same(a, a[:, None])


@pytest.mark.gpu
@pytest.mark.parametrize("T", [0, 6, 5000])
def test_same_outputs(monkeypatch, T):
    say(f"native marshalling: T={T}")
    side = torch.cuda.Stream()
    for stream in (torch.cuda.current_stream(), side):
        with torch.cuda.stream(stream):
            x = _inputs(T, "cuda")
            status = torch.zeros(1, dtype=torch.int32, device="cuda")
            native, python = _both(monkeypatch, _calls(x, status))
            stream.synchronize()
            for k in native:
                assert native[k][0] == python[k][0] == "ok", (k, native[k], python[k])
                for a, b in zip(native[k][1], python[k][1]):
                    assert (a is None) == (b is None), k
                    assert a is None or _same(a, b), k


@pytest.mark.gpu
def test_plain_calls_are_taken():
    x = _inputs(100, "cuda")
    f = binding._fast()
    assert f.advantage(x["f"], x["r"], x["m"], x["cu"], 1.0, 1.0, 0.0, None, True) is not None
    assert f.ppo_loss(x["f"], x["r"], None, x["f"], x["m"], 0.2, 0.2, None) is not None
    with torch.overrides.TorchFunctionMode():
        assert f.advantage(x["f"], x["r"], x["m"], x["cu"], 1.0, 1.0, 0.0, None, True) is None


@pytest.mark.gpu
@pytest.mark.parametrize("change", [
    dict(f=lambda t: t.double()), dict(f=lambda t: torch.stack([t, t], 1)[:, 0]), dict(m=lambda t: t.bool()),
    dict(m=lambda t: t[:50]), dict(r=lambda t: t.cpu()), dict(cu=lambda t: t.long()), dict(cu=lambda t: t[:1]),
    dict(cu=lambda t: t[:4].contiguous()), dict(f=lambda t: None), dict(n=lambda t: t.int())])
def test_same_refusals(monkeypatch, change):
    x = _inputs(100, "cuda")
    x.update({k: f(x[k]) for k, f in change.items()})
    native, python = _both(monkeypatch, _calls(x))
    for k in native:
        if native[k][0] == "ok":
            assert python[k][0] == "ok", k
        else:
            assert native[k] == python[k], k


def test_host_tensors_are_refused_alike(monkeypatch):
    native, python = _both(monkeypatch, _calls(_inputs(100, "cpu")))
    assert all(n[0] != "ok" and n == p for n, p in zip(native.values(), python.values())), (native, python)
