"""Host-side argument checks of the Python binding (no GPU needed).

The binding marshals raw pointers, so it rejects tensors of the wrong dtype,
layout, device or length before any library call: such a tensor would make a
kernel read past its end or misread its elements.
"""
import pytest
import torch

import paper_2607_07508_amd as sao


def _adv_args(T=64, B=2):
    values = torch.zeros(T, dtype=torch.float32)
    rewards = torch.zeros(T, dtype=torch.float32)
    mask = torch.ones(T, dtype=torch.uint8)
    cu = torch.tensor([0, T // 2, T], dtype=torch.int32)
    return values, rewards, mask, cu


@pytest.mark.parametrize("which,bad,err", [
    ("mask", torch.ones(64, dtype=torch.int32), TypeError),           # wrong dtype
    ("rewards", torch.zeros(63, dtype=torch.float32), ValueError),      # one element short
    ("rewards", torch.zeros(128, dtype=torch.float32)[::2], ValueError),  # strided view
    ("cu", torch.tensor([0, 32, 64], dtype=torch.int64), TypeError),   # int64 boundaries
])
def test_advantage_rejects_bad_arrays(which, bad, err):
    values, rewards, mask, cu = _adv_args()
    args = dict(values=values, rewards=rewards, mask=mask, cu=cu)
    args[which] = bad
    with pytest.raises(err):
        sao.advantage(args["values"], args["rewards"], args["mask"], args["cu"])


def test_clipped_loss_rejects_bad_arrays():
    T = 32
    lp = torch.zeros(T, dtype=torch.float32)
    mask = torch.ones(T, dtype=torch.uint8)
    with pytest.raises(TypeError):
        sao.clipped_loss(lp, torch.zeros(T, dtype=torch.float64), lp, mask, 0.2, 0.2)
    with pytest.raises(ValueError):
        sao.clipped_loss(lp, lp, torch.zeros(T - 1, dtype=torch.float32), mask, 0.2, 0.2)
    with pytest.raises(TypeError):
        sao.clipped_loss(lp, lp, lp, mask, 0.2, 0.2, n_tokens=torch.zeros(1, dtype=torch.int32))


def test_head_calls_reject_host_tensors_and_mismatched_shapes():
    h = torch.zeros(8, 16, dtype=torch.float32)
    w = torch.zeros(10, 16, dtype=torch.float32)
    tgt = torch.zeros(8, dtype=torch.int32)
    with pytest.raises(ValueError):       # host memory is not device memory
        sao.token_logprob(h, w, tgt)
    with pytest.raises(TypeError):
        sao.token_logprob(h, w.to(torch.bfloat16), tgt)
    with pytest.raises(ValueError):       # H differs
        sao.loss_backward(h, torch.zeros(10, 8), tgt, torch.zeros(8), torch.zeros(8))


def test_comparison_and_estimator_calls_reject_bad_arrays():
    T = 32
    lp = torch.zeros(T, dtype=torch.float32)
    mask = torch.ones(T, dtype=torch.uint8)
    with pytest.raises(TypeError):        # the decoupled weight's log-probs must be float32
        sao.ppo_loss(lp, lp, lp, mask, 0.2, 0.28, logp_behav=torch.zeros(T, dtype=torch.float64))
    with pytest.raises(ValueError):
        sao.ppo_loss(lp, lp, torch.zeros(T - 1), mask, 0.2, 0.28)
    with pytest.raises(TypeError):
        sao.explained_variance(lp, lp, mask, moments=torch.zeros(5, dtype=torch.float32))
    with pytest.raises(ValueError):
        sao.explained_variance(lp, lp, mask, moments=torch.zeros(4, dtype=torch.float64))
    values, rewards, mask, cu = _adv_args()
    with pytest.raises(ValueError):       # only "average" and "last"
        sao.step_advantage(values, rewards, mask, cu, step_value="median")
    with pytest.raises(TypeError):
        sao.step_advantage(values, rewards, mask.to(torch.int32), cu)
    with pytest.raises(TypeError):
        sao.group_advantage(rewards.double(), mask, cu, 2, 1e-6)
    history, seen = torch.zeros(3, 8, dtype=torch.float64), torch.zeros(3, dtype=torch.int64)
    with pytest.raises(ValueError):       # history is [n_keys, window]
        sao.running_mean_advantage(rewards, mask, cu, history.flatten(), seen)
    with pytest.raises(ValueError):
        sao.running_mean_advantage(rewards, mask, cu, history, seen[:2])
    with pytest.raises(TypeError):
        sao.running_mean_advantage(rewards, mask, cu, history, seen, keys=torch.zeros(2, dtype=torch.int64))


def test_calls_without_the_native_marshalling(monkeypatch):
    """Without _fast.so, or with one built for another torch, the same calls go through Python."""
    import sys
    import types

    from paper_2607_07508_amd import binding
    values, rewards, mask, cu = _adv_args()
    name = "paper_2607_07508_amd._fast"
    for module in (None, types.SimpleNamespace(torch="0.0"), types.SimpleNamespace()):  # None: its import fails
        with monkeypatch.context() as mp:
            mp.setitem(sys.modules, name, module)
            mp.setattr(binding, "_fast_module", None)
            assert binding._load_fast() is None
            assert binding._fast().advantage(values, rewards, mask, cu) is None
            with pytest.raises(TypeError):    # the Python code's own check
                sao.advantage(values, rewards.double(), mask, cu)


def test_build_does_without_the_native_marshalling(monkeypatch, tmp_path):
    """What _fast.so needs beyond the C library may be missing; a compile error is an error."""
    import sysconfig

    from paper_2607_07508_amd import build as B
    monkeypatch.setattr(B, "FAST_MODULE", str(tmp_path / "_fast.so"))
    with monkeypatch.context() as mp:
        mp.setattr(B.shutil, "which", lambda name: None)
        assert "g++" in B._build_fast()
    if B.shutil.which("g++") is None:
        pytest.skip("no C++ compiler")
    with monkeypatch.context() as mp:
        mp.setattr(sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
        assert "Python.h" in B._build_fast()
    monkeypatch.setattr(B, "CSRC", str(tmp_path))
    (tmp_path / "fast.cpp").write_text("not C++\n")
    with pytest.raises(RuntimeError):
        B._build_fast()
    assert not (tmp_path / "_fast.so").exists()
