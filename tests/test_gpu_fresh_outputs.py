"""The loss, explained-variance and critic entry points that write their accumulated
outputs (sao_*_store) against the ones that add to zeros: the same kernels, so every
value must agree, whatever the buffers held before. Through the binding, which stores
when it makes the outputs and adds when the caller brings them; fresh allocations are
primed with NaN so that a value left unwritten shows."""
import pytest
import torch

import paper_2607_07508_amd as sao
from tests.gpu_common import say

pytestmark = pytest.mark.gpu

SIZES = [1, 255, 1024, 1025, 4099, 262147, 2097152 + 5]  # up to past one quad of tokens per thread


def _inputs(T, off=0):
    gen = torch.Generator(device="cuda").manual_seed(T + off)
    r = lambda: torch.randn(T + off, generator=gen, device="cuda")[off:]  # noqa: E731
    lp = -r().abs() - 0.1
    mask = (torch.rand(T + off, generator=gen, device="cuda") < 0.6).to(torch.uint8)[off:]
    return lp, lp - 0.3 * r(), r(), r(), mask


def _prime():
    """Leaves NaN bit patterns in the allocator's small blocks."""
    junk = [torch.full((n,), float("nan"), dtype=torch.float64, device="cuda") for n in (1, 2, 5, 64) for _ in range(8)]
    del junk


@pytest.mark.parametrize("off", [0, 3])  # 3: no vector access, a mask without whole words
@pytest.mark.parametrize("T", SIZES)
def test_store_equals_add(T, off):
    say(f"fresh outputs: T={T} offset={off}")
    lp, old, adv, val, mask = _inputs(T, off)
    zeros = lambda n, d: torch.zeros(n, dtype=d, device="cuda")  # noqa: E731
    n = mask.sum(dtype=torch.int64).reshape(1)
    for kw in ({}, {"n_tokens": n}):
        for fn, nl in ((sao.clipped_loss, 2), (sao.ppo_loss, 1)):
            _prime()
            a = fn(lp, old, adv, mask, 0.2, 0.28, **kw)
            b = fn(lp, old, adv, mask, 0.2, 0.28, loss=zeros(nl, torch.float64), counts=zeros(5, torch.int64), **kw)
            c = fn(lp, old, adv, mask, 0.2, 0.28, counts=zeros(5, torch.int64), **kw)
            d = fn(lp, old, adv, mask, 0.2, 0.28, loss=zeros(nl, torch.float64), **kw)
            for x in (b, c, d):
                assert all(torch.equal(p, q) for p, q in zip(a, x))
            assert int(a[3][0]) == int(n) and int(a[3][1:].sum()) == int(n)
    _prime()
    ev, m = sao.explained_variance(val, adv, mask)
    ev2, m2 = sao.explained_variance(val, adv, mask, moments=zeros(5, torch.float64))
    assert torch.equal(m, m2) and (torch.equal(ev, ev2) or (ev.isnan() & ev2.isnan()).all())
    assert float(m[0]) == int(n)


@pytest.mark.parametrize("T,H", [(1, 8), (300, 72), (5000, 1032)])
def test_value_loss_store_equals_add(T, H):
    say(f"fresh outputs: critic T={T} H={H}")
    gen = torch.Generator(device="cuda").manual_seed(T)
    h = torch.randn((T, H), generator=gen, device="cuda")
    w = torch.randn(H, generator=gen, device="cuda")
    _, _, ret, v, mask = _inputs(T)
    for m in (mask, torch.zeros_like(mask)):
        a = sao.value_loss(h, w, v, ret, m)
        b = sao.value_loss(h, w, v, ret, m, loss=torch.zeros(1, dtype=torch.float64, device="cuda"),
                           dw_value=torch.zeros(H, device="cuda"))
        assert all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("dtype,T", [(torch.bfloat16, 32769), (torch.bfloat16, 65535), (torch.float32, 16385)])
def test_value_loss_over_the_cache(dtype, T):
    """One call whose hidden states and their gradient exceed 128 MiB (non-temporal stores) against the same rows
    in two calls that don't: each row's gradient comes from that row alone, so it is the same bit for bit."""
    H = 1024
    say(f"critic over the cache: T={T} {dtype}")
    gen = torch.Generator(device="cuda").manual_seed(T)
    h = torch.randn((T, H), generator=gen, device="cuda").to(dtype)
    w = torch.randn(H, generator=gen, device="cuda").to(dtype)
    _, _, ret, v, mask = _inputs(T)
    n = mask.sum(dtype=torch.int64).reshape(1)
    loss, dh, dw = sao.value_loss(h, w, v, ret, mask, n_tokens=n)
    loss2 = torch.zeros(1, dtype=torch.float64, device="cuda")
    dw2 = torch.zeros(H, device="cuda")
    dh2 = torch.empty_like(h)
    for a, b in ((0, T // 2), (T // 2, T)):
        sao.value_loss(h[a:b], w, v[a:b], ret[a:b], mask[a:b], n_tokens=n, loss=loss2, dw_value=dw2, dhidden=dh2[a:b])
    assert torch.equal(dh, dh2)
    # fp32 sums of T terms in another order
    assert float((loss - loss2).abs()) <= 1e-12 * float(loss) and float((dw - dw2).norm() / dw.norm()) <= 1e-5


def test_empty_calls():
    f = torch.empty(0, device="cuda")
    m = torch.empty(0, dtype=torch.uint8, device="cuda")
    for fn in (sao.clipped_loss, sao.ppo_loss):
        loss, _, _, counts = fn(f, f, f, m, 0.2, 0.2)
        assert (loss == 0).all() and (counts == 0).all()
    ev, moments = sao.explained_variance(f, f, m)
    assert ev.isnan().all() and (moments == 0).all()
