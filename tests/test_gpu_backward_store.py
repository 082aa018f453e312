"""The weight gradient stored by sao_loss_backward_store against the one that
sao_loss_backward adds to zeros: the same tiles without the read, so every element
must agree, whatever the buffer held before (NaN here)."""
import numpy as np
import pytest
import torch

import paper_2607_07508_amd as sao
from tests.gpu_common import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("T,H,V,active", [
    (1, 8, 1, 1),           # one element-wide edge tile
    (300, 264, 1000, 200),  # whole tiles and edges on both sides
    (520, 512, 512, 257),   # whole tiles only, K past one tile of rows
    (700, 72, 70000, 90),   # several tiles of vocabulary and an edge
    (500, 64, 700, 0),      # no row with a gradient: zeros
])
def test_store_equals_add_to_zeros(T, H, V, active, dtype):
    say(f"dW store: T={T} H={H} V={V} rows with a gradient={active} {dtype}")
    gen = torch.Generator(device="cuda").manual_seed(T + V)
    h = torch.randn((T, H), generator=gen, device="cuda").to(dtype)
    w = (0.05 * torch.randn((V, H), generator=gen, device="cuda")).to(dtype)
    y = torch.randint(0, V, (T,), generator=gen, device="cuda", dtype=torch.int32)
    g = torch.zeros(T, device="cuda")
    rows = np.sort(np.random.default_rng(V).choice(T, active, replace=False))
    g[torch.from_numpy(rows).cuda()] = 1.0 / T
    lse = torch.logsumexp(h.float() @ w.float().t(), 1)
    added = torch.zeros((V, H), device="cuda")
    dh0, _ = sao.loss_backward(h, w, y, lse, g, dw_head=added)
    stored = torch.full((V, H), float("nan"), device="cuda")
    dh1 = torch.empty_like(h)
    L = sao.lib()
    code = 0 if dtype == torch.bfloat16 else 1
    ws = torch.empty(sao.workspace_size(3, T, H, V, code), dtype=torch.uint8, device="cuda")
    assert L.sao_loss_backward_store(h.data_ptr(), H, w.data_ptr(), H, y.data_ptr(), lse.data_ptr(), g.data_ptr(), T, H,
                                     V, code, dh1.data_ptr(), stored.data_ptr(), ws.data_ptr(), ws.numel(),
                                     torch.cuda.current_stream().cuda_stream) == 0
    assert torch.equal(added, stored) and torch.equal(dh0, dh1)
    dh2, fresh = sao.loss_backward(h, w, y, lse, g)
    assert torch.equal(added, fresh) and torch.equal(dh0, dh2)
    if active == 0:
        assert (stored == 0).all()


def test_empty_call_gives_zeros():
    h = torch.empty((0, 64), dtype=torch.bfloat16, device="cuda")
    w = torch.ones((100, 64), dtype=torch.bfloat16, device="cuda")
    f = torch.empty(0, device="cuda")
    dh, dw = sao.loss_backward(h, w, torch.empty(0, dtype=torch.int32, device="cuda"), f, f)
    assert dh.shape == (0, 64) and (dw == 0).all()
