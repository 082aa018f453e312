"""Log-probs of a batch of at most 10,240 token rows, whose partials are merged by 8-row
blocks, against the same rows inside a larger batch (64-row blocks) and against float64."""
import pytest
import torch

import paper_2607_07508_amd as sao
from tests.gpu_common import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("H,V", [
    (8, 200),       # one vocabulary tile, one chunk per row
    (264, 8300),    # 33 tiles: one more than a row's threads; a ragged last chunk
    (1032, 70000),  # 274 tiles: a whole batch of loads and a remainder
])
def test_few_rows_against_many(H, V, dtype):
    say(f"few rows: H={H} V={V} {dtype}")
    gen = torch.Generator(device="cuda").manual_seed(H + V)
    h = torch.randn((32769, H), generator=gen, device="cuda").to(dtype)
    w = (0.1 * torch.randn((V, H), generator=gen, device="cuda")).to(dtype)
    y = torch.randint(0, V, (32769,), generator=gen, device="cuda", dtype=torch.int32)
    mask = (torch.rand(32769, generator=gen, device="cuda") < 0.7).to(torch.uint8)
    logp, lse = sao.token_logprob(h, w, y, mask)
    # fp32 sums in another order: 594-term sums of exponentials and H-term dot products
    tol = 4e-6
    for n in (1, 7, 8, 9, 300, 10240, 10241):
        lp, ls = sao.token_logprob(h[:n], w, y[:n], mask[:n])
        assert (lp - logp[:n]).abs().max() <= tol * (1 + logp[:n].abs().max())
        assert (ls - lse[:n]).abs().max() <= tol * (1 + lse[:n].abs().max())
        assert ((lp == 0) | (mask[:n] != 0)).all()
    z = h[:300].double() @ w.double().t()
    ref = torch.logsumexp(z, 1)
    on = mask[:300] != 0
    assert (lse[:300].double() - ref)[on].abs().max() <= tol * (1 + ref.abs().max())
    zy = z.gather(1, y[:300].long()[:, None])[:, 0] - ref
    assert (logp[:300].double() - zy)[on].abs().max() <= tol * (1 + zy.abs().max())
