"""The backward's dH product over token counts whose output tiles are cut into K
pieces in different ways (one token tile and many pieces, pieces shorter than a
piece length, several vocabulary blocks, no gradient row at all), against the
same products of the oracle's logit gradient."""
import numpy as np
import pytest
import torch

import oracle
import paper_2607_07508_amd as sao
from synth import bf16_round
from synth.rollouts import bf16_bits
from tests.gpu_common import check_grad, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,H,V,active", [
    (1, 8, 300, 1),          # one tile of one row; K shorter than the pieces allow
    (300, 64, 4100, 300),    # two token tiles, one column tile: the most pieces
    (2600, 520, 3000, 700),  # three of eleven token tiles hold rows; a ragged column tile
    (900, 2056, 900, 513),   # nine column tiles: two groups, the last one tile wide
    (700, 72, 70000, 90),    # two vocabulary blocks, the second shorter
    (500, 64, 700, 0),       # no row has a gradient
])
def test_dh_pieces(T, H, V, active):
    rng = np.random.default_rng(T + V)
    h = bf16_round(rng.standard_normal((T, H)).astype(np.float32))
    w = bf16_round((0.05 * rng.standard_normal((V, H))).astype(np.float32))
    y = rng.integers(0, V, T).astype(np.int32)
    g = np.zeros(T, dtype=np.float32)
    rows = np.sort(rng.choice(T, active, replace=False))
    g[rows] = rng.standard_normal(active) / T
    say(f"dH pieces: T={T} H={H} V={V} rows with a gradient={active}")
    dev = lambda x: torch.from_numpy(bf16_bits(x)).view(torch.bfloat16).cuda()  # noqa: E731
    _, lse = oracle.token_logprob(h, w, y, (g != 0).astype(np.uint8))
    args = (dev(h), dev(w), torch.from_numpy(y).cuda(), torch.from_numpy(lse.astype(np.float32)).cuda(),
            torch.from_numpy(g).cuda())
    dh, dw = sao.loss_backward(*args)
    dh2, dw2 = sao.loss_backward(*args)
    torch.cuda.synchronize()
    assert torch.equal(dh, dh2) and torch.equal(dw, dw2)
    ref_h, ref_w = oracle.loss_backward(h, w, y, lse, g)
    zero = np.nonzero(g == 0)[0]
    if active == 0:
        assert (dh == 0).all() and (dw == 0).all()
        return
    check_grad(dh.float().cpu().numpy(), ref_h, zero, "dh")
    check_grad(dw.cpu().numpy(), ref_w, None, "dw")
