"""Step-level and group advantages on both sides of their launch rules (256 trajectories and a
mean length of 1536 tokens for the step-level workgroups, 512 trajectories for the fused group
launches), against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2607_07508_amd as sao
from tests.gpu_common import TOL_ADV, say

pytestmark = pytest.mark.gpu


def _batch(B, T, seed):
    rng = np.random.default_rng(seed)
    cuts = np.sort(rng.integers(0, T + 1, B - 1))  # some trajectories empty
    cu = np.concatenate([[0], cuts, [T]]).astype(np.int32)
    mask = np.zeros(T, dtype=np.uint8)
    pos = 0
    while pos < T:
        n = int(rng.integers(1, 40))
        mask[pos:pos + n] = rng.random() < 0.6
        pos += n
    return rng.normal(0.5, 0.2, T).astype(np.float32), rng.normal(0.0, 0.5, T).astype(np.float32), mask, cu


def _t(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("B,T", [(1, 8191), (1, 8193), (2, 50_000), (256, 30_000), (257, 30_000), (1, 1535), (1, 1536),
                                 (40, 61_439), (40, 61_440)])
def test_step_forms(B, T):
    say(f"step forms: B={B} T={T}")
    v, r, m, cu = _batch(B, T, B + T)
    adv, ret, last, n = sao.step_advantage(_t(v), _t(r), _t(m), _t(cu), 0.99, 0.9, 1.5)
    ra, rg, rl, rn = oracle.step_advantage(v, r, m, cu, 0.99, 0.9, 1.5, "average")
    assert int(n) == rn == int(m.sum())
    assert np.array_equal(last.cpu().numpy(), rl)
    for x, y in ((adv, ra), (ret, rg)):
        assert (np.abs(x.cpu().numpy() - y) <= TOL_ADV * np.maximum(1.0, np.abs(y))).all()
    assert sao.step_advantage(_t(v), _t(r), _t(m), _t(cu), want_count=False)[3] is None


@pytest.mark.parametrize("B,G", [(4, 4), (1024, 8), (1028, 4), (512, 512), (512, 64), (520, 520), (513, 27)])
def test_group_forms(B, G):
    T = 30_000
    say(f"group forms: B={B}")
    v, r, m, cu = _batch(B, T, B)
    adv, traj, rew, n = sao.group_advantage(_t(r), _t(m), _t(cu), G, 1e-6)
    R = np.array([r[a:b].astype(np.float64).sum() for a, b in zip(cu[:-1], cu[1:])])
    g = R.reshape(-1, G)
    A = ((g - g.mean(1, keepdims=True)) / np.sqrt(g.var(1, keepdims=True) + 1e-6)).reshape(-1)
    assert int(n) == int(m.sum())
    assert np.abs(rew.cpu().numpy() - R).max() <= 1e-12 * max(1.0, np.abs(R).max())
    assert np.abs(traj.cpu().numpy() - A).max() <= 1e-9
    want = np.where(m != 0, np.repeat(A, np.diff(cu)), 0.0).astype(np.float32)
    assert np.abs(adv.cpu().numpy() - want).max() <= 1e-6
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    bad = cu.copy()
    bad[1] = T + 7
    adv, traj, rew, n = sao.group_advantage(_t(r), _t(m), _t(bad), G, 1e-6, status=status)
    assert adv.isnan().all() and traj.isnan().all() and rew.isnan().all() and int(n) == int(m.sum())
    assert int(status) == 2
    assert sao.group_advantage(_t(r), _t(m), _t(cu), G, 1e-6, want_count=False)[3] is None


@pytest.mark.parametrize("B,T", [(3, 2000), (16, 9000), (1024, 9000), (1025, 9000), (3000, 9000)])
def test_scan_finds_its_segments(B, T):
    """The flat scan's search for a tile's trajectories, with few and with many of them and
    empty ones among them; then with malformed segments."""
    say(f"scan segments: B={B} T={T}")
    v, r, m, cu = _batch(B, T, B)
    adv, ret, n = sao.advantage(_t(v), _t(r), _t(m), _t(cu), 0.99, 0.9, 1.5)
    ra, rr, rn = oracle.advantage(v, r, m, cu, 0.99, 0.9, 1.5)
    assert int(n) == rn
    for x, y in ((adv, ra), (ret, rr)):
        assert (np.abs(x.cpu().numpy() - y) <= TOL_ADV * np.maximum(1.0, np.abs(y))).all()
    for i, x in ((1, T + 9), (B // 2, -5), (0, 3)):
        bad = cu.copy()
        bad[i] = x
        status = torch.zeros(1, dtype=torch.int32, device="cuda")
        adv, ret, n = sao.advantage(_t(v), _t(r), _t(m), _t(bad), status=status)
        assert adv.isnan().all() and ret.isnan().all() and int(n) == rn and int(status) == 2
