"""The flat advantage scan (tiles of 2048 tokens whatever trajectories they hold)
around its edges: one tile and a few more, trajectories that end at, before and
after tile and thread boundaries, empty ones, a single one over hundreds of tiles,
and the switch to one workgroup per trajectory; and non-finite inputs, which stay
inside their trajectory."""
import numpy as np
import pytest
import torch

import oracle
import paper_2607_07508_amd as sao
from tests.gpu_common import TOL_ADV, say

pytestmark = pytest.mark.gpu


def _batch(lengths, seed):
    rng = np.random.default_rng(seed)
    cu = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    T = int(cu[-1])
    mask = (rng.random(T) < 0.6).astype(np.uint8)
    v = rng.normal(0.5, 0.2, T).astype(np.float32)
    r = rng.normal(0.0, 0.1, T).astype(np.float32)
    return v, r, mask, cu


def _run(v, r, mask, cu, gamma, lam, alpha):
    out = sao.advantage(*[torch.from_numpy(x).cuda() for x in (v, r, mask, cu)], gamma, lam, alpha)
    torch.cuda.synchronize()
    return [x.cpu().numpy() for x in out]


CASES = {
    "one token": [1],
    "one tile exactly": [2048],
    "tile and one": [2049],
    "ends on tile edges": [2048, 4096, 2048],
    "ends beside tile edges": [2047, 2, 2047, 4097, 1, 2046],
    "short in one tile": [3, 1, 0, 0, 8, 7, 9, 250, 0, 1],
    "empty at both ends": [0, 0, 5000, 0, 0, 1, 3000, 0],
    "many short": [int(x) for x in np.random.default_rng(3).integers(0, 40, 700)],
    "hundreds of tiles": [13, 700_001, 5],
    "brief, one long": [30] * 300 + [20_000] + [17] * 300,  # mean below 128: one workgroup per trajectory
    "brief": [128] * 256,                                   # on the rule's edge
    "not brief": [129] * 250,
    "more than 1024 brief": [3, 0, 11, 1] * 300,
    "per trajectory": [4097] * 1030,  # over the token and trajectory limits of the flat scan
}


@pytest.mark.parametrize("name", CASES)
@pytest.mark.parametrize("gamma,lam,alpha", [(1.0, 1.0, 1.5), (0.97, 0.9, 0.0), (0.0, 0.5, 0.0)])
def test_flat_scan(name, gamma, lam, alpha):
    v, r, mask, cu = _batch(CASES[name], len(name))
    if len(mask) > 1_000_000 and (gamma, alpha) != (1.0, 1.5):
        pytest.skip("one setting is enough at this size")
    say(f"flat scan: {name}, T={len(mask)} gamma={gamma}")
    adv, ret, n = _run(v, r, mask, cu, gamma, lam, alpha)
    ra, rr, N = oracle.advantage(v, r, mask, cu, gamma, lam, alpha)
    assert int(n[0]) == N
    assert (np.abs(adv - ra) <= TOL_ADV * np.maximum(1.0, np.abs(ra))).all()
    assert (np.abs(ret - rr) <= TOL_ADV * np.maximum(1.0, np.abs(rr))).all()


def _run_small_workspace(v, r, mask, cu, gamma, lam, alpha, off=0):
    """sao_advantage with the 768 bytes that every T takes (one workgroup per trajectory), the arrays `off`
    elements into their storage. Also that nothing past those bytes is written."""
    dev = []
    for x in (v, r, mask):
        t = torch.zeros(len(x) + off, dtype=torch.from_numpy(x[:0]).dtype, device="cuda")
        t[off:] = torch.from_numpy(x).cuda()
        dev.append(t[off:])
    cud = torch.from_numpy(cu).cuda()
    out = [torch.full((len(v) + off,), 7.0, device="cuda")[off:] for _ in range(2)]
    n = torch.full((1,), -1, dtype=torch.int64, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.full((4096,), 0x5a, dtype=torch.uint8, device="cuda")
    code = sao.lib().sao_advantage(*[t.data_ptr() for t in dev], cud.data_ptr(), len(cu) - 1, len(v), gamma, lam, alpha,
                                   out[0].data_ptr(), out[1].data_ptr(), n.data_ptr(), status.data_ptr(),
                                   ws.data_ptr(), 768, torch.cuda.current_stream().cuda_stream)
    assert code == 0, sao.lib().sao_last_error_message()
    assert (ws[768:] == 0x5a).all()
    return [x.cpu().numpy() for x in (*out, n)] + [int(status)]


@pytest.mark.parametrize("name", [k for k in CASES if k not in ("per trajectory",)])
@pytest.mark.parametrize("off", [0, 1])
def test_small_workspace(name, off):
    v, r, mask, cu = _batch(CASES[name], len(name))
    say(f"per-trajectory scan: {name}, T={len(mask)} offset={off}")
    adv, ret, n, status = _run_small_workspace(v, r, mask, cu, 0.97, 0.9, 1.5, off)
    ra, rr, N = oracle.advantage(v, r, mask, cu, 0.97, 0.9, 1.5)
    assert int(n[0]) == N and status == 0
    assert (np.abs(adv - ra) <= TOL_ADV * np.maximum(1.0, np.abs(ra))).all()
    assert (np.abs(ret - rr) <= TOL_ADV * np.maximum(1.0, np.abs(rr))).all()
    for i, x in ((len(cu) - 1, len(v) + 5), (0, 1)):
        bad = cu.copy()
        bad[i] = x
        adv, ret, n, status = _run_small_workspace(v, r, mask, bad, 0.97, 0.9, 1.5, off)
        assert np.isnan(adv).all() and np.isnan(ret).all() and int(n[0]) == N and status == 2


@pytest.mark.parametrize("off", [0, 1])
def test_per_trajectory_rule(off):
    """Over both limits of the flat scan with the whole workspace: unaligned arrays, then malformed segments."""
    v, r, mask, cu = _batch([4097] * 300, 6)
    say(f"per-trajectory scan: T={len(v)} B=300 offset={off}")
    pad = lambda x: torch.from_numpy(np.concatenate([x[:off], x])).cuda()[off:]  # noqa: E731
    args = [pad(v), pad(r), pad(mask)]
    adv, ret, n = sao.advantage(*args, torch.from_numpy(cu).cuda(), 0.97, 0.9, 1.5)
    ra, rr, N = oracle.advantage(v, r, mask, cu, 0.97, 0.9, 1.5)
    assert int(n) == N
    assert (np.abs(adv.cpu().numpy() - ra) <= TOL_ADV * np.maximum(1.0, np.abs(ra))).all()
    assert (np.abs(ret.cpu().numpy() - rr) <= TOL_ADV * np.maximum(1.0, np.abs(rr))).all()
    bad = cu.copy()
    bad[150] = bad[149] - 1
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    adv, ret, n = sao.advantage(*args, torch.from_numpy(bad).cuda(), 0.97, 0.9, 1.5, status=status)
    assert adv.isnan().all() and ret.isnan().all() and int(n) == N and int(status) == 2


@pytest.mark.parametrize("lengths", [[500, 20, 600], [3000, 20, 5000, 2000]])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_nonfinite_stays_in_its_trajectory(lengths, bad):
    v, r, mask, cu = _batch(lengths, 9)
    hit = [2] if len(lengths) == 3 else [1, 3]
    for b in hit:
        v[cu[b] + 7] = bad
        r[cu[b] + 9] = bad
        mask[cu[b] + 7] = 1
    say(f"flat scan, {bad} in trajectories {hit} of {lengths}")
    adv, ret, _ = _run(v, r, mask, cu, 1.0, 1.0, 1.5)
    for b in range(len(lengths)):
        s, e = cu[b], cu[b + 1]
        if b in hit:
            assert not np.isfinite(adv[s + 7])
            continue
        ra, rr, _ = oracle.advantage(v[s:e], r[s:e], mask[s:e], np.array([0, e - s], np.int32), 1.0, 1.0, 1.5)
        assert (np.abs(adv[s:e] - ra) <= TOL_ADV * np.maximum(1.0, np.abs(ra))).all()
        assert (np.abs(ret[s:e] - rr) <= TOL_ADV * np.maximum(1.0, np.abs(rr))).all()


@pytest.mark.parametrize("lengths", [
    [1] + [0] * 200_000 + [4096],                    # between two tokens of one thread
    [2045, 0, 0, 5] + [0] * 70_000 + [1, 2000, 0],   # across a tile edge
    [0] * 100_000 + [300, 0, 0, 1, 1],               # before the first token of a one-tile batch
])
def test_many_empty_trajectories(lengths):
    """Empty trajectories change nothing and cost a search, not a walk: well under 5 ms a call (tens of
    milliseconds when a thread steps over them one by one)."""
    v, r, mask, cu = _batch(lengths, 4)
    full = [n for n in lengths if n]
    say(f"flat scan: {len(lengths) - len(full)} empty trajectories among {len(full)}")
    a = _run(v, r, mask, cu, 1.0, 0.9, 1.5)
    b = _run(v, r, mask, np.concatenate([[0], np.cumsum(full)]).astype(np.int32), 1.0, 0.9, 1.5)
    assert all(np.array_equal(x, y) for x, y in zip(a, b))
    args = [torch.from_numpy(x).cuda() for x in (v, r, mask, cu)]
    times = []
    for _ in range(5):
        start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        sao.advantage(*args, 1.0, 0.9, 1.5)
        stop.record()
        stop.synchronize()
        times.append(start.elapsed_time(stop))
    say(f"median {sorted(times)[2]:.3f} ms")
    assert sorted(times)[2] < 5.0
