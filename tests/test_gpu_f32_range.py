"""fp32 head products over the whole range of fp32 operands, against float64: magnitudes down to
subnormals and up to fp32's largest in the forward and in both gradients, on both sides of what
the three-term split holds (operands below 2^104, sums below 2^80; the kernel multiplies a tile
beyond them with fp32 MFMAs), and the bias of long sums.

Bounds as for ordinary operands: each of the 6 ceil(K / 16) MFMAs of a sum rounds twice (4 allowed)
by 2^-24 of at most sum |a b|; the terms that the split leaves out reach 2^-24 of |a b|, one more.
"""
import numpy as np
import pytest
import torch

import paper_2607_07508_amd as sao
from tests.gpu_common import say

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24
TINY = 2.0 ** -149


def _inputs(T, H, V, seed):
    rng = np.random.default_rng(seed)
    h = rng.standard_normal((T, H)).astype(np.float32)
    w = (rng.standard_normal((V, H)) / np.sqrt(H)).astype(np.float32)
    y = rng.integers(0, V, T).astype(np.int32)
    g = (rng.standard_normal(T) / T).astype(np.float32)
    return h, w, y, g


def _gpu(*xs):
    return [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in xs]


def _steps(k):
    return 24 * -(-k // 16) + 4


def _check(h, w, y, g):
    """Forward and backward against float64, element by element."""
    (T, H), V = h.shape, w.shape[0]
    hd, wd, yd, gd = _gpu(h, w, y, g)
    logp, lse = sao.token_logprob(hd, wd, yd)
    dh, dw = sao.loss_backward(hd, wd, yd, lse, gd)
    torch.cuda.synchronize()
    h, w, g = h.astype(np.float64), w.astype(np.float64), g.astype(np.float64)
    z = h @ w.T
    m = z.max(1, keepdims=True)
    ref_lse = (m + np.log(np.exp(z - m).sum(1, keepdims=True)))[:, 0]
    ref_lp = z[np.arange(T), y] - ref_lse
    z_err = (_steps(H) * EPS * (np.abs(h) @ np.abs(w).T)).max(1)
    tol = 2 * z_err + (V / 64 + 16) * EPS + 4 * EPS * np.abs(ref_lp)
    assert (np.abs(lse.cpu().numpy() - ref_lse) <= tol).all()
    assert (np.abs(logp.cpu().numpy() - ref_lp) <= tol).all()
    p = np.exp(z - lse.cpu().numpy().astype(np.float64)[:, None])
    dz = -p * g[:, None]
    dz[np.arange(T), y] += g
    # the logit's error, a few roundings of exp, and dz's own rounding (absolute where it is subnormal)
    dz_err = np.abs(g[:, None] * p) * (z_err + 8 * EPS)[:, None] + 2 * EPS * np.abs(dz) + 2 * TINY
    tol_h = dz_err @ np.abs(w) + _steps(V) * (EPS * (np.abs(dz) @ np.abs(w)) + TINY)
    tol_w = dz_err.T @ np.abs(h) + _steps(T) * (EPS * (np.abs(dz).T @ np.abs(h)) + TINY)
    assert (np.abs(dh.cpu().numpy() - dz @ w) <= tol_h).all()
    assert (np.abs(dw.cpu().numpy() - dz.T @ h) <= tol_w).all()


# factor of one column of the hidden states, and the weights' value there
PAIRS = [
    (1e-38, 3.4e38),       # a weight that rounds to a bf16 infinity
    (1e-38, 3.3e38),       # finite in bf16, beyond the split's 2^104; half the hidden values subnormal
    (1e-32, 2.0 ** 104),   # on the limit
    (1e-32, 2.0 ** 103),   # below it: partners that three unscaled bf16 terms would hold in part
    (1e-36, 1e25),
    (1e-44, 1e30),         # subnormals
    (1e-20, 1e20),
    (1.0, 1e-38),
]


@pytest.mark.parametrize("small,large", PAIRS)
@pytest.mark.parametrize("swap", [False, True])
def test_wide_operands(small, large, swap):
    """Tiny times huge gives ordinary logits; `swap` puts the huge values in the hidden states."""
    T, H, V = 300, 72, 4100  # two token tiles, ragged sides, several K pieces of dH
    say(f"f32 range: {small:g} x {large:g} swap={swap}")
    h, w, y, g = _inputs(T, H, V, 11)
    a, b = (w, h) if swap else (h, w)
    a[:, 1] = (a[:, 1].astype(np.float64) * small).astype(np.float32)
    b[::7, 1] = large
    b[3::7, 1] = -large
    b[1::7, 1] = 0.0
    _check(h, w, y, g)


@pytest.mark.parametrize("scale", [1e-20, 1e-30, 1e-34, 1e-37])
def test_tiny_gradients(scale):
    """The relative accuracy of gradients does not depend on the size of g."""
    say(f"f32 range: g times {scale:g}")
    h, w, y, g = _inputs(257, 72, 1000, 12)
    _check(h, w, y, (g * scale).astype(np.float32))


def test_nonfinite_operands_in_later_tiles():
    """A workgroup that takes one tile after another: -inf vocabulary rows drop out, a NaN and an infinite
    hidden row give NaN, everything else is as without them."""
    T, H, V = 300, 64, 90_000  # 704 tiles for 256 workgroups
    say("f32 range: non-finite operands in streamed tiles")
    h, w, y, _ = _inputs(T, H, V, 13)
    h[:, 0] = 0.25 + np.abs(h[:, 0])
    out = np.arange(1000, V, 9973)
    y[np.isin(y, out)] = 0
    hd, wd, yd = _gpu(h, w, y)
    wd[torch.from_numpy(out).cuda(), 0] = -float("inf")
    logp, lse = sao.token_logprob(hd, wd, yd)
    bad = hd.clone()
    bad[41] = float("nan")
    bad[270, 5] = float("inf")
    logp2, lse2 = sao.token_logprob(bad, wd, yd)
    torch.cuda.synchronize()
    z = hd.double() @ wd.double().t()
    ref = torch.logsumexp(z, 1).cpu().numpy()
    lp = z.gather(1, yd.long()[:, None])[:, 0].cpu().numpy() - ref
    z_err = _steps(H) * EPS * (np.abs(h).astype(np.float64) @ np.abs(w).astype(np.float64).max(0))
    tol = 2 * z_err + (V / 64 + 16) * EPS + 4 * EPS * np.abs(lp)
    assert (np.abs(lse.cpu().numpy() - ref) <= tol).all()
    assert (np.abs(logp.cpu().numpy() - lp) <= tol).all()
    keep = torch.ones(T, dtype=torch.bool, device="cuda")
    keep[41] = keep[270] = False
    assert not lse2[~keep].isfinite().any()
    # other rows of the same tiles come from fp32 MFMAs there: equal within the same bound
    assert (np.abs((lse2 - lse)[keep].cpu().numpy()) <= 2 * tol[keep.cpu().numpy()]).all()
    assert (np.abs((logp2 - logp)[keep].cpu().numpy()) <= 2 * tol[keep.cpu().numpy()]).all()


@pytest.mark.parametrize("H", [2048, 6144])
def test_long_sums_have_no_bias(H):
    """The mean error of logits (log Z over a vocabulary of one) of unit scale. The matrix cores floor what they
    align, each of a logit's 12 H / 16 sums by up to about 2^-9 of its last place, one way: -1.6e-7 and -8.4e-7 if
    they added up. A fifth of that is allowed, and 4 standard errors of the mean."""
    T, rows = 512, 64
    say(f"f32 range: bias at H={H}")
    gen = torch.Generator(device="cuda").manual_seed(H)
    h = torch.randn((T, H), generator=gen, device="cuda")
    w = 0.02 * torch.randn((rows, H), generator=gen, device="cuda")
    y = torch.zeros(T, dtype=torch.int32, device="cuda")
    z = torch.stack([sao.token_logprob(h, w[v:v + 1], y)[1] for v in range(rows)])
    err = (z.double() - w.double() @ h.double().t()).cpu().numpy()
    say(f"mean {err.mean():+.2e}, rms {err.std():.2e}")
    shift = 12 * H / 16 * 2.0 ** -9 * EPS * 0.02 * np.sqrt(H)
    assert abs(err.mean()) <= shift / 5 + 4 * err.std() / np.sqrt(err.size)
