"""fp32 head products on the bf16 matrix cores (three-term splits): error against
float64 at tile edges and K remainders, and operands that a bf16 split cannot
hold (infinities, magnitudes that round to a bf16 infinity), which the kernel
multiplies with fp32 MFMAs instead.

Bound on a logit: a tile's sum takes 6 ceil(K / 16) MFMAs, each rounding its
fp32 accumulator a few times (allowed here: 4) by 2^-24 of at most sum |a b|; the
product terms left out reach 2^-24 of |a b|, one more rounding.
"""
import numpy as np
import pytest
import torch

import paper_2607_07508_amd as sao
from tests.gpu_common import say

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24


def _inputs(T, H, V, seed):
    rng = np.random.default_rng(seed)
    h = rng.standard_normal((T, H)).astype(np.float32)
    w = (rng.standard_normal((V, H)) / np.sqrt(H)).astype(np.float32)
    y = rng.integers(0, V, T).astype(np.int32)
    g = (rng.standard_normal(T) / T).astype(np.float32)
    return h, w, y, g


def _gpu(*xs):
    return [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in xs]


@pytest.mark.parametrize("T,H,V", [(1, 8, 1), (257, 40, 255), (300, 72, 513), (129, 2048, 300), (513, 136, 1000)])
def test_f32_products_against_float64(T, H, V):
    h, w, y, g = _inputs(T, H, V, T + H + V)
    say(f"f32 split: T={T} H={H} V={V}")
    hd, wd, yd, gd = _gpu(h, w, y, g)
    logp, lse = sao.token_logprob(hd, wd, yd)
    dh, dw = sao.loss_backward(hd, wd, yd, lse, gd)
    torch.cuda.synchronize()
    h64, w64 = h.astype(np.float64), w.astype(np.float64)
    z = h64 @ w64.T
    m = z.max(1, keepdims=True)
    ref_lse = (m + np.log(np.exp(z - m).sum(1, keepdims=True)))[:, 0]
    ref_lp = z[np.arange(T), y] - ref_lse
    # logits: 4 roundings in each of 6 ceil(K / 16) MFMAs; the log-sum-exp averages them and adds about V / 64
    # roundings of its own sum plus the exp's and log's (a few ulp), and the float32 result rounds once
    dz_max = (24 * -(-H // 16) + 4) * EPS * (np.abs(h64) @ np.abs(w64).T).max(1)
    tol = 2 * dz_max + (V / 64 + 16) * EPS + 4 * EPS * np.abs(ref_lp)
    assert (np.abs(lse.cpu().numpy() - ref_lse) <= tol).all()
    assert (np.abs(logp.cpu().numpy() - ref_lp) <= tol).all()
    # the backward from the same lse and g
    p = np.exp(z - lse.cpu().numpy().astype(np.float64)[:, None])
    dz = -p * g[:, None].astype(np.float64)
    dz[np.arange(T), y] += g
    # dz carries its logit's error and a few roundings of exp; then a product over V (or T) as above
    dz_err = np.abs(g[:, None] * p) * (dz_max + 8 * EPS)[:, None] + 2 * EPS * np.abs(dz)
    tol_h = dz_err @ np.abs(w64) + (24 * -(-V // 16) + 4) * EPS * (np.abs(dz) @ np.abs(w64))
    tol_w = dz_err.T @ np.abs(h64) + (24 * -(-T // 16) + 4) * EPS * (np.abs(dz).T @ np.abs(h64))
    assert (np.abs(dh.cpu().numpy() - dz @ w64) <= tol_h + 1e-30).all()
    assert (np.abs(dw.cpu().numpy() - dz.T @ h64) <= tol_w + 1e-30).all()


def test_f32_operands_beyond_bf16():
    """-inf logits drop out of the log-sum-exp, products of huge and tiny values stay finite, and the rows and
    columns beside them are unaffected."""
    T, H, V = 300, 64, 600
    h, w, y, _ = _inputs(T, H, V, 5)
    h[:, 0] = 0.25 + np.abs(h[:, 0])
    w[17, 0] = -np.inf           # a vocabulary row that is masked out
    w[300, 1] = 3.4e38           # rounds to a bf16 infinity
    h[:, 1] *= 1e-38
    h[41, 1] = 0.0
    w[301] *= 1e-42              # subnormal
    y[y == 17] = 18
    hd, wd, yd = _gpu(h, w, y)
    logp, lse = sao.token_logprob(hd, wd, yd)
    torch.cuda.synchronize()
    h64, w64 = h.astype(np.float64), w.astype(np.float64)
    keep = np.arange(V) != 17
    z = h64 @ w64[keep].T
    m = z.max(1, keepdims=True)
    ref = (m + np.log(np.exp(z - m).sum(1, keepdims=True)))[:, 0]
    tol = 2 * (24 * -(-H // 16) + 4) * EPS * (np.abs(h64) @ np.abs(w64[keep]).T).max(1) + 64 * EPS
    assert (np.abs(lse.cpu().numpy() - ref) <= tol).all()
    lp = np.einsum("th,th->t", h64, w64[y]) - ref
    assert (np.abs(logp.cpu().numpy() - lp) <= tol + 4 * EPS * np.abs(lp)).all()
