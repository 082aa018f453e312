// Skip-observation token-level GAE (Sec. 3.2, Eq. 4-5) as a segmented reverse scan.
//
// Walking right to left, the state after a token is
//   s = (Vn, R, A, G): value of the next action, reward pending since the next
// action, and that action's advantage and return. Token t maps the state that
// enters from its right to the state that leaves to its left:
//   action (value v, reward r):  Vn' = v, R' = 0,
//                                A'  = (r + R) + gamma Vn - v + gamma lambda_b A,
//                                G'  = (r + R) + gamma G            (and A', G' are its outputs)
//   observation (reward r):      R' = R + r, everything else unchanged
// starting from s = 0 after the last token (no bootstrap after the last action;
// rewards before the first action leave through the left end and are dropped).
// Every such map, and every composition of them, has the form
//   Vn' = z Vn + cV,  R' = z R + cR,
//   A'  = cA + X (R + gamma Vn) + (kappa X + z) A,   kappa = gamma lambda_b,
//   G'  = cG + Y R + (gamma Y + z) G,
// where z = 1 for a run of observations only (then cV = cA = cG = X = Y = 0) and
// z = 0 once the run holds an action (then X = kappa^(n-1) and Y = gamma^(n-1) for
// its n actions). So a thread summarises its contiguous tokens by 7 numbers, the
// block scans the summaries (DPP lane moves inside each wave, then across waves
// through LDS), and each thread replays its tokens from the exact state that
// enters it. Arithmetic is float64. Tiles of 2048 tokens aligned to the global
// index give every thread 8 tokens that it reads and writes with 16-byte vector
// accesses.
#include "common.hpp"
#include "launch.hpp"
#include "layout.hpp"
#include "segments.hpp"

#include "../../include/sao.h"

namespace sao {

struct Aff {
  double z, cV, cR, X, cA, Y, cG;
};

__device__ __forceinline__ Aff aff_identity() { return Aff{1.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0}; }

// (F o G)(s) = F(G(s)). The coefficients of A and G in F are kappa F.X + F.z and
// gamma F.Y + F.z; products of them with G's come out in the same form.
__device__ __forceinline__ Aff compose(const Aff& F, const Aff& G, double gamma, double kappa) {
  const double fa = fma(kappa, F.X, F.z), fg = fma(gamma, F.Y, F.z);
  Aff r;
  r.z = F.z * G.z;
  r.cV = fma(F.z, G.cV, F.cV);
  r.cR = fma(F.z, G.cR, F.cR);
  r.X = fma(F.X, G.z, fa * G.X);
  r.cA = fma(F.X, fma(gamma, G.cV, G.cR), fma(fa, G.cA, F.cA));
  r.Y = fma(F.Y, G.z, fg * G.Y);
  r.cG = fma(F.Y, G.cR, fma(fg, G.cG, F.cG));
  return r;
}

// M o F for the map M of one token, F covering the tokens to its right
// (compose() with M's constants substituted: an action is z = 0, cV = v, cR = 0,
// X = Y = 1, cA = r - v, cG = r; an observation is the identity plus cR = r).
__device__ __forceinline__ void push_action(Aff& F, double v, double r, double gamma, double kappa) {
  const Aff G = F;
  F.z = 0.0;
  F.cV = v;
  F.cR = 0.0;
  F.X = fma(kappa, G.X, G.z);
  F.cA = fma(kappa, G.cA, fma(gamma, G.cV, G.cR + (r - v)));
  F.Y = fma(gamma, G.Y, G.z);
  F.cG = fma(gamma, G.cG, G.cR + r);
}
__device__ __forceinline__ void push_observation(Aff& F, double r) { F.cR += r; }

// A double moved across lanes by DPP (CTRL, ROW_MASK); lanes without a source keep `old`.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_f64(double old, double x) {
  const uint2 o = __builtin_bit_cast(uint2, old), v = __builtin_bit_cast(uint2, x);
  const int lo = __builtin_amdgcn_update_dpp(static_cast<int>(o.x), static_cast<int>(v.x), CTRL, ROW_MASK, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(static_cast<int>(o.y), static_cast<int>(v.y), CTRL, ROW_MASK, 0xf, false);
  return __builtin_bit_cast(double, make_uint2(static_cast<uint32_t>(lo), static_cast<uint32_t>(hi)));
}
// The map of another lane (identity where there is none).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ Aff dpp_aff(const Aff& x) {
  Aff o;
  o.z = dpp_f64<CTRL, ROW_MASK>(1.0, x.z);
  o.cV = dpp_f64<CTRL, ROW_MASK>(0.0, x.cV);
  o.cR = dpp_f64<CTRL, ROW_MASK>(0.0, x.cR);
  o.X = dpp_f64<CTRL, ROW_MASK>(0.0, x.X);
  o.cA = dpp_f64<CTRL, ROW_MASK>(0.0, x.cA);
  o.Y = dpp_f64<CTRL, ROW_MASK>(0.0, x.Y);
  o.cG = dpp_f64<CTRL, ROW_MASK>(0.0, x.cG);
  return o;
}

// Inclusive scan over the wave in lane order, S_l = F_l o F_{l-1} o ... o F_0:
// shifts by 1, 2, 4, 8 inside each row of 16 lanes (row_shr), then the last lane
// of row 0 into row 1 and of row 2 into row 3 (row_bcast:15), then lane 31 into
// rows 2 and 3 (row_bcast:31). DPP moves are VALU operations, so no step waits
// on the LDS crossbar.
__device__ __forceinline__ Aff wave_scan(Aff S, double gamma, double kappa) {
  S = compose(S, dpp_aff<0x111, 0xf>(S), gamma, kappa);
  S = compose(S, dpp_aff<0x112, 0xf>(S), gamma, kappa);
  S = compose(S, dpp_aff<0x114, 0xf>(S), gamma, kappa);
  S = compose(S, dpp_aff<0x118, 0xf>(S), gamma, kappa);
  S = compose(S, dpp_aff<0x142, 0xa>(S), gamma, kappa);
  S = compose(S, dpp_aff<0x143, 0xc>(S), gamma, kappa);
  return S;
}

constexpr int kScanThreads = 256;
constexpr int kScanPer = 8;                               // tokens per thread per tile
static_assert(kScanPer % 4 == 0, "whole blocks are read as 16-byte vectors");
constexpr int kScanTile = kScanThreads * kScanPer;        // tokens per tile
static_assert(kScanTile == kScanTileTokens, "the layout counts tiles");

// State after applying map M to (Vn, R, A, G).
struct St {
  double Vn, R, A, G;
};
__device__ __forceinline__ St apply(const Aff& M, const St& s, double gamma, double kappa) {
  St o;
  o.Vn = fma(M.z, s.Vn, M.cV);
  o.R = fma(M.z, s.R, M.cR);
  o.A = fma(M.X, fma(gamma, s.Vn, s.R), fma(fma(kappa, M.X, M.z), s.A, M.cA));
  o.G = fma(M.Y, s.R, fma(fma(gamma, M.Y, M.z), s.G, M.cG));
  return o;
}

// One workgroup per trajectory. The trajectory is walked right to left in tiles
// of kScanTile tokens aligned to the global token index (so that each thread's
// kScanPer tokens are one aligned vector load per array); the state leaving a
// tile on the left enters the next tile from the right. Inside a tile each
// thread composes the maps of its tokens, the block scans the compositions,
// and each thread replays its tokens from the exact entering state.
__global__ __launch_bounds__(kScanThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_advantage(
    const float* values, const float* rewards, const uint8_t* mask, const int32_t* cu, int32_t B,
    int64_t T, double gamma, double lam, double alpha, float* adv, float* ret, int64_t* slots,
    const int32_t* bad, bool vec_ok) {
  __shared__ Aff s_agg[2][kScanThreads / 64];  // alternate tiles use alternate halves
  __shared__ int64_t s_cnt[kScanThreads / 64];
  // The state entering the next tile from the right, double-buffered so that a
  // tile's writer never waits for the previous tile's readers.
  __shared__ St s_carry[2];
  // Each thread's values and rewards wait here, in its own slots, while the block
  // scans: holding them in registers instead would cost a wave per SIMD.
  __shared__ f32x4_t s_in[2 * kScanPer / 4][kScanThreads];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b = blockIdx.x;
  if (*bad) {
    malformed_slice<kScanThreads, kCountSlots>(mask, B, T, adv, ret, nullptr, slots);
    return;
  }
  const int64_t s = cu[b], e = cu[b + 1];
  const int64_t L = e - s;
  if (L <= 0) return;
  double lam_b = lam;
  if (alpha > 0.0) {
    lam_b = 1.0 - 1.0 / (alpha * static_cast<double>(L));
    if (lam_b < 0.0) lam_b = 0.0;
  }
  const double kappa = gamma * lam_b;
  const int64_t first = s / kScanTile * kScanTile;           // aligned tile containing s
  int64_t total = 0;
  if (tid == 0) s_carry[0] = St{0.0, 0.0, 0.0, 0.0};         // nothing after the last token
  int buf = 0;
  // Thread i takes block 255 - i of each tile, so lane order runs right to left
  // and the reverse scan over tokens is a forward scan over lanes. Whole blocks
  // inside [s, e) use vector access (when the array bases allow it).
  for (int64_t t0 = (e - 1) / kScanTile * kScanTile; t0 >= first; t0 -= kScanTile) {
    const int64_t c0 = t0 + static_cast<int64_t>(kScanThreads - 1 - tid) * kScanPer;
    const bool full = vec_ok && c0 >= s && c0 + kScanPer <= e;
    float v[kScanPer], r[kScanPer];
    bool act[kScanPer];
    if (full) {
      const f32x4_t* pv = reinterpret_cast<const f32x4_t*>(values + c0);
      const f32x4_t* pr = reinterpret_cast<const f32x4_t*>(rewards + c0);
      const uint32_t* pm = reinterpret_cast<const uint32_t*>(mask + c0);
#pragma unroll
      for (int q = 0; q < kScanPer / 4; ++q) {
        const f32x4_t vq = pv[q], rq = pr[q];
        const uint32_t mq = pm[q];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          v[4 * q + j] = vq[j];
          r[4 * q + j] = rq[j];
          act[4 * q + j] = ((mq >> (8 * j)) & 0xffu) != 0;
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < kScanPer; ++j) {
        const int64_t t = c0 + j;
        const bool in = t >= s && t < e;
        v[j] = in ? values[t] : 0.0f;
        r[j] = in ? rewards[t] : 0.0f;
        act[j] = in && mask[t] != 0;
      }
    }
#pragma unroll
    for (int q = 0; q < kScanPer / 4; ++q) {
      s_in[q][tid] = f32x4_t{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
      s_in[kScanPer / 4 + q][tid] = f32x4_t{r[4 * q], r[4 * q + 1], r[4 * q + 2], r[4 * q + 3]};
    }
    // Pass 1: this thread's tokens as one map (tokens outside [s, e) are identities).
    Aff F = aff_identity();
    int64_t cnt = 0;
#pragma unroll
    for (int j = kScanPer - 1; j >= 0; --j) {
      const bool in = full || (c0 + j >= s && c0 + j < e);
      if (!in) continue;
      if (act[j]) {
        ++cnt;
        push_action(F, v[j], r[j], gamma, kappa);
      } else {
        push_observation(F, r[j]);
      }
    }
    total += cnt;
    const Aff S = wave_scan(F, gamma, kappa);                     // this lane and the lanes to its right
    const Aff E = dpp_aff<0x138, 0xf>(S);          // wave_shr:1, the lanes to its right only
    // One barrier per tile: the half of s_agg written here was last read two tiles
    // ago, and the carry written at the end of the previous tile is published by it.
    if (lane == 63) s_agg[buf][wave] = S;
    __syncthreads();
    // State entering this wave: the carry through the waves to its right (lower waves).
    St sw = s_carry[buf];
    for (int w = 0; w < wave; ++w) sw = apply(s_agg[buf][w], sw, gamma, kappa);
    St st = apply(E, sw, gamma, kappa);
    // Pass 2: replay the tokens from that state and write the outputs.
#pragma unroll
    for (int q = 0; q < kScanPer / 4; ++q) {
      const f32x4_t vq = s_in[q][tid], rq = s_in[kScanPer / 4 + q][tid];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        v[4 * q + j] = vq[j];
        r[4 * q + j] = rq[j];
      }
    }
    float oa[kScanPer], og[kScanPer];
#pragma unroll
    for (int j = kScanPer - 1; j >= 0; --j) {
      oa[j] = 0.0f;
      og[j] = 0.0f;
      const bool in = full || (c0 + j >= s && c0 + j < e);
      if (!in) continue;
      const double rr = r[j];
      if (act[j]) {
        const double vv = v[j];
        const double rt = rr + st.R;
        const double An = fma(kappa, st.A, fma(gamma, st.Vn, rt - vv));
        const double Gn = fma(gamma, st.G, rt);
        oa[j] = static_cast<float>(An);
        og[j] = static_cast<float>(Gn);
        st.Vn = vv;
        st.R = 0.0;
        st.A = An;
        st.G = Gn;
      } else {
        st.R += rr;
      }
    }
    if (full) {
      f32x4_t* qa = reinterpret_cast<f32x4_t*>(adv + c0);
      f32x4_t* qg = reinterpret_cast<f32x4_t*>(ret + c0);
#pragma unroll
      for (int q = 0; q < kScanPer / 4; ++q) {
        qa[q] = f32x4_t{oa[4 * q], oa[4 * q + 1], oa[4 * q + 2], oa[4 * q + 3]};
        qg[q] = f32x4_t{og[4 * q], og[4 * q + 1], og[4 * q + 2], og[4 * q + 3]};
      }
    } else {
#pragma unroll
      for (int j = 0; j < kScanPer; ++j) {
        const int64_t t = c0 + j;
        if (t >= s && t < e) {
          adv[t] = oa[j];
          ret[t] = og[j];
        }
      }
    }
    // The state leaving this tile on the left (the last thread's final state) enters
    // the next tile; the other buffer's readers finished before this tile's barrier.
    buf ^= 1;
    if (tid == kScanThreads - 1) s_carry[buf] = st;
  }
  const int64_t wcnt = wave_sum(total);
  __syncthreads();
  if (lane == 0) s_cnt[wave] = wcnt;
  __syncthreads();
  if (tid == 0) {
    int64_t tot = 0;
    for (int w = 0; w < kScanThreads / 64; ++w) tot += s_cnt[w];
    add_count<kCountSlots>(slots, tot);
  }
}

// ------------------------------------------------------------------------- //
// The flat scan: one workgroup per tile of kScanTile tokens, whatever trajectories
// the tile holds
// ------------------------------------------------------------------------- //
// A trajectory's last token forgets the state entering from its right: a map that
// covers such a token is marked `cut`, has no coefficients (z = X = Y = 0), and its
// composition with anything on its right is itself, selected rather than multiplied,
// so that NaN or infinite inputs stay inside their trajectory. A map that is not cut
// lies in one trajectory, whose kappa the composition takes. Tile maps of a first
// launch (k_scan_tiles) go to the workspace, 64 bytes each; in the second
// (k_scan_flat) every tile composes the maps to its right, up to the end of its last
// token's trajectory, and replays its tokens. A batch of one tile needs no first
// launch, and the same workgroup checks the segments and counts the mask.
//
// Bound by launches and one tile's latency (load, compose, block scan, replay, about
// 5 us) instead of by the longest trajectory's chain of tiles at 2.6 us each.
struct CutMap {
  Aff f;
  int cut;
};
__device__ __forceinline__ CutMap cut_identity() { return CutMap{aff_identity(), 0}; }
__device__ __forceinline__ CutMap compose_cut(const CutMap& F, const CutMap& G, double gamma, double kappa) {
  const Aff c = compose(F.f, G.f, gamma, kappa);
  CutMap r;
  r.f.z = F.cut ? F.f.z : c.z;
  r.f.cV = F.cut ? F.f.cV : c.cV;
  r.f.cR = F.cut ? F.f.cR : c.cR;
  r.f.X = F.cut ? F.f.X : c.X;
  r.f.cA = F.cut ? F.f.cA : c.cA;
  r.f.Y = F.cut ? F.f.Y : c.Y;
  r.f.cG = F.cut ? F.f.cG : c.cG;
  r.cut = F.cut | G.cut;
  return r;
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ CutMap dpp_cut(const CutMap& x) {
  return CutMap{dpp_aff<CTRL, ROW_MASK>(x.f), __builtin_amdgcn_update_dpp(0, x.cut, CTRL, ROW_MASK, 0xf, false)};
}
__device__ __forceinline__ CutMap wave_scan_cut(CutMap S, double gamma, double kappa) {
  S = compose_cut(S, dpp_cut<0x111, 0xf>(S), gamma, kappa);
  S = compose_cut(S, dpp_cut<0x112, 0xf>(S), gamma, kappa);
  S = compose_cut(S, dpp_cut<0x114, 0xf>(S), gamma, kappa);
  S = compose_cut(S, dpp_cut<0x118, 0xf>(S), gamma, kappa);
  S = compose_cut(S, dpp_cut<0x142, 0xa>(S), gamma, kappa);
  S = compose_cut(S, dpp_cut<0x143, 0xc>(S), gamma, kappa);
  return S;
}
__device__ __forceinline__ St apply_cut(const CutMap& M, const St& s, double gamma, double kappa) {
  return M.cut ? St{M.f.cV, M.f.cR, M.f.cA, M.f.cG} : apply(M.f, s, gamma, kappa);
}

struct TileMap {
  Aff f;
  int32_t cut;
  int32_t count;  // loss-mask tokens
};
static_assert(sizeof(TileMap) == kScanMapBytes, "the layout counts these");

// The trajectory holding token t, at or after trajectory lo (a batch whose segments
// are malformed gives some trajectory in [lo, hi]).
__device__ __forceinline__ int find_segment(const int32_t* cu, int lo, int hi, int64_t t) {
  while (lo < hi) {  // the last b in [lo, hi] with cu[b] <= t
    const int mid = lo + (hi - lo + 1) / 2;
    if (static_cast<int64_t>(cu[mid]) <= t)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

__device__ __forceinline__ double segment_kappa(int64_t L, double gamma, double lam, double alpha) {
  double lam_b = lam;
  if (alpha > 0.0) {
    lam_b = 1.0 - 1.0 / (alpha * static_cast<double>(L));
    if (lam_b < 0.0) lam_b = 0.0;
  }
  return gamma * lam_b;
}

// One thread's kScanPer tokens [c0, c0 + kScanPer) and the trajectory of its last one.
struct ScanTokens {
  float v[kScanPer], r[kScanPer];
  bool act[kScanPer];
  int n;              // tokens below T
  int seg;            // trajectory of token c0 + n - 1
  int64_t s, e;       // its range
  double kappa;

  __device__ __forceinline__ void load(const float* values, const float* rewards, const uint8_t* mask, int64_t c0,
                                       int64_t T, bool vec_ok) {
    n = T - c0 >= kScanPer ? kScanPer : (T > c0 ? static_cast<int>(T - c0) : 0);
    if (vec_ok && n == kScanPer) {
      const f32x4_t* pv = reinterpret_cast<const f32x4_t*>(values + c0);
      const f32x4_t* pr = reinterpret_cast<const f32x4_t*>(rewards + c0);
      const uint64_t m8 = *reinterpret_cast<const uint64_t*>(mask + c0);
#pragma unroll
      for (int q = 0; q < kScanPer / 4; ++q) {
        const f32x4_t vq = pv[q], rq = pr[q];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          v[4 * q + j] = vq[j];
          r[4 * q + j] = rq[j];
          act[4 * q + j] = ((m8 >> (8 * (4 * q + j))) & 0xffu) != 0;
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < kScanPer; ++j) {
        const bool in = j < n;
        v[j] = in ? values[c0 + j] : 0.0f;
        r[j] = in ? rewards[c0 + j] : 0.0f;
        act[j] = in && mask[c0 + j] != 0;
      }
    }
  }
  __device__ __forceinline__ void locate(const int32_t* cu, int lo, int hi, int64_t c0, double gamma, double lam,
                                         double alpha) {
    seg = find_segment(cu, lo, hi, c0 + (n > 0 ? n - 1 : 0));
    s = cu[seg];
    e = cu[seg + 1];
    kappa = segment_kappa(e - s, gamma, lam, alpha);
  }
  // Right to left over the tokens: end() before the last token of a trajectory, then
  // act(j, kappa) or obs(j). The trajectory changes at most once per token.
  template <class End, class Act, class Obs>
  __device__ __forceinline__ void walk(const int32_t* cu, int64_t c0, double gamma, double lam, double alpha, End&& end,
                                       Act&& action, Obs&& obs) const {
    int b = seg;
    int64_t bs = s, be = e;
    double k = kappa;
#pragma unroll
    for (int j = kScanPer - 1; j >= 0; --j) {
      if (j >= n) continue;
      const int64_t t = c0 + j;
      if (t < bs) {  // rarely: into the trajectory on the left, past empty ones by bisection (200,000 of
                     // them between two tokens: 0.12 ms a call, 50 ms one after another)
        if (b > 0) --b;
        be = bs;
        bs = cu[b];
        if (t < bs) {
          b = find_segment(cu, 0, b, t);
          bs = cu[b];
          be = cu[b + 1];
        }
        k = segment_kappa(be - bs, gamma, lam, alpha);
      }
      if (t + 1 == be) end();
      if (act[j])
        action(j, k);
      else
        obs(j);
    }
  }
};

// This thread's tokens as one map, and their loss-mask count.
__device__ __forceinline__ CutMap thread_map(const ScanTokens& x, const int32_t* cu, int64_t c0, double gamma, double lam,
                                             double alpha, int& cnt) {
  CutMap F = cut_identity();
  int c = 0;
  x.walk(
      cu, c0, gamma, lam, alpha, [&]() { F = CutMap{Aff{0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0}, 1}; },
      [&](int j, double k) {
        ++c;
        push_action(F.f, x.v[j], x.r[j], gamma, k);
      },
      [&](int j) { push_observation(F.f, x.r[j]); });
  cnt = c;
  return F;
}

// Trajectories of the first and last token of the tile at t0 (uniform): each by 64 probes
// at a time, both searches' loads together, so that 4096 trajectories take two rounds of
// loads where halving takes 24 (131,072 tokens in 512 trajectories 17.7 -> 15.7 us). As
// find_segment, some trajectory in [0, B) if the segments are malformed.
__device__ __forceinline__ void tile_segments(const int32_t* cu, int32_t B, int64_t T, int64_t t0, int& lo, int& hi) {
  const int64_t last = t0 + kScanTile < T ? t0 + kScanTile - 1 : T - 1;
  const int lane = threadIdx.x & 63;
  int a0 = 0, z0 = B - 1, a1 = 0, z1 = B - 1;
  while (a0 < z0 || a1 < z1) {  // uniform
    const int s0 = (z0 - a0) / 64 + 1, s1 = (z1 - a1) / 64 + 1;
    const int64_t i0 = a0 + static_cast<int64_t>(lane) * s0, i1 = a1 + static_cast<int64_t>(lane) * s1;
    const int32_t c0 = cu[i0 < z0 ? i0 : z0], c1 = cu[i1 < z1 ? i1 : z1];
    // The last probe at or before the token; lane 0's counts as one.
    const int l0 = 63 - __builtin_clzll(__ballot(i0 <= z0 && c0 <= t0) | 1);
    const int l1 = 63 - __builtin_clzll(__ballot(i1 <= z1 && c1 <= last) | 1);
    a0 += l0 * s0;
    a1 += l1 * s1;
    z0 = z0 - a0 < s0 ? z0 : a0 + s0 - 1;
    z1 = z1 - a1 < s1 ? z1 : a1 + s1 - 1;
  }
  lo = a0;
  hi = a1;
}

// First launch: block i's tile map; the block after the last tile checks the segments.
__global__ __launch_bounds__(kScanThreads) void k_scan_tiles(const float* values, const float* rewards,
                                                             const uint8_t* mask, const int32_t* cu, int32_t B,
                                                             int64_t T, double gamma, double lam, double alpha,
                                                             TileMap* maps, int32_t* bad, int32_t* status, bool vec_ok) {
  __shared__ CutMap s_agg[kScanThreads / 64];
  __shared__ double s_kap[kScanThreads / 64];
  __shared__ int s_cnt[kScanThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (blockIdx.x == gridDim.x - 1) {
    const bool b = segments_bad<kScanThreads>(cu, B, T);
    if (tid == 0) {
      *bad = b ? 1 : 0;
      if (b && status) atomicOr(status, SAO_STATUS_SEGMENTS);
    }
    return;
  }
  const int64_t t0 = static_cast<int64_t>(blockIdx.x) * kScanTile;
  const int64_t c0 = t0 + static_cast<int64_t>(kScanThreads - 1 - tid) * kScanPer;
  ScanTokens x;
  x.load(values, rewards, mask, c0, T, vec_ok);
  int lo, hi;
  tile_segments(cu, B, T, t0, lo, hi);
  x.locate(cu, lo, hi, c0, gamma, lam, alpha);
  int cnt;
  const CutMap S = wave_scan_cut(thread_map(x, cu, c0, gamma, lam, alpha, cnt), gamma, x.kappa);
  cnt = wave_sum(cnt);
  if (lane == 63) {
    s_agg[wave] = S;
    s_kap[wave] = x.kappa;
  }
  if (lane == 0) s_cnt[wave] = cnt;
  __syncthreads();
  if (tid == 0) {
    CutMap m = s_agg[0];
    int c = s_cnt[0];
    for (int w = 1; w < kScanThreads / 64; ++w) {
      m = compose_cut(s_agg[w], m, gamma, s_kap[w]);
      c += s_cnt[w];
    }
    maps[blockIdx.x] = TileMap{m.f, m.cut, c};
  }
}

// Second launch: outputs of one tile; block 0 adds the tiles' loss-mask counts. With
// kSingle the batch is one tile and this is the only launch.
template <bool kSingle>
__global__ __launch_bounds__(kScanThreads) void k_scan_flat(const float* values, const float* rewards,
                                                            const uint8_t* mask, const int32_t* cu, int32_t B,
                                                            int64_t T, double gamma, double lam, double alpha,
                                                            float* adv, float* ret, int64_t* n_tokens, TileMap* maps,
                                                            const int32_t* bad, int32_t* status, bool vec_ok) {
  constexpr int kWaves = kScanThreads / 64;
  __shared__ CutMap s_agg[kWaves];
  __shared__ double s_kap[kWaves];
  __shared__ CutMap s_right[kWaves];
  __shared__ int64_t s_cnt[kWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t t0 = static_cast<int64_t>(blockIdx.x) * kScanTile;
  const int64_t c0 = t0 + static_cast<int64_t>(kWaves * 64 - 1 - tid) * kScanPer;
  ScanTokens x;
  x.load(values, rewards, mask, c0, T, vec_ok);
  bool is_bad;
  if constexpr (kSingle) {
    is_bad = segments_bad<kScanThreads>(cu, B, T);
    if (tid == 0 && is_bad && status) atomicOr(status, SAO_STATUS_SEGMENTS);
  } else {
    is_bad = *bad != 0;
  }
  if (!kSingle && blockIdx.x == 0 && n_tokens) {
    int64_t c = 0;
    for (int i = tid; i < static_cast<int>(gridDim.x); i += kScanThreads) c += maps[i].count;
    c = wave_sum(c);
    if (lane == 0) s_cnt[wave] = c;
    __syncthreads();
    if (tid == 0) {
      int64_t tot = 0;
      for (int w = 0; w < kWaves; ++w) tot += s_cnt[w];
      *n_tokens = tot;
    }
  }
  int lo = 0, hi = 0;
  if (!is_bad) tile_segments(cu, B, T, t0, lo, hi);
  int cnt = 0;
  float oa[kScanPer], og[kScanPer];
  if (is_bad) {
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) {
      cnt += x.act[j] ? 1 : 0;
      oa[j] = og[j] = __builtin_nanf("");
    }
  } else {
    x.locate(cu, lo, hi, c0, gamma, lam, alpha);
    const CutMap S = wave_scan_cut(thread_map(x, cu, c0, gamma, lam, alpha, cnt), gamma, x.kappa);
    const CutMap E = dpp_cut<0x138, 0xf>(S);  // the lanes to the right only (identity at lane 0)
    if (lane == 63) {
      s_agg[wave] = S;
      s_kap[wave] = x.kappa;
    }
    // The state entering the tile from the right: the maps of the tiles to the right,
    // 64 per wave and 256 per round, up to the one that ends this tile's last trajectory.
    St right{0.0, 0.0, 0.0, 0.0};
    if constexpr (!kSingle) {
      const int64_t e_hi = cu[hi + 1];
      const double k_hi = segment_kappa(e_hi - static_cast<int64_t>(cu[hi]), gamma, lam, alpha);
      const int n_right = e_hi > t0 + kScanTile ? static_cast<int>((e_hi - 1) / kScanTile - blockIdx.x) : 0;
      CutMap all = cut_identity();
      for (int i0 = 0; i0 < n_right; i0 += kScanThreads) {  // uniform
        // Scan order is right to left, so lane 63 takes the tile nearest to this one.
        const int i = i0 + 64 * wave + 63 - lane;
        CutMap M = cut_identity();
        if (i < n_right) M = CutMap{maps[blockIdx.x + 1 + i].f, maps[blockIdx.x + 1 + i].cut};
        M = wave_scan_cut(M, gamma, k_hi);
        __syncthreads();  // the previous round's s_right has been read
        if (lane == 63) s_right[wave] = M;
        __syncthreads();
        for (int w = 0; w < kWaves; ++w) all = compose_cut(all, s_right[w], gamma, k_hi);
      }
      right = apply_cut(all, St{0.0, 0.0, 0.0, 0.0}, gamma, k_hi);
    }
    __syncthreads();
    // ... then the waves to the right (lower waves), then the lanes to the right.
    St st = right;
    for (int w = 0; w < wave; ++w) st = apply_cut(s_agg[w], st, gamma, s_kap[w]);
    st = apply_cut(E, st, gamma, dpp_f64<0x138, 0xf>(x.kappa, x.kappa));
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) oa[j] = og[j] = 0.0f;
    x.walk(
        cu, c0, gamma, lam, alpha, [&]() { st = St{0.0, 0.0, 0.0, 0.0}; },
        [&](int j, double k) {
          const double vv = x.v[j];
          const double rt = static_cast<double>(x.r[j]) + st.R;
          const double An = fma(k, st.A, fma(gamma, st.Vn, rt - vv));
          const double Gn = fma(gamma, st.G, rt);
          oa[j] = static_cast<float>(An);
          og[j] = static_cast<float>(Gn);
          st = St{vv, 0.0, An, Gn};
        },
        [&](int j) { st.R += static_cast<double>(x.r[j]); });
  }
  if (vec_ok && x.n == kScanPer) {
    f32x4_t* qa = reinterpret_cast<f32x4_t*>(adv + c0);
    f32x4_t* qg = reinterpret_cast<f32x4_t*>(ret + c0);
#pragma unroll
    for (int q = 0; q < kScanPer / 4; ++q) {
      qa[q] = f32x4_t{oa[4 * q], oa[4 * q + 1], oa[4 * q + 2], oa[4 * q + 3]};
      qg[q] = f32x4_t{og[4 * q], og[4 * q + 1], og[4 * q + 2], og[4 * q + 3]};
    }
  } else {
#pragma unroll
    for (int j = 0; j < kScanPer; ++j)
      if (j < x.n) {
        adv[c0 + j] = oa[j];
        ret[c0 + j] = og[j];
      }
  }
  if (kSingle && n_tokens) {
    const int64_t wcnt = wave_sum(cnt);
    __syncthreads();
    if (lane == 0) s_cnt[wave] = wcnt;
    __syncthreads();
    if (tid == 0) {
      int64_t tot = 0;
      for (int w = 0; w < kWaves; ++w) tot += s_cnt[w];
      *n_tokens = tot;
    }
  }
}

// The flat scan reads its inputs twice and keeps fewer waves per SIMD, so it moves
// half as many tokens per second as one workgroup per trajectory when those fill the
// GPU and are long (2^22 tokens: 48 us against 27 us with 512 trajectories or more;
// 2^24: 134 us against 70 us with 1024, 134 us either way with 256). Up to 2^20
// tokens both take a few launches' time whatever the lengths (23 us per call from
// Python), but for one trajectory among few: 131,071 tokens in one took 183 us with
// one workgroup and 19 us flat. So trajectories by the CU-full over 2^20 tokens take
// one workgroup each, everything else the flat scan, if the workspace holds its tile maps.
// Not batches of brief trajectories, at most 1024 of a mean of up to 128 tokens within 16
// tiles: the flat scan's threads step over a trajectory's end at almost every token (per
// trajectory / flat, kernels and gaps: 4096 tokens in 255 trajectories 14.3 / 19.0 us,
// 8192 in 64 14.3 / 15.9, 16,384 in 1024 17.2 / 19.0, in 2048 20.1 / 18.8, 32,768 in 255
// 14.8 / 16.0, in 64 14.9 / 13.8, 65,536 in 512 16.2 / 16.9). One long trajectory among
// them takes 2.6 us per tile there, so 16 tiles bound what the rule can lose to 30 us.
constexpr int64_t kScanFlatTokens = int64_t{1} << 20;
constexpr int32_t kScanFlatMaxB = 256;
constexpr int64_t kScanBriefTokens = 16 * kScanTileTokens;
constexpr int32_t kScanBriefMaxB = 1024;
constexpr int64_t kScanBriefMeanTokens = 128;

int launch_advantage(const float* values, const float* rewards, const uint8_t* mask,
                            const int32_t* cu_seqlens, int32_t B, int64_t T, double gamma, double lam,
                            double alpha, float* adv, float* ret, int64_t* n_tokens, int32_t* status,
                            void* ws, size_t ws_bytes, hipStream_t st) {
  const SegHead H = seg_head();
  char* w8 = static_cast<char*>(ws);
  int32_t* bad = reinterpret_cast<int32_t*>(w8 + H.bad);
  int64_t* slots = reinterpret_cast<int64_t*>(w8 + H.slots);
  // Vector access needs 16-byte aligned float arrays and an 8-byte aligned mask.
  const uintptr_t f = reinterpret_cast<uintptr_t>(values) | reinterpret_cast<uintptr_t>(rewards) |
                      reinterpret_cast<uintptr_t>(adv) | reinterpret_cast<uintptr_t>(ret);
  const bool vec_ok = (f & 15u) == 0 && (reinterpret_cast<uintptr_t>(mask) & 7u) == 0;
  if (T <= kScanTile) {
    hipLaunchKernelGGL(k_scan_flat<true>, dim3(1), dim3(kScanThreads), 0, st, values, rewards, mask, cu_seqlens, B, T,
                       gamma, lam, alpha, adv, ret, n_tokens, nullptr, nullptr, status, vec_ok);
    return hipGetLastError();
  }
  const bool brief = T <= kScanBriefTokens && B <= kScanBriefMaxB && T <= kScanBriefMeanTokens * B;
  if ((T <= kScanFlatTokens || B < kScanFlatMaxB) && !brief && ws_bytes >= advantage_workspace(T)) {
    TileMap* maps = reinterpret_cast<TileMap*>(w8 + H.total);
    const unsigned tiles = static_cast<unsigned>(ceil_div(T, kScanTile));
    hipLaunchKernelGGL(k_scan_tiles, dim3(tiles + 1), dim3(kScanThreads), 0, st, values, rewards, mask, cu_seqlens, B, T,
                       gamma, lam, alpha, maps, bad, status, vec_ok);
    hipLaunchKernelGGL(k_scan_flat<false>, dim3(tiles), dim3(kScanThreads), 0, st, values, rewards, mask, cu_seqlens, B,
                       T, gamma, lam, alpha, adv, ret, n_tokens, maps, bad, status, vec_ok);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((k_check_segments<256, kCountSlots>), dim3(1), dim3(256), 0, st, cu_seqlens, B, T, bad, slots,
                     status, nullptr);
  hipLaunchKernelGGL(k_advantage, dim3(B), dim3(kScanThreads), 0, st, values, rewards, mask, cu_seqlens,
                     B, T, gamma, lam, alpha, adv, ret, slots, bad, vec_ok);
  if (n_tokens) hipLaunchKernelGGL(k_slots_total<kCountSlots>, dim3(1), dim3(64), 0, st, slots, n_tokens);
  return hipGetLastError();
}

}  // namespace sao
