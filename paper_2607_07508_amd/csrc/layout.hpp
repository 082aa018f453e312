// Host-side workspace layouts shared by sao_workspace_size and the launchers.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace sao {

constexpr int64_t kTile = 256;
constexpr int64_t kRowsPerCountBlock = 1024;  // rows per block of the compaction count
constexpr int64_t kVocabBlock = 32768;        // vocabulary rows per backward dZ block (at least)
constexpr int64_t kVocabBlockMax = 65536;     // ... and at most
constexpr int kLossThreads = 256;
constexpr int kLossPerThread = 4;             // tokens per thread before blocks take a second turn
constexpr int kLossMaxBlocks = 2048;
// Threads take one quad of tokens at a time up to this many tokens (every thread then has
// one), two beyond, for the loads in flight.
constexpr int64_t kLossOneQuadTokens = int64_t{kLossMaxBlocks} * kLossThreads * kLossPerThread;
static_assert(kLossPerThread == 4, "one quad");

inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }
inline int64_t ceil_div(int64_t x, int64_t m) { return (x + m - 1) / m; }
inline size_t align256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

struct Carve {
  size_t off = 0;
  size_t take(size_t bytes) {
    const size_t o = off;
    off = align256(off + bytes);
    return o;
  }
};

// sao_token_logprob
struct LogprobLayout {
  int64_t t_pad, n_count_blocks, m_tiles;
  size_t blk_counts, count, next, idx, hc, part, total;
};

inline LogprobLayout logprob_layout(int64_t T, int64_t H, int64_t V, size_t esize) {
  LogprobLayout L{};
  L.t_pad = round_up(T, kTile);
  L.n_count_blocks = ceil_div(T, kRowsPerCountBlock);
  L.m_tiles = ceil_div(V, kTile);
  Carve c;
  L.blk_counts = c.take(4 * static_cast<size_t>(L.n_count_blocks));
  L.count = c.take(4);
  L.next = c.take(4 * 8);  // the forward's tile counters, one per XCD
  L.idx = c.take(4 * static_cast<size_t>(L.t_pad));
  L.hc = c.take(esize * static_cast<size_t>(L.t_pad) * static_cast<size_t>(H));
  L.part = c.take(8 * static_cast<size_t>(L.m_tiles) * static_cast<size_t>(L.t_pad));
  L.total = c.off;
  return L;
}

// sao_loss_backward
struct BackwardLayout {
  int64_t t_pad, n_count_blocks, vc, n_vblocks;
  int64_t dh_cap;  // token tiles of dH accumulators (dh_cap_tiles)
  size_t blk_counts, count, next, idx, pos, g_c, lse_c, y_c, hg, dh, dz, total;
};

// K pieces of the dH product. Its output tiles (token tiles with a gradient row x
// ceil(H / 256)) can be fewer than the CUs, so K (the block's vocabulary rows) is cut
// into pieces, each adding into its own fp32 accumulator. Only the device knows how
// many token tiles hold rows, so the kernels choose: of up to kMaxDhPieces pieces
// whose accumulators fit `cap` token tiles, the number whose rounds of tiles over the
// CUs take least, a round costing its K slabs and kDhRoundSlabs slabs' time of
// prologue, epilogue and of the accumulators' later sum (25k cycles and 5k, a slab
// taking about 2k). 24 tiles run as 10 pieces, 128 as 2, 136 as 7. The first
// vocabulary block's K decides for all blocks.
constexpr int kMaxDhPieces = 32;
constexpr float kDhRoundSlabs = 16.0f;
constexpr int dh_pieces(int m_tiles, int n_tiles, int64_t cap, int k_slabs) {
  int best = 1;
  float least = 0.0f;
  for (int p = 1; p <= kMaxDhPieces && p <= k_slabs && (p == 1 || static_cast<int64_t>(p) * m_tiles <= cap); ++p) {
    const int64_t rounds = (static_cast<int64_t>(m_tiles) * n_tiles * p + 255) / 256;
    const float cost = static_cast<float>(rounds) * (static_cast<float>(k_slabs) / static_cast<float>(p) + kDhRoundSlabs);
    if (p == 1 || cost < least) {
      best = p;
      least = cost;
    }
  }
  return best;
}
// Token tiles of accumulators: every piece of up to 1024 output tiles (four per CU).
constexpr int64_t dh_cap_tiles(int64_t m_tiles, int64_t n_tiles) {
  int64_t c = (1024 + n_tiles - 1) / n_tiles;
  if (c > m_tiles * kMaxDhPieces) c = m_tiles * kMaxDhPieces;
  return c > m_tiles ? c : m_tiles;
}
// K rows per piece when `k` rows go into `pieces`: a multiple of 64.
constexpr int64_t dh_piece_rows(int64_t k, int pieces) { return ((k + pieces - 1) / pieces + 63) / 64 * 64; }

// MI355X's memory-side (Infinity) cache, shared by the XCDs, and its compute units.
constexpr int64_t kMemorySideCacheBytes = int64_t{256} << 20;
constexpr int64_t kGpuCus = 256;

inline int64_t gcd64(int64_t a, int64_t b) { return b == 0 ? a : gcd64(b, a % b); }

// Vocabulary rows per backward block. The target size is kVocabBlock, doubled up
// to kVocabBlockMax while one block's dz product would have fewer than 8192 tiles
// (32 per CU) at the host bound of token rows, so that short token chunks still
// give each launch many rounds of tiles and take fewer launches. V is then cut
// into as many blocks as that target size needs, as equal as possible.
// A block's dW product has (block tiles) x ceil(H / 256) output tiles, each as
// long as the whole token range, so a block whose dW tiles leave a partial last
// round idles part of the GPU for one long tile. Where the block's rows of W fit
// the memory-side cache, the block is therefore rounded up to a multiple of
// kGpuCus / gcd(kGpuCus, ceil(H / 256)) tiles (32 at H = 2048), which leaves
// only the last block with a partial round. (Measured: 1.4 % off c2's backward,
// 1.9 % off c3's.) Where the rounded-up block's rows of W would not fit the
// cache (H = 6144), the larger blocks slowed the logit recompute by more than
// dW gained; there the block is rounded down to that multiple instead (0.7 %
// off c4's backward).
inline int64_t vocab_block(int64_t t_pad, int64_t V, int64_t H, size_t esize) {
  int64_t vc = kVocabBlock;
  while (vc < kVocabBlockMax && (t_pad / kTile) * (vc / kTile) < 8192) vc *= 2;
  const int64_t blocks = ceil_div(V, vc);
  int64_t tiles = ceil_div(ceil_div(V, blocks), kTile);
  const int64_t align = kGpuCus / gcd64(kGpuCus, ceil_div(H, kTile));
  const int64_t rounded = round_up(tiles, align);
  if (blocks > 1 && rounded <= vc / kTile &&
      rounded * kTile * H * static_cast<int64_t>(esize) <= kMemorySideCacheBytes)
    tiles = rounded;
  else if (blocks > 1 && tiles >= align)
    tiles = tiles / align * align;
  return tiles * kTile;
}

inline BackwardLayout backward_layout(int64_t T, int64_t H, int64_t V, size_t esize) {
  BackwardLayout L{};
  L.t_pad = round_up(T, kTile);
  L.n_count_blocks = ceil_div(T, kRowsPerCountBlock);
  L.vc = vocab_block(L.t_pad, V, H, esize);
  L.n_vblocks = ceil_div(V, L.vc);
  L.dh_cap = dh_cap_tiles(L.t_pad / kTile, ceil_div(H, kTile));
  Carve c;
  const size_t tp = static_cast<size_t>(L.t_pad);
  L.blk_counts = c.take(4 * static_cast<size_t>(L.n_count_blocks));
  L.count = c.take(4);
  L.next = c.take(4 * 8 * static_cast<size_t>(L.n_vblocks));  // the recompute's tile counters
  L.idx = c.take(4 * tp);
  L.pos = c.take(4 * static_cast<size_t>(T));
  L.g_c = c.take(4 * tp);
  L.lse_c = c.take(4 * tp);
  L.y_c = c.take(4 * tp);
  L.hg = c.take(esize * tp * static_cast<size_t>(H));
  L.dh = c.take(4 * static_cast<size_t>(kTile) * static_cast<size_t>(H) * static_cast<size_t>(L.dh_cap));
  L.dz = c.take(esize * tp * static_cast<size_t>(L.vc));
  L.total = c.off;
  return L;
}

// Head of every advantage kernel's workspace: the int32 segments flag, then
// kCountSlots int64 slots that spread the loss-mask count's atomic adds (one
// slot per workgroup, modulo kCountSlots) before a one-block total.
constexpr int kCountSlots = 64;
struct SegHead {
  size_t bad, slots, total;
};
inline SegHead seg_head() {
  SegHead H{};
  Carve c;
  H.bad = c.take(4);
  H.slots = c.take(8 * kCountSlots);
  H.total = c.off;
  return H;
}

// The critic-free baselines need only the head.
inline size_t baseline_workspace() { return seg_head().total; }

// sao_advantage: the head, then (for more than one tile) a map per tile of tokens.
constexpr int64_t kScanTileTokens = 2048;
constexpr size_t kScanMapBytes = 64;
inline size_t advantage_workspace(int64_t T) {
  return seg_head().total +
         (T > kScanTileTokens ? align256(kScanMapBytes * static_cast<size_t>(ceil_div(T, kScanTileTokens))) : 0);
}

// sao_clipped_loss
struct LossLayout {
  int64_t blocks;
  size_t part_f, part_i, part_n, total;
};

inline LossLayout loss_layout(int64_t T) {
  LossLayout L{};
  int64_t blocks = ceil_div(T, static_cast<int64_t>(kLossThreads) * kLossPerThread);
  if (blocks > kLossMaxBlocks) blocks = kLossMaxBlocks;
  if (blocks < 1) blocks = 1;
  L.blocks = blocks;
  Carve c;
  L.part_f = c.take(16 * static_cast<size_t>(blocks));   // two doubles per block
  L.part_i = c.take(40 * static_cast<size_t>(blocks));   // five int64 per block
  L.part_n = c.take(8 * static_cast<size_t>(blocks));    // the mask count's partials
  L.total = c.off;
  return L;
}

// The largest sao_clipped_loss workspace (kLossMaxBlocks blocks; the pieces are
// 256-byte multiples), the size of sao_clipped_loss_noalloc's static scratch.
// Every T fits, since the block count is capped.
constexpr size_t kLossScratchBytes = (16 + 40 + 8) * kLossMaxBlocks;
static_assert(8 * kLossMaxBlocks % 256 == 0, "pieces stay aligned");

// The recurrence over a trajectory's n steps runs over kStepChunks chunks of equal length;
// chunk i is [step_chunk_begin(n, i), step_chunk_begin(n, i + 1)), empty from kStepChunks on.
// In 64 bits: with 1024 threads i x length passes 2^31 from 537 million steps.
constexpr int kStepChunks = 256;
constexpr int step_chunk_len(int n) {
  return static_cast<int>((static_cast<int64_t>(n) + kStepChunks - 1) / kStepChunks);
}
constexpr int step_chunk_begin(int n, int i) {
  const int64_t p = static_cast<int64_t>(i) * step_chunk_len(n);
  return p < n ? static_cast<int>(p) : n;
}

// sao_step_advantage: the head, then a step table of T entries (a trajectory's
// steps sit at its own token offset): start and end (int32), and two doubles
// (the step's value and reward, later its advantage and return).
struct StepLayout {
  size_t tab_a, tab_z, tab_v, tab_r, total;
};

inline StepLayout step_layout(int64_t T) {
  StepLayout L{};
  Carve c;
  c.take(seg_head().total);
  L.tab_a = c.take(4 * static_cast<size_t>(T));
  L.tab_z = c.take(4 * static_cast<size_t>(T));
  L.tab_v = c.take(8 * static_cast<size_t>(T));
  L.tab_r = c.take(8 * static_cast<size_t>(T));
  L.total = c.off;
  return L;
}

// sao_group_advantage / sao_running_mean_advantage need only the head.

// sao_ppo_loss shares the loss layout.

// sao_explained_variance: five doubles per block
struct EvLayout {
  int64_t blocks;
  size_t part, total;
};

inline EvLayout ev_layout(int64_t T) {
  EvLayout L{};
  L.blocks = loss_layout(T).blocks;
  Carve c;
  L.part = c.take(40 * static_cast<size_t>(L.blocks));
  L.total = c.off;
  return L;
}

// sao_value_loss (sao_value_forward needs none)
constexpr int kValueThreads = 256;
constexpr int64_t kValueRows = 128;           // rows per block of the value-loss pass
constexpr int64_t kValueCountBlocks = 1024;   // blocks of the mask count when N is not given

struct ValueLayout {
  int64_t row_blocks, count_blocks;
  size_t part_cnt, part_loss, part_dw, total;
};

inline ValueLayout value_layout(int64_t T, int64_t H) {
  ValueLayout L{};
  L.row_blocks = ceil_div(T, kValueRows);
  L.count_blocks = ceil_div(T, static_cast<int64_t>(kValueThreads) * 8);
  if (L.count_blocks > kValueCountBlocks) L.count_blocks = kValueCountBlocks;
  if (L.count_blocks < 1) L.count_blocks = 1;
  Carve c;
  L.part_cnt = c.take(8 * static_cast<size_t>(L.count_blocks));
  L.part_loss = c.take(8 * static_cast<size_t>(L.row_blocks));
  L.part_dw = c.take(4 * static_cast<size_t>(L.row_blocks) * static_cast<size_t>(H));
  L.total = c.off;
  return L;
}

}  // namespace sao
