// The host's choices between the forms of a kernel: rules on sizes alone, free
// of HIP, so that they can be looked at without a device.
#ifndef APB_PLAN_H_
#define APB_PLAN_H_

#include <stdint.h>

#include <algorithm>

namespace apb {

constexpr int kCus = 256;  // MI355X; the kernels below run one workgroup per CU

constexpr int kAttnRows = 256;       // query rows per workgroup of the 256-row form
constexpr int kAttnSplitRows = 128;  // of the key-split form

// Whether attention over M rows (La of them anchor rows), Lp passed keys in blocks
// of lp and n_q heads takes the key-split form.  In the 256-row form a problem of at most one
// round of workgroups takes as long as its longest row block, whose keys it walks
// alone; past one round the chip is full either way and that form does less work
// per key (a K or V tile serves twice the rows).  The key-split form takes about
// 1 / 1.7 of the time per key and row block, over twice the row blocks:
//  * all of them in one round: 1024 rows of the last of 8 hosts with every local
//    row passed on, 32 / 8 heads of d = 128, 183 -> 125 us; 300 rows 17.0 ->
//    12.5; 8192 rows of 4 / 1 heads of d = 64 (128 workgroups) 126 -> 79;
//  * more: the grid has the longest first, and the longest block of the second
//    round was seen to end up to as late as if it had waited for the longest of
//    the first.  So the keys of both, and what a second workgroup costs by itself
//    in keys, are held against the longest block's, by the ratio of the forms'
//    times per key: 1.6 where 160 CUs run the 256-row form, 1.84 (d = 64: 1.76)
//    where all do (the chip's clock gives way).  Triangles are well below it
//    (1324 rows and 381 passed keys 54.6 -> 44.4 us, 2048 rows 55.5 -> 45.7);
//    blocks whose keys are nearly all passed on are not (2048 rows and 14336
//    passed keys 444 against 471 us, 1280 and 8960 227 against 254).  Near the
//    line: 2048 rows and 3136 passed keys, 138 -> 129 us (256 CUs, 1.83 against
//    1.84); 1959 and 3556, 139 against 146 (256 CUs, 1.85 against 1.84); 1792 and
//    5376, 166 against 178 (224 CUs, 1.88 against 1.78); 4520 and 7620, 8 / 2
//    heads of d = 64, 191 against 202 (144 CUs, 1.71 against 1.58); 4508 and
//    5944, 14 / 2 heads, 171 against 194 (252 CUs, 1.84 against 1.76).
// It needs keys for both groups: 100 rows of d = 64, one tile, 8.2 against 9.1.
// And a tile that holds a passed block whole has its rows looked up one by one,
// which the 256-row form does half as often per key: such a key counts 0.85 more
// (many hosts that pass on less than a tile each: 63 blocks of 20 keys before 550
// rows of 8 / 2 heads of d = 64 47.7 against 53.7 us, 125 of 20 before 1900 rows of
// 32 / 8 heads of d = 128 120 against 214; 15 of 20 before 550 rows 38.3 -> 30.3).
inline bool attention_key_split(int64_t M, int64_t La, int64_t Lp, int64_t lp, int64_t n_q,
                                int64_t head_dim) {
  const int64_t total = M + Lp, tile = 8192 / head_dim;  // keys of the last row, of a tile
  const int64_t row_wgs = (M + kAttnRows - 1) / kAttnRows * n_q;
  if (row_wgs > kCus || total <= tile) return false;
  // passed keys in such tiles: all up to lp = tile / 2, none from a tile on
  const int64_t looked = Lp > 0 ? Lp * std::min(std::max<int64_t>(tile - lp, 0), lp) / lp : 0;
  const int64_t more = looked * 17 / 20;
  const int64_t tiles = (M + kAttnSplitRows - 1) / kAttnSplitRows;
  if (tiles * n_q <= kCus) return 100 * (total + more) <= (head_dim == 128 ? 160 : 145) * total;
  // the first block of the second round, and the keys of its last row
  const int64_t r = std::min((tiles - kCus / n_q) * kAttnSplitRows, M) - 1;
  const int64_t second = (r < La ? r : r + Lp) + 1, fixed = head_dim == 128 ? 128 : 512;
  const int64_t rate = std::min<int64_t>(461 + row_wgs, head_dim == 128 ? 707 : 676);  // x 384
  return 384 * (total + second + fixed + 2 * more) <= rate * total;
}

// How a decode call splits its keys; the workspace holds one partial per
// split and row: fp32 O and LSE (one or four row blocks), or fp16 O with a
// per-row power-of-two scale and the LSE (eight).
struct DecodePlan {
  int n_split;
  int blocks_per_split;
  int row_blocks;      // workgroups along the rows (each waves * 32 rows)
  int waves;           // 32-row blocks of a workgroup that share its key blocks (1, 4 or 8)
  bool one_launch;     // few keys: one split, its key blocks shared among a workgroup's waves
  uint64_t workspace_bytes;
};

// Rows and keys of a decode MFMA block, and the 32-key blocks of an eight-wave
// workgroup's tile.
constexpr int kRows = 32;
constexpr int kKeys = 32;
constexpr int kTileBlocks = 4;
constexpr int kWgPerCu = 3;  // one-wave workgroups per CU (LDS: 3 x 48 KiB at d = 128)

// Most key blocks of the one-launch form, whose waves share them: the step is then
// launches and latency.  Against split and merge, 32 / 8 heads of d = 128: 4 blocks
// 8.9 -> 6.9 us, 8 8.6 -> 7.9, 12 8.6 -> 8.5, 16 9.6 against 9.8 (turns of four
// blocks); 4 / 1 heads of d = 64: 4 blocks 7.0 -> 4.9, 20 7.2 -> 6.2, 28 7.1 ->
// 7.0, 30 7.0 against 7.7 (turns of eight, and the next splits are longer at 32).
constexpr int one_launch_blocks(int d) { return d == 128 ? 12 : 28; }

// max_workspace_bytes caps the splits; a plan with n_split == 0 does not fit.
inline DecodePlan plan_decode(int64_t n_q, int64_t n_kv, int head_dim, int64_t cache_len,
                              int64_t n_new, bool append, uint64_t max_workspace_bytes) {
  DecodePlan pl;
  const int64_t keys = cache_len + (append ? n_new : 0);
  const int64_t R = n_q / n_kv * n_new;
  // A GQA group of at least four 32-row blocks shares each K/V tile among the 8
  // waves of a workgroup (one workgroup per CU: its registers), else one wave
  // per 32-row block (kWgPerCu per CU: their LDS).
  pl.waves = R >= 4 * kRows ? 8 : 1;
  const int64_t bk = pl.waves == 8 ? kTileBlocks * kKeys : kKeys;
  const int64_t nblk = (keys + bk - 1) / bk;
  int64_t n_rb = (R + kRows * pl.waves - 1) / (kRows * pl.waves);
  // one round of workgroups, at least two key blocks each
  const int64_t target = pl.waves == 1 ? kCus * kWgPerCu : kCus;
  int64_t n_split = target / (n_kv * n_rb);
  if (n_split > nblk / 2) n_split = nblk / 2;
  if (n_split < 1) n_split = 1;
  int64_t bps = nblk > 0 ? (nblk + n_split - 1) / n_split : 0;
  if (bps > 0) n_split = (nblk + bps - 1) / bps;
  // Three or four row blocks: the same splits (256 workgroups, or 192 with four),
  // but two groups of four waves per workgroup in place of a workgroup per row
  // block, each reading the keys again.  85 rows x 30001 keys x 8 heads of d = 128:
  // 39.5 -> 31.7 us; 124 rows x 16384: 30.9 -> 25.6.  Short splits end before the
  // groups' start and merge are made up for.  By blocks per split, three row
  // blocks of d = 128 (96 rows x 8 heads): 4 18.7 against 19.3 us, 6 19.0 against
  // 20.0, 8 20.3 -> 20.2, 12 23.6 -> 22.5; four (124 rows): 4 18.6 against 19.3, 6
  // 20.4 against 20.5, 8 22.0 -> 21.8; d = 64 (124 rows x 2 heads): 4 14.0 against
  // 14.4, 6 15.5 -> 15.3.  With two row blocks the second read comes from cache
  // and the groups gain nothing.
  if (pl.waves == 1 && n_rb > 2 && bps >= (head_dim == 128 ? 9 : 6)) {
    pl.waves = 4;
    n_rb = 1;
  }
  // a workspace limit caps the splits (longer splits, the same kernels)
  const int64_t rows_total = n_q * n_new;
  // per (split, row): fp32 O and LSE, or fp16 O, its scale and the LSE
  const uint64_t per_row = pl.waves == 8 ? (uint64_t)head_dim * 2 + 8 : (uint64_t)(head_dim + 1) * 4;
  const uint64_t per_split = (uint64_t)rows_total * per_row;
  pl.one_launch = false;
  if ((uint64_t)n_split * per_split > max_workspace_bytes) {
    const int64_t cap = (int64_t)(max_workspace_bytes / per_split);
    if (cap < 1) {
      pl.n_split = 0;  // does not fit
      pl.blocks_per_split = 0;
      pl.row_blocks = (int)n_rb;
      pl.workspace_bytes = per_split;
      return pl;
    }
    bps = (nblk + cap - 1) / cap;
    n_split = (nblk + bps - 1) / bps;
  }
  pl.workspace_bytes = (uint64_t)n_split * per_split;
  // (the workspace keeps the size of the splits)
  if (pl.waves == 1 && n_split > 1 && nblk <= one_launch_blocks(head_dim)) {
    pl.one_launch = true;
    n_split = 1;
    bps = nblk;
  }
  pl.n_split = (int)n_split;
  pl.blocks_per_split = (int)bps;
  pl.row_blocks = (int)n_rb;
  return pl;
}

// How the token tiles of one matrix product (apb_gemm.h) are cut: `full` tiles of
// 256 tokens (nb = 8), then tiles of 32 * nb tokens for the rest.  The chip runs
// one workgroup per CU, so a product takes whole rounds of 256 tiles, and one with
// fewer or not quite a multiple of them leaves CUs idle: 80 tiles of 256 tokens
// (1256 tokens x 4096 features) take as long as 256.  Smaller tiles cost more per
// token (a step's copies of the weight slab do not shrink), so the cut is the
// cheapest by kTiles: the time of one round in units of a 256-token round,
// measured at K = 4096 to 14336 (O projection of 1256 tokens: 109 us in 80 tiles
// of 256 tokens, 65 us in 160 of 128, 57 us in 224 of 96, 45 us per round of 64).
// A second launch costs its ramp (kSecond).
struct GemmSplit {
  int full, nb;
};

// Rounds of workgroups (one per CU; every XCD gets an eighth of the tiles).
inline int64_t gemm_rounds(int64_t tiles) { return (tiles + kCus - 1) / kCus; }

inline GemmSplit gemm_split(int64_t T, int64_t nfy) {
  static const struct { int nb; double cost; } kTiles[] = {{8, 1.0}, {4, 0.54}, {3, 0.50}, {2, 0.43}};
  constexpr double kSecond = 0.08;
  const int64_t most = T / 256;  // whole 256-token tiles
  GemmSplit best{0, 8};
  double best_cost = (double)gemm_rounds((T + 255) / 256 * nfy);
  for (const auto& k : kTiles) {
    if (k.nb == 8) continue;
    // whole rounds of 256-token tiles first, as many as fit or fewer
    const int64_t all = gemm_rounds(most * nfy);
    for (int64_t r = all > 2 ? all - 2 : 0; r <= all; ++r) {
      const int64_t full = std::min<int64_t>(most, r * kCus / nfy);
      const int64_t rest = (T - 256 * full + 32 * k.nb - 1) / (32 * k.nb);
      const double cost = (double)gemm_rounds(full * nfy) + (double)gemm_rounds(rest * nfy) * k.cost +
                          (full > 0 && rest > 0 ? kSecond : 0.0);
      if (cost < best_cost) {
        best_cost = cost;
        best = GemmSplit{(int)full, k.nb};
      }
    }
  }
  return best;
}

}  // namespace apb

#endif  // APB_PLAN_H_
