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

// Whether attention over M rows (La of them anchor rows), Lp passed keys and n_q
// heads takes the key-split form.  In the 256-row form a problem of at most one
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
inline bool attention_key_split(int64_t M, int64_t La, int64_t Lp, int64_t n_q, int64_t head_dim) {
  const int64_t total = M + Lp;  // keys of the last row
  const int64_t row_wgs = (M + kAttnRows - 1) / kAttnRows * n_q;
  if (row_wgs > kCus || total <= 8192 / head_dim) return false;
  const int64_t tiles = (M + kAttnSplitRows - 1) / kAttnSplitRows;
  if (tiles * n_q <= kCus) return true;
  // the first block of the second round, and the keys of its last row
  const int64_t r = std::min((tiles - kCus / n_q) * kAttnSplitRows, M) - 1;
  const int64_t second = (r < La ? r : r + Lp) + 1, fixed = head_dim == 128 ? 128 : 512;
  const int64_t rate = std::min<int64_t>(461 + row_wgs, head_dim == 128 ? 707 : 676);  // x 384
  return 384 * (total + second + fixed) <= rate * total;
}

}  // namespace apb

#endif  // APB_PLAN_H_
