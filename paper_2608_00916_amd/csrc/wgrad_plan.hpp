// Schedule of the weight-gradient products, built on the device per
// backward from the expert offsets.
//
// Every tile of an expert's weight gradient reduces over that expert's rows
// (K = n_e), so under skewed routing tile lengths differ by an order of
// magnitude and equal tile counts per XCD are far from equal work.  The plan
// orders the experts by descending rows (ties to the lower index) and numbers
// the tiles expert by expert in that order; XCD x takes the tiles whose
// cumulative work (K steps plus kTileFixed per tile) starts in
// [x W / 8, (x + 1) W / 8), W the total, and the workgroups of an XCD take its
// tiles round-robin, longest first.  An expert's tiles stay on one or two
// XCDs, so its rows are fetched into few L2s.  Each tile is still computed
// whole by one workgroup: the schedule changes no result.
//
// Tile height.  A weight gradient that may (WgradTiles::tall) runs on
// 256 x 256 tiles, half as many: at 128 experts x 512 rows, H = 2048, F = 768
// the down product took 246-250 us against 276 with 128 x 256, the gate/up
// product 536-542 against 555.  It stays on 128-row tiles
//  * where the longest tile is more than half of a workgroup's mean work, as
//    halving the tile count then costs more in balance (hottest expert at 10x
//    the mean, T = 32768: the down product 1010 us against 970; at 0.39 of the
//    mean work, the gate/up product 1870 against 1950);
//  * for a mean of 25 to 41 rows per expert: many experts then take two 32-row
//    steps where 128-row tiles take one of 64 rows (same widths, gate/up: 171
//    us against 180 at 24 rows, 2-4% slower at 26 to 40, 2% faster at 42);
//  * for a mean under 3: many experts then have no rows, and their tiles, which take
//    nearly as long as short ones but count 2 steps against 3 below, leave the
//    XCDs uneven (1 row: gate/up 10% slower; 192 experts, 1536 x 768, 2 rows: down 5%);
//  * with fewer than 12 tall tiles per workgroup for any mean under 48: the stores
//    of a tile's last 64 rows, which nothing overlaps, then weigh more (at 8
//    rows: 256 experts of 512 x 512, 4 per workgroup, down 41 us against 36;
//    232 of 256 x 1152, 8 per workgroup, gate/up 9% slower; at 42 rows 7% and 9%).
// With 8 to 10 per workgroup and H = 256 the gate/up product is up to 6% slower
// at 56 to 256 rows too, where the last round of tiles is nearly empty, and 3-5%
// faster from 384 on: the rule does not look at rounds.
// The order of the experts and the XCDs' shares count 64-row steps for either height.
//
// Layout (wgrad_plan_ints(E) ints): plan[0, E) the expert at each position of
// the order; then, per weight gradient q (0: down, 1: gate/up), the first
// tile of XCD x at plan[E + q (kPlanXcds + 1) + x], x = 0..kPlanXcds; then
// per q whether its tiles are tall (plan_tall).
#pragma once

#include "common.hpp"
#include "launch.hpp"
#include "moe.h"

namespace moe {

constexpr int kPlanXcds = 8;
constexpr int kPlanBK = 64;    // K steps are 64 rows deep
constexpr int kPlanWgs = 256;   // workgroups of the persistent grid (one per CU)
constexpr int kTileFixed = 2;  // a tile's fixed cost (setup, epilogue) in K steps
// Tile height (above): mean rows per expert from which, up to which and again
// from which on tiles are tall with kTallMany of them per workgroup, and from
// which on with fewer.
constexpr int kTallMany = 12;
constexpr int kTallFrom = 3, kTallUpTo = 24, kTallAgain = 42, kTallFew = 48;

__host__ __device__ constexpr int plan_tall(int E, int q) { return E + 2 * (kPlanXcds + 1) + q; }

// Whether weight gradient q runs on tall tiles: `longest` and `total` are the
// work of the longest tile and of one tile of every expert, `rows` the rows of
// all E experts.
__device__ __forceinline__ bool use_tall(const WgradTiles& t, int q, int E, int rows, int longest, int64_t total) {
  const int tpe = t.tpe[q] / 2;
  const bool many = E * tpe >= kTallMany * kPlanWgs;
  const bool depth = rows >= kTallFew * E || (many && (rows >= kTallAgain * E ||
                                                       (rows >= kTallFrom * E && rows <= kTallUpTo * E)));
  return t.tall[q] && depth && 2LL * kPlanWgs * longest <= tpe * total;
}

// One workgroup of 256 threads (E <= 256) builds the plan.
__device__ __forceinline__ void build_wgrad_plan(const int32_t* __restrict__ offsets, int E, const WgradTiles& tiles,
                                                 int32_t* __restrict__ plan) {
  static_assert(MOE_MAX_EXPERTS <= 256, "one thread per expert");
  constexpr int kPairs = 2 * (kPlanXcds + 1);
  __shared__ int rows[MOE_MAX_EXPERTS];
  __shared__ int wave_tot[4];
  __shared__ int64_t bound[kPairs];
  __shared__ int cum_at[MOE_MAX_EXPERTS];
  __shared__ int steps_at[MOE_MAX_EXPERTS];
  __shared__ int cnt[4][kPairs];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  if (tid < E) rows[tid] = offsets[tid + 1] - offsets[tid];
  __syncthreads();
  // position of expert tid in the order: experts with more rows, or as many
  // and a lower index, come first
  int pos = 0, steps = 0;
  if (tid < E) {
    const int ne = rows[tid];
    int rank = 0;
#pragma unroll 8
    for (int f = 0; f < E; ++f) {
      const int nf = rows[f];
      rank += (nf > ne || (nf == ne && f < tid)) ? 1 : 0;
    }
    pos = rank;
    steps = cdiv(ne, kPlanBK) + kTileFixed;
    plan[pos] = tid;
    steps_at[pos] = steps;
  }
  __syncthreads();
  // exclusive prefix sum of the steps over positions (thread p holds position p)
  int v = tid < E ? steps_at[tid] : 0;
  int incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(incl, o, 64);
    incl += lane >= o ? u : 0;
  }
  if (lane == 63) wave_tot[wv] = incl;
  __syncthreads();
  int before = 0;
  for (int w = 0; w < wv; ++w) before += wave_tot[w];
  const int cum = before + incl - v;  // work of the positions before tid, per tile of each
  if (tid < E) cum_at[tid] = cum;
  const int total = wave_tot[0] + wave_tot[1] + wave_tot[2] + wave_tot[3];
  const int all_rows = offsets[E] - offsets[0];
  const bool tall0 = use_tall(tiles, 0, E, all_rows, steps_at[0], total);
  const bool tall1 = use_tall(tiles, 1, E, all_rows, steps_at[0], total);
  const int tpe0 = tall0 ? tiles.tpe[0] / 2 : tiles.tpe[0];
  const int tpe1 = tall1 ? tiles.tpe[1] / 2 : tiles.tpe[1];
  if (tid == 0) {
    plan[plan_tall(E, 0)] = tall0;
    plan[plan_tall(E, 1)] = tall1;
  }
  if (tid < kPairs) {
    const int q = tid / (kPlanXcds + 1), x = tid % (kPlanXcds + 1);
    const int64_t tpe = q == 0 ? tpe0 : tpe1;
    bound[tid] = x * (tpe * total) / kPlanXcds;  // work before XCD x's first tile
  }
  __syncthreads();
  // for each (q, x): the last position whose first tile starts at or before
  // the bound (positions 0..E-1; cum strictly increases)
#pragma unroll
  for (int i = 0; i < kPairs; ++i) {
    const int64_t tpe = i < kPlanXcds + 1 ? tpe0 : tpe1;
    const bool le = tid < E && tpe * cum <= bound[i];
    const int c = __popcll(__ballot(le));
    if (lane == 0) cnt[wv][i] = c;
  }
  __syncthreads();
  if (tid < kPairs) {
    const int q = tid / (kPlanXcds + 1), x = tid % (kPlanXcds + 1);
    const int64_t tpe = q == 0 ? tpe0 : tpe1;
    int64_t t = static_cast<int64_t>(E) * tpe;
    if (x < kPlanXcds) {
      const int p = cnt[0][tid] + cnt[1][tid] + cnt[2][tid] + cnt[3][tid] - 1;
      // first tile of position p whose start is at or past the bound
      const int64_t local = cdiv64(bound[tid] - tpe * cum_at[p], steps_at[p]);
      t = static_cast<int64_t>(p) * tpe + (local < tpe ? local : tpe);
    }
    plan[E + q * (kPlanXcds + 1) + x] = static_cast<int32_t>(t);
  }
}

}  // namespace moe
