// Launch planning of the HiF8 GEMM kernels: which launches cover a problem, and which tile a workgroup takes
// (plain C++, no HIP types; `__host__ __device__` are the only annotations, defined away in host-only builds).
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace hif8gemm {

// A ragged last round of 256 x 256 tiles leaves most compute units idle for a whole tile time.  When that
// round would be at most half full, the large tiles get as many whole tile columns as fill complete rounds
// (columns [0, *split)) and the remaining columns go to 128 x 128 tiles -- a quarter of the work each, two
// workgroups per compute unit, one round -- in a second launch.  Returns false where one launch is better.
inline bool ragged_round_split(size_t M, size_t N, size_t cus, uint32_t* split) {
  const size_t tm = (M + 255) / 256, tn = (N + 255) / 256, tiles = tm * tn;
  if (cus == 0 || tiles <= cus || tiles % cus == 0) return false;
  const size_t cols_big = tiles / cus * cus / tm;  // whole tile columns within the complete rounds
  if (cols_big < 1 || cols_big >= tn || (tn - cols_big) * tm * 2 > cus) return false;
  *split = (uint32_t)(cols_big * 256);
  return true;
}

// Tiles of the expanded-operand kernel: 256 x 256 or 256 x 192, one workgroup per compute unit, or 128 x 128, two.  A launch
// takes as long as its rounds of resident workgroups, so the tile with the shortest sum of rounds is taken.  A round
// costs, relative to each other, 13 (256 x 256), 10 (256 x 192), 7.6 (128 x 128, two per compute unit) or 6.2 (128 x 128,
// one), 4.0 (128 x 128 on at most one per compute unit, with four LDS stages): measured 84, 63.8, 47.7, 40.7 and 25.7 us
// at K = 4096.  The column split adds a launch (a twelfth of a large round).
// Measured in us (256 x 256 / 256 x 192 / 128 x 128): 2048 x 11008 x 4096 151 / 128 / 138, 2048 x 4096 x 11008
// 183 / 164 / 131, 11008 x 4096 x 2048 132 / 142 / 148, 4096^3 84 / 126 / 99.
enum : int { TILE_256 = 0, TILE_192 = 1, TILE_128 = 2, TILE_SPLIT = 3 };
inline uint64_t tile_count(int tile, size_t M, size_t N, size_t pairs) {
  const uint64_t bm = tile == TILE_128 ? 128 : 256, bn = tile == TILE_256 ? 256 : tile == TILE_192 ? 192 : 128;
  return ((M + bm - 1) / bm) * ((N + bn - 1) / bn) * (uint64_t)pairs;
}
// LDS stages of a launch: four for 128 x 128 tiles where every workgroup has a compute unit to itself.  What is priced and
// what is launched ask here (columns behind a split with two stages / four, us: 4096 x 5000 x 4096 124 / 116, 1792 x 9472 x
// 4096 120 / 107).
inline int tile_stages(int tile, uint64_t tiles, size_t cus) { return tile == TILE_128 && tiles <= cus ? 4 : 2; }
inline uint64_t tile_cost(int tile, size_t M, size_t N, size_t pairs, size_t cus) {
  const uint64_t tiles = tile_count(tile, M, N, pairs);
  if (tile != TILE_128) return (tiles + cus - 1) / cus * (tile == TILE_256 ? 130u : 100u);
  if (tile_stages(tile, tiles, cus) == 4) return 40u;
  const uint64_t rest = tiles % (2 * cus);
  return tiles / (2 * cus) * 76u + (rest == 0 ? 0u : rest <= cus ? 62u : 76u);
}
inline int tile_plan(size_t M, size_t N, size_t pairs, size_t cus, uint32_t* split) {
  int best = TILE_256;
  uint64_t cost = tile_cost(TILE_256, M, N, pairs, cus);
  for (int t = TILE_192; t <= TILE_128; ++t) {
    const uint64_t c = tile_cost(t, M, N, pairs, cus);
    if (c < cost) {
      cost = c;
      best = t;
    }
  }
  // complete rounds of 256 x 256 tiles, then the remaining columns in 128 x 128 tiles
  if (pairs == 1 && ragged_round_split(M, N, cus, split) &&
      tile_cost(TILE_256, M, *split, 1, cus) + tile_cost(TILE_128, M, N - *split, 1, cus) + 10u < cost)
    best = TILE_SPLIT;
  return best;
}

// The launches of a plan, one after the other on columns [begin, end) each; returns how many (one or two).
struct TileLaunch {
  int tile, stages;
  uint32_t begin, end;
};
inline int tile_launches(int plan, size_t M, size_t N, size_t pairs, size_t cus, uint32_t split, TileLaunch (&out)[2]) {
  auto one = [&](int tile, size_t begin, size_t end) {
    return TileLaunch{tile, tile_stages(tile, tile_count(tile, M, end - begin, pairs), cus), (uint32_t)begin, (uint32_t)end};
  };
  if (plan != TILE_SPLIT) {
    out[0] = one(plan, 0, N);
    return 1;
  }
  out[0] = one(TILE_256, 0, split);
  out[1] = one(TILE_128, split, N);
  return 2;
}

// Most tiles of a launch: its threads, 256 for each workgroup, are counted in 32 bits, and its workgroups are dealt out in
// whole rounds of the dies (kXcds).  The squared error in 256 x 256 tiles walks over tiles with one workgroup per compute unit,
// so that there only the tile number is limited.
constexpr uint64_t kMaxWorkgroups = 0xFFFFFFFFull / 256 / 8 * 8;
inline uint64_t most_tiles(int tile, bool sqerr) { return tile == TILE_256 && sqerr ? 0x7FFFFFF0ull : kMaxWorkgroups; }

// Pairs of a scale search (na x nb error products) that one launch takes: all of them, one row of nb, or a single one
// (0: not even that).  tile: the tile asked for, or -1 for the plan's own choice, which goes by the pairs of the launch.
inline uint32_t pairs_per_launch(int tile, size_t M, size_t N, uint32_t na, uint32_t nb, size_t cus) {
  auto fits = [&](size_t pairs) {
    uint32_t split = 0;
    const int t = tile >= 0 ? tile : tile_plan(M, N, pairs, cus, &split);
    return t == TILE_SPLIT || tile_count(t, M, N, pairs) <= most_tiles(t, true);  // a split: one part walks, the other has at most two rounds
  };
  return fits((size_t)na * nb) ? na * nb : fits(nb) ? nb : fits(1) ? 1u : 0u;
}

// Products with at most this many rows on one side run straight from the codes in hif8_gemm_ws_* when they go to the
// small-tile kernel; above it expanding first is faster (128 x 11008 x 4096: 52 us against 55; 384 x 4096 x 4096:
// 50 against 44; 512 x 4096 x 11008: 150 against 100).
constexpr size_t kSmallCodesRows = 128;

// Which problems go to the small-tile kernel (hif8_gemm_s.hip) although the tiled kernels could run them.  The tiled
// kernels take a whole K walk however few tiles there are (K = 4096: 85 us on codes, 25.7 us expanded), the small-tile
// kernel's time goes with M N.  On codes (us, small tiles / 128 x 128): 192 x 11008 x 4096 75 / 85, 256 x 11008 x 4096 94 /
// 85, 384 x 11008 135 / 120, 1024 x 4096 112 / 91; K = 1024 1500 x 1500 28.5 / 27.4, K = 512
// 700 x 3000 19.4 / 18.6, K = 256 1000 x 2000 14.0 / 13.1 (below K = 1024 up to 1.6 M); K = 11008 512 x 4096 150 / 231, 1024 x 4096 278 / 232.
// On expanded operands (us, small tiles / 128 x 128): 256 x 4096 x 4096 19.6 / 25.7, 384 x 4096 x 4096 29.2 / 25.9, 64 x
// 11008 x 4096 21.2 / 24.6, 100 x 11008 x 4096 29.1 / 25.4; K = 11008 256 x 4096 38 / 64, 512 x 4096 80 / 65; K = 2048 512 x
// 2048 12.5 / 14.3; K = 1024 300 x 5000 12.6 / 9.5.  With up to 32 rows on either side three quarters of a tile would be
// padding, so such products stay with the small tiles whatever the other side is.
inline bool small_problem(size_t M, size_t N, bool codes, size_t K = 4096) {
  const size_t s = M < N ? M : N, l = M < N ? N : M;
  if (s <= 32) return true;
  return codes ? l <= (size_t)(K < 1024 ? 24 : 33) * 65536 / s : l <= (size_t)5 * 262144 / ((s + 31) / 32 * 32);
}

// Tile (16 tm x 16 tn) and wavefronts per workgroup of the small-tile kernel.  The wavefronts split K, so a wavefront
// count is part of the result's rounding: below 128 rows it is the same for code and for expanded operands (there
// hif8_gemm_ws_* runs on the codes what hif8_gemm_expanded_* runs on expanded operands).  The smallest tiles win while
// one operand has few rows (8 x 11008 x 4096 on codes: 1 x 1 14 us, 1 x 2 17, 2 x 4 20); more rows want the operand
// reuse of larger ones, and fewer wavefronts once the tiles alone fill the chip (64 x 4096 x 4096: 2 x 2 with 16
// wavefronts 14.2 us, with 8 16.2; 64 x 11008 x 4096: 4 wavefronts 33.6, 16 41.8).
// With more than 256 tiles no more wavefronts than K has shares of kShareK elements: one without a share adds nothing to the
// sum, and its staging area takes LDS that other workgroups could have (codes, us, all wavefronts / as many as shares:
// 8 x 200000 x 64 42.1 / 14.7, 32 x 200000 x 256 80 / 29.5); with few tiles its lanes help with the table and the sum
// (128 x 512 x 16 6.9 / 9.1).
struct SmallPlan {
  uint32_t tm, tn, waves;
};
constexpr size_t kShareK = 128;
inline SmallPlan small_plan(size_t M, size_t N, size_t K, bool codes) {
  auto tiles = [&](size_t tm, size_t tn) { return ((M + 16 * tm - 1) / (16 * tm)) * ((N + 16 * tn - 1) / (16 * tn)); };
  const size_t s = M < N ? M : N, shares = K > kShareK ? (K + kShareK - 1) / kShareK : 1;
  auto plan = [&](uint32_t tm, uint32_t tn, uint32_t waves) {
    return SmallPlan{tm, tn, waves < shares || tiles(tm, tn) <= 256 ? waves : (uint32_t)shares};
  };
  if (s <= 16) return plan(1, 1, 8);
  if (s <= 32) return tiles(2, 4) >= 128 ? plan(2, 4, 8) : plan(1, 2, 8);
  if (s <= 64) return plan(2, 2, tiles(2, 2) <= 256 ? 16 : 4);
  if (s <= kSmallCodesRows || (codes && small_problem(M, N, true))) return plan(2, 4, tiles(2, 4) <= 256 ? 8 : 4);
  return plan(4, 4, !codes && tiles(4, 4) <= 256 ? 8 : 4);
}

// Workgroup -> tile of the expanded-operand kernel.  The hardware deals consecutive workgroups round-robin over the
// kXcds accelerator dies (XCDs), each with its own L2.  Workgroup b therefore takes tile number
// (b % kXcds) * per_xcd + b / kXcds of a tile order that walks groups of kGroupM tile rows column by column: the
// workgroups resident on one die at a time then cover a compact kGroupM x (a few) block of tiles and share their
// operand panels in that die's L2, whatever tiles_n is.  The launch has tile_order_grid() workgroups; returns false
// for the few at the end of the last die's share that have no tile.
constexpr uint32_t kXcds = 8;    // accelerator dies, each with an L2 of its own
constexpr uint32_t kGroupM = 8;  // tile rows per group of the tile order
__host__ __device__ inline uint32_t tile_order_grid(uint32_t n_tiles) { return (n_tiles + kXcds - 1u) / kXcds * kXcds; }
__host__ __device__ inline bool tile_order(uint32_t b, uint32_t tiles_m, uint32_t tiles_n, uint32_t* tile_m, uint32_t* tile_n) {
  const uint32_t n_tiles = tiles_m * tiles_n, per_xcd = (n_tiles + kXcds - 1u) / kXcds;
  const uint32_t t = (b % kXcds) * per_xcd + b / kXcds;
  if (t >= n_tiles) return false;
  const uint32_t grp = t / (kGroupM * tiles_n), first_m = grp * kGroupM;
  const uint32_t grp_rows = tiles_m - first_m < kGroupM ? tiles_m - first_m : kGroupM;
  const uint32_t in_grp = t - grp * (kGroupM * tiles_n);
  *tile_n = in_grp / grp_rows;
  *tile_m = first_m + (in_grp - *tile_n * grp_rows);
  return true;
}

}  // namespace hif8gemm
