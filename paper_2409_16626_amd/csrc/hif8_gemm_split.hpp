// Launch planning of the HiF8 GEMM kernels: which launches cover a problem, and which tile a workgroup takes
// (plain C++, no HIP types; `__host__ __device__` are the only annotations, defined away in host-only builds).
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <cmath>

namespace hif8gemm {

// A ragged last round of 256 x 256 tiles leaves most compute units idle for a whole tile time.  When that
// round would be at most half full, the large tiles get as many whole tile columns as fill complete rounds
// (columns [0, *split)) and the remaining columns may go to smaller tiles in a second launch: of expanded operands 128 x 128 -- a quarter
// of the work each, two workgroups per compute unit, one round --, of code operands the tile with the lowest price, one workgroup per compute unit
// and one round or two.  Returns false where there is no such round; the callers compare prices.
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
// at K = 4096, in two LDS stages.  The forms that run now (tile_form) keep these proportions: on another machine 89, 68.3, 49.9 (as 256 x 128
// tiles), 37 and 30.3 us at K = 4096, 165, 130, 94 and 66 at 8192, 49.5, 39, 28.3 and 20.4 at 2048.  The column split adds a launch (a twelfth of a
// large round).
// Measured in us (256 x 256 / 256 x 192 / 128 x 128, two stages): 2048 x 11008 x 4096 151 / 128 / 138, 2048 x 4096 x 11008
// 183 / 164 / 131, 11008 x 4096 x 2048 132 / 142 / 148, 4096^3 84 / 126 / 99.
enum : int { TILE_256 = 0, TILE_192 = 1, TILE_128 = 2, TILE_SPLIT = 3 };
inline uint64_t tile_count(int tile, size_t M, size_t N, size_t pairs) {
  const uint64_t bm = tile == TILE_128 ? 128 : 256, bn = tile == TILE_256 ? 256 : tile == TILE_192 ? 192 : 128;
  return ((M + bm - 1) / bm) * ((N + bn - 1) / bn) * (uint64_t)pairs;
}
// LDS stages that a launch is priced with: four for 128 x 128 tiles where every workgroup has a compute unit to itself.  The price and the
// form that is launched (tile_form) ask here (columns behind a split with two stages / four, us: 4096 x 5000 x 4096 124 / 116,
// 1792 x 9472 x 4096 120 / 107); a price holds for every form that a tile and a number of stages can run in.
inline int tile_stages(int tile, uint64_t tiles, size_t cus) { return tile == TILE_128 && tiles <= cus ? 4 : 2; }
// With K below 1024 a round's epilogue counts as much as its MFMAs, and two 128 x 128 tiles on a compute unit hide it from each
// other: there a round of single products costs a part that goes with the output and one that goes with K, in tenths of a us
// (256 x 256 / 256 x 192 / 128 x 128: 8192 x 8192 x 128 46 / 52 / 38 bfloat16, 64 / 67 / 53 binary32, 71 / 80 / 66 squared error; x
// 512 71 / 85 / 70 bfloat16; 4096 x 4096 x 512 21 / 29 / 21 bfloat16, 22.4 / 29 / 24 binary32; squared error
// 4096 x 4096 x 128 19 / 26 / 21, with edge tiles 1500 x 9000 x 128 24 / 26 / 20).
enum : int { OUT_16 = 0, OUT_32 = 1, OUT_ERR = 2 };
struct TileProblem {
  size_t M, N, K, pairs;
  int out;
};
inline uint64_t tile_cost(int tile, const TileProblem& p, size_t cus) {
  const uint64_t tiles = tile_count(tile, p.M, p.N, p.pairs), rest = tiles % (2 * cus);
  uint64_t round[5] = {130, 100, 76, 62, 40};  // 256 x 256, 256 x 192, 128 x 128: two per compute unit, one, one with four stages
  if (p.K < 1024 && p.pairs == 1) {
    constexpr uint64_t kOut[3][5] = {{90, 70, 35, 32, 38}, {125, 95, 60, 45, 42}, {156, 125, 84, 55, 60}}, kPerStep[5] = {111, 87, 68, 59, 34};
    for (int i = 0; i < 5; ++i) round[i] = kOut[p.out][i] + (p.K + 63) / 64 * kPerStep[i] / 10;
    if (p.out == OUT_ERR && (p.M % 256 != 0 || p.N % 256 != 0)) round[0] += 40;  // edge tiles
  }
  if (tile != TILE_128) return (tiles + cus - 1) / cus * round[tile];
  if (tile_stages(tile, tiles, cus) == 4) return round[4];
  return tiles / (2 * cus) * round[2] + (rest == 0 ? 0u : rest <= cus ? round[3] : round[2]);
}
inline int tile_plan(const TileProblem& p, size_t cus, uint32_t* split) {
  int best = TILE_256;
  uint64_t cost = tile_cost(TILE_256, p, cus);
  for (int t = TILE_192; t <= TILE_128; ++t) {
    const uint64_t c = tile_cost(t, p, cus);
    if (c < cost) {
      cost = c;
      best = t;
    }
  }
  // complete rounds of 256 x 256 tiles, then the remaining columns in 128 x 128 tiles
  if (p.pairs == 1 && ragged_round_split(p.M, p.N, cus, split)) {
    TileProblem left = p, right = p;
    left.N = *split;
    right.N = p.N - *split;
    if (tile_cost(TILE_256, left, cus) + tile_cost(TILE_128, right, cus) + (p.K < 1024 ? 25u : 10u) < cost) best = TILE_SPLIT;
  }
  return best;
}

// The launches of a plan, one after the other on columns [begin, end) each; returns how many (one or two).
struct TileLaunch {
  int tile, stages;
  uint32_t begin, end;
};
inline int tile_launches(int plan, const TileProblem& p, size_t cus, uint32_t split, TileLaunch (&out)[2]) {
  auto one = [&](int tile, size_t begin, size_t end) {
    return TileLaunch{tile, tile_stages(tile, tile_count(tile, p.M, end - begin, p.pairs), cus), (uint32_t)begin, (uint32_t)end};
  };
  if (plan != TILE_SPLIT) {
    out[0] = one(plan, 0, p.N);
    return 1;
  }
  out[0] = one(TILE_256, 0, split);
  out[1] = one(TILE_128, split, p.N);
  return 2;
}

// The kernel that a launch runs.  The large tiles use the ring of operand slots, but for a single round of 256 x 192 tiles with a short K, which
// has no next tile to request and is over before the ring's earlier requests pay (us, two stages / ring: 4096 x 3072 x 512 17.1 / 18.6, 1537 x
// 6197 x 704 19.2 / 19.7, 2048 x 5888 x 768 20.9 / 21.6, 1000 x 8000 x 512 16.4 / 16.5, 2048 x 6144 x 512 16.2 / 16.2; 4096 x 3072 x 960 24.0 / 23.9; more than
// a round, 4096 x 4000 x 512 29.1 / 27.6).  128 x 128 tiles run with four LDS stages or two, or two of them
// as a 256 x 128 tile, one to a compute unit with three stages.  That is three quarters of the tile loads, but an epilogue that nothing
// hides, so where K is long (us, 128 x 128 / 256 x 128: 2048 x 4096 x 1024 18.2 / 18.9, 1500 x 5000 x
// 2048 27.1 / 28.2, 1000 x 7000 x 3000 36.0 / 36.1, 2048 x 4096 x 4096 51.1 / 50.5, x 11008 135.7 / 123.8; as the remaining columns of 8192 x
// 11008 x 4096 500 / 486), and where that takes no more rounds (M of 128 more than a multiple of 256).
enum : int { FORM_RING = 0, FORM_TWO = 2, FORM_PAIRED = 3, FORM_FOUR = 4 };
inline int tile_form(const TileProblem& p, const TileLaunch& l, size_t cus) {
  if (l.tile == TILE_192 && p.K <= 768 && tile_count(TILE_192, p.M, l.end - l.begin, p.pairs) <= cus) return FORM_TWO;
  if (l.tile != TILE_128) return FORM_RING;
  if (l.stages == 4) return FORM_FOUR;
  if (p.K < 4096) return FORM_TWO;
  const uint64_t cols = (l.end - l.begin + 127) / 128 * p.pairs, ones = (p.M + 127) / 128 * cols, twos = (p.M + 255) / 256 * cols;
  return (twos + cus - 1) / cus <= (ones + 2 * cus - 1) / (2 * cus) ? FORM_PAIRED : FORM_TWO;
}

// The tile that a launch of FORM_FOUR runs: 64 x 64 or 128 x 64 where each of them still has a compute unit to itself.  us, weights from memory,
// 128 x 128 / 128 x 64 / 64 x 64 and two of these on some compute units: 512 x 2006 x 1024 10.7 / 8.2 / 6.4, x 8000 44.9 / 34.4 / 25.1; 1000 x 2000 x 256
// binary32 6.5 / 5.3, x 4096 26.3 / 21.2; 900 x 1100 (270 tiles of 64 x 64) x 1024 10.7 / 8.2 / 8.0, x 4096 26.2 / 19.4 / 21.9; 128 x 64 two to a
// compute unit 472 x 5928 x 2102 17.1 / 20.4.
enum : int { FINE_128 = 0, FINE_HALF = 1, FINE_64 = 2 };
inline int fine_tile(const TileProblem& p, const TileLaunch& l, size_t cus) {
  const uint64_t cols = (l.end - l.begin + 63) / 64 * p.pairs;
  return (p.M + 63) / 64 * cols <= cus ? FINE_64 : (p.M + 127) / 128 * cols <= cus ? FINE_HALF : FINE_128;
}

// Most tiles of a launch: its threads, 256 for each workgroup, are counted in 32 bits, and its workgroups are dealt out in
// whole rounds of the dies (kXcds).  The large tiles walk with one workgroup per compute unit, so that there only the tile number would be
// limited; that is made use of for the squared error in 256 x 256 tiles, which has several products to a launch, and what other launches
// refuse stays as it is.
constexpr uint64_t kMaxWorkgroups = 0xFFFFFFFFull / 256 / 8 * 8;
inline uint64_t most_tiles(int tile, bool sqerr) { return tile == TILE_256 && sqerr ? 0x7FFFFFF0ull : kMaxWorkgroups; }

// Pairs of a scale search (na x nb error products) that one launch takes: all of them, one row of nb, or a single one
// (0: not even that).  tile: the tile asked for, or -1 for the plan's own choice, which goes by the pairs of the launch.
inline uint32_t pairs_per_launch(int tile, size_t M, size_t N, size_t K, uint32_t na, uint32_t nb, size_t cus) {
  auto fits = [&](size_t pairs) {
    uint32_t split = 0;
    const int t = tile >= 0 ? tile : tile_plan(TileProblem{M, N, K, pairs, OUT_ERR}, cus, &split);
    return t == TILE_SPLIT || tile_count(t, M, N, pairs) <= most_tiles(t, true);  // a split: one part walks, the other has at most two rounds
  };
  return fits((size_t)na * nb) ? na * nb : fits(nb) ? nb : fits(1) ? 1u : 0u;
}

// Products with at most this many rows on one side run straight from the codes in hif8_gemm_ws_* when the expanded operands
// would go to the small-tile kernel: up to here both operand kinds have one K split (small_choice) and so the same bits.  Above it
// the codes are expanded first, which is faster for large products, or asked for the expanded operands' split, by price (small_from_codes).
constexpr size_t kSmallCodesRows = 128;

// Which problems go to the small-tile kernel (hif8_gemm_s.hip) although the tiled kernels could run them.  The tiled kernels
// walk all of K however few tiles there are, so their time is a few us plus K (up to 256 tiles of 128 x 128: 5.9 us + 0.013
// us * K on codes, 3.8 us + 0.005 us * K on expanded operands with their four LDS stages); the small-tile kernel's goes with
// M N K.  s: the shorter side, l: the longer one.  These lines were drawn with small_plan()'s tiles against 128 x 128 tiles that took a quarter longer on
// codes; both kernels are faster now, and small_route() moves products across them by price.  In us, small tiles / tiled, on either side
// of each line, as it was drawn:
//   codes        64 x 16384 x 64 8.2 / 8.2, 32000 9.6 / 8.9; 128 x 5120 x 64 7.8 / 8.2, 10240 13.4 / 8.4; 64 x 26624 x 512 14.7 /
//                17.2; 256 x 10240 x 1024 36 / 28; 512 x 3328 x 4096 64 / 90, 5120 104 / 89; 32 x 200000 x 64 20 / 32
//   expanded     256 x 4096 x 512 9.2 / 7.0, x 1024 10.1 / 9.4, x 2048 13.6 / 14.4, 5120 19.4 / 14.8; 128 x 2560 x 512
//                6.4 / 6.8; 128 x 8192 x 4096 23.4 / 26; 32 x 20480 x 1024 10.5 / 10.6
// Up to 128 rows hif8_gemm_ws_* goes by the line of the expanded operands, whose bits it gives, and saves the expansion on this
// side of it (expansion and tiled kernel / codes in small tiles: 64 x 20480 x 512 24 / 12, 128 x 8192 x 1024 24.5 / 12.3, 128 x 8192 x
// 128 9.2 / 7.9), so the line lies farther out there: 128 x 8192 x 128 expanded 6.1 / 4.9, 64 x 2048 x 64 5.1 / 4.0, 64 x 20480 x
// 512 8.7 / 7.1.
// The squared error costs the small-tile kernel an atomic per workgroup, all on one address (10 us for the thousand workgroups
// that walk), so there it wants a larger K:
//   codes        8 x 8000 x 64 9.9 / 10.1; 8 x 32000 x 256 17.2 / 15.9, x 512 17.9 / 20.5; 32 x 10240 x 64 9.5 / 10.3, 20480 x 256
//                14.8 / 14.8; 64 x 8000 x 128 12.7 / 11.4, x 256 12.9 / 13.7; 128 x 5120 x 64 11.9 / 9.9, x 256 11.8 / 13.8; 256 x
//                5120 x 512 20.5 / 19.2, x 1024 24.9 / 29.0
//   expanded     8 x 8000 x 512 9.9 / 7.8, x 1024 10.1 / 10.2; 32 x 10240 x 512 8.8 / 8.4, x 1024 9.3 / 10.8; 48 x 5120 x 256 8.4 /
//                8.1, x 1024 9.6 / 11.7; 128 x 5120 x 1024 12.2 / 10.0, x 2048 15.4 / 15.0; 512 x 2048 x 2048 17.1 / 15.2, x 4096
//                24.7 / 26.7
inline bool small_problem(size_t M, size_t N, size_t K, bool codes, bool sqerr) {
  const size_t s = M < N ? M : N, l = M < N ? N : M;
  auto tiles = [&](size_t tm, size_t tn) { return ((M + 16 * tm - 1) / (16 * tm)) * ((N + 16 * tn - 1) / (16 * tn)); };
  if (codes) {
    if (s > 32 && l > (size_t)(K < 1024 ? 24 : 33) * 65536 / s) return false;
    if (sqerr) {
      if (s <= 16) return l <= 6144 || l > 65536 || K >= (l < 25600 ? l / 64 : 400);
      if (s <= 32) return l <= 6144 || (l > 8192 && l <= 16384) || K >= (l <= 8192 ? 128 : 400);
      if (s <= 64) return K >= (l <= 1024 ? 0 : l <= 2048 ? 64 : l <= 5632 ? 128 : l / 36);
      return K >= (s * l <= (size_t)1 << 17 ? 0 : s * l <= (size_t)1 << 19 ? 64 : s * l <= 900000 ? 200 : s * l <= (size_t)1 << 20 ? 400 : 1024);
    }
    return s <= 32 || K > 64 || (s <= 64 ? l <= 16384 : tiles(2, 4) <= 512);
  }
  if (s <= 32) {
    if (!sqerr || l <= 2048) return true;
    if (K >= 2048 && l >= ((size_t)160 << 20) / K) return true;  // 320 MB of the longer operand: more than the last-level cache
    return s <= 16 ? K * 8 >= l : K * 10 >= l && l <= 12288;
  }
  if (s <= 64) return sqerr ? l <= 1024 || (K >= 256 && K * 6 >= l && l <= 12288) : l <= 20480;
  if (s <= kSmallCodesRows) return sqerr ? l <= 1024 || (K >= 384 && K * 7 >= l * 2 && tiles(2, 4) <= 512) : l <= 1310720 / ((s + 31) / 32 * 32);
  return K >= (sqerr ? 2048 : 1024) && tiles(4, 4) <= (sqerr && K < 3072 ? 170 : 256);
}

// Tile (16 tm x 16 tn) and wavefronts per workgroup of the small-tile kernel.  The wavefronts split K, so a wavefront
// count is part of the result's rounding: below 128 rows it is the same for code and for expanded operands (there
// hif8_gemm_ws_* runs on the codes what hif8_gemm_expanded_* runs on expanded operands).  The smallest tiles win while
// one operand has few rows (8 x 11008 x 4096 on codes: 1 x 1 14 us, 1 x 2 17, 2 x 4 20); more rows want the operand
// reuse of larger ones, and fewer wavefronts once the tiles alone fill the chip (64 x 4096 x 4096: 2 x 2 with 16
// wavefronts 14.2 us, with 8 16.2; 64 x 11008 x 4096: 4 wavefronts 33.6, 16 41.8; 32 rows, 2 x 4 with 8 wavefronts / 2 x 2 with 4,
// codes and expanded: 32 x 40960 x 1024 25.3, 22.7 / 20.4, 16.3, 32 x 53248 x 2048 48, 45 / 38, 35, but 32 x 10240 x 11008 43, 41 /
// 70, 45, 32 x 32768 x 11008 96, 139 / 104, 149; 128 rows, 2 x 4 / 2 x 2 with 4: 128 x 8192 x 256 7.7, 6.3 / 8.0, 5.8, 128 x 10240 x 512
// 13.7, 8.7 / 12.6, 8.6, but x 4096 50, 30 / 55, 33).
// A workgroup has no more wavefronts than K has shares of kShareK elements, in powers of two, but at least four: one without a
// share adds nothing to the sum, and its staging area takes LDS that another workgroup could have, while its lanes help with the
// table and the sum (codes, expanded, us: 32 x 10240 x 128 in 1 x 2 tiles with 8 wavefronts / 4 6.7, 5.3 / 5.1, 3.8; 128 x 8192 x
// 64 with 4 / 1 7.8 / 9.7 on codes).  Where there are more tiles than the chip holds workgroups at a time, fewer than four, too
// (codes, 8 / as many as shares: 8 x 200000 x 64 42.1 / 14.7; 64 x 32000 x 64 13.8 / 9.3).
struct SmallPlan {
  uint32_t tm, tn, waves;
};
constexpr size_t kShareK = 128;
// Workgroups that 256 compute units hold at a time: 160 KiB of LDS (table; per wavefront a staging area of 2 KiB for each
// 16-row block), and on each of the four SIMDs as many wavefronts as the registers of a tile allow.
inline size_t small_resident(uint32_t tm, uint32_t tn, uint32_t waves, bool codes) {
  const uint32_t by_lds = 160u * 1024u / (512u + waves * (tm + tn) * 2048u), blocks = tm * tn;
  const uint32_t by_regs = 4u * (blocks == 1u ? 6u : blocks == 2u ? 5u : blocks == 4u ? 4u : blocks == 8u && !codes ? 3u : 2u) / waves;
  return 256u * (by_lds < by_regs ? by_lds : by_regs);
}
// The same on one compute unit, for the price: by the registers of the kernels that store as they are built now.  small_plan()'s wavefronts, which are part
// of a result's rounding, stay with the number above, from earlier kernels.  By the registers that they take (a wavefront's, codes / expanded: 1 x 1 67 (half-row form 75) / 60, 1 x 2 87 / 76, 1 x 3 107 /
// 96, 2 x 2 120 / 112, 2 x 3 140 / 130, 2 x 4 160 / 152, 3 x 4, 4 x 3 and 4 x 4 192 to 236).
constexpr uint32_t small_resident_stored(const SmallPlan& p, bool codes) {
  const uint32_t by_lds = 160u * 1024u / (512u + p.waves * (p.tm + p.tn) * 2048u), blocks = p.tm * p.tn;
  const uint32_t per_simd = blocks == 1u ? (codes ? 6u : 8u) : blocks == 2u ? (codes ? 5u : 6u) : blocks == 3u ? (codes ? 4u : 5u) : blocks == 4u ? 4u : blocks <= 8u ? 3u : 2u;
  const uint32_t by_regs = 4u * per_simd / p.waves, most = by_lds < by_regs ? by_lds : by_regs;
  return most == 0u ? 1u : most;
}
// What a kernel can be launched with: 1024 lanes up to four blocks, 768 up to eight, 512 above, and LDS for the wavefronts' areas.
constexpr bool small_fits(const SmallPlan& p) {
  return p.waves <= (p.tm * p.tn <= 4u ? 16u : p.tm * p.tn <= 8u ? 12u : 8u) && 512u + p.waves * (p.tm + p.tn) * 2048u <= 160u * 1024u;
}
// The wavefronts' shares of K in pairs of units of 64, 128 codes: whole cache lines for every wavefront, unless single units give the longest
// share fewer of them (us, single units / pairs, the weight from memory, eight wavefronts: 2 x 4096 x 11008, 172 units, 14.7 / 14.4, 8 x 4096 x 2624, 41,
// 6.2 / 6.0, but 8 x 4096 x 5200, 82, 9.1 / 9.3, 509 x 1003 x 2049, 33, 15.7 / 18).
inline bool small_by_pairs(size_t K, uint32_t waves) {
  const size_t units = (K + 63) / 64, pairs = (units + 1) / 2;
  return (units + waves - 1) / waves >= 2 * ((pairs + waves - 1) / waves);
}
inline SmallPlan small_plan(size_t M, size_t N, size_t K, bool codes, bool sqerr) {
  auto tiles = [&](size_t tm, size_t tn) { return ((M + 16 * tm - 1) / (16 * tm)) * ((N + 16 * tn - 1) / (16 * tn)); };
  const size_t s = M < N ? M : N, l = M < N ? N : M, ld = (K + 63) / 64 * 64;  // codes plan as their expansion does
  auto plan = [&](uint32_t tm, uint32_t tn, uint32_t waves) {
    auto spare = [&] { return waves / 2u * kShareK >= ld; };
    while (waves > 4u && spare()) waves /= 2u;
    if (tiles(tm, tn) > small_resident(tm, tn, waves, codes))
      while (waves > 1u && spare()) waves /= 2u;
    return SmallPlan{tm, tn, waves};
  };
  const bool short_k = ld <= 4 * kShareK && !sqerr;  // four wavefronts have all of K: the smaller tiles (fewer atomics with the larger ones)
  if (s <= 16) return plan(1, 1, 8);
  if (s <= 32) {
    if (tiles(2, 4) < 128) return plan(1, 2, 8);
    return (tiles(2, 4) <= 256 && !short_k) || l * ld >= (size_t)300 << 20 ? plan(2, 4, 8) : plan(2, 2, 4);
  }
  if (s <= 64) return plan(2, 2, tiles(2, 2) <= 256 ? 16 : 4);
  if (s <= kSmallCodesRows && short_k) return plan(2, 2, 4);
  if (s <= kSmallCodesRows || (codes && M * N <= (size_t)33 * 65536)) return plan(2, 4, tiles(2, 4) <= 256 ? 8 : 4);
  return plan(4, 4, !codes && tiles(4, 4) <= 256 ? 8 : 4);
}

// Time of the small-tile kernel with stored results, us, as far as the tile and the wavefronts decide it.  A compute unit has `turns` tiles at most.
// Either its LDS (stages, look-ups, fragments) is busy with all their rows; or, with few wavefronts on it, each of them works off its share of
// K one stage after the other, and as many tiles as fit at a time go side by side; then the partial tiles are added.  The constants
// are a least-squares fit, in the logarithm, to 296 shapes of 4 to 1000 rows on codes and 178 on expanded operands, weights from memory, each in up to 40
// tiles and numbers of wavefronts: 13 and 12 % off on average.
constexpr size_t kPricedUnits = 256;  // compute units of the chip that the prices of the small tiles, and of what they are compared with, were measured on
struct SmallRates {
  double base, lds, wave, unit, turn, add, memory;
};
constexpr SmallRates kSmallRates[2] = {{1.88, 0.024, 0.078, 0.048, 1.49, 0.042, 1.36}, {2.2, 0.036, 0.2125, 0.0, 1.36, 0.054, 0.97}};  // expanded, codes
struct SmallCost {
  size_t M, N;
  bool codes;
  uint32_t units, tiles_m[5], tiles_n[5];  // of 16 to 64 rows and columns
  double memory;                           // fourth power of the memory's part

  SmallCost(size_t m, size_t n, size_t k, bool c) : M(m), N(n), codes(c), units((uint32_t)((k + 63) / 64)) {
    auto count = [](uint32_t (&t)[5], size_t rows) {
      t[1] = (uint32_t)((rows + 15) / 16);
      t[2] = (t[1] + 1) / 2;
      t[3] = (t[1] + 2) / 3;
      t[4] = (t[1] + 3) / 4;
    };
    count(tiles_m, m);
    count(tiles_n, n);
    memory = fourth((double)(m + n) * units * (codes ? 64.0 : 128.0) / 6e6 * kSmallRates[c ? 1 : 0].memory);
  }
  static double fourth(double x) { return x * x * x * x; }
  // what plans are compared by: the largest of the parts, more where two are close.  In two steps, the tile's and the wavefronts'
  struct Tile {
    double rows, lds;  // in blocks of 16 (the half-row form); fourth power
    uint32_t turns;
  };
  Tile tile(uint32_t tm, uint32_t tn) const {
    const uint64_t tiles = (uint64_t)tiles_m[tm] * tiles_n[tn], of_unit = (tiles + (kPricedUnits - 1)) / kPricedUnits;
    const uint32_t turns = of_unit > 0xFFFFFF00u ? 0xFFFFFF00u : (uint32_t)of_unit;
    const double rows = (codes && M <= 8 && tm * tn == 1u ? 0.5 : (double)tm) + tn;
    return Tile{rows, fourth((double)turns * units * rows * kSmallRates[codes ? 1 : 0].lds), turns};
  }
  double score(const Tile& t, const SmallPlan& p, uint32_t share, uint32_t resident) const {
    const SmallRates& r = kSmallRates[codes ? 1 : 0];
    const uint32_t rounds = t.turns <= resident ? 1u : (t.turns + resident - 1) / resident;
    return t.lds + fourth((double)rounds * (share * (t.rows * r.wave + r.unit) + r.turn + r.add * p.waves * (p.tm * p.tn))) + memory;
  }
  double score(const SmallPlan& p) const { return score(tile(p.tm, p.tn), p, (units + p.waves - 1) / p.waves, small_resident_stored(p, codes)); }
  double us(const SmallPlan& p) const { return kSmallRates[codes ? 1 : 0].base + std::sqrt(std::sqrt(score(p))); }
};

// Tile and wavefronts: the cheapest by SmallCost of the tiles that are built.  What that changes against small_plan(), whose lines were measured at
// few sizes: a number of tiles just below that of the compute units, or with each of them two, instead of a little more; small tiles with many
// wavefronts where there are few tiles and a long K; three blocks of columns or rows.  Measured (us, small_plan / now, weights from memory): codes 42 x 816 x 3693
// 14.2 / 7.7, 46 x 5162 x 7536 38 / 28, 48 x 10642 x 8528 63 / 45, 106 x 6133 x 7600 61 / 41, 173 x 3951 x 6832 53 / 36; expanded 80 x 1644 x 2528 10.0 /
// 6.9, 128 x 674 x 7456 18.8 / 10, 200 x 594 x 4176 18.6 / 7.1, 400 x 835 x 3456 16.9 / 10.  Over the shapes above it is 1.8 % (codes) and 3 %
// (expanded) behind the best tile for each; small_plan 22 and 26 %.
// The wavefronts decide the bits.  Up to kSmallCodesRows rows they are those of the code operands, for both kinds; the squared error takes the wavefronts that the stored product has here, with
// the tiles of its kernels and 0.01 us for each workgroup's atomic.  With fewer than four wavefronts (more tiles than the chip holds, a short K)
// small_plan() stands.  waves != 0: that number is asked for.
// Another plan than small_plan()'s has to promise 7 % (the fit's own error; without that 12 of 296 shapes on codes lost 4 to 10 %, with it 2).  No 16
// wavefronts up to 16 rows: 5 to 7 % better or worse from shape to shape.
constexpr double kSmallGain = 0.93;
// 16 wavefronts have to promise 12 % over 8 (here fourth powers): where they do less, codes gain nothing and expanded operands, which take over the
// split, lose 8 to 10 % (24 x 3398 x 5600 12.9 / 13.0 and 9.0 / 10.0).
constexpr double kSixteen = 1.6;
// A ninth wavefront where that takes a quarter or more of the stages off the longest share: 17, 33 or 49 units of K and a few more, in tiles of six or eight blocks, of
// which a compute unit has one (codes above kSmallCodesRows rows; us, 2 x 4 tiles with eight / nine: 509 x 1003 x 1081 10.7 / 9.9, x 2049 15.2 / 14.0, x 3100 17.5 / 16.6, 700 x 1400 x 2100
// 26.9 / 24.6; one stage of five less, x 4100, 20.8 / 21.2).
constexpr double kNineGain = 0.92;
inline bool ninth_wave(const SmallPlan& p, size_t K) {
  auto stages = [&](size_t waves) { return ((K + 63) / 64 + 2 * waves - 1) / (2 * waves); };
  return p.waves == 8u && p.tm * p.tn > 4u && p.tm * p.tn <= 8u && stages(9) * 4 <= stages(8) * 3;
}
// What the host takes for a launch: with less on the GPU nothing is gained, and the look at all tiles would come on top.
// Up to 16 rows it pays from larger products on (16 x 4447 x 7104 16.9 us, now 14.7, 16 x 10257 x 10453 41.8, 33.5; 16 x 1131 x 4272 8.0, 8.0).
constexpr double kLaunchBound = 5.2, kFewRowsBound = 9.0;
constexpr uint32_t kSmallWaveCounts = 4, kSmallTileCount = 9;
constexpr uint32_t kSmallWaves[kSmallWaveCounts] = {16, 9, 8, 4};
constexpr uint32_t kSmallTiles[kSmallTileCount][2] = {{1, 1}, {1, 2}, {1, 3}, {2, 2}, {2, 3}, {2, 4}, {3, 4}, {4, 3}, {4, 4}};
struct SmallResident {  // workgroups of a compute unit; 0: cannot be launched
  uint32_t of[2][kSmallTileCount][kSmallWaveCounts];
  constexpr SmallResident() : of{} {
    for (uint32_t c = 0; c < 2; ++c)
      for (uint32_t n = 0; n < kSmallTileCount; ++n)
        for (uint32_t i = 0; i < kSmallWaveCounts; ++i) {
          const SmallPlan p{kSmallTiles[n][0], kSmallTiles[n][1], kSmallWaves[i]};
          of[c][n][i] = small_fits(p) ? small_resident_stored(p, c == 1) : 0u;
        }
  }
};
constexpr SmallResident kSmallResident;
inline double atomics(const SmallCost& c, const SmallPlan& p, size_t K) {  // of a squared error, see launch_s
  const double wgs = (double)c.tiles_m[p.tm] * c.tiles_n[p.tn];
  return K < 4096 && wgs > 1024.0 ? 1024.0 : wgs;
}
inline SmallPlan small_choice(size_t M, size_t N, size_t K, bool codes, bool sqerr = false, uint32_t waves = 0) {
  const size_t s = M < N ? M : N, ld = (K + 63) / 64 * 64;
  const SmallPlan base = small_plan(M, N, K, codes, sqerr);
  if (waves == 0u) {
    const bool both = s <= kSmallCodesRows;  // kinds that have to agree
    if ((both || codes) && small_plan(M, N, K, true, false).waves < 4u) return base;
    if ((both || !codes) && small_plan(M, N, K, false, false).waves < 4u) return base;
    if (both && (!codes || sqerr)) waves = small_choice(M, N, K, true).waves;
    else if (sqerr) waves = small_choice(M, N, K, codes).waves;
  }
  const SmallCost cost(M, N, ld, codes);
  const bool may_stay = waves == 0u || waves == base.waves;
  const double base_us = cost.us(base);
  if (may_stay && base_us < (s <= 16 ? kFewRowsBound : kLaunchBound)) return base;
  SmallPlan best = base;
  double least = 1e300;
  uint32_t share[kSmallWaveCounts];
  for (uint32_t i = 0; i < kSmallWaveCounts; ++i) share[i] = (cost.units + kSmallWaves[i] - 1) / kSmallWaves[i];
  for (uint32_t n = 0; n < kSmallTileCount; ++n) {
    const uint32_t tm = kSmallTiles[n][0], tn = kSmallTiles[n][1];
    if (16u * (tm - 1u) >= M || 16u * (tn - 1u) >= N || (sqerr && (tm == 3u || tn == 3u))) continue;  // a block outside the matrix; tiles not built
    const SmallCost::Tile t = cost.tile(tm, tn);
    if (t.lds + cost.memory >= least) continue;
    for (uint32_t i = 0; i < kSmallWaveCounts; ++i) {
      const uint32_t w = kSmallWaves[i], resident = kSmallResident.of[codes ? 1 : 0][n][i];
      if (resident == 0u || (w == 9u ? waves != 9u : w == 16u && s <= 16)) continue;
      if (waves != 0u ? w != waves : w > 4u && w / 2u * kShareK >= ld) continue;  // no wavefronts without a share
      const SmallPlan p{tm, tn, w};
      const double c = (cost.score(t, p, share[i], resident) + (sqerr ? SmallCost::fourth(0.01 * atomics(cost, p, K)) : 0.0)) * (w == 16u ? kSixteen : 1.0);
      if (c < least) {
        best = p;
        least = c;
      }
    }
  }
  const bool nine = codes && !sqerr && waves == 0u && s > kSmallCodesRows;
  if (may_stay && cost.us(best) > kSmallGain * base_us * (nine && ninth_wave(base, K) ? kNineGain : 1.0)) best = base;
  if (nine && ninth_wave(best, K)) best.waves = 9;
  return best;
}

// Tiles of the code-operand kernel, one workgroup per compute unit: the shortest sum of rounds of 256 workgroups, a round at the price
// below, fitted to 206 shapes with weights from memory (4 % rms error; from the caches a round at K = 4096 takes 60, 86 and 126 us).  Where
// the complete rounds of 256 x 256 tiles leave some columns over, those may go to smaller tiles in a second launch.
enum : int { CODES_128 = 0, CODES_TALL = 1, CODES_WIDE = 2, CODES_256 = 3 };  // 128 x 128, 256 x 128, 128 x 256, 256 x 256
struct CodesLaunch {
  int tile;
  uint32_t begin, end;  // columns
};
inline double codes_tile_us(int tile, size_t M, size_t N, size_t K, size_t cus) {
  const uint64_t bm = tile == CODES_TALL || tile == CODES_256 ? 256 : 128, bn = tile == CODES_WIDE || tile == CODES_256 ? 256 : 128;
  const uint64_t rounds = (((M + bm - 1) / bm) * ((N + bn - 1) / bn) + cus - 1) / cus;
  const double k = (double)K;
  return (double)rounds * (tile == CODES_128 ? 5.9 + 0.013 * k : tile == CODES_256 ? 13.0 + 0.0303 * k : 10.2 + 0.0195 * k);
}
inline int codes_tile(size_t M, size_t N, size_t K, size_t cus, double* us) {
  int best = CODES_128;
  *us = codes_tile_us(CODES_128, M, N, K, cus);
  for (int tile = CODES_TALL; tile <= CODES_256; ++tile) {
    const double t = codes_tile_us(tile, M, N, K, cus);
    if (t < *us) *us = t, best = tile;
  }
  return best;
}
inline int codes_launches(size_t M, size_t N, size_t K, size_t cus, CodesLaunch (&out)[2]) {
  double us = 0.0, right = 0.0;
  out[0] = CodesLaunch{codes_tile(M, N, K, cus, &us), 0u, (uint32_t)N};
  uint32_t split = 0;
  if (!ragged_round_split(M, N, cus, &split)) return 1;
  const int tile = codes_tile(M, N - split, K, cus, &right);
  if (codes_tile_us(CODES_256, M, split, K, cus) + right + 4.0 >= us) return 1;
  out[0] = CodesLaunch{CODES_256, 0u, split};
  out[1] = CodesLaunch{tile, split, (uint32_t)N};
  return 2;
}

// Products that go to the small-tile kernel: small_problem()'s, whose lines were drawn with small_plan() and 128 x 128 tiles, but for the stored ones on the far side of
// those lines whose price is below the tiled kernels'.
// Codes: by price on either side (us, weights from memory, tiled / small tiles: 370 x 1071 x 6608 107 / 29, but 1428 x
// 2166 x 3792 66 / 75, 840 x 2996 x 6896 110 / 118); of 260 shapes the choice loses 0.3 % to the better one in the mean.
// Expanded operands of more than kSmallCodesRows rows: by price on either side where 64 x 64 tiles have a compute unit each (3.0 + 0.00275 K us; tiled / small
// tiles: 512 x 2006 x 4096 14.7 / 19.9, 256 x 3163 x 2048 8.9 / 13.0, but 512 x 1000 x 8000 24 / 21, 200 x 594 x 4176 14 / 7.1).  Where the two are within 15 % the
// product through the workspace, which has to give the same bits, decides: from the codes, or expanded first.  With more tiles the lines hold, beyond which
// the small tiles' price is up to a third too low for tiles of six and more blocks (tiled / small tiles: 187 x 8860 x 400 7.7 / 10.2, 283 x 6438 x 3776 29.4 /
// 36.1, 148 x 10790 x 5968 44.7 / 54.0, 258 x 4012 x 992 7.7 / 10.9, 582 x 1998 x 462 6.4 / 8.5).
// The squared error leaves the small tiles where the stored product does: it is that of the same bits, and faster (expanded, small tiles / tiled: 762 x 1119 x
// 5760 28.4 / 20.9, 1915 x 312 x 3136 19.1 / 13.2, 635 x 1081 x 8896 34.8 / 28.1, 2352 x 349 x 11200 49.6 / 49.8).  It does not follow into them, where its
// atomics come on top (expanded 501 x 951 x 832 11.3 / 7.2, 618 x 338 x 832 7.6 / 6.3; codes 591 x 3051 x 624 22.6 / 15.8, 415 x 8977 x 9856 210 / 213), so there
// it is the error of the tiled kernels' sum, whose rounding differs.
inline double expand_us(size_t M, size_t N, size_t ld) { return 2.5 + (double)(M + N) * (double)ld * 3.0 / 5.5e6; }
// The plan that the prices are of comes with the answer, so that a call searches once (0.15 to 0.3 us on the host, next to products of a few us).
struct SmallRoute {
  bool small;
  SmallPlan plan;        // where small
  SmallPlan from_codes;  // of the workspace's product, with the wavefronts of `plan`; waves 0: not looked for
};
inline SmallRoute small_route(size_t M, size_t N, size_t K, bool codes, bool sqerr) {
  const SmallPlan none{0, 0, 0};
  const bool small = small_problem(M, N, K, codes, sqerr);
  const size_t s = M < N ? M : N;
  auto tiles = [&](size_t side) { return ((M + side - 1) / side) * ((N + side - 1) / side); };
  auto by_lines = [&] { return small ? SmallRoute{true, small_choice(M, N, K, codes, sqerr), none} : SmallRoute{false, none, none}; };
  if (s <= (codes ? 32 : kSmallCodesRows) || (codes ? tiles(128) > 2 * kPricedUnits : tiles(64) > kPricedUnits) || K < 320) return by_lines();  // a shorter K gains little (256 x 1048 x 240 5.6 / 5.1)
  if (sqerr) {
    if (codes || !small || !small_problem(M, N, K, false, false) || small_route(M, N, K, false, false).small) return by_lines();
    return SmallRoute{false, none, none};
  }
  SmallRoute r{true, small_choice(M, N, K, codes), none};
  if (codes && small) return r;
  const double us = SmallCost(M, N, K, codes).us(r.plan);
  if (codes) {
    double tiled = 0.0;
    codes_tile(M, N, K, kPricedUnits, &tiled);
    r.small = us < tiled;
    return r;
  }
  const double tiled = 3.0 + 0.00275 * (double)K;
  if (us <= 0.87 * tiled || us >= 1.15 * tiled || r.plan.waves < 4u) {
    r.small = us < tiled;
    return r;
  }
  r.from_codes = small_choice(M, N, K, true, false, r.plan.waves);
  r.small = SmallCost(M, N, K, true).us(r.from_codes) < tiled + expand_us(M, N, K);
  return r;
}

// A product through the workspace, of operands whose expansions would go to the small-tile kernel (x) with more than kSmallCodesRows rows: straight from the codes with
// the expansions' wavefronts, which gives their bits, where that is faster than writing them (2.5 us and 3 bytes an element; us, expanded first / from
// the codes: 130 x 1477 x 2730 20.2 / 11.4, 168 x 981 x 1216 14.6 / 8, 454 x 1143 x 5168 28 / 25).  False: expand.
inline bool small_from_codes(size_t M, size_t N, size_t K, const SmallRoute& x, SmallPlan* plan) {
  if (x.plan.waves < 4u) return false;
  const size_t ld = (K + 63) / 64 * 64;
  *plan = x.from_codes.waves != 0u ? x.from_codes : small_choice(M, N, K, true, false, x.plan.waves);
  return SmallCost(M, N, K, true).us(*plan) < SmallCost(M, N, ld, false).us(x.plan) + expand_us(M, N, ld);
}

// Workgroup -> tile of the expanded-operand kernel.  The hardware deals consecutive workgroups round-robin over the
// kXcds accelerator dies (XCDs), each with its own L2.  Workgroup b therefore takes tile number
// (b % kXcds) * per_xcd + b / kXcds of a tile order that walks groups of `group` tile rows column by column: the
// workgroups resident on one die at a time then cover a compact group x (a few) block of tiles and share their
// operand panels in that die's L2, whatever tiles_n is.  Of 256 x 128 tiles a die holds 32: 4 x 8 of them take 2048 operand rows, 8 x 4
// 2560, and a row of the first operand is asked for by fewer dies at a time (2048 x 4096 x 11008 from cold memory 159 us with groups of 8, 155
// with 4).  The wider tiles stay with 8: groups of 4 gave 1 % at 8192^3, but a product with a short K right behind its expansions took
// longer (with expansions, groups of 8 / 4: 1537 x 6197 x 688 31.5 / 34.5, 2011 x 4511 x 1168 38.7 / 42.5).
// 128 x 64 tiles, one to a compute unit, take the same with either (60 drawn products, groups of 8 over 4: 0.94 to 1.03, 1.001 in the mean).
// The launch has tile_order_grid() workgroups; returns false
// for the few at the end of the last die's share that have no tile.
constexpr uint32_t kXcds = 8;    // accelerator dies, each with an L2 of its own
constexpr uint32_t kGroupM = 8, kGroupPaired = 4;  // tile rows per group of the tile order; of 256 x 128 tiles
__host__ __device__ inline uint32_t tile_order_grid(uint32_t n_tiles) { return (n_tiles + kXcds - 1u) / kXcds * kXcds; }
__host__ __device__ inline bool tile_order(uint32_t b, uint32_t tiles_m, uint32_t tiles_n, uint32_t* tile_m, uint32_t* tile_n,
                                           uint32_t group = kGroupM) {
  const uint32_t n_tiles = tiles_m * tiles_n, per_xcd = (n_tiles + kXcds - 1u) / kXcds;
  const uint32_t t = (b % kXcds) * per_xcd + b / kXcds;
  if (t >= n_tiles) return false;
  const uint32_t grp = t / (group * tiles_n), first_m = grp * group;
  const uint32_t grp_rows = tiles_m - first_m < group ? tiles_m - first_m : group;
  const uint32_t in_grp = t - grp * (group * tiles_n);
  *tile_n = in_grp / grp_rows;
  *tile_m = first_m + (in_grp - *tile_n * grp_rows);
  return true;
}

}  // namespace hif8gemm
