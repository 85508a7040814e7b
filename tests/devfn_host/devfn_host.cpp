// CPU build of the HIP library's device-side bit logic (hif8_device.hpp), for tests that
// run where there is no GPU.  Test infrastructure: it lets the encode / decode bit
// manipulation be compared with the oracle on the CPU before (and besides) the GPU parity
// tests.  Not part of the product and never loaded by it.
#include <stdint.h>
#include <stddef.h>
#include <chrono>
#define HIF8_DEVICE_HOST_SHIM 1
#define __device__
#define __host__
#define __forceinline__ inline
static inline int __clz(int x) { return x == 0 ? 32 : __builtin_clz((unsigned)x); }
#include "../../paper_2409_16626_amd/csrc/hif8_device.hpp"
#include "../../paper_2409_16626_amd/csrc/hif8_axis_plan.hpp"
#include "../../paper_2409_16626_amd/csrc/hif8_gemm_split.hpp"
#include "../../paper_2409_16626_amd/csrc/hif8_multi_plan.hpp"

template <typename F>
static double fastest(int rounds, F call) {  // ns a call
  static volatile uint32_t sink;
  double best = 1e300;
  for (int r = 0; r < rounds; ++r) {
    const auto t0 = std::chrono::steady_clock::now();
    for (int i = 0; i < 200; ++i) sink = call();
    const double ns = std::chrono::duration<double, std::nano>(std::chrono::steady_clock::now() - t0).count() / 200;
    if (ns < best) best = ns;
  }
  return best;
}

extern "C" {
// per-tensor scale from an amax (the arithmetic of the scale kernels)
void devfn_scale_from_amax(const float* amax, float* out, size_t n, float target, int pow2) {
  for (size_t i = 0; i < n; ++i) out[i] = hif8dev::scale_from_amax_value(amax[i], target, pow2);
}
// whether the scale of a sample's amax holds for an amax, and that scale
int devfn_sample_holds(uint32_t sample, uint32_t amax, float target, float* scale) { return hif8dev::sample_holds(sample, amax, target, scale); }
// first tile of the piece that a sample reads, and the number of tiles from which on a tensor is sampled
uint64_t devfn_sampled_piece(uint64_t offset, uint64_t tiles) { return hif8conv::sampled_piece(offset, tiles); }
uint32_t devfn_sample_period() { return hif8conv::kSamplePeriod; }
// whether a per-channel call goes to the element kernels (what: 0 maxima, 1 encode, 2 decode)
int devfn_axis_by_elements(int what, int axis, size_t rows, size_t cols, size_t ve, uint64_t grid, uint32_t mode, int aligned) {
  return hif8calib::axis_by_elements(what, axis, rows, cols, ve, grid, mode, aligned != 0);
}
// which way a list is cast: 0 by sample, 1 in groups, 2 in four launches
int devfn_multi_cast_way(size_t count, uint64_t tiles, int host, int pow2, uint32_t mode) {
  return hif8conv::multi_cast_way(count, tiles, host != 0, pow2 != 0, mode);
}
// generic element-wise form (any rounding method, any source kind)
void devfn_encode_bits(const uint32_t* ybits, uint8_t* dst, size_t n, uint32_t mode, int srck,
                       uint64_t seed) {
  for (size_t i = 0; i < n; ++i) {
    const uint32_t t = hif8dev::sr_threshold(seed, (uint64_t)i);
    uint32_t c;
    if (srck == 0) c = hif8dev::encode_any<0>(ybits[i], mode, t);
    else if (srck == 1) c = hif8dev::encode_any<1>(ybits[i], mode, t);
    else c = hif8dev::encode_any<2>(ybits[i], mode, t);
    dst[i] = (uint8_t)c;
  }
}
// table-driven hybrid rounding (or simplified SR everywhere) of binary32 sources, then the TA code of
// the (representable) result
void devfn_encode_bits_hr_table(const uint32_t* ybits, uint8_t* dst, size_t n, uint32_t mode) {
  const bool ssr = (mode & 0xF) == hif8dev::kRmSSR;
  for (size_t i = 0; i < n; ++i) {
    const uint32_t y = ybits[i];
    if ((y & 0x7FFFFFFFu) > 0x7F800000u) { dst[i] = (uint8_t)hif8dev::nan_code(mode); continue; }
    const uint32_t r = hif8dev::hr_round_bits<0>(y, hif8dev::hr_exp_entry((y >> 23) & 0xFFu, ssr));
    dst[i] = (uint8_t)hif8dev::encode_alu<false, 0>(r & 0xFFF80000u, mode);
  }
}
// 16-bit sources, streaming form: clamped sum, then the truncating table's entry (the TA code of
// trunc_table_pattern())
void devfn_encode_bits_hr16_stream(const uint32_t* ybits, uint8_t* dst, size_t n, uint32_t mode, int srck) {
  const bool ssr = (mode & 0xF) == hif8dev::kRmSSR;
  for (size_t i = 0; i < n; ++i) {
    const uint32_t y = ybits[i];
    const hif8dev::HrExp16 p = hif8dev::hr16_exp_entry((y >> 23) & 0xFFu, ssr);
    const uint32_t lsb = srck == 1 ? hif8dev::hr16_lsb<1>(y) : hif8dev::hr16_lsb<2>(y);
    const uint32_t r = hif8dev::hr16_round_sum(y, lsb ? p.add1 : p.add0);
    dst[i] = (uint8_t)hif8dev::encode_alu<false, 0>(hif8dev::trunc_table_pattern(r >> 19), mode);
  }
}
// standard SR, streaming form: per-exponent table entry, add-and-truncate, then the TA code of the
// (representable) result
void devfn_encode_bits_sr_table(const uint32_t* ybits, uint8_t* dst, size_t n, uint32_t mode, uint64_t seed) {
  for (size_t i = 0; i < n; ++i) {
    const uint32_t y = ybits[i];
    if ((y & 0x7FFFFFFFu) > 0x7F800000u) { dst[i] = (uint8_t)hif8dev::nan_code(mode); continue; }
    const uint32_t r = hif8dev::sr_round_bits(y, hif8dev::sr_threshold(seed, (uint64_t)i), hif8dev::sr_exp_entry((y >> 23) & 0xFFu));
    dst[i] = (uint8_t)hif8dev::encode_alu<false, 0>(r & 0xFFF80000u, mode);
  }
}
void devfn_decode_bits(const uint8_t* codes, uint32_t* dst, size_t n) {
  for (size_t i = 0; i < n; ++i) dst[i] = hif8dev::decode_bits(codes[i]);
}
void devfn_narrow_bf16(const uint32_t* bits, uint16_t* dst, size_t n) {
  for (size_t i = 0; i < n; ++i) dst[i] = (uint16_t)hif8dev::narrow_bf16(bits[i]);
}
// workgroup -> tile of the expanded-operand GEMM: tile_m * tiles_n + tile_n, or 0xFFFFFFFF for a workgroup without a tile
uint32_t devfn_tile_order(uint32_t b, uint32_t tiles_m, uint32_t tiles_n) {
  uint32_t tm = 0, tn = 0;
  return hif8gemm::tile_order(b, tiles_m, tiles_n, &tm, &tn) ? tm * tiles_n + tn : 0xFFFFFFFFu;
}
uint32_t devfn_tile_order_paired(uint32_t b, uint32_t tiles_m, uint32_t tiles_n) {  // the same for 256 x 128 tiles
  uint32_t tm = 0, tn = 0;
  return hif8gemm::tile_order(b, tiles_m, tiles_n, &tm, &tn, hif8gemm::kGroupPaired) ? tm * tiles_n + tn : 0xFFFFFFFFu;
}
uint32_t devfn_tile_order_grid(uint32_t n_tiles) { return hif8gemm::tile_order_grid(n_tiles); }
// host-side launch planning of the GEMM kernels: returns the split column, or 0 for a single launch
uint32_t devfn_ragged_round_split(size_t M, size_t N, size_t cus) {
  uint32_t split = 0;
  return hif8gemm::ragged_round_split(M, N, cus, &split) ? split : 0u;
}
// code-operand GEMM: the launches of its plan, 3 numbers each: tile (0 = 128 x 128, 1 = 256 x 128, 2 = 128 x 256, 3 = 256 x 256), first column,
// end; returns how many
int devfn_codes_launches(size_t M, size_t N, size_t K, size_t cus, uint32_t* out) {
  hif8gemm::CodesLaunch l[2];
  const int n = hif8gemm::codes_launches(M, N, K, cus, l);
  for (int i = 0; i < n; ++i) {
    out[3 * i] = (uint32_t)l[i].tile;
    out[3 * i + 1] = l[i].begin;
    out[3 * i + 2] = l[i].end;
  }
  return n;
}
double devfn_codes_tile_us(int tile, size_t M, size_t N, size_t K, size_t cus) { return hif8gemm::codes_tile_us(tile, M, N, K, cus); }
// small-tile GEMM kernel: 100 * tile rows + 10 * tile columns (in blocks of 16) and wavefronts; whether a problem goes there
uint32_t devfn_small_plan(size_t M, size_t N, size_t K, int codes, int sqerr, uint32_t* waves) {
  const hif8gemm::SmallPlan p = hif8gemm::small_plan(M, N, K, codes != 0, sqerr != 0);
  *waves = p.waves;
  return p.tm * 100 + p.tn * 10;
}
// the kernel's choice (waves_asked != 0: that many wavefronts); whether a product goes there; wavefronts with which a product through
// the workspace is taken from the codes
uint32_t devfn_small_choice(size_t M, size_t N, size_t K, int codes, int sqerr, uint32_t waves_asked, uint32_t* waves) {
  const hif8gemm::SmallPlan p = hif8gemm::small_choice(M, N, K, codes != 0, sqerr != 0, waves_asked);
  *waves = p.waves;
  return p.tm * 100 + p.tn * 10;
}
int devfn_small_route(size_t M, size_t N, size_t K, int codes, int sqerr) { return hif8gemm::small_route(M, N, K, codes != 0, sqerr != 0).small; }
// the plan that comes with the route: as devfn_small_choice, 0 where the product does not go there
uint32_t devfn_small_route_plan(size_t M, size_t N, size_t K, int codes, int sqerr, uint32_t* waves) {
  const hif8gemm::SmallRoute r = hif8gemm::small_route(M, N, K, codes != 0, sqerr != 0);
  *waves = r.plan.waves;
  return r.small ? r.plan.tm * 100 + r.plan.tn * 10 : 0u;
}
uint32_t devfn_small_codes_waves(size_t M, size_t N, size_t K) {
  const hif8gemm::SmallRoute r{true, hif8gemm::small_choice(M, N, (K + 63) / 64 * 64, false), {0, 0, 0}};
  hif8gemm::SmallPlan p{0, 0, 0};
  return hif8gemm::small_from_codes(M, N, K, r, &p) ? p.waves : 0u;
}
// shortest time of a call, ns, over `rounds` of 200: the route with its plan (of the product, and of the workspace's where it is taken from the codes) / one search
double devfn_small_route_ns(size_t M, size_t N, size_t K, int codes, int rounds) {
  return fastest(rounds, [&] {
    const hif8gemm::SmallRoute r = hif8gemm::small_route(M, N, K, codes != 0, false);
    hif8gemm::SmallPlan p = r.plan;
    if (codes == 0 && r.small) hif8gemm::small_from_codes(M, N, K, r, &p);
    return p.waves;
  });
}
double devfn_small_choice_ns(size_t M, size_t N, size_t K, int codes, int rounds) {
  return fastest(rounds, [&] { return hif8gemm::small_choice(M, N, K, codes != 0).waves; });
}
int devfn_small_by_pairs(size_t K, uint32_t waves) { return hif8gemm::small_by_pairs(K, waves); }
int devfn_small_problem(size_t M, size_t N, size_t K, int codes, int sqerr) { return hif8gemm::small_problem(M, N, K, codes != 0, sqerr != 0); }
// the finest tile with which a launch of 128 x 128 tiles, one to a compute unit, keeps that: 0 = 128 x 128, 1 = 128 x 64, 2 = 64 x 64
int devfn_fine_tile(size_t M, uint32_t begin, uint32_t end, size_t pairs, size_t cus) {
  return hif8gemm::fine_tile(hif8gemm::TileProblem{M, end, 4096, pairs, 0}, hif8gemm::TileLaunch{hif8gemm::TILE_128, 4, begin, end}, cus);
}
// expanded-operand GEMM: the launches of its plan, 4 numbers each: tile (0 = 256 x 256, 1 = 256 x 192, 2 = 128 x 128), LDS
// stages, first column, end; returns how many
int devfn_tile_launches(size_t M, size_t N, size_t K, size_t pairs, size_t cus, int kind, uint32_t* out) {
  uint32_t split = 0;
  const hif8gemm::TileProblem p{M, N, K, pairs, kind};
  const int plan = hif8gemm::tile_plan(p, cus, &split);
  hif8gemm::TileLaunch l[2];
  const int n = hif8gemm::tile_launches(plan, p, cus, split, l);
  for (int i = 0; i < n; ++i) {
    out[4 * i] = (uint32_t)l[i].tile;
    out[4 * i + 1] = (uint32_t)l[i].stages;
    out[4 * i + 2] = l[i].begin;
    out[4 * i + 3] = l[i].end;
  }
  return n;
}
// the kernel that launch i of that plan runs: 0 = ring, 2 / 4 = so many LDS stages, 3 = 256 x 128
int devfn_tile_form(size_t M, size_t N, size_t K, size_t pairs, size_t cus, int kind, int asked, int i) {
  uint32_t split = 0;
  const hif8gemm::TileProblem p{M, N, K, pairs, kind};
  const int plan = asked >= 0 ? asked : hif8gemm::tile_plan(p, cus, &split);
  hif8gemm::TileLaunch l[2];
  return i < hif8gemm::tile_launches(plan, p, cus, split, l) ? hif8gemm::tile_form(p, l[i], cus) : -1;
}
uint32_t devfn_pairs_per_launch(int tile, size_t M, size_t N, size_t K, uint32_t na, uint32_t nb, size_t cus) {
  return hif8gemm::pairs_per_launch(tile, M, N, K, na, nb, cus);
}
}
