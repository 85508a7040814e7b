// Simulated HiF8 GEMM for problems with few output tiles (a handful of tokens against a weight matrix, small products)
// and for code matrices of any K and any alignment.
//
// The tiled kernels (hif8_gemm.hip, hif8_gemm_x.hip) need a 128 x 128 output tile for every compute unit and 16-byte
// aligned rows; with eight rows of activations their launch has one tile row, most of the chip idles and each
// workgroup walks the whole of K alone, one memory round trip per step.  Here an output tile is small (16 TM x 16 TN)
// and the wavefronts of a workgroup split K between them: no barrier in the K loop, a wavefront's loads only ever
// wait for themselves, and the partial products meet in LDS once, added in a fixed order (the result does not
// depend on timing).
//
// A wavefront reads 128 bytes of 8 rows with one load (8 lanes x 16 bytes a row: whole cache lines; fragments taken
// straight from global memory, 16 rows in 16 neighbouring lanes, ran at half the speed on rows that are not 16-byte
// aligned), passes them through its own 2 KiB of LDS per 16-row block, with the loads of the next 128 bytes in flight
// meanwhile, and expands codes on their way from there into the fragments of v_mfma_f32_16x16x32_bf16 through a
// 256-entry table in LDS.  That table look-up, one LDS read and two vector instructions per element, is the larger part of
// the code form: 8 x 11008 x 4096 took 14 us, without it 11, without the loads 14, and takes 12.6 with the shorter one; the LDS is active 56 % of
// the cycles, a fifth of them bank conflicts, the vector ALUs half (with three vector instructions 55 %).  Conflicts weigh more than
// instructions: without table_slots(), half an instruction less per element, it is 4 to 6 % slower.  With one workgroup per compute unit (509 x 1003 x 2049) both
// are busy a quarter of the time, and the chain of loads, stages and the sum counts.  (8 x 11008 x 4096: 45 MB, 7.5 us at
// the memory's rate); 128 x 128 tiles of the code-operand kernel take 67 us.  Measured against 128 x 128 and finer tiles (us per call, codes /
// expanded operands): 8 x 4096 x 4096 6.5 / 5.9 (61 / 13), 64 x 4096 x 4096 13.5 / 10.2 (62 / 14), 256 x 4096 x 4096 26 / 20
// (64 / 14), 512 x 4096 x 11008 107 / 74 (179 / 52); odd K, 509 x 1003 x 2049: 13.7 (3810 with one output per lane).
//
// The element order of a K share is the same for both operand kinds, so that one product gives the same bits whether
// its operands come as codes or expanded.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <type_traits>

#include "hif8.h"
#include "hif8_device.hpp"
#include "hif8_gemm_common.hpp"
#include "hif8_host.hpp"

namespace hif8gemm {

using namespace hif8dev;
using namespace hif8host;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Operand kinds
enum : int { OP_CODES = 0, OP_BF16 = 1 };

// K is shared out in units of 64 elements, one pass of fragments.  In units of 128, a stage of codes, 509 x 1003 x 2049 with eight
// wavefronts gave one of them three stages and the others two (64 x 2048 x 129 7.3 us, now 6.3; with all loads of a row's end in flight 4.7;
// 509 x 1003 x 2049 17.9, 15.5; 1200 x 1200 x 3000 44, 36).  Where that shortens no wavefront's share it is counted in pairs of units
// (small_by_pairs).
constexpr uint32_t kUnitK = 64;

// 16 bytes from any address
__device__ __forceinline__ u32x4 load16(const uint8_t* p) {
  u32x4 v;
  __builtin_memcpy(&v, p, 16);
  return v;
}

// The last bytes of a row: v holds the 16 bytes that end with the row, `past` of them before the ones asked for; those move down and zero
// codes follow.
__device__ __forceinline__ u32x4 drop_bytes(u32x4 v, uint32_t past) {
  const uint32_t words = past >> 2;
  u32x4 w;
#pragma unroll
  for (uint32_t i = 0; i < 4u; ++i) {
    w[i] = 0u;
#pragma unroll
    for (uint32_t j = i; j < 4u; ++j) w[i] = j - i == words ? v[j] : w[i];
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = __builtin_amdgcn_alignbyte(i < 3 ? w[i + 1] : 0u, w[i], past);
  return v;
}

// 16 codes of a row with fewer than 16, from k on.
__device__ __forceinline__ u32x4 load_short_row(const uint8_t* row, uint32_t k, uint32_t K) {
  u32x4 v = {0u, 0u, 0u, 0u};
  for (uint32_t j = k; j < K; ++j) v[(j - k) >> 2] |= (uint32_t)row[j] << (8u * ((j - k) & 3u));
  return v;
}

// Position of a code in the table: bit 4 flipped for negative codes, so that the magnitudes a tensor uses most and
// their negatives (codes 0x40.., 0x60.., 0xC0.., 0xE0.. of values above 2^4) sit in different LDS banks.
__device__ __forceinline__ uint32_t table_slots(uint32_t w) { return w ^ ((w >> 3) & 0x10101010u); }

// Twice the lowest byte of w, the LDS address of that code's element: the table is the first thing in the kernel's only LDS, which is dynamic,
// at LDS address 0 (a CPU test holds the kernel to that); from the array's own address an index costs an addition more (3 % more
// instructions in the kernel).  The compiler takes one instruction for the other bytes of a word, but a shift and a mask for this one, a ninth
// of all that an expansion takes (us: 64 x 11008 x 4096 26.0, so 25.6; 173 x 3951 x 6832 37.2, 36.3; 509 x 1003 x 2049 14.3, 14.0; with the eight rows'
// words selected before the look-ups, not the elements behind them, 8 x 11008 x 4096 14.85, 14.6).
__device__ __forceinline__ uint32_t twice_lowest(uint32_t w) {
  uint32_t r;
  asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_0" : "=v"(r) : "v"(1u), "v"(w));
  return r;
}

// Two neighbouring elements, by their addresses
__device__ __forceinline__ uint32_t lookup2(uint32_t lo, uint32_t hi) {
  typedef const __attribute__((address_space(3))) uint16_t* lds_u16;
  return (uint32_t)*(lds_u16)lo | ((uint32_t)*(lds_u16)hi << 16);
}

// 8 codes -> one MFMA fragment
__device__ __forceinline__ u32x4 expand8(uint32_t w0, uint32_t w1) {
  w0 = table_slots(w0);
  w1 = table_slots(w1);
  auto second = [](uint32_t w) { return ((w >> 8) & 0xFFu) << 1; };
  auto upper = [](uint32_t w) { return lookup2(((w >> 16) & 0xFFu) << 1, (w >> 24) << 1); };
  return u32x4{lookup2(twice_lowest(w0), second(w0)), upper(w0), lookup2(twice_lowest(w1), second(w1)), upper(w1)};
}

// 16 codes -> two fragments
__device__ __forceinline__ void expand16(const u32x4& c, bf16x8 (&f)[2]) {
  f[0] = __builtin_bit_cast(bf16x8, expand8(c[0], c[1]));
  f[1] = __builtin_bit_cast(bf16x8, expand8(c[2], c[3]));
}

// Rows of a 16-row operand block are staged 128 bytes at a time: 128 codes or 64 bfloat16.
constexpr uint32_t kRowStage = 128;

// K: codes per row (OP_CODES) or row pitch, a multiple of 64 (OP_BF16).  HALF: at most 8 rows of A (codes): the lanes
// of the upper eight rows expand the second half of a fragment pair for the lower eight, half the look-ups for A.  It is held to six
// wavefronts on a SIMD, which its work fills at the sizes it is for: aiming at seven, the compiler waits for look-ups one pair
// after the other to save registers (4 x 4096 x 4096 7.1 us, 7.7 so; 5 x 7001 x 1999 7.6, 7.85).
template <int OP, int TM, int TN, int HALF, int EPI>
__global__ void __launch_bounds__(TM * TN <= 4 ? 1024 : TM * TN <= 8 ? 768 : 512) __attribute__((amdgpu_waves_per_eu(TM * TN <= 4 ? 4 : TM * TN <= 8 ? 3 : 2, HALF != 0 ? 6 : 8)))
k_gemm_s(const uint8_t* __restrict__ A, const uint8_t* __restrict__ B, void* __restrict__ out,
         const float* __restrict__ ref, double* __restrict__ err, uint32_t M, uint32_t N, uint32_t K, float descale,
         uint32_t tiles_m, uint32_t tiles_n, uint32_t share) {
  constexpr int kPitch = TN * 16 + 4;  // floats per row of the reduction buffer: the four lane groups start 16 banks apart
  constexpr uint32_t kElem = OP == OP_CODES ? 1u : 2u, kBlocks = TM + TN, kStageUnits = OP == OP_CODES ? 2u : 1u;
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];  // [512] table, then one area per wavefront, reused by the reduction
  const uint32_t tid = threadIdx.x, lane = tid & 63u, threads = blockDim.x;
  const uint32_t waves = threads >> 6, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t r16 = lane & 15u, q = lane >> 4;
  uint8_t* const area = smem + 512 + wave * (kBlocks * 16u * kRowStage);
  float* const red = reinterpret_cast<float*>(smem + 512);  // [wavefronts][16][kPitch]
  if constexpr (OP == OP_CODES) {
    auto entry = [&](uint32_t c) { reinterpret_cast<uint16_t*>(smem)[table_slots(c)] = (uint16_t)(decode_bits(c) >> 16); };
    if (tid < 256u) entry(tid);
    if (threads < 256u)
      for (uint32_t c = tid + threads; c < 256u; c += threads) entry(c);
  }
  // this wavefront's share of K: units [u0, u1), staged kStageUnits at a time, kRowStage bytes per row.  share: units it is counted in.
  // The 64-bit division is for the compiler's sake: behind a 32-bit one it keeps a running address for every row, and the larger tiles are
  // slower for the registers (16 x 4096 x 11008 16.5 us, 18.2 so; 509 x 1003 x 2049 15.8, 19); up to eight rows it only saves 0.07 us of 6.9.
  const uint32_t row_bytes = K * kElem, units = (K + kUnitK - 1u) / kUnitK, shares = share == 1u ? units : units - (units >> 1);
  using Wide = std::conditional_t<HALF != 0, uint32_t, uint64_t>;
  const uint32_t u0 = (uint32_t)((Wide)shares * wave / waves) * share, end = (uint32_t)((Wide)shares * (wave + 1u) / waves) * share, u1 = end < units ? end : units;
  // staging: 8 lanes x 16 bytes per row, 8 rows per load; chunk c of row r sits at position c ^ ((r >> 1) & 7)
  const uint32_t lrow = lane >> 3, lchunk = lane & 7u;
  double e2 = 0.0;

  const uint32_t total = tile_order_grid(tiles_m * tiles_n);
  for (uint32_t b = blockIdx.x; b < total; b += gridDim.x) {  // gridDim.x is a multiple of the number of dies
    uint32_t tile_m, tile_n;
    if (!tile_order(b, tiles_m, tiles_n, &tile_m, &tile_n)) continue;  // the whole workgroup skips
    const uint32_t m0 = tile_m * (16 * TM), n0 = tile_n * (16 * TN);
    // rows past the edge repeat the last one; what they produce is not stored
    const uint8_t* rows[kBlocks][2];
#pragma unroll
    for (int i = 0; i < (int)kBlocks; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t r = (i < TM ? m0 + i * 16u : n0 + (i - TM) * 16u) + h * 8u + lrow, last = (i < TM ? M : N) - 1u;
        rows[i][h] = (i < TM ? A : B) + (size_t)(r < last ? r : last) * row_bytes;
      }
    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    u32x4 raw[kBlocks][2];
    bool tail = false;   // of the stage in `raw`: it reaches past the rows' end;
    uint32_t past = 0u;  // bytes before the ones asked for
    auto load_stage = [&](uint32_t u) {
      const uint32_t first = u * (kUnitK * kElem), left = (u1 - u) * (kUnitK * kElem);
      // of a stage of one unit of codes the lanes of the second half repeat the first: no other wavefront's codes
      const uint32_t at = first + (left < kRowStage ? lchunk & 3u : lchunk) * 16u;
      tail = first + (left < kRowStage ? left : kRowStage) > row_bytes;
      if (!tail || row_bytes >= 16u) {
        // past a row's end its last 16 bytes, put right on the way into LDS: all loads are in flight together (with a load and its shift
        // behind a branch each, the last stage waited for one row after the other)
        uint32_t from = at;
        if (OP == OP_CODES && tail) from = at + 16u <= row_bytes ? at : row_bytes - 16u;
        past = at - from;
#pragma unroll
        for (int i = 0; i < (int)kBlocks; ++i)
#pragma unroll
          for (int h = 0; h < 2; ++h) raw[i][h] = load16(rows[i][h] + from);
      } else {
#pragma unroll
        for (int i = 0; i < (int)kBlocks; ++i)
#pragma unroll
          for (int h = 0; h < 2; ++h) raw[i][h] = load_short_row(rows[i][h], at, row_bytes);
      }
    };
    auto stage_to_lds = [&]() {
      if (OP == OP_CODES && tail && row_bytes >= 16u) {
#pragma unroll
        for (int i = 0; i < (int)kBlocks; ++i)
#pragma unroll
          for (int h = 0; h < 2; ++h) raw[i][h] = drop_bytes(raw[i][h], past);
      }
      // through the wavefront's own LDS: a wavefront's LDS operations run in order, so only the compiler needs fences
#pragma unroll
      for (int i = 0; i < (int)kBlocks; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint32_t r = h * 8u + lrow;
          *reinterpret_cast<u32x4*>(area + (i * 16u + r) * kRowStage + ((lchunk ^ ((r >> 1) & 7u)) * 16u)) = raw[i][h];
        }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
    };
    auto compute_stage = [&](uint32_t u) {
      auto frag = [&](int block, uint32_t chunk) {
        return *reinterpret_cast<const u32x4*>(area + (block * 16u + r16) * kRowStage + ((chunk ^ ((r16 >> 1) & 7u)) * 16u));
      };
      // element order within a unit: 16 q + 0..7, then 16 q + 8..15
#pragma unroll
      for (uint32_t p = 0; p < kStageUnits; ++p) {
        if (u + p >= u1) break;  // a stage of one unit
        bf16x8 fa[TM][2], fb[2];
        auto get = [&](int block, bf16x8 (&f)[2]) {
          if constexpr (OP == OP_CODES) {
            expand16(frag(block, p * 4 + q), f);
          } else {
            f[0] = __builtin_bit_cast(bf16x8, frag(block, 2 * q));
            f[1] = __builtin_bit_cast(bf16x8, frag(block, 2 * q + 1));
          }
        };
        if constexpr (HALF != 0) {
          static_assert(OP == OP_CODES && TM == 1, "one row block of codes");
          const uint32_t r8 = r16 & 7u;
          const u32x4 c = *reinterpret_cast<const u32x4*>(area + r8 * kRowStage + (((p * 4 + q) ^ (r8 >> 1)) * 16u));
          const u32x4 own = expand8(r16 < 8u ? c[0] : c[2], r16 < 8u ? c[1] : c[3]);
          u32x4 other;
#pragma unroll
          for (int v = 0; v < 4; ++v) other[v] = __builtin_amdgcn_update_dpp(0, own[v], 0x128, 0xF, 0xF, true);  // row_ror:8
          fa[0][0] = __builtin_bit_cast(bf16x8, own);
          fa[0][1] = __builtin_bit_cast(bf16x8, other);
        } else {
#pragma unroll
          for (int i = 0; i < TM; ++i) get(i, fa[i]);
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          get(TM + j, fb);
#pragma unroll
          for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < TM; ++i)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i][h], fb[h], acc[i][j], 0, 0, 0);
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    };
    if (u0 < u1) load_stage(u0);
    __syncthreads();  // table written; reduction buffer of the previous tile read
    for (uint32_t u = u0; u < u1; u += kStageUnits) {
      stage_to_lds();
      if (u + kStageUnits < u1) load_stage(u + kStageUnits);
      compute_stage(u);
    }
    __syncthreads();  // staging areas free: the reduction uses the same LDS

    // the wavefronts' partial tiles, 16 rows at a time, four by four in a fixed order: with more wavefronts, which a plan may take for its speed, a sum of
    // one after the other has more roundings than it saves in their shorter chains (relative error of binary32 results, 20 x 1284 x 2614: eight wavefronts
    // 4.6e-8, sixteen 4.9e-8, added so 4.2e-8; 612 x 788 x 785 from codes: four 2.5e-8, eight 2.6e-8, 2.4e-8; the times are the same)
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if (i > 0) __syncthreads();
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[(wave * 16u + q * 4u + v) * kPitch + j * 16 + r16] = acc[i][j][v];
      __syncthreads();
      auto finish = [&](auto sum_of) {
        for (uint32_t e = tid; e < 16u * (TN * 16); e += threads) {
          const uint32_t r = e / (TN * 16), c = e % (TN * 16), row = m0 + i * 16u + r, col = n0 + c;
          const float sum = sum_of([&](uint32_t w) { return red[(w * 16u + r) * kPitch + c]; });
          if (row < M && col < N) {
            const float o = __fmul_rn(sum, descale);
            if constexpr (EPI == EPI_ERR) {
              const double d = (double)o - (double)ref[(size_t)row * N + col];
              e2 = fma(d, d, e2);
            } else {
              store_one<EPI>(out, (size_t)row * N + col, o);
            }
          }
        }
      };
      // with one wavefront or two, which many tiles of a short K have, the sum is a good part of the time: no loop
      // (us, the loop below for all / so: 511 x 4297 x 70 17.7 / 15.1, 391 x 6197 x 178 16.6 / 14.4, 64 x 20000 x 128 expanded 7.0 / 6.4)
      if (waves == 1u)
        finish([](auto of) { return 0.0f + of(0u); });
      else if (waves == 2u)
        finish([](auto of) { return 0.0f + (of(0u) + of(1u)); });
      else
        finish([&](auto of) {
          float sum = 0.0f;
          uint32_t w = 0;
          for (; w + 4u <= waves; w += 4u) sum += (of(w) + of(w + 1u)) + (of(w + 2u) + of(w + 3u));
          for (; w < waves; ++w) sum += of(w);
          return sum;
        });
    }
    __syncthreads();
  }
  if constexpr (EPI == EPI_ERR) {
    double* scratch = reinterpret_cast<double*>(red);  // free: every tile ends with a barrier
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) e2 += __shfl_xor(e2, off, 64);
    if (lane == 0) scratch[wave] = e2;
    __syncthreads();
    if (tid == 0) {
      double t = 0.0;
      for (uint32_t w = 0; w < waves; ++w) t += scratch[w];
      unsafeAtomicAdd(err, t);
    }
  }
}

// ====================================================================================
// host side
// ====================================================================================
template <int OP, int TM, int TN, int HALF, int EPI>
static hif8_status launch_s(const void* A, const void* B, void* out, const float* ref, double* err, uint32_t M, uint32_t N,
                            uint32_t K, float descale, uint32_t waves, int cus, hipStream_t st) {
  const uint64_t tiles_m = ((uint64_t)M + 16 * TM - 1) / (16 * TM), tiles_n = ((uint64_t)N + 16 * TN - 1) / (16 * TN);
  if (tiles_m * tiles_n > 0x7FFFFFF0ull) return HIF8_ERR_ARG;
  const uint32_t total = tile_order_grid((uint32_t)(tiles_m * tiles_n));
  // threads of a launch are counted in 32 bits.  The squared error ends each workgroup with an atomic on one address, and those
  // are served one after the other (10 ns each), so there four workgroups per compute unit walk over the tiles (codes, us, a
  // workgroup per tile / 256, 512, 1024 workgroups: 8 x 200000 x 64 158 / 81, 46, 35; 64 x 32000 x 64 34 / 54, 32, 27).  With a long
  // K the atomics come slowly enough, and dealing out the tiles evenly counts more (16 x 53248 x 4096 84 / 94 with 1024).
  const uint32_t most = EPI == EPI_ERR && K < 4096u ? tile_order_grid((uint32_t)cus * 4u) : 1u << 20;
  const size_t stage = (size_t)waves * (TM + TN) * 16 * kRowStage, red = (size_t)waves * 16 * (TN * 16 + 4) * 4;
  const size_t smem = 512 + (stage > red ? stage : red);
  if (smem > 65536) {
    static bool attr_set[64] = {};
    int dev = 0;
    if (!hip_ok(hipGetDevice(&dev))) return HIF8_ERR_HIP;
    if (dev < 0 || dev >= 64) return HIF8_ERR_ARG;
    if (!attr_set[dev]) {
      if (!hip_ok(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_s<OP, TM, TN, HALF, EPI>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024)))
        return HIF8_ERR_HIP;
      attr_set[dev] = true;
    }
  }
  hipLaunchKernelGGL((k_gemm_s<OP, TM, TN, HALF, EPI>), dim3(total < most ? total : most), dim3(64 * waves), smem, st,
                     reinterpret_cast<const uint8_t*>(A), reinterpret_cast<const uint8_t*>(B), out, ref, err, M, N, K, descale,
                     (uint32_t)tiles_m, (uint32_t)tiles_n, small_by_pairs(K, waves) ? 2u : 1u);
  return finish_launch();
}

template <int OP, int EPI>
static hif8_status gemm_small_op(const void* A, const void* B, void* out, const float* ref, double* err, size_t M, size_t N,
                                 size_t K, const SmallPlan& p, float descale, hipStream_t st) {
  const uint32_t m = (uint32_t)M, n = (uint32_t)N, k = (uint32_t)K;
  int cus = 0;
  const hif8_status s = ensure_init(&cus, nullptr);
  if (s != HIF8_OK) return s;
  auto run = [&](auto launch) { return launch(A, B, out, ref, err, m, n, k, descale, p.waves, cus, st); };
  switch (p.tm * 10 + p.tn) {
    case 11:
      if constexpr (OP == OP_CODES) {
        if (M <= 8) return run(launch_s<OP, 1, 1, 1, EPI>);
      }
      return run(launch_s<OP, 1, 1, 0, EPI>);
    case 12: return run(launch_s<OP, 1, 2, 0, EPI>);
    case 22: return run(launch_s<OP, 2, 2, 0, EPI>);
    case 24: return run(launch_s<OP, 2, 4, 0, EPI>);
    case 44: return run(launch_s<OP, 4, 4, 0, EPI>);
  }
  if constexpr (EPI != EPI_ERR) {
    switch (p.tm * 10 + p.tn) {
      case 13: return run(launch_s<OP, 1, 3, 0, EPI>);
      case 23: return run(launch_s<OP, 2, 3, 0, EPI>);
      case 34: return run(launch_s<OP, 3, 4, 0, EPI>);
      case 43: return run(launch_s<OP, 4, 3, 0, EPI>);
    }
  }
  return HIF8_ERR_ARG;  // no such tile in the plans
}

template <int EPI>
hif8_status gemm_small(const void* A, const void* B, bool expanded, void* out, const float* ref, double* err, size_t M, size_t N,
                       size_t K, const SmallPlan& plan, float descale, hipStream_t st) {
  return expanded ? gemm_small_op<OP_BF16, EPI>(A, B, out, ref, err, M, N, K, plan, descale, st)
                  : gemm_small_op<OP_CODES, EPI>(A, B, out, ref, err, M, N, K, plan, descale, st);
}

template hif8_status gemm_small<EPI_F32>(const void*, const void*, bool, void*, const float*, double*, size_t, size_t, size_t, const SmallPlan&, float, hipStream_t);
template hif8_status gemm_small<EPI_BF16>(const void*, const void*, bool, void*, const float*, double*, size_t, size_t, size_t, const SmallPlan&, float, hipStream_t);
template hif8_status gemm_small<EPI_F16>(const void*, const void*, bool, void*, const float*, double*, size_t, size_t, size_t, const SmallPlan&, float, hipStream_t);
template hif8_status gemm_small<EPI_ERR>(const void*, const void*, bool, void*, const float*, double*, size_t, size_t, size_t, const SmallPlan&, float, hipStream_t);

}  // namespace hif8gemm
