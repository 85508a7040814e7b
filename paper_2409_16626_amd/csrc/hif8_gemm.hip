// Simulated HiF8 GEMM on the matrix cores of gfx950, and Algorithm 1's per-layer scale search.
//
// The paper's experiments cast the GEMM inputs (activations, weights, activation gradients) to
// HiF8 and run the GEMM on the represented values (Sec. 4, Sec. 5); Algorithm 1 ("MatMul &
// Restore") descales the product by the two input scales.  Every HiF8 value is exact in
// bfloat16 (at most 3 mantissa bits, exponents -22..15), so the product is computed with bf16
// MFMA instructions and FP32 accumulation; the u8 codes are expanded to bf16 on their way from
// HBM into LDS (one table lookup per element, table replicated per LDS bank so that lookups of a
// wavefront never conflict), which halves the operand traffic against a bf16 GEMM.
//
//   O[M, N] = (value(A[M, K]) x value(B[N, K])^T) * descale        (both operands K-contiguous)
//
// Tiling: a workgroup of WM x WN wavefronts owns a (WM TM 32) x (WN TN 32) tile of O; each
// wavefront TM x TN blocks of v_mfma_f32_32x32x16_bf16; K advances in steps of BK through a
// double-buffered LDS tile, with the next tile's codes in flight in registers during the MFMAs.  What bounds it is the LDS: of a
// step of a 256 x 128 x 64 tile the table look-ups take 768 cycles, the fragments 512 and the expanded codes' stores 384, the MFMAs 1024 on
// each SIMD and the vector instructions (3.7 a code) as much; 1024 x 8192 x 4096 keeps the LDS 54 %, the vector ALUs 46 % and the
// matrix cores 33 % busy and takes 86 to 105 us, by the clock of the chip.  A look-up is needed per row or column and K of a workgroup's tile, so a larger tile needs fewer per MFMA;
// BK = 64 makes fewer, longer steps (256 x 128 with BK = 32: 120 us).  16 wavefronts do no better (93 us), two workgroups of 128 x 128 tiles
// on a compute unit need a third more look-ups (121 us).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <mutex>

#include "hif8.h"
#include "hif8_diag.h"
#include "hif8_conv_api.hpp"
#include "hif8_device.hpp"
#include "hif8_gemm_common.hpp"
#include "hif8_host.hpp"

namespace hif8gemm {

using namespace hif8dev;
using namespace hif8host;

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

#ifndef HIF8_GEMM_PAD
#define HIF8_GEMM_PAD 8
#endif
constexpr int kPad = HIF8_GEMM_PAD;  // bf16 elements of padding per LDS row
constexpr int kLutCopies = 32;    // one copy of the code -> bf16 table per LDS bank

// code -> bfloat16 pattern (the top half of the binary32 pattern; exact for every code)
static __device__ __attribute__((aligned(16))) uint16_t g_bf16_lut[256];
__global__ void k_build_gemm_lut() {
  const uint32_t i = threadIdx.x;
  if (i < 256u) g_bf16_lut[i] = (uint16_t)(decode_bits(i) >> 16);
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// 16 codes (one 16-byte chunk) -> 16 bf16, written to LDS as two 16-byte stores.
// lut16: this lane's column of the replicated table, indexed by code * (2 * kLutCopies).
__device__ __forceinline__ void decode_chunk_to_lds(const u32x4& c, const uint16_t* lut16, uint4* dst) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    uint32_t o[4];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const uint32_t w = c[2 * h + j];
      u16x2 p0, p1;
      p0.x = lut16[(w & 0xFFu) * (2 * kLutCopies)];
      p0.y = lut16[((w >> 8) & 0xFFu) * (2 * kLutCopies)];
      p1.x = lut16[((w >> 16) & 0xFFu) * (2 * kLutCopies)];
      p1.y = lut16[(w >> 24) * (2 * kLutCopies)];
      o[2 * j] = __builtin_bit_cast(uint32_t, p0);
      o[2 * j + 1] = __builtin_bit_cast(uint32_t, p1);
    }
    dst[h] = make_uint4(o[0], o[1], o[2], o[3]);
  }
}

// 16 codes of row `row` at column k; rows / columns outside the matrix read as zero codes.  The address is selected, not the value:
// a value that is selected behind its load gets loaded under a branch, which cut the K step into blocks, kept the look-ups of one
// from the MFMAs of the next and made a step wait for the loads that it had just issued (3006 x 8074 x 7664 602 us, so 493).
static __device__ __attribute__((aligned(16))) const uint8_t g_zero_codes[16] = {};
__device__ __forceinline__ u32x4 load_chunk(const uint8_t* __restrict__ P, uint32_t row, uint32_t rows, uint32_t k, uint32_t K) {
  const uint8_t* at = row < rows && k < K ? P + (size_t)row * K + k : g_zero_codes;
  return *(const __attribute__((address_space(1))) u32x4*)(uintptr_t)at;  // global memory, which the compiler no longer sees
}

// Epilogue of one wavefront, straight from the accumulators: TM x TN blocks of v_mfma_f32_32x32x16_bf16 whose top-left
// element is (row0, col0).  Element v of a 32 x 32 block sits at row (v / 4) * 8 + (lane / 32) * 4 + v % 4,
// column lane % 32.  EPI_ERR adds the squared differences to *err in fp64: the wavefronts of the workgroup
// combine through `wg_scratch` (LDS, at least one double per wavefront, free of other use by now; every
// wavefront of the workgroup must make this call) and issue one atomic per workgroup.  The K loop here leaves the memory
// path idle, so whole lines through LDS (the epilogue of the expanded-operand kernel) gain little, 48.9 -> 46.2 us at 512 x
// 6000 x 2048, and lose on rows that are not 16-byte aligned, 27.4 -> 30.1 us at 1501 x 1503 x 1024.
template <int EPI, int TM, int TN>
__device__ __forceinline__ void epilogue_direct(const f32x16 (&acc)[TM][TN], void* __restrict__ out,
                                         const float* __restrict__ ref, double* __restrict__ err, uint32_t M,
                                         uint32_t N, uint32_t row0, uint32_t col0, uint32_t lane, float descale,
                                         double* wg_scratch, uint32_t wave, uint32_t n_waves) {
  double e2 = 0.0;
  // the whole wavefront tile inside the matrix (the usual case): no per-element bounds checks
  const bool inside = row0 + TM * 32 <= M && col0 + TN * 32 <= N;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const uint32_t col = col0 + j * 32 + (lane & 31u);
      const uint32_t rbase = row0 + i * 32 + (lane >> 5) * 4;
      if constexpr (EPI == EPI_ERR) {
        // all 16 reference values of the block are requested before the first is used; positions
        // outside the matrix read element 0 and contribute nothing
        float r[16];
        bool ok[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const uint32_t row = rbase + (v >> 2) * 8 + (v & 3);
          ok[v] = inside || (row < M && col < N);
          r[v] = ref[ok[v] ? (size_t)row * N + col : (size_t)0];
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const double d = (double)__fmul_rn(acc[i][j][v], descale) - (double)r[v];
          e2 = ok[v] ? fma(d, d, e2) : e2;
        }
      } else if (inside) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
          store_one<EPI>(out, (size_t)(rbase + (v >> 2) * 8 + (v & 3)) * N + col, __fmul_rn(acc[i][j][v], descale));
      } else {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const uint32_t row = rbase + (v >> 2) * 8 + (v & 3);
          if (row < M && col < N) store_one<EPI>(out, (size_t)row * N + col, __fmul_rn(acc[i][j][v], descale));
        }
      }
    }
  }
  if constexpr (EPI == EPI_ERR) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) e2 += __shfl_xor(e2, off, 64);
    if (lane == 0) wg_scratch[wave] = e2;
    __syncthreads();
    if (wave == 0 && lane == 0) {
      double t = 0.0;
      for (uint32_t w = 0; w < n_waves; ++w) t += wg_scratch[w];
      unsafeAtomicAdd(err, t);  // hardware fp64 add at the L2, no compare-and-swap loop
    }
  }
}

template <int WM, int WN, int TM, int TN, int BK, int EPI>
__global__ void __launch_bounds__(64 * WM * WN)
k_gemm_nt(const uint8_t* __restrict__ A, const uint8_t* __restrict__ B, void* __restrict__ out,
          const float* __restrict__ ref, double* __restrict__ err, uint32_t M, uint32_t N, uint32_t K,
          float descale, const uint16_t* __restrict__ g_lut, uint32_t tiles_n, uint32_t col_begin) {
  constexpr int kThreads = 64 * WM * WN;
  constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
  constexpr int LDA = BK + kPad;                       // LDS row stride in bf16
  constexpr int CPR = BK / 16;                         // 16-code chunks per tile row
  constexpr int CA = BM * CPR / kThreads, CB = BN * CPR / kThreads;  // chunks per thread
  static_assert(BM * CPR % kThreads == 0 && BN * CPR % kThreads == 0, "tile / thread mismatch");

  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  uint32_t* lut32 = reinterpret_cast<uint32_t*>(smem);                     // [256][kLutCopies]
  __bf16* As = reinterpret_cast<__bf16*>(smem + 256 * kLutCopies * 4);     // [2][BM][LDA]
  __bf16* Bs = As + 2 * BM * LDA;                                          // [2][BN][LDA]

  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint32_t wm = wave / WN, wn = wave % WN;
  const uint32_t tile_m = blockIdx.x / tiles_n, tile_n = blockIdx.x - tile_m * tiles_n;
  const uint32_t m0 = tile_m * BM, n0 = col_begin + tile_n * BN;  // the launch covers columns from col_begin on

  // replicated table: entry (code, copy) at dword code * 32 + copy; lane l reads copy l % 32
  for (uint32_t i = tid; i < 256u * kLutCopies; i += kThreads) {
    const uint32_t v = g_lut[i / kLutCopies];
    lut32[i] = v | (v << 16);
  }
  const uint16_t* lut16 = reinterpret_cast<const uint16_t*>(lut32) + 2 * (lane & (kLutCopies - 1));

  // this thread's chunks of the A and B tiles.  Chunk q -> (row, 16-code column): 8 consecutive
  // lanes take 8 consecutive rows of the same column, so that their 16-byte LDS stores (row
  // stride 16 bytes more than a power of two) fall into 8 different groups of 4 banks; the lanes
  // 8 apart take the neighbouring columns, so a wavefront still loads whole 16 * CPR byte runs.
  auto chunk_row = [](uint32_t q) { return 8u * (q / (8u * CPR)) + (q & 7u); };
  auto chunk_col = [](uint32_t q) { return (q >> 3) % CPR; };
  // Two register sets: one holds the codes of the tile being expanded into LDS during this K step,
  // the other receives the loads for the tile after it, so a load has a whole K step to arrive.
  u32x4 ra[2][CA], rb[2][CB];
  auto load_tiles = [&](int set, uint32_t k0) {
#pragma unroll
    for (int i = 0; i < CA; ++i) {
      const uint32_t q = tid + i * kThreads, r = chunk_row(q), kc = chunk_col(q);
      ra[set][i] = load_chunk(A, m0 + r, M, k0 + kc * 16, K);
    }
#pragma unroll
    for (int i = 0; i < CB; ++i) {
      const uint32_t q = tid + i * kThreads, r = chunk_row(q), kc = chunk_col(q);
      rb[set][i] = load_chunk(B, n0 + r, N, k0 + kc * 16, K);
    }
  };
  auto store_tiles = [&](int set, int buf) {
#pragma unroll
    for (int i = 0; i < CA; ++i) {
      const uint32_t q = tid + i * kThreads, r = chunk_row(q), kc = chunk_col(q);
      decode_chunk_to_lds(ra[set][i], lut16, reinterpret_cast<uint4*>(As + ((size_t)buf * BM + r) * LDA + kc * 16));
    }
#pragma unroll
    for (int i = 0; i < CB; ++i) {
      const uint32_t q = tid + i * kThreads, r = chunk_row(q), kc = chunk_col(q);
      decode_chunk_to_lds(rb[set][i], lut16, reinterpret_cast<uint4*>(Bs + ((size_t)buf * BN + r) * LDA + kc * 16));
    }
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

  const uint32_t frag_row = lane & 31u, frag_k = (lane >> 5) * 8u;
  // formed once, not from the buffer's number in each step: 128 x 128 tiles 512 x 4096 x 4096 67 -> 60 us, 256 x 256 3006 x 8074 x 7664 512 -> 484, the
  // others the same
  const __bf16* const a_frag = As + (size_t)(wm * TM * 32 + frag_row) * LDA + frag_k;
  const __bf16* const b_frag = Bs + (size_t)(wn * TN * 32 + frag_row) * LDA + frag_k;
  // one K step: MFMAs on LDS buffer `buf` (tile kt) while the codes in register set `set`
  // (tile kt + 1) are expanded into the other buffer and tile kt + 2 is requested from memory
  auto k_step = [&](uint32_t kt, int buf, int set) {
    load_tiles(set ^ 1, (kt + 2) * BK);  // past the last tile this reads zeros (k >= K); never used
    const __bf16 *a_base = a_frag + buf * BM * LDA, *b_base = b_frag + buf * BN * LDA;
#pragma unroll
    for (int s = 0; s < BK / 16; ++s) {
      bf16x8 fa[TM], fb[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[i] = *reinterpret_cast<const bf16x8*>(a_base + (size_t)i * 32 * LDA + s * 16);
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[j] = *reinterpret_cast<const bf16x8*>(b_base + (size_t)j * 32 * LDA + s * 16);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
    }
    store_tiles(set, buf ^ 1);
    // The look-ups spread evenly over the MFMAs, so that neither the LDS nor the matrix core waits while the other works; left to itself
    // the compiler puts half of them behind the last MFMA (256 x 128 tiles, us with / without: 1024 x 8192 x 4096 86 / 97, 3006 x 8074 x
    // 7664 462 / 509).  128 x 128 tiles have four look-ups per MFMA and wave and a shorter step, where a fixed order costs (512 x 4096^2 65 / 59).
    if constexpr (TM * TN * WM * WN > 16) {
      constexpr int kMfma = TM * TN * (BK / 16), kFirst = TM + TN;
      constexpr int kReads = (TM + TN) * (BK / 16) + 16 * (CA + CB);  // fragments and look-ups
      __builtin_amdgcn_sched_group_barrier(0x100, kFirst, 0);
#pragma unroll
      for (int i = 0; i < kMfma; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, (kReads - kFirst + kMfma - 1) / kMfma, 0);
      }
    }
    __syncthreads();
  };

  const uint32_t nk = (K + BK - 1) / BK;
  load_tiles(0, 0);
  load_tiles(1, BK);
  __syncthreads();  // table staged
  store_tiles(0, 0);
  __syncthreads();
  // register sets alternate with the LDS buffers: tile kt + 1 sits in set (kt + 1) & 1
  uint32_t kt = 0;
  for (; kt + 1 < nk; kt += 2) {
    k_step(kt, 0, 1);
    k_step(kt + 1, 1, 0);
  }
  if (kt < nk) k_step(kt, 0, 1);

  // the last K step ended with a barrier: the tile buffers (behind the table) are free for the epilogue
  epilogue_direct<EPI, TM, TN>(acc, out, ref, err, M, N, m0 + wm * TM * 32, n0 + wn * TN * 32, lane, descale,
                               reinterpret_cast<double*>(As), wave, WM * WN);
}

// ====================================================================================
// host side
// ====================================================================================
constexpr int kMaxDevices = 64;
static const uint16_t* g_lut_ptr[kMaxDevices] = {};

static hif8_status gemm_init(const uint16_t** lut_out, int* cus_out) {
  int cus = 0;
  hif8_status s = ensure_init(&cus, nullptr);
  if (s != HIF8_OK) return s;
  int dev = 0;
  if (!hip_ok(hipGetDevice(&dev))) return HIF8_ERR_HIP;
  if (dev < 0 || dev >= kMaxDevices) return HIF8_ERR_ARG;
  static std::mutex mu;
  std::lock_guard<std::mutex> lock(mu);
  if (!g_lut_ptr[dev]) {
    void* p = nullptr;
    if (!hip_ok(hipGetSymbolAddress(&p, HIP_SYMBOL(g_bf16_lut)))) return HIF8_ERR_HIP;
    hipLaunchKernelGGL(k_build_gemm_lut, dim3(1), dim3(256), 0, (hipStream_t)0);
    if (!hip_ok(hipGetLastError())) return HIF8_ERR_HIP;
    if (!hip_ok(hipStreamSynchronize((hipStream_t)0))) return HIF8_ERR_HIP;
    g_lut_ptr[dev] = reinterpret_cast<const uint16_t*>(p);
  }
  *lut_out = g_lut_ptr[dev];
  if (cus_out) *cus_out = cus;
  return HIF8_OK;
}

template <int WM, int WN, int TM, int TN, int BK>
constexpr size_t smem_bytes() {
  return 256 * kLutCopies * 4 + (size_t)2 * (WM * TM * 32 + WN * TN * 32) * (BK + kPad) * 2;
}

template <int WM, int WN, int TM, int TN, int BK, int EPI>
static hif8_status launch_tiled(const uint8_t* A, const uint8_t* B, void* out, const float* ref, double* err,
                                uint32_t M, uint32_t N, uint32_t K, float descale, const uint16_t* lut,
                                hipStream_t st, uint32_t col_begin, uint32_t col_end) {
  if (col_begin >= col_end) return HIF8_OK;
  constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
  constexpr size_t smem = smem_bytes<WM, WN, TM, TN, BK>();
  static bool attr_set[kMaxDevices] = {};
  int dev = 0;
  if (!hip_ok(hipGetDevice(&dev))) return HIF8_ERR_HIP;
  if (!attr_set[dev]) {
    if (!hip_ok(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_nt<WM, WN, TM, TN, BK, EPI>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem)))
      return HIF8_ERR_HIP;
    attr_set[dev] = true;
  }
  const uint32_t tiles_m = (M + BM - 1) / BM, tiles_n = (col_end - col_begin + BN - 1) / BN;
  if ((uint64_t)tiles_m * tiles_n > 0x7FFFFFFFull) return HIF8_ERR_ARG;
  hipLaunchKernelGGL((k_gemm_nt<WM, WN, TM, TN, BK, EPI>), dim3(tiles_m * tiles_n), dim3(64 * WM * WN), smem, st,
                     A, B, out, ref, err, M, N, K, descale, lut, tiles_n, col_begin);
  return finish_launch();
}

static int g_gemm_variant = 0;  // 0 = default choice; tuning knob HIF8_TUNE_GEMM_TILE

template <int EPI>
static hif8_status gemm_dispatch(const uint8_t* A, const uint8_t* B, void* out, const float* ref, double* err,
                                 size_t M, size_t N, size_t K, float scale_a, float scale_b, hipStream_t st) {
  float inv_a = 1.0f, inv_b = 1.0f;
  if (!valid_scale(scale_a, &inv_a) || !valid_scale(scale_b, &inv_b)) return HIF8_ERR_SCALE;
  volatile float ds = inv_a * inv_b;
  const float descale = ds;
  if (!(descale > 0.0f) || std::isinf(descale)) return HIF8_ERR_SCALE;
  if (M == 0 || N == 0) return HIF8_OK;
  if (M > 0x7FFFFFFFu || N > 0x7FFFFFFFu || K > 0x7FFFFFFFu) return HIF8_ERR_ARG;
  if ((!A || !B) && K != 0) return HIF8_ERR_NULL;
  if (EPI == EPI_ERR ? (!ref || !err) : !out) return HIF8_ERR_NULL;
  if (EPI == EPI_ERR && !aligned_to(err, 8)) return HIF8_ERR_ARG;  // fp64 atomics need naturally aligned doubles
  const uint16_t* lut = nullptr;
  int cus = 0;
  hif8_status s = gemm_init(&lut, &cus);
  if (s != HIF8_OK) return s;
  const uint32_t m = (uint32_t)M, n = (uint32_t)N, k = (uint32_t)K;
  const bool fast = K != 0 && (K % 16) == 0 && aligned_to(A, 16) && aligned_to(B, 16);
  if (!fast || g_gemm_variant == 12)
    return gemm_small<EPI>(A, B, false, out, ref, err, M, N, K, small_choice(M, N, K, true, EPI == EPI_ERR), descale, st);
  if (g_gemm_variant == 0) {
    const SmallRoute route = small_route(M, N, K, true, EPI == EPI_ERR);
    if (route.small) return gemm_small<EPI>(A, B, false, out, ref, err, M, N, K, route.plan, descale, st);
  }
  CodesLaunch launch[2] = {{g_gemm_variant == 5 ? CODES_256 : CODES_128, 0u, n}, {CODES_128, 0u, 0u}};
  const int launches = g_gemm_variant == 0 ? codes_launches(M, N, K, (size_t)cus, launch) : 1;
  for (int i = 0; i < launches && s == HIF8_OK; ++i) {
    auto go = [&](auto launch_one) { return launch_one(A, B, out, ref, err, m, n, k, descale, lut, st, launch[i].begin, launch[i].end); };
    switch (launch[i].tile) {
      case CODES_256: s = go(launch_tiled<4, 2, 2, 4, 32, EPI>); break;
      case CODES_TALL: s = go(launch_tiled<4, 2, 2, 2, 64, EPI>); break;
      case CODES_WIDE: s = go(launch_tiled<2, 4, 2, 2, 64, EPI>); break;
      default: s = go(launch_tiled<2, 4, 2, 1, 64, EPI>); break;
    }
  }
  return s;
}

// hif8_gemm_* through a workspace: expand both operands, then the expanded-operand kernel.
static size_t gemm_ws_bytes(size_t M, size_t N, size_t K) {
  if (M == 0 || N == 0 || K == 0) return 0;
  const size_t ld = expanded_ld(K);
  if (ld > kMaxLd || M > 0x7FFFFFFFu || N > 0x7FFFFFFFu) return 0;
  return 2 * (M + N) * ld;
}

template <int EPI>
static hif8_status gemm_ws(const uint8_t* A, const uint8_t* B, void* out, const float* ref, double* err, size_t M,
                           size_t N, size_t K, float scale_a, float scale_b, void* ws, size_t ws_bytes, hipStream_t st) {
  const size_t need = gemm_ws_bytes(M, N, K);
  if (need == 0)  // nothing to expand, or a shape beyond the expanded-operand kernel's limits
    return gemm_dispatch<EPI>(A, B, out, ref, err, M, N, K, scale_a, scale_b, st);
  float inv_a = 1.0f, inv_b = 1.0f;
  if (!valid_scale(scale_a, &inv_a) || !valid_scale(scale_b, &inv_b)) return HIF8_ERR_SCALE;
  volatile float ds = inv_a * inv_b;
  const float descale = ds;
  if (!(descale > 0.0f) || std::isinf(descale)) return HIF8_ERR_SCALE;
  if (!A || !B || !ws) return HIF8_ERR_NULL;
  if (EPI == EPI_ERR ? (!ref || !err) : !out) return HIF8_ERR_NULL;
  if (ws_bytes < need || !aligned_to(ws, 16)) return HIF8_ERR_ARG;
  if (EPI == EPI_ERR && !aligned_to(err, 8)) return HIF8_ERR_ARG;
  // few rows: straight from the codes, which gives the bits that the expanded operands would give (see small_choice)
  if (expanded_variant() == 0 && (M < N ? M : N) <= kSmallCodesRows && small_problem(M, N, expanded_ld(K), false, EPI == EPI_ERR))
    return gemm_small<EPI>(A, B, false, out, ref, err, M, N, K, small_choice(M, N, K, true, EPI == EPI_ERR), descale, st);
  const size_t ld = expanded_ld(K);
  SmallRoute route{false, {0, 0, 0}, {0, 0, 0}};
  const bool routed = EPI != EPI_ERR && expanded_variant() == 0;
  if (routed) {
    route = small_route(M, N, ld, false, false);
    SmallPlan plan;
    if (route.small && (M < N ? M : N) > kSmallCodesRows && small_from_codes(M, N, K, route, &plan))
      return gemm_small<EPI>(A, B, false, out, ref, err, M, N, K, plan, descale, st);
  }
  uint16_t* xa = reinterpret_cast<uint16_t*>(ws);
  uint16_t* xb = xa + M * ld;  // M * ld * 2 bytes is a multiple of 128: still 16-byte aligned
  const hif8_status s = expand_rows(A, M, B, N, K, xa, ld, st);
  if (s != HIF8_OK) return s;
  if (route.small) return gemm_small<EPI>(xa, xb, true, out, ref, err, M, N, ld, route.plan, descale, st);
  return gemm_expanded<EPI>(xa, xb, out, ref, err, M, N, ld, descale, st, Batch{}, routed);
}

// position of the smallest finite entry of err[rows * cols] -> best[0] = e_row_lo + row,
// best[1] = e_col_lo + col (first minimum in row-major order; {e_row_lo, e_col_lo} if none is finite).  One wavefront.
__global__ void __launch_bounds__(64)
k_argmin_pair(const double* __restrict__ err, int rows, int cols, int e_row_lo, int e_col_lo, int32_t* __restrict__ best) {
  int bi = 0x7FFFFFFF;
  double bv = INFINITY;
  for (int i = (int)threadIdx.x; i < rows * cols; i += 64) {
    const double v = err[i];
    if (v < bv) { bv = v; bi = i; }  // NaN and +Inf never compare below
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const double v = __shfl_xor(bv, off, 64);
    const int i = __shfl_xor(bi, off, 64);
    if (v < bv || (v == bv && i < bi)) { bv = v; bi = i; }
  }
  if (threadIdx.x != 0) return;
  if (bi == 0x7FFFFFFF) bi = 0;
  best[0] = e_row_lo + bi / cols;
  best[1] = e_col_lo + bi % cols;
}

static size_t calibrate_bytes(size_t M, size_t N, size_t K, int ea_count, int ew_count) {
  const size_t ld = expanded_ld(K);
  return ((M > N ? M : N) * K + 15) / 16 * 16 + 2 * ld * (M * (size_t)ea_count + N * (size_t)ew_count);
}

// Algorithm 1 for one layer: casts at every scale of the search square (each expanded to bfloat16
// once), then one error GEMM per pair.
template <int SRCK>
static hif8_status calibrate_layer(const void* a, const void* w, const float* o_ref, size_t M, size_t N, size_t K,
                                   int ea_lo, int ea_count, int ew_lo, int ew_count, uint32_t mode, void* workspace,
                                   size_t workspace_bytes, double* d_err, int32_t* d_best, hipStream_t st) {
  if (!valid_mode(mode)) return HIF8_ERR_MODE;
  if (ea_count < 1 || ew_count < 1 || ea_count > 64 || ew_count > 64 || ea_lo < -60 || ew_lo < -60 ||
      ea_lo + ea_count - 1 > 60 || ew_lo + ew_count - 1 > 60)
    return HIF8_ERR_ARG;
  if (!a || !w || !o_ref || !workspace || !d_err) return HIF8_ERR_NULL;
  if (!aligned_to(d_err, 8) || (d_best && !aligned_to(d_best, 4))) return HIF8_ERR_ARG;
  if (M == 0 || N == 0 || K == 0) return HIF8_ERR_ARG;
  if (M > 0x7FFFFFFFu || N > 0x7FFFFFFFu || K > kMaxLd) return HIF8_ERR_ARG;
  // workspace: every cast operand expanded to bfloat16 for the matrix cores, behind room for one code matrix that
  // hif8_calibrate_workspace_bytes has always counted
  const size_t ld = expanded_ld(K);
  const size_t code_bytes = ((M > N ? M : N) * K + 15) / 16 * 16;
  const size_t a_elems = M * ld, w_elems = N * ld;  // multiples of 64 elements: every matrix stays 128-byte aligned
  if (workspace_bytes < calibrate_bytes(M, N, K, ea_count, ew_count) || !aligned_to(workspace, 16)) return HIF8_ERR_ARG;
  uint16_t* ws_a = reinterpret_cast<uint16_t*>(reinterpret_cast<uint8_t*>(workspace) + code_bytes);
  uint16_t* ws_w = ws_a + a_elems * ea_count;
  hif8_status s = launch_fill_u32(reinterpret_cast<uint32_t*>(d_err), 0u, 2u * (uint32_t)(ea_count * ew_count), st);
  if (s != HIF8_OK) return s;
  s = hif8conv::cast_scales<SRCK>(a, M, K, ea_lo, ea_count, mode, ws_a, ld, a_elems, st);
  if (s != HIF8_OK) return s;
  s = hif8conv::cast_scales<SRCK>(w, N, K, ew_lo, ew_count, mode, ws_w, ld, w_elems, st);
  if (s != HIF8_OK) return s;
  // all pairs in one launch
  const Batch batch{(uint32_t)ea_count, (uint32_t)ew_count, ea_lo + ew_lo, a_elems, w_elems};
  s = gemm_expanded<EPI_ERR>(ws_a, ws_w, nullptr, o_ref, d_err, M, N, ld, 1.0f, st, batch);
  if (s != HIF8_OK) return s;
  if (d_best) {
    hipLaunchKernelGGL(k_argmin_pair, dim3(1), dim3(64), 0, st, d_err, ea_count, ew_count, ea_lo, ew_lo, d_best);
    return finish_launch();
  }
  return HIF8_OK;
}

}  // namespace hif8gemm

using namespace hif8gemm;

extern "C" {

hif8_status hif8_gemm_set_variant(int variant) {
  if (variant != 0 && variant != 5 && variant != 6 && (variant < 9 || variant > 12)) return HIF8_ERR_ARG;
  if (variant == 0) {
    g_gemm_variant = 0;
    expanded_variant() = 0;
  } else if (variant == 12) {
    g_gemm_variant = 12;
    expanded_variant() = 12;
  } else if (variant <= 6) {
    g_gemm_variant = variant;
  } else {
    expanded_variant() = variant;
  }
  return HIF8_OK;
}

size_t hif8_calibrate_workspace_bytes(size_t M, size_t N, size_t K, int ea_count, int ew_count) {
  if (ea_count < 0 || ew_count < 0) return 0;
  return calibrate_bytes(M, N, K, ea_count, ew_count);
}

#define HIF8_DEFINE_CALIBRATE(SFX, T, KIND)                                                                       \
  hif8_status hif8_calibrate_layer_##SFX(const T* a, const T* w, const float* o_ref, size_t M, size_t N,          \
                                         size_t K, int ea_lo, int ea_count, int ew_lo, int ew_count,              \
                                         uint32_t mode, void* workspace, size_t workspace_bytes, double* d_err,   \
                                         int32_t* d_best_or_null, hif8_stream_t stream) {                         \
    return calibrate_layer<KIND>(a, w, o_ref, M, N, K, ea_lo, ea_count, ew_lo, ew_count, mode, workspace,         \
                                 workspace_bytes, d_err, d_best_or_null, (hipStream_t)stream);                    \
  }
HIF8_DEFINE_CALIBRATE(f32, float, kSrcF32)
HIF8_DEFINE_CALIBRATE(bf16, uint16_t, kSrcBF16)
HIF8_DEFINE_CALIBRATE(f16, uint16_t, kSrcF16)
#undef HIF8_DEFINE_CALIBRATE

size_t hif8_gemm_workspace_bytes(size_t M, size_t N, size_t K) { return gemm_ws_bytes(M, N, K); }
hif8_status hif8_gemm_ws_f32(const uint8_t* a_codes, const uint8_t* b_codes, float* out, size_t M, size_t N, size_t K,
                             float scale_a, float scale_b, void* workspace, size_t workspace_bytes, hif8_stream_t stream) {
  return gemm_ws<EPI_F32>(a_codes, b_codes, out, nullptr, nullptr, M, N, K, scale_a, scale_b, workspace, workspace_bytes,
                          (hipStream_t)stream);
}
hif8_status hif8_gemm_ws_bf16(const uint8_t* a_codes, const uint8_t* b_codes, uint16_t* out, size_t M, size_t N, size_t K,
                              float scale_a, float scale_b, void* workspace, size_t workspace_bytes, hif8_stream_t stream) {
  return gemm_ws<EPI_BF16>(a_codes, b_codes, out, nullptr, nullptr, M, N, K, scale_a, scale_b, workspace, workspace_bytes,
                           (hipStream_t)stream);
}
hif8_status hif8_gemm_ws_f16(const uint8_t* a_codes, const uint8_t* b_codes, uint16_t* out, size_t M, size_t N, size_t K,
                             float scale_a, float scale_b, void* workspace, size_t workspace_bytes, hif8_stream_t stream) {
  return gemm_ws<EPI_F16>(a_codes, b_codes, out, nullptr, nullptr, M, N, K, scale_a, scale_b, workspace, workspace_bytes,
                          (hipStream_t)stream);
}
hif8_status hif8_gemm_ws_sqerr(const uint8_t* a_codes, const uint8_t* b_codes, const float* ref, size_t M, size_t N,
                               size_t K, float scale_a, float scale_b, double* d_err, void* workspace,
                               size_t workspace_bytes, hif8_stream_t stream) {
  return gemm_ws<EPI_ERR>(a_codes, b_codes, nullptr, ref, d_err, M, N, K, scale_a, scale_b, workspace, workspace_bytes,
                          (hipStream_t)stream);
}

hif8_status hif8_gemm_f32(const uint8_t* a_codes, const uint8_t* b_codes, float* out, size_t M, size_t N, size_t K,
                          float scale_a, float scale_b, hif8_stream_t stream) {
  return gemm_dispatch<EPI_F32>(a_codes, b_codes, out, nullptr, nullptr, M, N, K, scale_a, scale_b, (hipStream_t)stream);
}
hif8_status hif8_gemm_bf16(const uint8_t* a_codes, const uint8_t* b_codes, uint16_t* out, size_t M, size_t N,
                           size_t K, float scale_a, float scale_b, hif8_stream_t stream) {
  return gemm_dispatch<EPI_BF16>(a_codes, b_codes, out, nullptr, nullptr, M, N, K, scale_a, scale_b, (hipStream_t)stream);
}
hif8_status hif8_gemm_f16(const uint8_t* a_codes, const uint8_t* b_codes, uint16_t* out, size_t M, size_t N,
                          size_t K, float scale_a, float scale_b, hif8_stream_t stream) {
  return gemm_dispatch<EPI_F16>(a_codes, b_codes, out, nullptr, nullptr, M, N, K, scale_a, scale_b, (hipStream_t)stream);
}
hif8_status hif8_gemm_sqerr(const uint8_t* a_codes, const uint8_t* b_codes, const float* ref, size_t M, size_t N,
                            size_t K, float scale_a, float scale_b, double* d_err, hif8_stream_t stream) {
  return gemm_dispatch<EPI_ERR>(a_codes, b_codes, nullptr, ref, d_err, M, N, K, scale_a, scale_b, (hipStream_t)stream);
}

}  // extern "C"
