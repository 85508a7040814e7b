// Declarations of the simulated-HiF8 GEMM kernels (u8 code operands expanded in the kernel, operands already expanded to
// bfloat16, small tiles of either) and what they share: accumulator types, output kinds, the batched-launch descriptor of
// Algorithm 1's scale search, the store of one element.  Then the epilogue of the expanded-operand kernel (descale, then
// store or score against a reference in whole lines); the other two store from their own sums.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "hif8.h"
#include "hif8_device.hpp"
#include "hif8_gemm_split.hpp"

namespace hif8gemm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

enum : int { EPI_F32 = 0, EPI_BF16 = 1, EPI_F16 = 2, EPI_ERR = 3 };

// Batched launches (Algorithm 1's scale search): every pair (i, j), i < na, j < nb, of matrices A + i * a_stride and
// B + j * b_stride (strides in operand elements) against one reference, err[i * nb + j], descale 2^-(e_base + i + j).
// na == 0: a single GEMM.  Tiles are numbered over a grid of tiles_m * na x tiles_n * nb with i and j the fast indexes,
// so that the tiles a die works on at a time are many pairs at few places of the matrix: they share a few tiles of the
// reference in that die's L2 (a tile of 256 KiB per workgroup otherwise, 67 MB a round from the last-level cache).
struct Batch {
  uint32_t na, nb;
  int e_base;
  size_t a_stride, b_stride;
};

// One output element.
template <int EPI>
__device__ __forceinline__ void store_one(void* __restrict__ out, size_t idx, float o) {
  if constexpr (EPI == EPI_F32) reinterpret_cast<float*>(out)[idx] = o;
  else if constexpr (EPI == EPI_BF16) reinterpret_cast<uint16_t*>(out)[idx] = (uint16_t)hif8dev::narrow_bf16(__float_as_uint(o));
  else reinterpret_cast<_Float16*>(out)[idx] = (_Float16)o;
}

// 16-byte accesses at any element's address (a row of a matrix with an odd N starts anywhere; the hardware takes them).
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef f32x4 f32x4_any __attribute__((aligned(4)));
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));

// Two values -> two 16-bit floats in one dword, by the hardware's conversions.
template <int EPI>
__device__ __forceinline__ uint32_t pack16(float a, float b) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
  const f32x2 f = {a, b};
  if constexpr (EPI == EPI_BF16) return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
  else return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, f16x2));
}

// Epilogue of one wavefront of the expanded-operand kernel: TM x TN blocks of 32 x 32, each of 2 x 2 accumulators of
// v_mfma_f32_16x16x32_bf16, multiplied as B x A^T so that a lane holds runs of four neighbouring columns (row lane % 16,
// columns (lane / 16) * 4 .. + 3).  (row0, col0): top-left element of the wavefront's tile.
//
// What bounds it is the number of memory instructions and the lines each of them touches: stored element by element from
// the accumulators, a 256 x 256 tile takes 1024 store instructions, and a round of such tiles spent 11 us (bfloat16), 13
// us (binary32), 24 us (squared error, whose loads were waited for block by block) outside its K loop; 16 bytes per lane
// straight from the accumulators, 32 bytes of a row at a time, more than doubled the binary32 time.  So CB blocks at a time
// pass through LDS (32 rows of CB * 32 values in an area of the wavefront's own, rows 4 banks apart) and leave in whole
// lines: 64 lanes x 16 bytes = CB * 128 (binary32) or CB * 64 bytes of a row.
//
// Edge tiles do the same: blocks outside the matrix are skipped, everything is read from LDS before the first store, and the
// last run of a row leaves as 8, 4 and 2 bytes (a loop over rows and over the elements of that run, or reference values
// requested only when their block is due, waited for each: bfloat16 512 x 967 x 128 7.8 us -> 5.9, binary32 1201 x 1203 x
// 256 8.5 -> 7.0, squared error 700 x 6194 x 64 9.8 -> 8.2).
//
// EPI_ERR adds the squared differences to *err in fp64; the reference values of the next blocks are requested before
// those of the current ones are used, and the wavefronts of the workgroup combine into one atomic per workgroup.
// lds: epilogue_lds(CB) bytes per wavefront, free of other use by now.  Every wavefront of the workgroup must call.
constexpr int epilogue_lds(int cb) { return 32 * (cb * 32 + 4) * 4; }

template <typename F, int... C>
__device__ __forceinline__ void for_each_chunk(F&& f, std::integer_sequence<int, C...>) {
  (f(std::integral_constant<int, C>{}), ...);
}
// The blocks of a row of TN, at most CB (a power of two) at a time: how many from block j on, and which chunk that is.
template <int TN, int CB>
struct EpilogueChunks {
  static constexpr int width(int j) {
    int w = CB;
    while (w > TN - j) w /= 2;
    return w;
  }
  static constexpr int per_row() {
    int n = 0;
    for (int j = 0; j < TN; j += width(j)) ++n;
    return n;
  }
  static constexpr int first(int c) {  // first block of chunk c of a row
    int j = 0;
    for (; c > 0; --c) j += width(j);
    return j;
  }
};

// W blocks of 32 x 32 from block (I, J) on, descaled, into LDS.
template <int I, int J, int W, int TM2, int TN2>
__device__ __forceinline__ void blocks_to_lds(const f32x4 (&acc)[TM2][TN2], float* stage, int pitch, uint32_t lane, float descale) {
  float* const at = stage + (lane & 15u) * pitch + (lane >> 4) * 4u;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2 * W; ++j) {
      const f32x4& a = acc[2 * I + i][2 * J + j];
      *reinterpret_cast<f32x4*>(at + i * 16 * pitch + j * 16) = f32x4{__fmul_rn(a[0], descale), __fmul_rn(a[1], descale),
                                                                      __fmul_rn(a[2], descale), __fmul_rn(a[3], descale)};
    }
}

// Columns of a lane on the way out, and the 16-byte stores that a wavefront of TM x TN blocks issues where its part lies inside the matrix.  A
// kernel that goes on to another tile counts these stores behind the loads it waits for (k_gemm_x), so the epilogue may issue more
// of them, but never fewer; a test counts them in the built code.
constexpr int epilogue_width(int epi) { return epi == EPI_BF16 || epi == EPI_F16 ? 8 : 4; }
constexpr int epilogue_stores(int epi, int tm, int tn) { return epi == EPI_ERR ? 0 : 32 * tm * 32 * tn / (64 * epilogue_width(epi)); }

template <int EPI, int TM, int TN, int CB, typename Acc>
__device__ __forceinline__ void epilogue(const Acc& acc, void* __restrict__ out,
                                         const float* __restrict__ ref, double* __restrict__ err, uint32_t M,
                                         uint32_t N, uint32_t row0, uint32_t col0, uint32_t lane, float descale,
                                         uint8_t* lds, uint32_t wave, uint32_t n_waves) {
  using Chunks = EpilogueChunks<TN, CB>;
  constexpr int kWidth = epilogue_width(EPI);
  constexpr int kChunks = TM * Chunks::per_row();
  float* const stage = reinterpret_cast<float*>(lds + wave * epilogue_lds(CB));
  const bool inside = row0 + TM * 32 <= M && col0 + TN * 32 <= N;  // the usual case: no bounds checks

  // chunk C: blocks (I, J) .. (I, J + W - 1) as 32 rows of W * 32 values
  auto with = [&](auto chunk, auto&& f) {
    constexpr int C = decltype(chunk)::value, I = C / Chunks::per_row(), J = Chunks::first(C % Chunks::per_row()), W = Chunks::width(J);
    constexpr int kPitch = W * 32 + 4, kLanes = W * 32 / kWidth, kRows = 64 / kLanes, kSteps = 32 / kRows;  // lanes per row, rows per step
    f(std::integral_constant<int, I>{}, std::integral_constant<int, J>{}, std::integral_constant<int, W>{},
      std::integral_constant<int, kPitch>{}, std::integral_constant<int, kLanes>{}, std::integral_constant<int, kRows>{},
      std::integral_constant<int, kSteps>{});
  };
  auto to_lds = [&](auto chunk) {
    with(chunk, [&](auto i, auto j0, auto w, auto pitch, auto, auto, auto) {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // a wavefront's LDS operations run in order: only the
      __builtin_amdgcn_wave_barrier();                        // compiler has to keep them so
      blocks_to_lds<i, j0, w>(acc, stage, pitch, lane, descale);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    });
  };
  // f(step, row, column, LDS address) for the runs of kWidth columns this lane has of a chunk
  auto runs = [&](auto chunk, auto&& f) {
    with(chunk, [&](auto i, auto j0, auto, auto pitch, auto lanes, auto rows, auto steps) {
      const uint32_t r = lane / lanes, c = lane % lanes * kWidth;
#pragma unroll
      for (int s = 0; s < steps; ++s)
        f(s, row0 + (uint32_t)(i * 32 + s * rows) + r, col0 + (uint32_t)(j0 * 32) + c, stage + (s * rows + r) * pitch + c);
    });
  };
  // nothing of a chunk lies inside the matrix (the same for all lanes)
  auto outside = [&](auto chunk) {
    bool none = false;
    with(chunk, [&](auto i, auto j0, auto, auto, auto, auto, auto) { none = row0 + i * 32u >= M || col0 + j0 * 32u >= N; });
    return none;
  };
  auto each = [&](auto&& f) { for_each_chunk(f, std::make_integer_sequence<int, kChunks>{}); };

  if constexpr (EPI == EPI_ERR) {
    double e2[4] = {0.0, 0.0, 0.0, 0.0};  // one chain of additions per column of a lane
    if (inside) {
      f32x4 r[2][CB * 4];
      auto request = [&](auto chunk) {
        runs(chunk, [&](int s, uint32_t row, uint32_t col, const float*) {
          r[chunk & 1][s] = *reinterpret_cast<const f32x4_any*>(ref + (size_t)row * N + col);
        });
      };
      request(std::integral_constant<int, 0>{});
      each([&](auto chunk) {
        constexpr int C = decltype(chunk)::value;
        if constexpr (C + 1 < kChunks) request(std::integral_constant<int, C + 1>{});
        to_lds(chunk);
        runs(chunk, [&](int s, uint32_t, uint32_t, const float* at) {
          const f32x4 o = *reinterpret_cast<const f32x4*>(at);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const double d = (double)o[k] - (double)r[C & 1][s][k];
            e2[k] = fma(d, d, e2[k]);
          }
        });
      });
    } else {
      // whole runs are read wherever the row has four columns: a run past its end from the last four, moved down
      const uint32_t last = N < 4u ? 0u : N - 4u;
      f32x4 r[2][CB * 4];
      auto request = [&](auto chunk) {
        if (outside(chunk)) return;
        runs(chunk, [&](int s, uint32_t row, uint32_t col, const float*) {
          const float* p = ref + (size_t)(row < M ? row : M - 1u) * N;
          if (N >= 4u) r[chunk & 1][s] = *reinterpret_cast<const f32x4_any*>(p + (col < last ? col : last));
          else
            for (uint32_t k = 0; k < N; ++k) r[chunk & 1][s][k] = p[k];
        });
      };
      request(std::integral_constant<int, 0>{});
      each([&](auto chunk) {
        constexpr int C = decltype(chunk)::value;
        if constexpr (C + 1 < kChunks) request(std::integral_constant<int, C + 1>{});
        if (outside(chunk)) return;
        to_lds(chunk);
        runs(chunk, [&](int s, uint32_t row, uint32_t col, const float* at) {
          const f32x4 o = *reinterpret_cast<const f32x4*>(at), q = r[C & 1][s];
          const uint32_t shift = col > last ? col - last : 0u;
          const f32x4 v = shift == 0u ? q : shift == 1u ? __builtin_shufflevector(q, q, 1, 2, 3, 3)
                          : shift == 2u ? __builtin_shufflevector(q, q, 2, 3, 3, 3) : __builtin_shufflevector(q, q, 3, 3, 3, 3);
#pragma unroll
          for (uint32_t k = 0; k < 4u; ++k) {
            const double d = (double)o[k] - (double)v[k];
            if (row < M && col + k < N) e2[k] = fma(d, d, e2[k]);
          }
        });
      });
    }
    double e = (e2[0] + e2[1]) + (e2[2] + e2[3]);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) e += __shfl_xor(e, off, 64);
    __syncthreads();  // the wavefronts' areas are read: the sums use the end of the same LDS
    double* const sums = reinterpret_cast<double*>(lds + n_waves * (epilogue_lds(CB) - (uint32_t)sizeof(double)));
    if (lane == 0) sums[wave] = e;
    __syncthreads();
    if (wave == 0 && lane == 0) {
      double t = 0.0;
      for (uint32_t w = 0; w < n_waves; ++w) t += sums[w];
      unsafeAtomicAdd(err, t);  // hardware fp64 add at the L2, no compare-and-swap loop
    }
  } else {
    // a run as the dwords that are stored: 4 binary32 or 8 16-bit values
    auto packed = [&](const float* from) -> u32x4_any {
      if constexpr (EPI == EPI_F32) {
        return __builtin_bit_cast(u32x4_any, *reinterpret_cast<const f32x4*>(from));
      } else {
        float o[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) o[k] = (*reinterpret_cast<const f32x4*>(from + k / 4 * 4))[k % 4];
        if constexpr (EPI == EPI_BF16) {
          bool nan = false;
#pragma unroll
          for (int k = 0; k < 8; k += 2) nan |= (bool)__builtin_isunordered(o[k], o[k + 1]);
          if (nan) {  // the hardware conversion keeps a NaN's sign and payload, the result is 0x7FC0
#pragma unroll
            for (int k = 0; k < 8; ++k) o[k] = o[k] == o[k] ? o[k] : __uint_as_float(0x7FC00000u);
          }
        }
        u32x4_any w;
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] = pack16<EPI>(o[2 * k], o[2 * k + 1]);
        return w;
      }
    };
    constexpr uint32_t kSize = EPI == EPI_F32 ? 4 : 2;
    auto address = [&](uint32_t row, uint32_t col) { return reinterpret_cast<uint8_t*>(out) + ((size_t)row * N + col) * kSize; };
    auto put = [&](uint32_t row, uint32_t col, const u32x4_any& w) { *reinterpret_cast<u32x4_any*>(address(row, col)) = w; };
    // a run with fewer than 16 bytes inside the row: 8, 4 and 2 of them
    auto put_part = [&](uint32_t row, uint32_t col, const u32x4_any& w, uint32_t bytes) {
      uint8_t* const p = address(row, col);
      if (bytes & 8u) {
        const uint32_t v[2] = {w[0], w[1]};
        __builtin_memcpy(p, v, 8);
      }
      if (bytes & 4u) {
        const uint32_t v = bytes & 8u ? w[2] : w[0];
        __builtin_memcpy(p + (bytes & 8u), &v, 4);
      }
      if constexpr (kSize == 2) {
        if (bytes & 2u) {
          const uint16_t v = (uint16_t)(bytes & 8u ? (bytes & 4u ? w[3] : w[2]) : (bytes & 4u ? w[1] : w[0]));
          __builtin_memcpy(p + (bytes & 12u), &v, 2);
        }
      }
    };
    each([&](auto chunk) {
      if (inside) {
        to_lds(chunk);
        runs(chunk, [&](int, uint32_t row, uint32_t col, const float* from) { put(row, col, packed(from)); });
      } else if (!outside(chunk)) {
        to_lds(chunk);
        u32x4_any w[CB * 4];  // all read before the first branch: one wait for the LDS, not one per run
        runs(chunk, [&](int s, uint32_t, uint32_t, const float* from) { w[s] = packed(from); });
        runs(chunk, [&](int s, uint32_t row, uint32_t col, const float*) {
          if (row >= M || col >= N) return;
          if (col + kWidth <= N) put(row, col, w[s]);
          else put_part(row, col, w[s], (N - col) * kSize);
        });
      }
    });
  }
}

// ---- operands expanded to bfloat16 (hif8_gemm_x.hip) ----
// Row pitch of an expanded operand: K rounded up to the K step of the kernel.
constexpr size_t kExpandK = 64;
inline size_t expanded_ld(size_t K) { return (K + kExpandK - 1) / kExpandK * kExpandK; }
// Largest pitch the GEMM accepts: 256 rows x pitch x 2 bytes must fit the 32-bit lane offsets of its tile loads.
constexpr size_t kMaxLd = (size_t)1 << 22;

// tile of the expanded-operand kernel: 0 = by problem size, 9 = 128 x 128, 10 = 256 x 256, 11 = 256 x 192, 12 = the
// small-tile kernel (set through hif8_gemm_set_variant)
int& expanded_variant();

// codes of a, then of b (rows_b may be 0), to bfloat16 rows of pitch ld that follow each other in dst
hif8_status expand_rows(const uint8_t* a, size_t rows_a, const uint8_t* b, size_t rows_b, size_t K, uint16_t* dst, size_t ld,
                        hipStream_t st);
hif8_status expand_cols(const uint8_t* codes, size_t rows, size_t cols, uint16_t* dst, size_t ld, hipStream_t st);

// out = (A x B^T) * descale on operands of pitch ld (zero beyond K); batch.na != 0: the na x nb products of a scale search; tiled: the caller has asked
// small_route(), which said no
template <int EPI>
hif8_status gemm_expanded(const uint16_t* A, const uint16_t* B, void* out, const float* ref, double* err, size_t M,
                          size_t N, size_t ld, float descale, hipStream_t st, const Batch& batch = Batch{}, bool tiled = false);

// ---- few output tiles, any K and alignment of code operands (hif8_gemm_s.hip) ----
// out = (A x B^T) * descale; expanded: operands are bfloat16 of pitch K (a multiple of 64), else codes of pitch K, in the tiles of `plan`
template <int EPI>
hif8_status gemm_small(const void* A, const void* B, bool expanded, void* out, const float* ref, double* err, size_t M,
                       size_t N, size_t K, const SmallPlan& plan, float descale, hipStream_t st);

}  // namespace hif8gemm
