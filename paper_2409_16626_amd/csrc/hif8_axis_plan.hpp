// Which per-channel kernels a matrix takes: those that work in vectors, or a lane per element (no HIP types: the CPU tests build it as it stands).
#pragma once

#include <stddef.h>
#include <stdint.h>

#include "hif8_device.hpp"

namespace hif8calib {

enum : int { AXIS_AMAX = 0, AXIS_ENCODE = 1, AXIS_DECODE = 2 };  // maxima; casts to codes; back to values

// Standard SR draws its thresholds with one key for each 2^32 elements, and the vector kernels one key for each vector.  Vectors of rows that end with a whole one
// begin at multiples of their width and lie within one such block; others may reach into the next one, where there is one.
inline bool vectors_in_blocks(size_t rows, size_t cols, size_t ve, uint32_t mode) {
  return (mode & 0xFu) != hif8dev::kRmSR || cols % ve == 0 || rows * cols <= (size_t)1 << 32;
}

// A matrix of fewer than `cols` columns, or of at most `values` values, goes to the element kernels.  The lines lie where 3900 drawn matrices of 60 Ki to 40 Mi values
// and 9 to 40000 columns, two thirds of them with an odd number, put them: the choice is 0.3 % behind the faster kernel in the mean (3.5 % with one line for all calls of an axis), and six
// are slower by more than 4.5 % than by vectors where those begin at multiples of 16 bytes, else by elements.  us, vectors / elements, below a line and beyond it:
//   axis 0: the vector kernels take a workgroup for each row, whatever its length, and stage their tables for it.  binary32, TA 38165 x 169 29.9 / 16.6, 19586 x 843 21.2 / 37.1; 101 x 4567
//     3.7 / 3.3, 295 x 4977 4.0 / 5.4; drawn thresholds 29650 x 343 35.2 / 30.4, 24764 x 463 30.7 / 33.5; decode 45263 x 829 51.2 / 44.0, 20511 x 976 23.7 / 25.2, 187 x 7125 4.8 / 3.9,
//     1052 x 3447 6.4 / 6.8.  16 bits, TA 59781 x 183 43 / 26, 28399 x 464 22.6 / 30.6; HR 41125 x 269 39 / 27, 22837 x 481 27.0 / 39.3; decode 73392 x 280 44.5 / 26.9, 30602 x 640
//     23.2 / 25.6, 669 x 4817 4.8 / 6.0
//   axis 1: a lane of the vector kernels keeps to its columns, so a wavefront has few lanes where there are few columns, and there are few rows for each in a small matrix.  binary32, TA
//     930197 x 39 85 / 82, 235342 x 53 24.2 / 29.8; 289 x 3153 5.6 / 4.4, 1571 x 1885 7.0 / 8.8; HR 254767 x 39 35.6 / 26.6, 69687 x 153 13.7 / 28.0, 779 x 1975 9.8 / 6.9, 1720 x 2377 11.0 /
//     13.7; decode 490913 x 40 46.8 / 26.4, 71540 x 176 16.5 / 18.5, 871 x 1904 6.1 / 4.6, 1720 x 11232 22.9 / 25.9, but 1721 x 9347 23.7 / 22.7.  16 bits, TA 531309 x 35 57 / 44, 195784 x
//     105 25.8 / 48.8; 669 x 2075 7.5 / 5.5, 3449 x 1913 9.0 / 17.4; SR 237192 x 71 86 / 60, HR 55804 x 169 16.3 / 24.6, 1138 x 2423 14.7 / 12.0, 2222 x 2189 15.2 / 19.0; decode 308647 x 61 38.5
//     / 26.9, 128699 x 189 22.0 / 34.0, 1215 x 1755 7.3 / 5.1, 3406 x 3000 11.0 / 14.8
// Vectors that begin at multiples of 16 bytes are faster than others, so the lines differ; of binary32 values by columns others never gain over the elements.
struct AxisLine {
  uint32_t cols, values;
};
constexpr AxisLine kAxisLines[2][2][3][2] = {  // vectors at any address, at multiples of 16 bytes; axis; rounding by value, thresholds drawn, decode; binary32, 16 bits
    {{{{384, 5u << 17}, {320, 5u << 17}}, {{448, 11u << 16}, {448, 11u << 16}}, {{1024, 3u << 20}, {640, 5u << 19}}},
     {{{48, 3u << 19}, {64, 9u << 18}}, {{80, 5u << 19}, {128, 13u << 18}}, {{0x80000000u, 0u}, {112, 15u << 18}}}},
    {{{{384, 1u << 19}, {320, 1u << 19}}, {{384, 1u << 19}, {288, 1u << 19}}, {{704, 11u << 16}, {512, 5u << 18}}},
     {{{48, 5u << 18}, {56, 1u << 21}}, {{80, 5u << 19}, {96, 3u << 20}}, {{80, 1u << 21}, {80, 5u << 19}}}}};

// True where the element kernels run.  ve: elements of a vector (16 bytes of binary32 or 16-bit values); grid: workgroups of 256 lanes that the vector kernel would take;
// aligned: the values begin at a multiple of 16 bytes.  A launch counts its lanes in 32 bits, and the element kernels walk.
// Maxima by elements, axis 0, are a lane for each row: up to 32 columns, with few rows up to 16 (us, vectors / elements, 64 Ki values: 16 columns 4.0 / 3.8, 32 3.3 / 5.3; 8 Mi: 32 107 / 17, binary32
// 107 / 32; 64 Mi binary32: 32 1010 / 970, 64 512 / 850); axis 1 they end with an atomic for each lane: only where a row is shorter than a vector.
inline bool axis_by_elements(int what, int axis, size_t rows, size_t cols, size_t ve, uint64_t grid, uint32_t mode, bool aligned) {
  if (cols < ve || !vectors_in_blocks(rows, cols, ve, mode) || grid * 256u > 0xFFFFFFFFull) return true;
  const size_t n = rows * cols;
  if (what == AXIS_AMAX) return axis == 0 && cols <= (n < (size_t)1 << 18 ? 16u : 32u);
  const uint32_t rm = mode & 0xFu;
  const bool whole = aligned && cols % ve == 0;
  const bool drawn = rm == hif8dev::kRmHR || rm == hif8dev::kRmSR || (rm == hif8dev::kRmSSR && !(whole && axis == 1));  // more instructions for each element
  AxisLine line = kAxisLines[whole ? 1 : 0][axis][what == AXIS_DECODE ? 2 : drawn ? 1 : 0][ve == 4 ? 0 : 1];
  const size_t last = (cols + ve - 1) / ve % 64;  // vectors of the last wavefront of a row
  if (axis == 1 && what == AXIS_ENCODE && drawn && ve == 8 && last != 0 && last <= 8) line.values = 1u << 22;  // 6336 x 568 HR 15.9 / 10.5
  return cols < line.cols || n <= line.values;
}

// Maximum, scale and codes of rows in three launches by elements instead of one pass in vectors, in which a wavefront has a row and few lanes at work on a narrow one (us, one pass / three
// launches: 223270 rows of 4 binary32 values TA 29 / 10, SR 61 / 11, of 16 32 / 22, 62 / 25, of 24 32.8 / 35.2; of 8 bfloat16 36 / 12, 93 / 15, of 24 39 / 26, of 32 38.8 / 37.7; 50000 rows of 8
// bfloat16 TA 10.2 / 10.2, SR 23.9 / 10.2; 5000 4.5 / 10.5).
inline bool rows_by_elements(size_t rows, size_t cols, size_t ve, uint32_t mode) {
  const uint32_t rm = mode & 0xFu;
  const bool drawn = rm == hif8dev::kRmHR || rm == hif8dev::kRmSSR || rm == hif8dev::kRmSR;
  return cols <= (ve == 4 ? 16u : 24u) && rows >= (drawn ? 60000u : 100000u);
}

}  // namespace hif8calib
