// Which per-channel kernels a matrix takes: those that work in vectors, or a lane per element (no HIP types: the CPU tests build it as it stands).
#pragma once

#include <stddef.h>
#include <stdint.h>

#include "hif8_device.hpp"

namespace hif8calib {

enum : int { AXIS_AMAX = 0, AXIS_CAST = 1 };  // maxima; encode or decode

// Standard SR draws its thresholds with one key for each 2^32 elements, and the vector kernels one key for each vector.  Vectors of rows that end with a whole one
// begin at multiples of their width and lie within one such block; others may reach into the next one, where there is one.
inline bool vectors_in_blocks(size_t rows, size_t cols, size_t ve, uint32_t mode) {
  return (mode & 0xFu) != hif8dev::kRmSR || cols % ve == 0 || rows * cols <= (size_t)1 << 32;
}

// True where the element kernels run.  ve: elements of a vector (16 bytes of binary32 or 16-bit values); grid: workgroups of 256 lanes that the vector kernel would take.
// A launch counts its lanes in 32 bits, and the element kernels walk.
// axis 0: the vector kernels take a workgroup for each row, whatever its length, and stage their tables for it (us, vectors / elements, 8 Mi
//   bfloat16 values: 17 columns, TA 344 / 20, maxima 239 / 11; 257, TA 23.8 / 19.9, HR 32 / 21.5, decode 23.3 / 17.9; 385, TA 16.1 / 20.2, HR 22.6 / 21.4, SR 25.6 / 25.8).
//   Maxima by elements are a lane for each row: up to 32 columns, with few rows up to 16 (64 Ki values: 16 columns 4.0 / 3.8, 32 3.3 / 5.3; 8 Mi: 32 107 / 17, binary32 107 / 32; 64 Mi
//   binary32: 32 1010 / 970, 64 512 / 850).
// axis 1: a lane of the vector kernels keeps to its columns, so a wavefront has few lanes where there are few columns, and there are few rows for each in a small
//   matrix (us, 8 Mi bfloat16: 17 columns, TA 45 / 22, SR 236 / 28; 33, TA 26.4 / 21.5; 65, TA 15.2 / 21.5, HR 29 / 23; 129, HR 18.1 / 22.8, SR 28.9 / 27.5; binary32: 33, TA 22.4 / 22.6,
//   HR 35.8 / 23.9, 65, HR 20.9 / 23.7; of any number of columns: 1 Mi bfloat16 TA 5.6 to 7.5 / 5.2, 2 Mi 5.8 to 7.9 / 7.5, HR 8.6 to 15.7 / 7.9, 4 Mi 9.1 to 10.9 / 12.8, but 15.9 where the last
//   wavefront of a row has a vector or a few, SR 25.9 / 15.6; binary32, 512 Ki TA 4.5 / 3.8, 1 Mi 4.5 / 5.2, HR 6.9 / 5.4, 2 Mi 7.5 / 7.8).
//   Maxima by elements end with an atomic for each lane: only where a row is shorter than a vector.
inline bool axis_by_elements(int what, int axis, size_t rows, size_t cols, size_t ve, uint64_t grid, uint32_t mode) {
  if (cols < ve || !vectors_in_blocks(rows, cols, ve, mode) || grid * 256u > 0xFFFFFFFFull) return true;
  const uint32_t rm = mode & 0xFu;
  const bool drawn = rm == hif8dev::kRmHR || rm == hif8dev::kRmSSR || rm == hif8dev::kRmSR;  // more instructions for each element
  const size_t n = rows * cols;
  if (what == AXIS_AMAX) return axis == 0 && cols <= (n < (size_t)1 << 18 ? 16u : 32u);
  if (axis == 0) return cols < (drawn ? 400u : 256u) || n <= (drawn ? (size_t)1 << 18 : (size_t)1 << 17);
  const size_t vecs = (cols + ve - 1) / ve, last = vecs % 64;  // of a row; of the last wavefront on it
  const size_t least = ve == 4 ? (drawn ? 56u : 32u) : (drawn ? 96u : 40u);
  return cols < least || n <= ((size_t)(!drawn ? 1u << 17 : last != 0 && last <= 8 ? 1u << 19 : 1u << 18)) * ve;
}

}  // namespace hif8calib
