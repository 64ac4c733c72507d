// Tile shapes of the FFT passes: lines and threads per workgroup by pass, type,
// length and variant (see fft_passes.hpp).
#pragma once

#include "common.hpp"

namespace fwi {

constexpr int NT = 256;
constexpr int kLdsMax = 160 * 1024;

// rows per workgroup of variant v: 2048 / 4096 / 8192 points
__host__ __device__ constexpr int row_lines(int L, int v, int es) {
  const int pts = v == 0 ? 2048 : v == 1 ? 4096 : 8192;
  const int nl0 = pts / L > 1 ? pts / L : 1;
  // keep the workgroup inside the LDS budget
  return nl0 * (L + L / 8) * es <= kLdsMax - 4096 ? nl0 : (nl0 / 2 > 0 ? nl0 / 2 : 1);
}
template <typename T, int L, int V>
__host__ __device__ constexpr int row_nl() {
  return row_lines(L, V, (int)sizeof(cplx<T>));
}
// strided-pass variants: (columns, threads) = (8, 256), (16, 256), (16, 512),
// with 32 columns instead of 16 for complex64 lines of length 256 (256-byte
// row segments: the 3D elevation passes measured 9% faster than with 16);
// columns are halved while the tile is over half the LDS (two workgroups per CU)
constexpr int kColLds = 80 * 1024;
template <int V>
__host__ __device__ constexpr int col_nt() {
  return V == 2 ? 512 : 256;
}
template <typename T, int L, int V>
__host__ __device__ constexpr int col_nl() {
  constexpr int nl0 = V == 0 ? 8 : (sizeof(T) == 4 && L == 256 ? 32 : 16);
  constexpr int lp = L + L / 8;
  constexpr int es = (int)sizeof(cplx<T>);
  return nl0 * lp * es <= kColLds ? nl0 : (nl0 / 2) * lp * es <= kColLds ? nl0 / 2 : nl0 / 4;
}

// Operator lengths between the tuned ones: one tile per pass (rows of 2048
// points; elevation passes (16, 256), complex128 (8, 256) and from 128 points on
// (16, 512)). The convolution takes (16, 256) and for 320 to 640 complex64 points
// (16, 512); the other tile costs, us per launch: 144 19 against 16, 288 30
// against 28, 432 75 against 64, 576 60 against 53, 640 74 against 69, 864 249
// against 185.
#define FWI_OP_LENGTHS(X) X(72) X(80) X(144) X(160) X(216) X(288) X(320) X(432) X(576) X(640) X(864)
template <typename T>
constexpr int op_conv_variant(int L) {
  return sizeof(T) == 4 && L >= 320 && L <= 640 ? 2 : 1;
}
template <typename T>
constexpr int op_strided_variant(int L) {
  return sizeof(T) == 4 ? 1 : L >= 128 ? 2 : 0;
}

}  // namespace fwi
