// Phase-tracked products of Pauli rows on the device, and the transpose of 64
// rows of 64 bits.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ccut {

// P = i^a X^x Z^z.
template <int W>
struct PAcc {
  uint64_t x[W], z[W];
  uint32_t a;
};

template <int W>
__device__ inline void pclear(PAcc<W> &L) {
#pragma unroll
  for (int w = 0; w < W; ++w) L.x[w] = L.z[w] = 0;
  L.a = 0;
}

template <int W, class R>
__device__ inline void pmul(PAcc<W> &L, R *row) {  // L <- L * row (a Hermitian row: x[W], z[W], sign)
  uint32_t cross = 0, pr = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    cross += __popcll(L.z[w] & row[w]);
    pr += __popcll(row[w] & row[W + w]);
  }
  L.a = (L.a + 2u * (uint32_t)row[2 * W] + pr + 2u * cross) & 3u;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    L.x[w] ^= row[w];
    L.z[w] ^= row[W + w];
  }
}

// A Pauli (I, X, Y, Z = 0..3) of a quantum output: rx its X row, its Z row
// right behind; Y = i X Z.
template <int W, class R>
__device__ inline void pmul_out(PAcc<W> &L, uint32_t P, R *rx) {
  if (P == 2) L.a = (L.a + 1u) & 3u;
  if (P == 1 || P == 2) pmul<W>(L, rx);
  if (P >= 2) pmul<W>(L, rx + 2 * W + 1);
}

template <int W>
__device__ inline uint32_t pbit(const uint64_t (&v)[W], uint32_t q) {
  uint64_t word = v[0];
#pragma unroll
  for (int w = 1; w < W; ++w)
    if ((q >> 6) == (uint32_t)w) word = v[w];
  return (uint32_t)(word >> (q & 63)) & 1u;
}

// The Pauli on qubit q.
template <int W>
__device__ inline uint32_t pdigit(const PAcc<W> &L, uint32_t q) {
  const uint32_t x = pbit<W>(L.x, q), z = pbit<W>(L.z, q);
  return x ? (z ? 2u : 1u) : (z ? 3u : 0u);
}

// The sign bit of a Hermitian product (a - x.z is 0 or 2).
template <int W>
__device__ inline uint32_t psign(const PAcc<W> &L) {
  uint32_t pxz = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) pxz += __popcll(L.x[w] & L.z[w]);
  return ((L.a - pxz) & 3u) >> 1;
}

// 64 x 64 bits held one row per lane, transposed: bit c of lane r goes to bit
// r of lane c (swaps of the index bits, one lane exchange each).
__device__ inline uint64_t transpose64(uint64_t v, uint32_t lane) {
  constexpr uint64_t low[6] = {0x5555555555555555ull, 0x3333333333333333ull, 0x0F0F0F0F0F0F0F0Full,
                               0x00FF00FF00FF00FFull, 0x0000FFFF0000FFFFull, 0x00000000FFFFFFFFull};
#pragma unroll
  for (int b = 5; b >= 0; --b) {
    const uint32_t j = 1u << b;
    const uint64_t p = __shfl_xor((unsigned long long)v, j);
    v = lane & j ? (v & ~low[b]) | ((p & ~low[b]) >> j) : (v & low[b]) | ((p & low[b]) << j);
  }
  return v;
}

}  // namespace ccut
