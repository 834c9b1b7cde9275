// Exact contractions through one Clifford fragment in the Heisenberg picture.
//
// Let C be a Clifford fragment whose carried-back observables are known
// (k_heis.hip).  For a subset S of its requested outputs and Paulis P_out on
// its quantum outputs, O = U^dag (Z_S (x) P_out) U is one Pauli: it fixes the
// Pauli of every quantum input, and its expectation is 0 or (-1)^s 2^n_in.  So
// of the 4^n_in Paulis its inputs could carry exactly one contributes, and
//   R[b_C, b] = 2^(n_in - r - k) sum_S (-1)^(b_C.S)
//               sum_free (-1)^s prod_{f != C} T_f[b_f; P(S, free)|f],
// where `free` runs over the Paulis of the cuts that are not inputs of C: no
// tensor of C is formed and 4^(k - n_in) terms are summed instead of 4^k.  The
// sum over S is a Walsh-Hadamard transform of the r requested bits in LDS.
//
// Bound by latency: a call is a few hundred KB of gathers from small tensors.
// The products over rows are rebuilt by every workgroup (a few thousand
// cycles) rather than kept from a launch before.  Measured on MI355X: the
// 16-qubit marginal of a 300-qubit circuit with 10 cuts, carry-back to result,
// 8300 us (C's 4^10 columns filled and transformed 1590 us, contracted densely
// 6700 us) -> 13 us; 64 strings over 6 cuts 95 -> 2.5 us.
#include <algorithm>

#include "common.hpp"
#include "pauli.hpp"

namespace ccut {

namespace {

typedef __attribute__((address_space(4))) const uint64_t c_u64;
typedef __attribute__((address_space(4))) const RecombArgs c_RecombArgs;
typedef __attribute__((address_space(1))) const double g_f64;

// Column of fragment f's tensor under cut term P (two bits per cut).
template <class F>
__device__ inline uint32_t frag_column(F &f, uint32_t P) {
  uint32_t p = 0;
  for (uint32_t j = 0; j < f.n_axes; ++j) p |= ((P >> (2 * f.axis_cut[j])) & 3u) << (2 * j);
  return p;
}

// The free Paulis' share of the cut term, and C's output Paulis among them
// applied to `acc`.
template <int W>
__device__ inline uint32_t free_paulis(const ExactArgs &A, uint32_t t, PAcc<W> &acc, c_u64 *rows) {
  uint32_t P = 0;
  for (uint32_t i = 0; i < A.n_free; ++i) {
    const uint32_t d = (t >> (2 * i)) & 3u;
    P |= d << (2 * A.free_cut[i]);
    if (A.free_row[i] != ~0u) pmul_out<W>(acc, d, rows + (size_t)A.free_row[i] * (2 * W + 1));
  }
  return P;
}

// C's input Paulis as bits of the cut term; false if a circuit input carries
// X or Y (the expectation vanishes).
template <int W>
__device__ inline bool input_paulis(const ExactArgs &A, const PAcc<W> &acc, uint32_t &P) {
  uint64_t bad = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) bad |= acc.x[w] & A.cin_mask[w];
  if (bad) return false;
  for (uint32_t i = 0; i < A.n_in; ++i) P |= pdigit<W>(acc, A.in_local[i]) << (2 * A.in_cut[i]);
  return true;
}

constexpr uint32_t kExactThreads = 256;

// Workgroup x: outcomes [x G, x G + G) of the other fragments' requested bits
// (G = 256 / 2^r, at least 1), every subset S.
template <int W>
__global__ __launch_bounds__(kExactThreads) void exact_marginal_kernel(const ExactArgs A, const RecombArgs *d_args,
                                                                       const uint64_t *d_rows, double *__restrict__ out) {
  extern __shared__ double h[];  // [G][2^r]
  c_RecombArgs &R = *(c_RecombArgs *)(uintptr_t)d_args;
  c_u64 *rows = (c_u64 *)(uintptr_t)d_rows;
  constexpr uint32_t RS = 2 * W + 1;
  const uint32_t tid = threadIdx.x, r = A.r, n = 1u << r;
  const uint32_t lg = r < 8 ? 8 - r : 0;  // log2 G
  const uint32_t rest = A.nq - r;         // requested bits of the other fragments
  const uint32_t grp = tid >> (8 - lg), s0 = tid & ((kExactThreads >> lg) - 1), step = kExactThreads >> lg;
  const uint32_t b = (blockIdx.x << lg) | grp;
  const bool live = b < 1u << rest;
  // S = s0 + step i: the product over the bits of s0 once, the higher bits
  // stepped through in Gray code order
  PAcc<W> acc;
  pclear(acc);
  const uint32_t lowbits = r < 8 ? r : 8;
  for (uint32_t j = 0; j < lowbits; ++j)
    if (s0 >> j & 1u) pmul<W>(acc, rows + (size_t)j * RS);
  uint32_t gray = 0;
  const uint32_t iters = r > 8 ? 1u << (r - 8) : 1u;
  for (uint32_t i = 0; i < iters; ++i) {
    if (i) {
      const uint32_t j = __ffs(i) - 1;
      gray ^= 1u << j;
      pmul<W>(acc, rows + (size_t)(8 + j) * RS);  // the rows commute: order and repeats only matter for the bits set
    }
    double sum = 0.0;
    for (uint32_t t = 0; t < 1u << (2 * A.n_free); ++t) {
      PAcc<W> o = acc;
      uint32_t P = free_paulis<W>(A, t, o, rows);
      if (!live || !input_paulis<W>(A, o, P)) continue;
      double v = psign<W>(o) ? -1.0 : 1.0;
      uint32_t shift = 0;
      for (uint32_t f = 0; f < R.n_frags; ++f) {
        if (f == A.frag) continue;
        auto &F = R.f[f];
        const uint32_t bf = (b >> shift) & (F.rows - 1);
        shift += F.n_req;
        v *= ((g_f64 *)(uintptr_t)F.T)[(size_t)frag_column(F, P) * F.rows + bf];
      }
      sum += v;
    }
    h[grp * n + (s0 | gray << 8)] = sum;
  }
  __syncthreads();
  // all G transforms at once: the group is the index above bit r
  const uint32_t total = n << lg;
  for (uint32_t s = 0; s < r; ++s) {
    for (uint32_t k = tid; k < total / 2; k += kExactThreads) {
      const uint32_t i0 = ((k >> s) << (s + 1)) | (k & ((1u << s) - 1)), i1 = i0 | (1u << s);
      const double x = h[i0], y = h[i1];
      h[i0] = x + y;
      h[i1] = x - y;
    }
    __syncthreads();
  }
  auto &C = R.f[A.frag];
  for (uint32_t k = tid; k < total; k += kExactThreads) {
    const uint32_t bc = k & (n - 1), bo = (blockIdx.x << lg) | (k >> r);
    if (bo >= 1u << rest) break;
    uint32_t idx = 0, shift = 0;
    for (uint32_t i = 0; i < r; ++i) idx |= ((bc >> i) & 1u) << C.req_user[i];
    for (uint32_t f = 0; f < R.n_frags; ++f) {
      if (f == A.frag) continue;
      auto &F = R.f[f];
      for (uint32_t i = 0; i < F.n_req; ++i) idx |= ((bo >> (shift + i)) & 1u) << F.req_user[i];
      shift += F.n_req;
    }
    out[idx] = ldexp(h[k], (int)A.n_in - (int)r - (int)R.k);
  }
}

// One string per thread.  F32 (no free cuts): the one term's product in fp32
// as the plain sum of that precision forms it, with its correction term when
// operands are split.
template <int W, bool F32>
__global__ __launch_bounds__(64) void exact_strings_kernel(const ExactArgs A, const RecombArgs *d_args,
                                                           const uint64_t *__restrict__ d_rows, uint32_t n_strings,
                                                           double *__restrict__ out) {
  c_RecombArgs &R = *(c_RecombArgs *)(uintptr_t)d_args;
  c_u64 *rows = (c_u64 *)(uintptr_t)d_rows;
  const uint32_t s = blockIdx.x * 64 + threadIdx.x;
  if (s >= n_strings) return;
  PAcc<W> acc;
  pclear(acc);
  pmul<W>(acc, d_rows + (size_t)s * (2 * W + 1));
  double sum = 0.0;
  for (uint32_t t = 0; t < 1u << (2 * A.n_free); ++t) {
    PAcc<W> o = acc;
    uint32_t P = free_paulis<W>(A, t, o, rows);
    if (!input_paulis<W>(A, o, P)) continue;
    double v = psign<W>(o) ? -1.0 : 1.0;
    float hi = (float)v, corr = 0.f;
    for (uint32_t f = 0; f < R.n_frags; ++f) {
      if (f == A.frag) continue;
      auto &F = R.f[f];
      const double x = ((g_f64 *)(uintptr_t)F.T)[(size_t)frag_column(F, P) * F.rows + s];
      if (F32) {
        const float th = (float)x, tl = R.lo_parts ? (float)(x - (double)th) : 0.f;
        corr = corr * th + hi * tl;
        hi *= th;
      } else {
        v *= x;
      }
    }
    sum += F32 ? (double)(hi + corr) : v;
  }
  out[s] = ldexp(sum, (int)A.n_in - (int)R.k);
}

}  // namespace

hipError_t launch_exact_marginal(const ExactArgs &A, const RecombArgs *d_args, uint32_t W, const uint64_t *rows,
                                 double *out, hipStream_t s) {
  if (A.r > kExactMaxReq || A.r > A.nq || A.n_free > kExactMaxFree || A.nq > 24) return hipErrorInvalidValue;
  const uint32_t lg = A.r < 8 ? 8 - A.r : 0, rest = A.nq - A.r;
  const dim3 grid(rest > lg ? 1u << (rest - lg) : 1u);
  const size_t lds = sizeof(double) << (A.r + lg);
  const void *kernel = W == 1 ? (const void *)exact_marginal_kernel<1>
                       : W == 2 ? (const void *)exact_marginal_kernel<2>
                       : W == 4 ? (const void *)exact_marginal_kernel<4>
                                : (const void *)exact_marginal_kernel<8>;
  hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  switch (W) {
    case 1: hipLaunchKernelGGL(exact_marginal_kernel<1>, grid, dim3(kExactThreads), lds, s, A, d_args, rows, out); break;
    case 2: hipLaunchKernelGGL(exact_marginal_kernel<2>, grid, dim3(kExactThreads), lds, s, A, d_args, rows, out); break;
    case 4: hipLaunchKernelGGL(exact_marginal_kernel<4>, grid, dim3(kExactThreads), lds, s, A, d_args, rows, out); break;
    case 8: hipLaunchKernelGGL(exact_marginal_kernel<8>, grid, dim3(kExactThreads), lds, s, A, d_args, rows, out); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int W>
static void strings_w(const ExactArgs &A, const RecombArgs *d_args, const uint64_t *rows, uint32_t n_strings, bool fp32,
                      double *out, hipStream_t s) {
  const dim3 grid((n_strings + 63) / 64), block(64);
  if (fp32)
    hipLaunchKernelGGL((exact_strings_kernel<W, true>), grid, block, 0, s, A, d_args, rows, n_strings, out);
  else
    hipLaunchKernelGGL((exact_strings_kernel<W, false>), grid, block, 0, s, A, d_args, rows, n_strings, out);
}

hipError_t launch_exact_strings(const ExactArgs &A, const RecombArgs *d_args, uint32_t W, const uint64_t *rows,
                                uint32_t n_strings, bool fp32, double *out, hipStream_t s) {
  if (n_strings == 0) return hipSuccess;
  if (A.n_free > (fp32 ? 0 : kExactMaxFree)) return hipErrorInvalidValue;
  switch (W) {
    case 1: strings_w<1>(A, d_args, rows, n_strings, fp32, out, s); break;
    case 2: strings_w<2>(A, d_args, rows, n_strings, fp32, out, s); break;
    case 4: strings_w<4>(A, d_args, rows, n_strings, fp32, out, s); break;
    case 8: strings_w<8>(A, d_args, rows, n_strings, fp32, out, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace ccut
