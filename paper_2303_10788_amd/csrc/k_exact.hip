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

// Column of fragment f's tensor under cut term P (two bits per cut; up to
// kMaxAxes + kExactMaxFree = 19 cuts pass through one fragment, so 38 bits).
template <class F>
__device__ inline uint32_t frag_column(F &f, uint64_t P) {
  uint32_t p = 0;
  for (uint32_t j = 0; j < f.n_axes; ++j) p |= ((uint32_t)(P >> (2 * f.axis_cut[j])) & 3u) << (2 * j);
  return p;
}

// The free Paulis' share of the cut term, and C's output Paulis among them
// applied to `acc`.
template <int W>
__device__ inline uint64_t free_paulis(const ExactArgs &A, uint32_t t, PAcc<W> &acc, c_u64 *rows) {
  uint64_t P = 0;
  for (uint32_t i = 0; i < A.n_free; ++i) {
    const uint32_t d = (t >> (2 * i)) & 3u;
    P |= (uint64_t)d << (2 * A.free_cut[i]);
    if (A.free_row[i] != ~0u) pmul_out<W>(acc, d, rows + (size_t)A.free_row[i] * (2 * W + 1));
  }
  return P;
}

// C's input Paulis as bits of the cut term; false if a circuit input carries
// X or Y (the expectation vanishes).
template <int W>
__device__ inline bool input_paulis(const ExactArgs &A, const PAcc<W> &acc, uint64_t &P) {
  uint64_t bad = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) bad |= acc.x[w] & A.cin_mask[w];
  if (bad) return false;
  for (uint32_t i = 0; i < A.n_in; ++i) P |= (uint64_t)pdigit<W>(acc, A.in_local[i]) << (2 * A.in_cut[i]);
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
      uint64_t P = free_paulis<W>(A, t, o, rows);
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
    uint64_t P = free_paulis<W>(A, t, o, rows);
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

// ------------------------------------------------- the nonzero columns
// Where the columns of C's tensor are needed themselves (fp32 contractions,
// whose sums of eight terms are rounded in cut-term order, and sampled term
// lists): one workgroup marks the column of every (subset, output Paulis) pair
// in a bit mask in LDS (4^10 terms: 128 KB), counts the bits below each thread's
// words and lists the columns in ascending order; a workgroup per column then
// gathers its pairs and transforms them.  A few of the 4^k columns are
// nonzero (1 to 16 in the 6- and 10-cut workloads).  Measured at 10 cuts: 19 +
// 4 us where filling and transforming every column took 1590 us, its column
// norms another 3400 us and each contraction of 16384 drawn terms 220 us
// (their counts 5, the columns' contraction 16 us); at 6 cuts, 1024 subsets of
// 7 words 20 + 6 us and an fp32 contraction of 15 + 5 us, for 94 us.
constexpr uint32_t kColThreads = 1024;

// Inclusive scan over the workgroup of two counts packed in one word.
__device__ inline uint32_t block_scan(uint32_t v, uint32_t *wave_sum) {
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (uint32_t o = 1; o < 64; o <<= 1) {
    const uint32_t p = __shfl_up(v, o);
    if (lane >= o) v += p;
  }
  __syncthreads();  // wave_sum is free
  if (lane == 63) wave_sum[wave] = v;
  __syncthreads();
  for (uint32_t w = 0; w < wave; ++w) v += wave_sum[w];
  return v;
}

// Words of the mask per thread, and a word's place in LDS: a thread walks its
// own words in order, so each thread's run is one word longer than its words
// (lanes on different banks).
__host__ __device__ inline uint32_t col_per(uint32_t k) { return 2 * k > 15 ? 1u << (2 * k - 15) : 1u; }
__device__ inline uint32_t col_at(uint32_t w, uint32_t per) { return per > 1 ? w + w / per : w; }

template <int W>
__global__ __launch_bounds__(kColThreads) void columns_kernel(const ExactArgs A, const ColumnSet S,
                                                              const uint64_t *d_rows) {
  extern __shared__ uint32_t mask[];  // [4^k / 32], col_at
  __shared__ uint32_t base[kColThreads], wave_sum[kColThreads / 64];
  c_u64 *rows = (c_u64 *)(uintptr_t)d_rows;
  const uint32_t tid = threadIdx.x;
  const uint32_t n_words = 1u << (2 * S.k - 5), per = col_per(S.k);
  for (uint32_t i = tid; i < n_words; i += kColThreads) mask[col_at(i, per)] = 0;
  __syncthreads();
  const uint32_t n_pairs = 1u << (A.r + 2 * A.n_free);
  constexpr uint32_t kMost = kMaxColumnEntries / kColThreads;
  uint32_t pair[kMost];  // this thread's pairs: sign << 31 | term, or ~0
#pragma unroll
  for (uint32_t i = 0; i < kMost; ++i) {
    const uint32_t e = tid + i * kColThreads;
    pair[i] = ~0u;
    if (e >= n_pairs) continue;
    PAcc<W> acc;
    pclear(acc);
    for (uint32_t j = 0; j < A.r; ++j)
      if (e >> j & 1u) pmul<W>(acc, rows + (size_t)j * (2 * W + 1));
    uint64_t term = free_paulis<W>(A, e >> A.r, acc, rows);
    if (!input_paulis<W>(A, acc, term)) continue;
    const uint32_t P = (uint32_t)term;  // (at most kMaxColumnCuts cuts here)
    pair[i] = P | psign<W>(acc) << 31;
    atomicOr(&mask[col_at(P >> 5, per)], 1u << (P & 31));
  }
  __syncthreads();
  // columns (low half) and 8-aligned groups (high half) in this thread's words
  uint32_t own = 0;
  const uint32_t w0 = tid * per, w1 = w0 < n_words ? w0 + per : w0;
  auto groups = [](uint32_t m) {  // nonzero bytes
    return ((m & 0xFFu) != 0) + ((m & 0xFF00u) != 0) + ((m & 0xFF0000u) != 0) + ((m & 0xFF000000u) != 0);
  };
  for (uint32_t w = w0; w < w1; ++w) {
    const uint32_t m = mask[col_at(w, per)];
    own += __popc(m) | (uint32_t)groups(m) << 16;
  }
  const uint32_t incl = block_scan(own, wave_sum);
  base[tid] = (incl - own) & 0xFFFFu;
  uint32_t col = (incl - own) & 0xFFFFu, grp = (incl - own) >> 16;
  if (tid == kColThreads - 1) {
    S.count[0] = incl & 0xFFFFu;
    S.count[1] = S.group8 ? 8ull * (incl >> 16) : incl & 0xFFFFu;
  }
  if (S.mask) {
    for (uint32_t i = tid; i < n_words; i += kColThreads) S.mask[i] = mask[col_at(i, per)];
    if (w0 < n_words) S.rank[tid] = col;
  }
  for (uint32_t w = w0; own && w < w1; ++w) {
    const uint32_t m = mask[col_at(w, per)];
    for (uint32_t g = 0; m && g < 4; ++g) {
      const uint32_t byte = m >> (8 * g) & 0xFFu;
      if (!byte) continue;
      for (uint32_t i = 0; i < 8; ++i) {
        const uint64_t P = 32ull * w + 8 * g + i;
        const bool in = byte >> i & 1u;
        if (S.group8) {
          S.terms[8 * grp + i] = P;
          S.term_col[8 * grp + i] = in ? col : S.zero;
        } else if (in) {
          S.terms[col] = P;
          S.term_col[col] = col;
        }
        if (in) S.cols[col++] = P;
      }
      ++grp;
    }
  }
  __syncthreads();
#pragma unroll
  for (uint32_t i = 0; i < kMost; ++i) {
    const uint32_t e = tid + i * kColThreads;
    if (e >= n_pairs) continue;
    uint32_t out = ~0u;
    if (pair[i] != ~0u) {
      const uint32_t P = pair[i] & 0x7FFFFFFFu, w = P >> 5, t = w / per;
      uint32_t c = base[t] + __popc(mask[col_at(w, per)] & ((1u << (P & 31)) - 1));
      for (uint32_t v = t * per; v < w; ++v) c += __popc(mask[col_at(v, per)]);
      out = 2 * c | pair[i] >> 31;
    }
    S.entries[e] = out;
  }
}

// Block c: column c (blocks past the columns end at once; block `zero` writes
// the zero column).
__global__ __launch_bounds__(256) void column_tensor_kernel(const ExactArgs A, const ColumnSet S,
                                                            double *__restrict__ T, double *__restrict__ norm) {
  extern __shared__ double h[];
  __shared__ uint32_t size;
  const uint32_t c = blockIdx.x, tid = threadIdx.x, r = A.r, n = 1u << r;
  double *row = T + (size_t)c * n;
  if (c == S.zero) {
    for (uint32_t i = tid; i < n; i += 256) row[i] = 0.0;
    return;
  }
  if (c >= S.count[0]) return;
  if (tid == 0) size = 0;
  for (uint32_t i = tid; i < n; i += 256) h[i] = 0.0;
  __syncthreads();
  const uint32_t n_pairs = n << (2 * A.n_free);
  const double v = ldexp(1.0, (int)A.n_in);
  uint32_t found = 0;
  for (uint32_t e = tid; e < n_pairs; e += 256) {
    const uint32_t x = S.entries[e];
    if (x >> 1 != c || x == ~0u) continue;
    h[e & (n - 1)] = x & 1u ? -v : v;  // (a column has one output Pauli combination: its subsets differ)
    ++found;
  }
  if (norm && found) atomicAdd(&size, found);
  __syncthreads();
  for (uint32_t s = 0; s < r; ++s) {
    for (uint32_t k = tid; k < n / 2; k += 256) {
      const uint32_t i0 = ((k >> s) << (s + 1)) | (k & ((1u << s) - 1)), i1 = i0 | (1u << s);
      const double a = h[i0], b = h[i1];
      h[i0] = a + b;
      h[i1] = a - b;
    }
    __syncthreads();
  }
  for (uint32_t i = tid; i < n; i += 256) row[i] = ldexp(h[i], -(int)r);
  // sum_b T[b]^2 = 2^-r sum_S tau[S]^2 (every value is a power of two times an
  // integer: the sum over b is exact too)
  if (norm && tid == 0) norm[S.cols[c]] = sqrt(ldexp((double)size, 2 * (int)A.n_in - (int)r));
}

__global__ __launch_bounds__(kColThreads) void column_support_kernel(const RecombArgs *d_args, const ExactArgs A,
                                                                     const SupportArgs sa,
                                                                     const uint8_t *__restrict__ nz, const ColumnSet S) {
  __shared__ uint32_t wave_sum[kColThreads / 64];
  c_RecombArgs &R = *(c_RecombArgs *)(uintptr_t)d_args;
  const uint32_t n = (uint32_t)S.count[0];
  uint32_t done = 0;
  for (uint32_t i0 = 0; i0 < n; i0 += kColThreads) {
    const uint32_t i = i0 + threadIdx.x;
    bool ok = i < n;
    const uint64_t P = ok ? S.cols[i] : 0;
    for (uint32_t f = 0; ok && f < R.n_frags; ++f) {
      if (f == A.frag) continue;
      auto &F = R.f[f];
      ok = nz[sa.off[f] + frag_column(F, P)] != 0;
    }
    const uint32_t incl = block_scan(ok ? 1u : 0u, wave_sum);
    uint32_t total = 0;
    __syncthreads();
    if (threadIdx.x == kColThreads - 1) wave_sum[0] = incl;
    __syncthreads();
    total = wave_sum[0];
    if (ok) {
      S.terms[done + incl - 1] = P;
      S.term_col[done + incl - 1] = i;
    }
    done += total;
  }
  if (threadIdx.x == 0) S.count[1] = done;
}

// Draws per column, counted in LDS first: most draws fall on a handful of
// columns (16384 global atomics on one counter took 178 us).
__global__ __launch_bounds__(kColThreads) void column_count_kernel(const ColumnSet S, const uint64_t *__restrict__ terms,
                                                                   uint64_t n, uint32_t *__restrict__ counts) {
  __shared__ uint32_t own[kMaxColumnEntries];
  for (uint32_t i = threadIdx.x; i < S.zero; i += kColThreads) own[i] = 0;
  __syncthreads();
  const uint32_t per = col_per(S.k);
  for (uint64_t j = (uint64_t)blockIdx.x * kColThreads + threadIdx.x; j < n; j += (uint64_t)gridDim.x * kColThreads) {
    const uint64_t P = terms[j];
    const uint32_t w = (uint32_t)(P >> 5), m = S.mask[w], b = 1u << (P & 31);
    if (!(m & b)) continue;
    uint32_t c = S.rank[w / per] + __popc(m & (b - 1));
    for (uint32_t v = w / per * per; v < w; ++v) c += __popc(S.mask[v]);
    atomicAdd(&own[c], 1u);
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < S.zero; i += kColThreads)
    if (own[i]) atomicAdd(&counts[i], own[i]);
}

__global__ void column_weight_kernel(const ColumnSet S, uint64_t n, const double *__restrict__ q,
                                     const uint32_t *__restrict__ counts, double *__restrict__ scale,
                                     double *__restrict__ scale2) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= S.count[0]) return;
  const double c = counts[i], s = counts[i] ? 1.0 / ((double)n * q[S.cols[i]]) : 0.0;
  scale[i] = c * s;
  scale2[i] = sqrt(c) * s;
}

}  // namespace

hipError_t launch_columns(const ExactArgs &A, const ColumnSet &S, uint32_t W, const uint64_t *rows, hipStream_t s) {
  if (S.k < 3 || S.k > kMaxColumnCuts || A.r + 2 * A.n_free > 12 || A.n_free > kExactMaxFree)
    return hipErrorInvalidValue;
  static_assert(kMaxColumnEntries == 1u << 12, "pairs per workgroup");
  const uint32_t n_words = 1u << (2 * S.k - 5);
  const size_t lds = sizeof(uint32_t) * (n_words + n_words / col_per(S.k));
  const void *kernel = W == 1 ? (const void *)columns_kernel<1>
                       : W == 2 ? (const void *)columns_kernel<2>
                       : W == 4 ? (const void *)columns_kernel<4>
                                : (const void *)columns_kernel<8>;
  hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  const dim3 grid(1), block(kColThreads);
  switch (W) {
    case 1: hipLaunchKernelGGL(columns_kernel<1>, grid, block, lds, s, A, S, rows); break;
    case 2: hipLaunchKernelGGL(columns_kernel<2>, grid, block, lds, s, A, S, rows); break;
    case 4: hipLaunchKernelGGL(columns_kernel<4>, grid, block, lds, s, A, S, rows); break;
    case 8: hipLaunchKernelGGL(columns_kernel<8>, grid, block, lds, s, A, S, rows); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_column_tensor(const ExactArgs &A, const ColumnSet &S, double *T, double *norm, hipStream_t s) {
  if (A.r + 2 * A.n_free > 12) return hipErrorInvalidValue;
  hipLaunchKernelGGL(column_tensor_kernel, dim3(S.zero + 1), dim3(256), sizeof(double) << A.r, s, A, S, T, norm);
  return hipGetLastError();
}

hipError_t launch_column_support(const RecombArgs *d_args, const ExactArgs &A, const SupportArgs &sa, const uint8_t *nz,
                                 const ColumnSet &S, hipStream_t s) {
  hipLaunchKernelGGL(column_support_kernel, dim3(1), dim3(kColThreads), 0, s, d_args, A, sa, nz, S);
  return hipGetLastError();
}

hipError_t launch_column_weights(const ColumnSet &S, const uint64_t *terms, uint64_t n, const double *q,
                                 uint32_t *counts, double *scale, double *scale2, hipStream_t s) {
  hipError_t e = launch_fill_u32(counts, S.zero, 0u, s);
  if (e != hipSuccess) return e;
  if (n) hipLaunchKernelGGL(column_count_kernel, dim3((unsigned)std::min<uint64_t>((n + kColThreads - 1) / kColThreads, 256)),
                       dim3(kColThreads), 0, s, S, terms, n, counts);
  hipLaunchKernelGGL(column_weight_kernel, dim3((S.zero + 255) / 256), dim3(256), 0, s, S, n, q, counts, scale, scale2);
  return hipGetLastError();
}

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
