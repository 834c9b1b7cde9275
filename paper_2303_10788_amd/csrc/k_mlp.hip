// Learned importance proposal over the 4^k cut terms of the recombination
// sum (Sec. V-C; its cost grows as 4^k, Sec. III-B): a small ReLU MLP maps
// per-term features to a predicted log-weight, trained and evaluated here
// with BF16 MFMA products and fp32 accumulation; the proposal
// q = (1 - eps) softmax + eps / K, its integer CDF, Philox inverse-CDF term
// sampling, and the per-term inputs (features, labels, support) computed
// from the fragment tensors.
#include <algorithm>
#include <cmath>
#include <mutex>

#include "bf16.hpp"
#include "ccut.h"
#include "common.hpp"

namespace ccut {

namespace {

constexpr int MG_T = 64, MG_K = 32, MG_PAD = 8, MG_THREADS = 256;

// C[m][n] = relu(sum_k A[m][k] B[n][k] + bias[n]) as bf16, fp32
// accumulation.  Rows m >= M read as zero and are not written; N % 64 == 0
// and K % 32 == 0.
__global__ __launch_bounds__(MG_THREADS) void mlp_gemm_kernel(const MlpGemm g) {
  __shared__ __attribute__((aligned(16))) uint16_t As[MG_T][MG_K + MG_PAD];  // [m][k]
  __shared__ __attribute__((aligned(16))) uint16_t Bs[MG_T][MG_K + MG_PAD];  // [n][k]
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t m0 = (uint64_t)blockIdx.x * MG_T;
  const uint32_t n0 = blockIdx.y * MG_T;
  const uint32_t wm = (wave & 1) * 32, wn = (wave >> 1) * 32;
  float4v acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = float4v{0.f, 0.f, 0.f, 0.f};
  for (uint32_t k0 = 0; k0 < g.K; k0 += MG_K) {
    // 64 rows x 32 k of each operand, eight contiguous elements per thread
    const uint32_t rr = tid >> 2, kc = (tid & 3) * 8;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (m0 + rr < g.M) v = *(const uint4 *)(g.A + (m0 + rr) * g.K + k0 + kc);
    *(uint4 *)&As[rr][kc] = v;
    *(uint4 *)&Bs[rr][kc] = *(const uint4 *)(g.B + (uint64_t)(n0 + rr) * g.K + k0 + kc);
    __syncthreads();
    u32x4 a[2], b[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) a[i] = *(const u32x4 *)&As[wm + 16 * i + (lane & 15)][8 * (lane >> 4)];
#pragma unroll
    for (int j = 0; j < 2; ++j) b[j] = *(const u32x4 *)&Bs[wn + 16 * j + (lane & 15)][8 * (lane >> 4)];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = mfma_bf16(a[i], b[j], acc[i][j]);
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint64_t m = m0 + wm + 16 * i + 4 * (lane >> 4) + r;
        const uint32_t n = n0 + wn + 16 * j + (lane & 15);
        if (m < g.M) g.C[m * g.N + n] = f2bf(fmaxf(acc[i][j][r] + g.bias[n], 0.f));
      }
}

// y[m] = scale (b + sum_n H[m][n] w[n]); 32 lanes per row, eight elements per lane,
// summed in a fixed butterfly order.
__global__ void head_forward_kernel(const uint16_t *__restrict__ H, uint32_t width, uint64_t rows,
                                    const uint16_t *__restrict__ w, const float *__restrict__ b, float scale,
                                    float *__restrict__ y) {
  const uint64_t row = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 5;
  const uint32_t l = threadIdx.x & 31;
  float s = 0.f;
  if (row < rows)
    for (uint32_t c = l * 8; c < width; c += 256) {
      const uint4 hv = *(const uint4 *)(H + row * width + c);
      const uint4 wv = *(const uint4 *)(w + c);
      const uint16_t *hp = (const uint16_t *)&hv, *wp = (const uint16_t *)&wv;
#pragma unroll
      for (int t = 0; t < 8; ++t) s += bf2f(hp[t]) * bf2f(wp[t]);
    }
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) s += __shfl_xor(s, o, 32);
  if (row < rows && l == 0) y[row] = scale * (s + b[0]);
}

// ------------------------------------------------------------ term model

__device__ inline uint64_t frag_index(const LearnedDev *__restrict__ L, uint32_t f, uint64_t P) {
  uint64_t p = 0;
  for (uint32_t j = 0; j < L->n_axes[f]; ++j) p |= ((P >> (2 * L->axis_cut[f][j])) & 3ull) << (2 * j);
  return p;
}

// n_f[p] = sqrt(sum_b T_f[p][b]^2), rows summed in order
__global__ void colnorm_kernel(const double *__restrict__ T, uint32_t rows, uint64_t ncols,
                               double *__restrict__ out) {
  const uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= ncols) return;
  double s = 0.0;
  for (uint32_t b = 0; b < rows; ++b) {
    const double t = T[p * rows + b];
    s += t * t;
  }
  out[p] = sqrt(s);
}

// The same for up to 64 rows per column: a wave stages 64 whole columns
// (contiguous in memory) through LDS with coalesced loads, all issued before
// the first store, then each lane sums its column in row order as above.  The
// tiles of all fragments are one launch, as those of their shares, whose ends
// make the phi tables too: a launch is 2 us of work, and the five fragments'
// were fourteen (ten-cut estimate 673 us; in three launches 644 us on MI355X).
__global__ __launch_bounds__(64) void colnorm_tile_kernel(const NormJob *__restrict__ jobs, uint32_t n_jobs) {
  __shared__ double tile[64 * 65];  // column c at c * 65 (padded against bank conflicts)
  uint32_t f = 0;
  while (f + 1 < n_jobs && blockIdx.x >= jobs[f + 1].tile0) ++f;
  const double *__restrict__ T = jobs[f].T;
  double *__restrict__ out = jobs[f].norm;
  const uint32_t rows = jobs[f].rows;
  const uint64_t ncols = 1ull << (2 * jobs[f].n_axes);
  const uint64_t p0 = (uint64_t)(blockIdx.x - jobs[f].tile0) * 64;
  const uint32_t lane = threadIdx.x;
  const uint64_t cols = ncols - p0 < 64 ? ncols - p0 : 64;
  const uint32_t n = (uint32_t)(cols * rows);  // <= 4096 doubles
  const double *src = T + p0 * rows;
  for (uint32_t i0 = 0; i0 < n; i0 += 64 * 16) {
    double v[16];
#pragma unroll
    for (uint32_t k = 0; k < 16; ++k) {
      const uint32_t i = i0 + 64 * k + lane;
      v[k] = i < n ? src[i] : 0.0;
    }
#pragma unroll
    for (uint32_t k = 0; k < 16; ++k) {
      const uint32_t i = i0 + 64 * k + lane;
      if (i < n) tile[(i / rows) * 65 + i % rows] = v[k];
    }
  }
  __syncthreads();
  if (lane < cols) {
    double s = 0.0;
    for (uint32_t b = 0; b < rows; ++b) {
      const double t = tile[lane * 65 + b];
      s += t * t;
    }
    out[p0 + lane] = sqrt(s);
  }
}

// shares[j][d] = sum_{p: digit j of p = d} n[p]^2 / sum_p n[p]^2 for each
// fragment: slot 4 j + d sums the 4^(a-1) columns with that digit, in
// chunks (partials in order, then a fixed-order tree), then the chunks in
// order.
constexpr uint32_t kShareChunk = 4096;
__global__ __launch_bounds__(256) void share_partial_kernel(const NormJob *__restrict__ jobs, uint32_t n_jobs) {
  __shared__ double red[256];
  uint32_t f = 0;
  while (f + 1 < n_jobs && blockIdx.x >= jobs[f + 1].block0) ++f;
  const double *__restrict__ norm = jobs[f].norm;
  const uint32_t local = blockIdx.x - jobs[f].block0, chunks = jobs[f].chunks;
  const uint32_t slot = local / chunks, chunk = local % chunks;
  const uint64_t per_slot = 1ull << (2 * (jobs[f].n_axes - 1));
  const uint32_t j = slot >> 2, d = slot & 3;
  const uint64_t low = (1ull << (2 * j)) - 1;
  const uint64_t e0 = (uint64_t)chunk * kShareChunk;
  const uint64_t e1 = e0 + kShareChunk < per_slot ? e0 + kShareChunk : per_slot;
  double acc = 0.0;
  for (uint64_t e = e0 + threadIdx.x; e < e1; e += 256) {
    const uint64_t p = ((e & ~low) << 2) | ((uint64_t)d << (2 * j)) | (e & low);
    acc += norm[p] * norm[p];
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (uint32_t w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) jobs[f].part[local] = red[0];
}

// The shares and, from them, the phi tables of every cut: phi(s) =
// max(ln s, -40) / 40 of the share of the fragment on each side (src.slot
// holds, per cut and side, the slot of that fragment's share row, or -1 when
// the side has no fragment).  One workgroup, a thread per slot.
__global__ __launch_bounds__(kPhiSlots) void phi_kernel(const NormJob *__restrict__ jobs, uint32_t n_jobs,
                                                        const PhiSrc src, uint32_t n_slots, uint32_t k,
                                                        double *__restrict__ phi) {
  __shared__ double tot[kPhiSlots], share[kPhiSlots];
  const uint32_t i = threadIdx.x;
  uint32_t f = 0;
  if (i < n_slots) {
    while (f + 1 < n_jobs && i >= jobs[f + 1].slot0) ++f;
    const uint32_t chunks = jobs[f].chunks;
    const double *__restrict__ part = jobs[f].part + (uint64_t)(i - jobs[f].slot0) * chunks;
    double sum = 0.0;
    uint32_t c = 0;
    for (; c + 16 <= chunks; c += 16) {  // sixteen loads in flight, added in order
      double v[16];
#pragma unroll
      for (uint32_t u = 0; u < 16; ++u) v[u] = part[c + u];
#pragma unroll
      for (uint32_t u = 0; u < 16; ++u) sum += v[u];
    }
    for (; c < chunks; ++c) sum += part[c];
    tot[i] = sum;
  }
  __syncthreads();
  if (i < n_slots) {
    const double *t = tot + jobs[f].slot0;
    const double total = t[0] + t[1] + t[2] + t[3];
    share[i] = tot[i] / total;
  }
  __syncthreads();
  if (i >= 8 * k) return;  // i = (c * 2 + side) * 4 + d
  const int o = src.slot[i >> 2];
  const double s = o < 0 ? 0.0 : share[o + (i & 3)];
  phi[i] = (s > 0.0 ? fmax(log(s), -40.0) : -40.0) / 40.0;
}

// Feature rows: columns 6c..6c+3 one-hot of P_c, 6c+4 phi_up(c, P_c),
// 6c+5 phi_dn(c, P_c), the rest zero (bf16).
__global__ void features_kernel(const LearnedDev *__restrict__ L, const uint64_t *__restrict__ terms,
                                uint64_t first, uint64_t n, uint32_t width, uint16_t *__restrict__ X) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * width) return;
  const uint64_t t = i / width;
  const uint32_t col = (uint32_t)(i % width);
  const uint64_t P = terms ? terms[t] : first + t;
  const uint32_t c = col / 6, r = col % 6;
  float v = 0.f;
  if (c < L->k) {
    const uint32_t p = (uint32_t)((P >> (2 * c)) & 3u);
    if (r < 4)
      v = r == p ? 1.f : 0.f;
    else
      v = (float)L->phi[(c * 2 + (r - 4)) * 4 + p];
  }
  X[i] = f2bf(v);
}

// Fused forward pass: a workgroup of four waves takes 128 term rows.  The
// rows' features are built in LDS (as features_kernel does); wave w then forms
// columns 64 w .. + 63 of each layer for all rows with increasing k, adds the
// bias, applies the ReLU and rounds to bf16 into the activation tile (in place,
// after a barrier); the head sums each row as head_forward_kernel does.
//
// The products are transposed (weights as the left operand), so that a lane
// holds four consecutive columns of a row and stores them at once.  No other
// wave of the workgroup reads a wave's weights: they come from L2 in lane order
// straight into registers, 4 KB a wave and 32 inner indices, loaded a step
// ahead, and the loop over k has no barrier.  Through LDS they would double its
// traffic, which at 64 columns by 128 rows a wave is 64 bytes a clock for the
// activations alone, half of what LDS delivers.  68 KB of LDS and at most 256
// registers let two workgroups share a CU: one's epilogue, features and head
// run beside the other's products.  2^20 rows (312 GFLOP), F 64, H 256: 358 us,
// 870 TFLOP/s (833 us with 16-deep products and the weights through LDS in
// chunks of 64 columns, a barrier on each side of a chunk).
constexpr uint32_t FF_TM = 128, FF_H = 256, FF_F = 64, FF_THREADS = 256;
constexpr uint32_t FF_AS = FF_H + 8;  // padded row stride (bf16)
constexpr uint32_t FF_LAYERS = 3;

struct FFWeights {
  u32x4 w[4];  // a wave's 64 columns, 32 inner indices
};

__device__ inline void ff_load(FFWeights &B, const uint16_t *__restrict__ W, uint32_t nc, uint32_t c, uint32_t tid) {
  const u32x4 *src = reinterpret_cast<const u32x4 *>(W) + ((size_t)(4 * (tid >> 6)) * nc + c) * 64 + (tid & 63);
#pragma unroll
  for (uint32_t i = 0; i < 4; ++i) B.w[i] = src[(size_t)i * nc * 64];
}

// acc[i][j] += the wave's columns 16 i .. + 15 by rows 16 j .. + 15
__device__ __attribute__((always_inline)) inline void ff_products(const FFWeights &B, const uint16_t *act,
                                                                  float4v (&acc)[4][8]) {
#pragma unroll
  for (uint32_t j = 0; j < 8; ++j) {
    const u32x4 x = *(const u32x4 *)(act + 16 * j * FF_AS);
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) acc[i][j] = mfma_bf16(B.w[i], x, acc[i][j]);
  }
}

__global__ __launch_bounds__(FF_THREADS, 2) void mlp_fused_forward_kernel(const LearnedDev *__restrict__ L,
                                                                          const MlpFused net, uint64_t first,
                                                                          uint64_t n, float scale,
                                                                          float *__restrict__ y) {
  extern __shared__ __attribute__((aligned(16))) uint16_t act[];  // [FF_TM][FF_AS]
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t r0 = (uint64_t)blockIdx.x * FF_TM;
  FFWeights cur;
  ff_load(cur, net.w[0], FF_F / 32, 0, tid);
  // features of rows r0 .. r0 + 127 (zero rows past n), a column per lane
  {
    const uint32_t c = lane / 6, rr = lane % 6;
    uint64_t v = 0;  // the feature's bf16 by P_c
    if (c < L->k) {
#pragma unroll
      for (uint32_t p = 0; p < 4; ++p)
        v |= (uint64_t)f2bf(rr < 4 ? (rr == p ? 1.f : 0.f) : (float)L->phi[(c * 2 + (rr - 4)) * 4 + p]) << (16 * p);
    }
    for (uint32_t t = wave; t < FF_TM; t += FF_THREADS / 64) {
      const uint32_t p = (uint32_t)((first + r0 + t) >> (2 * c)) & 3u;
      act[t * FF_AS + lane] = r0 + t < n ? (uint16_t)(v >> (16 * p)) : (uint16_t)0;
    }
  }
  __syncthreads();
  const uint16_t *in = act + (lane & 15) * FF_AS + 8 * (lane >> 4);
#pragma unroll 1
  for (uint32_t layer = 0; layer < FF_LAYERS; ++layer) {
    const uint16_t *W = net.w[layer];
    const uint32_t nc = layer ? FF_H / 32 : FF_F / 32;
    const uint32_t after = layer + 1 < FF_LAYERS ? layer + 1 : layer;  // (the last layer's own, unused)
    float4v acc[4][8];
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i)
#pragma unroll
      for (uint32_t j = 0; j < 8; ++j) acc[i][j] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (uint32_t c = 0; c < nc; c += 2) {
      FFWeights odd;
      ff_load(odd, W, nc, c + 1, tid);
      ff_products(cur, in + 32 * c, acc);
      const bool more = c + 2 < nc;
      ff_load(cur, more ? W : net.w[after], more ? nc : FF_H / 32, more ? c + 2 : 0, tid);
      ff_products(odd, in + 32 * c + 32, acc);
    }
    float4v b[4];
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i)
      b[i] = *(const float4v *)(net.b[layer] + 64 * wave + 16 * i + 4 * (lane >> 4));
    __syncthreads();  // every wave is done reading this layer's input
#pragma unroll
    for (uint32_t j = 0; j < 8; ++j)
#pragma unroll
      for (uint32_t i = 0; i < 4; ++i) {
        float r[4];
#pragma unroll
        for (uint32_t e = 0; e < 4; ++e) r[e] = fmaxf(acc[i][j][e] + b[i][e], 0.f);
        *(uint64_t *)(act + (16 * j + (lane & 15)) * FF_AS + 64 * wave + 16 * i + 4 * (lane >> 4)) =
            ((uint64_t)f2bf2(r[2], r[3]) << 32) | f2bf2(r[0], r[1]);
      }
    __syncthreads();
  }
  // head: 32 lanes per row, eight consecutive elements per lane, butterfly
  const uint32_t l = tid & 31;
  float w4[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) w4[e] = bf2f(net.w4[l * 8 + e]);
  const float b4 = net.b4[0];
#pragma unroll 4
  for (uint32_t t = tid >> 5; t < FF_TM; t += FF_THREADS / 32) {
    const u32x4 h = *(const u32x4 *)(act + t * FF_AS + l * 8);
    float sacc = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) sacc += bf2f((uint16_t)(h[e >> 1] >> (16 * (e & 1)))) * w4[e];
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) sacc += __shfl_xor(sacc, o, 32);
    if (l == 0 && r0 + t < n) y[r0 + t] = scale * (sacc + b4);
  }
}

// kind 0: labels y(P) = ln(2^-k prod_f n_f[P|f] + 2^-60) (fp64, stored
// fp32); kind 2: y(P) / kLabelScale, the network's regression target;
// kind 1: the product-of-shares log-weights sum_c 40 (phi_up + phi_dn).
__global__ void labels_kernel(const LearnedDev *__restrict__ L, const uint64_t *__restrict__ terms,
                              uint64_t first, uint64_t n, float *__restrict__ y, int kind) {
  const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const uint64_t P = terms ? terms[t] : first + t;
  if (kind == 1) {
    double s = 0.0;
    for (uint32_t c = 0; c < L->k; ++c) {
      const uint32_t p = (uint32_t)((P >> (2 * c)) & 3u);
      s += 40.0 * (L->phi[(c * 2) * 4 + p] + L->phi[(c * 2 + 1) * 4 + p]);
    }
    y[t] = (float)s;
    return;
  }
  double v = ldexp(1.0, -(int)L->k);
  for (uint32_t f = 0; f < L->n_frags; ++f) v *= L->norm[f][frag_index(L, f, P)];
  const double lab = log(v + ldexp(1.0, -60));
  y[t] = (float)(kind == 2 ? lab / kLabelScale : lab);
}

// flags[P] = 1 if every fragment column of P has a nonzero norm
__global__ void support_flags_kernel(const LearnedDev *__restrict__ L, uint64_t K, uint64_t *__restrict__ flags) {
  const uint64_t P = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (P >= K) return;
  uint64_t ok = 1;
  for (uint32_t f = 0; f < L->n_frags; ++f) ok &= L->norm[f][frag_index(L, f, P)] > 0.0 ? 1u : 0u;
  flags[P] = ok;
}
// out[pos - 1] = P for flagged P, pos = inclusive prefix count
__global__ void support_scatter_kernel(const uint64_t *__restrict__ flags, const uint64_t *__restrict__ pos,
                                       uint64_t K, uint64_t cap, uint64_t *__restrict__ out) {
  const uint64_t P = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (P >= K || !flags[P]) return;
  if (pos[P] - 1 < cap) out[pos[P] - 1] = P;
}

// ------------------------------------------------------------ proposal

constexpr uint32_t kRedBlock = 256;
// stats[0] = max of the logits, stats[1] = sum exp(x - max) (fp64), each
// from per-block partials reduced in a fixed order.
__global__ void max_partial_kernel(const float *__restrict__ x, uint64_t n, float *__restrict__ part) {
  __shared__ float red[kRedBlock];
  float m = -INFINITY;
  for (uint64_t i = (uint64_t)blockIdx.x * kRedBlock + threadIdx.x; i < n; i += (uint64_t)gridDim.x * kRedBlock)
    m = fmaxf(m, x[i]);
  red[threadIdx.x] = m;
  __syncthreads();
  for (uint32_t w = kRedBlock / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}
// final reductions: thread t takes partials t, t + 256, ... in order, then a
// fixed tree over the 256 threads (deterministic)
__global__ __launch_bounds__(kRedBlock) void max_final_kernel(const float *__restrict__ part, uint32_t np,
                                                              double *__restrict__ stats) {
  __shared__ float red[kRedBlock];
  float m = -INFINITY;
  for (uint32_t i = threadIdx.x; i < np; i += kRedBlock) m = fmaxf(m, part[i]);
  red[threadIdx.x] = m;
  __syncthreads();
  for (uint32_t w = kRedBlock / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0) stats[0] = (double)red[0];
}
__global__ void sumexp_partial_kernel(const float *__restrict__ x, uint64_t n, const double *__restrict__ stats,
                                      double *__restrict__ part) {
  __shared__ double red[kRedBlock];
  const double mx = stats[0];
  double s = 0.0;
  for (uint64_t i = (uint64_t)blockIdx.x * kRedBlock + threadIdx.x; i < n; i += (uint64_t)gridDim.x * kRedBlock)
    s += exp((double)x[i] - mx);
  red[threadIdx.x] = s;
  __syncthreads();
  for (uint32_t w = kRedBlock / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}
__global__ __launch_bounds__(kRedBlock) void sum_final_kernel(const double *__restrict__ part, uint32_t np,
                                                              double *__restrict__ stats) {
  __shared__ double red[kRedBlock];
  double s = 0.0;
  for (uint32_t i = threadIdx.x; i < np; i += kRedBlock) s += part[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (uint32_t w = kRedBlock / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) stats[1] = red[0];
}
// q = (1 - eps) exp(x - max) / S + eps / n; uniform 1 / n without logits
__global__ void proposal_kernel(const float *__restrict__ x, uint64_t n, const double *__restrict__ stats, double eps,
                                double *__restrict__ q) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  if (!x) {
    q[i] = 1.0 / (double)n;
    return;
  }
  q[i] = (1.0 - eps) * exp((double)x[i] - stats[0]) / stats[1] + eps / (double)n;
}

// integer weights floor(q 2^40)
__global__ void int_weights_kernel(const double *__restrict__ q, uint64_t n, uint64_t *__restrict__ w) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) w[i] = (uint64_t)floor(q[i] * 1099511627776.0);
}

// Inclusive scan of u64 in blocks of 1024 (four per thread), block totals
// out; a second level scans the totals and a third adds them back.
constexpr uint32_t kScanBlock = 256, kScanPer = 4, kScanTile = kScanBlock * kScanPer;
__global__ __launch_bounds__(kScanBlock) void scan_tile_kernel(uint64_t *__restrict__ x, uint64_t n,
                                                               uint64_t *__restrict__ totals) {
  __shared__ uint64_t s[kScanBlock];
  const uint64_t base = (uint64_t)blockIdx.x * kScanTile + threadIdx.x * kScanPer;
  uint64_t v[kScanPer];
  uint64_t run = 0;
#pragma unroll
  for (uint32_t i = 0; i < kScanPer; ++i) {
    run += base + i < n ? x[base + i] : 0;
    v[i] = run;
  }
  s[threadIdx.x] = run;
  __syncthreads();
  for (uint32_t o = 1; o < kScanBlock; o <<= 1) {
    const uint64_t add = threadIdx.x >= o ? s[threadIdx.x - o] : 0;
    __syncthreads();
    s[threadIdx.x] += add;
    __syncthreads();
  }
  const uint64_t before = threadIdx.x ? s[threadIdx.x - 1] : 0;
#pragma unroll
  for (uint32_t i = 0; i < kScanPer; ++i)
    if (base + i < n) x[base + i] = v[i] + before;
  if (threadIdx.x == kScanBlock - 1 && totals) totals[blockIdx.x] = s[kScanBlock - 1];
}
__global__ void scan_add_kernel(uint64_t *__restrict__ x, uint64_t n, const uint64_t *__restrict__ scanned_totals) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint64_t tile = i / kScanTile;
  if (i < n && tile > 0) x[i] += scanned_totals[tile - 1];
}

// Term j: u = (o1 2^32 + o0) mod C[K-1] from Philox(ctr = (j, 0, lo cid,
// hi cid), key = (lo seed ^ 0x7E570001, hi seed)); the term is the smallest
// P with C[P] > u.
__global__ void sample_terms_kernel(const uint64_t *__restrict__ cdf, uint64_t K, uint64_t n, uint64_t seed,
                                    uint64_t cid, uint64_t *__restrict__ out) {
  const uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  const U4 o = philox10((uint32_t)j, 0u, (uint32_t)cid, (uint32_t)(cid >> 32), (uint32_t)seed ^ 0x7E570001u,
                        (uint32_t)(seed >> 32));
  const uint64_t total = cdf[K - 1];
  if (total == 0) {  // every integer weight rounded to zero: no valid draw
    out[j] = 0;
    return;
  }
  const uint64_t u = (((uint64_t)o.w[1] << 32) | o.w[0]) % total;
  uint64_t lo = 0, hi = K - 1;  // cdf[hi] = total > u
  while (lo < hi) {
    const uint64_t mid = (lo + hi) >> 1;
    if (cdf[mid] > u)
      hi = mid;
    else
      lo = mid + 1;
  }
  out[j] = lo;
}

// importance weights 1 / (N q[P_j])
__global__ void is_scale_kernel(const uint64_t *__restrict__ terms, const double *__restrict__ q, uint64_t n,
                                double *__restrict__ scale) {
  const uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j < n) scale[j] = 1.0 / ((double)n * q[terms[j]]);
}

// the estimate's summed standard error: partial sums of a fixed stride, a
// fixed tree, then a tree over the blocks
__global__ __launch_bounds__(256) void stderr_partial_kernel(const double *__restrict__ e, const double *__restrict__ e2,
                                                             uint64_t bins, uint32_t k, double n,
                                                             double *__restrict__ part) {
  __shared__ double red[256];
  double s = 0.0;
  for (uint64_t b = (uint64_t)blockIdx.x * 256 + threadIdx.x; b < bins; b += (uint64_t)gridDim.x * 256)
    s += sqrt(fmax(0.0, ldexp(e2[b], -(int)k) - e[b] * e[b] / n));
  red[threadIdx.x] = s;
  __syncthreads();
  for (uint32_t w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}
__global__ __launch_bounds__(kStderrBlocks) void stderr_final_kernel(const double *__restrict__ part, uint32_t n,
                                                                     double *__restrict__ out) {
  __shared__ double red[kStderrBlocks];
  red[threadIdx.x] = threadIdx.x < n ? part[threadIdx.x] : 0.0;
  __syncthreads();
  for (uint32_t w = kStderrBlocks / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = red[0];
}

inline unsigned blocks(uint64_t n, uint32_t b) { return (unsigned)((n + b - 1) / b); }

}  // namespace

hipError_t launch_mlp_gemm(const MlpGemm &g, hipStream_t s) {
  if (g.N % MG_T || g.K % MG_K) return hipErrorInvalidValue;
  const uint64_t tm = (g.M + MG_T - 1) / MG_T;
  if (tm == 0) return hipSuccess;
  if (tm > 0x7FFFFFFFull) return hipErrorInvalidValue;
  hipLaunchKernelGGL(mlp_gemm_kernel, dim3((unsigned)tm, g.N / MG_T), dim3(MG_THREADS), 0, s, g);
  return hipGetLastError();
}

hipError_t launch_mlp_logits_fused(const LearnedDev *L, const MlpFused &net, uint64_t first, uint64_t n, float scale,
                                   float *y, hipStream_t s) {
  if (net.F != FF_F || net.H != FF_H) return hipErrorInvalidValue;
  if (n == 0) return hipSuccess;
  const size_t lds = (size_t)FF_TM * FF_AS * sizeof(uint16_t);
  hipError_t e = hipFuncSetAttribute((const void *)mlp_fused_forward_kernel,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  const uint64_t blocks_n = (n + FF_TM - 1) / FF_TM;
  if (blocks_n > 0x7FFFFFFFull) return hipErrorInvalidValue;
  hipLaunchKernelGGL(mlp_fused_forward_kernel, dim3((unsigned)blocks_n), dim3(FF_THREADS), lds, s, L, net, first, n,
                     scale, y);
  return hipGetLastError();
}

hipError_t launch_head_forward(const uint16_t *H, uint32_t width, uint64_t rows, const uint16_t *w, const float *b,
                               float scale, float *y, hipStream_t s) {
  if (width % 8 || rows == 0) return rows == 0 ? hipSuccess : hipErrorInvalidValue;
  hipLaunchKernelGGL(head_forward_kernel, dim3(blocks(rows * 32, 256)), dim3(256), 0, s, H, width, rows, w, b, scale,
                     y);
  return hipGetLastError();
}

hipError_t launch_norms(const NormJob *jobs, const NormJob *d_jobs, uint32_t n_jobs, const PhiSrc &src, uint32_t k,
                        double *phi, hipStream_t s) {
  uint32_t tiles = 0, parts = 0, slots = 0;
  for (uint32_t f = 0; f < n_jobs; ++f) {
    const NormJob &J = jobs[f];
    if (J.n_axes > (uint32_t)kMaxAxes || J.tile0 != tiles || J.block0 != parts || J.slot0 != slots)
      return hipErrorInvalidValue;
    const uint64_t ncols = 1ull << (2 * J.n_axes);
    tiles += norm_tiles(J);
    parts += 4 * J.n_axes * J.chunks;
    slots += 4 * J.n_axes;
    if (J.T && norm_tiles(J) == 0)
      hipLaunchKernelGGL(colnorm_kernel, dim3(blocks(ncols, 256)), dim3(256), 0, s, J.T, J.rows, ncols, J.norm);
  }
  if (slots > kPhiSlots || 8 * k > kPhiSlots) return hipErrorInvalidValue;
  if (tiles) hipLaunchKernelGGL(colnorm_tile_kernel, dim3(tiles), dim3(64), 0, s, d_jobs, n_jobs);
  if (parts) hipLaunchKernelGGL(share_partial_kernel, dim3(parts), dim3(256), 0, s, d_jobs, n_jobs);
  hipLaunchKernelGGL(phi_kernel, dim3(1), dim3(kPhiSlots), 0, s, d_jobs, n_jobs, src, slots, k, phi);
  return hipGetLastError();
}

uint32_t norm_tiles(const NormJob &J) {
  return J.T && J.rows <= 64 ? (uint32_t)(((1ull << (2 * J.n_axes)) + 63) / 64) : 0;
}

uint32_t share_chunks(uint32_t n_axes) {
  if (n_axes == 0) return 1;
  const uint64_t per_slot = 1ull << (2 * (n_axes - 1));
  return (uint32_t)((per_slot + kShareChunk - 1) / kShareChunk);
}

hipError_t launch_features(const LearnedDev *L, const uint64_t *terms, uint64_t first, uint64_t n, uint32_t width,
                           uint16_t *X, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(features_kernel, dim3(blocks(n * width, 256)), dim3(256), 0, s, L, terms, first, n, width, X);
  return hipGetLastError();
}

hipError_t launch_labels(const LearnedDev *L, const uint64_t *terms, uint64_t first, uint64_t n, float *y, int kind,
                         hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(labels_kernel, dim3(blocks(n, 256)), dim3(256), 0, s, L, terms, first, n, y, kind);
  return hipGetLastError();
}

hipError_t launch_support(const LearnedDev *L, uint64_t K, uint64_t *flags, uint64_t *pos, uint64_t *scratch,
                          uint64_t cap, uint64_t *out, hipStream_t s) {
  hipLaunchKernelGGL(support_flags_kernel, dim3(blocks(K, 256)), dim3(256), 0, s, L, K, flags);
  hipError_t e = hipMemcpyAsync(pos, flags, K * 8, hipMemcpyDeviceToDevice, s);
  if (e != hipSuccess) return e;
  if ((e = launch_scan_u64(pos, K, scratch, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(support_scatter_kernel, dim3(blocks(K, 256)), dim3(256), 0, s, flags, pos, K, cap, out);
  return hipGetLastError();
}

uint64_t scan_scratch_words(uint64_t n) {
  uint64_t w = 0;
  while (n > kScanTile) {
    n = (n + kScanTile - 1) / kScanTile;
    w += n;
  }
  return w + 1;
}

hipError_t launch_scan_u64(uint64_t *x, uint64_t n, uint64_t *scratch, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const uint64_t tiles = (n + kScanTile - 1) / kScanTile;
  if (tiles > 0x7FFFFFFFull) return hipErrorInvalidValue;
  if (tiles == 1) {
    hipLaunchKernelGGL(scan_tile_kernel, dim3(1), dim3(kScanBlock), 0, s, x, n, (uint64_t *)nullptr);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(scan_tile_kernel, dim3((unsigned)tiles), dim3(kScanBlock), 0, s, x, n, scratch);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if ((e = launch_scan_u64(scratch, tiles, scratch + tiles, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(scan_add_kernel, dim3(blocks(n, 256)), dim3(256), 0, s, x, n, scratch);
  return hipGetLastError();
}

uint32_t reduce_blocks(uint64_t n) {
  const uint64_t b = (n + kRedBlock - 1) / kRedBlock;
  return (uint32_t)(b < 1024 ? (b ? b : 1) : 1024);
}

hipError_t launch_proposal(const float *logits, uint64_t n, double eps, float *mpart, double *spart, double *stats,
                           double *q, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const uint32_t nb = reduce_blocks(n);
  if (logits) {
    hipLaunchKernelGGL(max_partial_kernel, dim3(nb), dim3(kRedBlock), 0, s, logits, n, mpart);
    hipLaunchKernelGGL(max_final_kernel, dim3(1), dim3(kRedBlock), 0, s, mpart, nb, stats);
    hipLaunchKernelGGL(sumexp_partial_kernel, dim3(nb), dim3(kRedBlock), 0, s, logits, n, stats, spart);
    hipLaunchKernelGGL(sum_final_kernel, dim3(1), dim3(kRedBlock), 0, s, spart, nb, stats);
  }
  hipLaunchKernelGGL(proposal_kernel, dim3(blocks(n, 256)), dim3(256), 0, s, logits, n, stats, eps, q);
  return hipGetLastError();
}

hipError_t launch_int_cdf(const double *q, uint64_t n, uint64_t *cdf, uint64_t *scratch, hipStream_t s) {
  hipLaunchKernelGGL(int_weights_kernel, dim3(blocks(n, 256)), dim3(256), 0, s, q, n, cdf);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_scan_u64(cdf, n, scratch, s);
}

hipError_t launch_sample_terms(const uint64_t *cdf, uint64_t K, uint64_t n, uint64_t seed, uint64_t cid,
                               uint64_t *out, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(sample_terms_kernel, dim3(blocks(n, 256)), dim3(256), 0, s, cdf, K, n, seed, cid, out);
  return hipGetLastError();
}

hipError_t launch_is_scale(const uint64_t *terms, const double *q, uint64_t n, double *scale, hipStream_t s) {
  hipLaunchKernelGGL(is_scale_kernel, dim3(blocks(n, 256)), dim3(256), 0, s, terms, q, n, scale);
  return hipGetLastError();
}

hipError_t launch_stderr_l1(const double *e, const double *e2, uint64_t bins, uint32_t k, double n, double *part,
                            double *out, hipStream_t s) {
  const unsigned nb = std::min(blocks(bins, 256), kStderrBlocks);
  hipLaunchKernelGGL(stderr_partial_kernel, dim3(nb), dim3(256), 0, s, e, e2, bins, k, n, part);
  hipLaunchKernelGGL(stderr_final_kernel, dim3(1), dim3(kStderrBlocks), 0, s, part, nb, out);
  return hipGetLastError();
}

}  // namespace ccut

// ------------------------------------------------ term draws without allocation
// ccut_sample_terms_noalloc keeps the integer CDF and the scan partials of a
// draw in one fixed device array instead of allocating them: up to
// kNoAllocMaxTerms cut terms (4^10, the ten-cut recombination) plus the scan
// partials of that size, 8 MiB + 16 KiB on each device the library runs on,
// held until the process ends.  Host code never uses the array's name as an
// address: its device address is looked up once per device with
// hipGetSymbolAddress (with that device current) and kept.
namespace {

constexpr uint64_t kNoAllocMaxTerms = 1ull << 20;
constexpr uint64_t kNoAllocScanWords = 2048;  // scan partials for up to kNoAllocMaxTerms entries (1025 words)
constexpr uint64_t kNoAllocWords = kNoAllocMaxTerms + kNoAllocScanWords;
constexpr int kNoAllocMaxDevices = 64;

static __device__ __align__(256) uint64_t noalloc_scratch[kNoAllocWords];

std::mutex g_noalloc_mu;
uint64_t *g_noalloc_ptr[kNoAllocMaxDevices] = {};

}  // namespace

extern "C" ccut_status ccut_sample_terms_noalloc(void *hip_stream, const double *q, uint64_t K, uint64_t n,
                                                 uint64_t seed, uint64_t cid, uint64_t *out) {
  using namespace ccut;
  if (!q || K == 0 || (n && !out)) {
    set_call_error("ccut_sample_terms_noalloc: NULL argument or K = 0");
    return CCUT_E_INVALID;
  }
  if (n > 0xFFFFFFFFull) {
    set_call_error("ccut_sample_terms_noalloc: at most 2^32 - 1 terms per draw");
    return CCUT_E_INVALID;
  }
  if (K > kNoAllocMaxTerms || scan_scratch_words(K) > kNoAllocScanWords) {
    set_call_error("ccut_sample_terms_noalloc: K above 2^20, the size of the fixed term buffer");
    return CCUT_E_UNSUPPORTED;
  }
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kNoAllocMaxDevices) {
    set_call_error("ccut_sample_terms_noalloc: no current HIP device");
    return CCUT_E_DEVICE;
  }
  uint64_t *base = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_noalloc_mu);
    if (!g_noalloc_ptr[dev]) {
      void *ptr = nullptr;
      if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(noalloc_scratch)) != hipSuccess || !ptr) {
        set_call_error("ccut_sample_terms_noalloc: hipGetSymbolAddress of the term buffer failed");
        return CCUT_E_DEVICE;
      }
      g_noalloc_ptr[dev] = static_cast<uint64_t *>(ptr);
    }
    base = g_noalloc_ptr[dev];
  }
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  // every CDF entry and scan partial is written before it is read: nothing
  // left by an earlier call is used
  uint64_t *cdf = base, *partials = base + K;
  if (launch_int_cdf(q, K, cdf, partials, s) != hipSuccess ||
      launch_sample_terms(cdf, K, n, seed, cid, out, s) != hipSuccess) {
    set_call_error("ccut_sample_terms_noalloc: kernel launch failed");
    return CCUT_E_DEVICE;
  }
  return CCUT_OK;
}
