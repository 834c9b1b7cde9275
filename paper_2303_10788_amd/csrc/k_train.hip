// Training of the term network (F -> H -> H -> H -> 1, ReLU): one step is two
// launches.
//
// * train_rows_kernel: everything that is local to a row of the batch.  A
//   workgroup of eight waves takes 16 rows: it gathers them, runs the three
//   layers and the head, forms the loss terms and carries the gradient back
//   to every layer's pre-activations, the activations staying in LDS.
// * train_grads_kernel: the sums over the batch, all independent of each
//   other: 32 x 32 tiles of the three weight gradients, the column sums of
//   the bias gradients and of the head's weights, and the two scalar sums.
//   Each parameter's gradient is complete in the workgroup that sums it, which
//   applies Adam to it and writes the bf16 copies.
//
// A step of 1024 rows is bound by latencies and the dependent chain of small
// products, not by their arithmetic (1 GFLOP) nor by memory (2 MB).  Rows are
// split finely (64 workgroups at 1024 rows; 32 rows a workgroup would leave more
// of the chip idle), and one 16-row workgroup runs five products of at most
// 256 x 256 weights after one another: 544 KB of weights through one CU's L1 at
// 64 bytes a clock, 3.6 us.  They are kept a second time in the order the lanes
// read them (16 bytes a lane, 1 KB a wave and load), and as a product uses its
// weights those of the product after the next take their registers, so that the
// loads never stop.  No sum is split over workgroups: every result has the bits
// of one launch per operation.  Measured at 1024 rows, F 64, H 256: 11 + 10
// us a step; with single-buffered weights, a launch of its own for Adam and one
// stage of rows ahead 20 + 9 + 5 us, and 411 us as 27 launches per step with a
// memory access per row and column in the column sums (58 us each) and 64 x 64
// tiles for the weight gradients (16 workgroups, 35 us each).
#include "bf16.hpp"
#include "common.hpp"

namespace ccut {

namespace {

constexpr uint32_t kRows = 16, kRowThreads = 512, kRowWaves = kRowThreads / 64;
constexpr uint32_t kPad = 8;       // row padding of the LDS tiles (bf16)
constexpr uint32_t kMaxChunks = 8; // 32-wide pieces of the inner index (at most 256)
constexpr uint32_t kProducts = 5, kMaxWidth = 256;

// A wave's share of one product's weights: columns 16 (wave + 8 t) .. + 15 for
// t < NT.
template <uint32_t NT>
struct WaveWeights {
  u32x4 w[NT][kMaxChunks];
};

// Chunk c of NC of the weights of 16 NTILES columns; of a tile beyond them, the
// last one's (in range, unused).
template <uint32_t NTILES, uint32_t NC, uint32_t NT>
__device__ __attribute__((always_inline)) inline void load_chunk(WaveWeights<NT> &B,
                                                                 const uint16_t *__restrict__ packed, uint32_t c,
                                                                 uint32_t wave, uint32_t lane) {
#pragma unroll
  for (uint32_t t = 0; t < NT; ++t) {
    uint32_t tile = wave + kRowWaves * t;
    if (tile >= NTILES) tile = NTILES - 1;
    B.w[t][c] = reinterpret_cast<const u32x4 *>(packed)[(size_t)(tile * NC + c) * 64 + lane];
  }
}

// What the stages of train_rows_kernel share.
struct RowTiles {
  uint16_t *xs, *a1;  // the rows; then h1, h2, h3, d3, d2, d1, a tile each
  float *w4, *bias;   // the head's weights; the three biases, kMaxWidth apart
  uint32_t wave, lane, m, l;
  uint64_t r0;
  float target, b4;
};

// A tile's rows r0 .. r0 + 15 to a global [rows][width] array, 32 lanes a row.
__device__ __attribute__((always_inline)) inline void store_rows(const RowTiles &T, const uint16_t *tile, uint32_t ld,
                                                                 uint32_t width, uint16_t *__restrict__ out) {
  if (T.l * 8 < width) *(u32x4 *)(out + (T.r0 + T.m) * width + T.l * 8) = *(const u32x4 *)(tile + T.m * ld + T.l * 8);
}

// Product P of the step: the three layers (the head after the third), then the
// gradient back through W3 and W2.  It reads the tile before its own (one
// further from the fourth on: the head lies between).  As its weights are used,
// those of product P + 2 take their registers.
template <uint32_t F, uint32_t H, uint32_t P, uint32_t NT>
__device__ __attribute__((always_inline)) inline void product(const TrainRows &g, const RowTiles &T,
                                                              WaveWeights<NT> &B) {
  constexpr bool back = P >= 3;
  constexpr uint32_t p = P, nc = (P ? H : F) / 32, ldx = F + kPad, ld = H + kPad, tile = kRows * ld;
  const uint16_t *in = P == 0 ? T.xs : T.a1 + (back ? P : P - 1) * tile;
  uint16_t *out = T.a1 + (back ? P + 1 : P) * tile;
  float4v acc[NT];
#pragma unroll
  for (uint32_t t = 0; t < NT; ++t) acc[t] = float4v{0.f, 0.f, 0.f, 0.f};
  const uint16_t *a = in + (T.lane & 15) * (P ? ld : ldx) + 8 * (T.lane >> 4);
#pragma unroll
  for (uint32_t c = 0; c < kMaxChunks; ++c) {
    if (c < nc) {
      const u32x4 av = *(const u32x4 *)(a + 32 * c);
#pragma unroll
      for (uint32_t t = 0; t < NT; ++t) acc[t] = mfma_bf16(B.w[t][c], av, acc[t]);
    }
    if (P + 2 < kProducts && c < H / 32) load_chunk<H / 16, H / 32>(B, g.w[P + 2], c, T.wave, T.lane);
  }
  // bias and ReLU, or the gradient where the layer below was positive
  const uint16_t *act = T.a1 + (back ? 4 - p : 0) * tile;
  const float *bias = T.bias + (back ? 0 : p) * kMaxWidth;
#pragma unroll
  for (uint32_t t = 0; t < NT; ++t) {
    const uint32_t n = 16 * (T.wave + kRowWaves * t) + 4 * (T.lane >> 4);
    if (n >= H) continue;
    const uint32_t i = (T.lane & 15) * ld + n;
    const uint64_t av = *(const uint64_t *)(act + i);
    const float4v b = *(const float4v *)(bias + n);
    float z[4];
#pragma unroll
    for (uint32_t e = 0; e < 4; ++e)
      z[e] = back ? (bf2f((uint16_t)(av >> (16 * e))) > 0.f ? acc[t][e] : 0.f) : fmaxf(acc[t][e] + b[e], 0.f);
    *(uint64_t *)(out + i) = ((uint64_t)f2bf2(z[2], z[3]) << 32) | f2bf2(z[0], z[1]);
  }
  __syncthreads();
  store_rows(T, out, ld, H, g.out[p]);
  if (p != 2) return;
  // head: 32 lanes per row, eight consecutive elements per lane, butterfly;
  // loss term and gradient at the last layer's pre-activations
  uint16_t *dz = out + tile;
  const bool in_row = T.l * 8 < H;
  u32x4 h{};
  float s = 0.f;
  if (in_row) {
    h = *(const u32x4 *)(out + T.m * ld + T.l * 8);
#pragma unroll
    for (uint32_t e = 0; e < 8; ++e) s += bf2f((uint16_t)(h[e >> 1] >> (16 * (e & 1)))) * T.w4[T.l * 8 + e];
  }
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) s += __shfl_xor(s, o, 32);
  const float y = s + T.b4;
  const float r = y - T.target;
  const float d = r * g.inv_b2;
  if (T.l == 0) {
    g.dy[T.r0 + T.m] = d;
    g.sq[T.r0 + T.m] = r * r;
  }
  if (in_row) {
    u32x4 v;
#pragma unroll
    for (uint32_t e = 0; e < 4; ++e) {
      const float lo = __uint_as_float(h[e] << 16), hi = __uint_as_float(h[e] & 0xFFFF0000u);
      v[e] = f2bf2(lo > 0.f ? d * T.w4[T.l * 8 + 2 * e] : 0.f, hi > 0.f ? d * T.w4[T.l * 8 + 2 * e + 1] : 0.f);
    }
    *(u32x4 *)(dz + T.m * ld + T.l * 8) = v;
  }
  __syncthreads();
  store_rows(T, dz, ld, H, g.d3);
}

// One instantiation for each supported pair of widths: a load under a branch
// would make the compiler wait for more of them than the next product needs.
template <uint32_t F, uint32_t H>
__global__ __launch_bounds__(kRowThreads) void train_rows_kernel(const TrainRows g) {
  extern __shared__ __attribute__((aligned(16))) uint16_t tr_smem[];
  constexpr uint32_t ldx = F + kPad, ld = H + kPad, NT = (H / 16 + kRowWaves - 1) / kRowWaves;
  const uint32_t tid = threadIdx.x;
  RowTiles T;
  T.lane = tid & 63;
  T.wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  T.m = tid >> 5;
  T.l = tid & 31;
  T.xs = tr_smem;
  T.a1 = T.xs + kRows * ldx;
  T.w4 = reinterpret_cast<float *>(T.a1 + 6 * kRows * ld);
  T.bias = T.w4 + kMaxWidth;
  T.r0 = (uint64_t)blockIdx.x * kRows;
  WaveWeights<NT> even, odd;
  float b[3], w4 = 0.f;
  if (tid < H) {
    for (uint32_t i = 0; i < 3; ++i) b[i] = g.b[i][tid];
    w4 = bf2f(g.w4[tid]);
  }
  // the rows: data row philox(i, step) mod n, or row i itself
  uint64_t src = T.r0 + T.m;
  if (g.gather) {
    const U4 o = philox10((uint32_t)src, g.step, 0x4D4C5000u, 0u, (uint32_t)g.seed, (uint32_t)(g.seed >> 32));
    src = ((uint64_t)o.w[1] << 32) | o.w[0];
    src -= __umul64hi(src, g.inv_n) * g.n;  // at most two too few
    if (src >= g.n) src -= g.n;
    if (src >= g.n) src -= g.n;
  }
  T.target = g.t[src];
  T.b4 = g.b4[0];
  uint16_t *row = T.xs + T.m * ldx;
  const bool wide = !g.xf && ((uintptr_t)g.x & 15) == 0, in_x = T.l * 8 < F;
  u32x4 x{};
  if (wide && in_x) x = *(const u32x4 *)(g.x + src * F + T.l * 8);
#pragma unroll
  for (uint32_t c = 0; c < F / 32; ++c) load_chunk<H / 16, F / 32>(even, g.w[0], c, T.wave, T.lane);
#pragma unroll
  for (uint32_t c = 0; c < H / 64; ++c) load_chunk<H / 16, H / 32>(odd, g.w[1], c, T.wave, T.lane);
  if (tid < H) {
    for (uint32_t i = 0; i < 3; ++i) T.bias[i * kMaxWidth + tid] = b[i];
    T.w4[tid] = w4;
  }
  if (wide) {
    if (in_x) *(u32x4 *)(row + T.l * 8) = x;
  } else if (g.xf) {  // fp32 rows, rounded here
    for (uint32_t c = T.l; c < F; c += 32) row[c] = f2bf(g.xf[src * F + c]);
  } else {  // a view whose rows are not 16-byte aligned
    for (uint32_t c = T.l; c < F; c += 32) row[c] = g.x[src * F + c];
  }
  __syncthreads();
  store_rows(T, T.xs, ldx, F, g.xb);
#pragma unroll
  for (uint32_t c = H / 64; c < H / 32; ++c) load_chunk<H / 16, H / 32>(odd, g.w[1], c, T.wave, T.lane);
  product<F, H, 0>(g, T, even);
  product<F, H, 1>(g, T, odd);
  product<F, H, 2>(g, T, even);
  product<F, H, 3>(g, T, odd);
  product<F, H, 4>(g, T, even);
}

// -------------------------------------------- sums over the batch, and Adam

// A parameter's bf16 copies: row-major in pb, and the three weight matrices
// once more in lane order (forward: rows n, inner k; W2 and W3 also
// transposed, for the gradient's way back).
__device__ inline void store_copies(const TrainParams &P, uint64_t i, float v) {
  const uint16_t h = f2bf(v);
  P.pb[i] = h;
  const uint32_t F = P.F, H = P.H;
  if (i < P.off_b1) {
    P.w1[lane_order((uint32_t)i / F, (uint32_t)i % F, F)] = h;
  } else if (i >= P.off_w2 && i < P.off_b2) {
    const uint32_t j = (uint32_t)(i - P.off_w2);
    P.w2[lane_order(j / H, j % H, H)] = h;
    P.w2t[lane_order(j % H, j / H, H)] = h;
  } else if (i >= P.off_w3 && i < P.off_b3) {
    const uint32_t j = (uint32_t)(i - P.off_w3);
    P.w3[lane_order(j / H, j % H, H)] = h;
    P.w3t[lane_order(j % H, j / H, H)] = h;
  }
}

// Parameter i (value p, moments m, v) once its gradient is known: Adam (Kingma
// & Ba), c1 = 1 - b1^t, c2 = 1 - b2^t, the fused multiply-adds written out; or
// the gradient alone.
__device__ inline void param_step(const TrainParams &P, const TrainAdam &A, uint64_t i, float p, float m, float v,
                                  float gi) {
  if (!A.update) {
    P.g[i] = gi;
    return;
  }
  const float mi = __builtin_fmaf(1.f - A.b1, gi, A.b1 * m);
  const float vi = __builtin_fmaf(gi, (1.f - A.b2) * gi, A.b2 * v);
  P.m[i] = mi;
  P.v[i] = vi;
  const float np = p - A.lr * (mi / A.c1) / (sqrtf(vi / A.c2) + A.eps);
  P.p[i] = np;
  store_copies(P, i, np);
}

constexpr uint32_t kGradThreads = 256;
constexpr uint32_t kGradK = 128;              // rows staged at a time
constexpr uint32_t kGradLd = kGradK + 8;      // padded LDS stride (bf16)
constexpr uint32_t kGradAhead = 4;            // stages in flight
constexpr uint32_t kColRows = kColChunkRows;  // rows of a column-sum chunk
constexpr uint32_t kColChunks = kGradThreads / 64;  // chunks at a time, one a wave

// 128 rows by 32 columns of a row-major [rows][width] array, as columns of
// consecutive rows: thread t (of 128) holds rows 4 (t / 4) .. + 3, columns
// 8 (t % 4) .. + 7.  Past the last row, that row again (not used).
struct GradRegs {
  u32x4 v[4];
};
__device__ inline void grad_load(GradRegs &R, const uint16_t *__restrict__ src, uint32_t width, uint64_t r0,
                                 uint64_t rows, uint32_t c0, uint32_t t) {
#pragma unroll
  for (uint32_t i = 0; i < 4; ++i) {
    const uint64_t r = r0 + 4 * (t >> 2) + i;
    R.v[i] = *(const u32x4 *)(src + (r < rows ? r : rows - 1) * width + c0 + 8 * (t & 3));
  }
}
__device__ inline void grad_store(const GradRegs &R, uint16_t *tile, uint32_t t) {
#pragma unroll
  for (uint32_t j = 0; j < 8; ++j) {
    const uint32_t sh = 16 * (j & 1);
    uint64_t p = 0;
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) p |= (uint64_t)((R.v[i][j >> 1] >> sh) & 0xFFFFu) << (16 * i);
    *(uint64_t *)(tile + (8 * (t & 3) + j) * kGradLd + 4 * (t >> 2)) = p;
  }
}

// sum over rows of D[row][m] X[row][n] for m0 <= m < m0 + 32, n0 <= n < n0 + 32:
// one 16 x 16 block per wave, rows ascending in steps of 32.  Bound by the chain
// of `rows` / 32 dependent products and the memory's latency: four stages of
// 128 rows are on their way at a time, loaded without a branch (the compiler
// would wait for all loads where branches meet).
__device__ inline float4v grad_tile(uint64_t rows, const uint16_t *__restrict__ D, uint32_t ldd,
                                    const uint16_t *__restrict__ X, uint32_t ldx, uint32_t m0, uint32_t n0,
                                    uint16_t *smem) {
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t half = tid >> 7, t = tid & 127;
  const uint16_t *src = half ? X : D;
  const uint32_t width = half ? ldx : ldd, c0 = half ? n0 : m0;
  const uint64_t stages = (rows + kGradK - 1) / kGradK;
  GradRegs R[kGradAhead];
#pragma unroll
  for (uint32_t j = 0; j < kGradAhead; ++j) grad_load(R[j], src, width, (uint64_t)j * kGradK, rows, c0, t);
  float4v acc = float4v{0.f, 0.f, 0.f, 0.f};
  for (uint64_t s0 = 0; s0 < stages; s0 += kGradAhead) {
#pragma unroll
    for (uint32_t j = 0; j < kGradAhead; ++j) {
      if (s0 + j >= stages) break;
      uint16_t *As = smem + (j & 1) * 64 * kGradLd, *Bs = As + 32 * kGradLd;
      grad_store(R[j], half ? Bs : As, t);
      __syncthreads();  // (two buffers: the other one's readers passed this barrier's predecessor)
      grad_load(R[j], src, width, (s0 + j + kGradAhead) * kGradK, rows, c0, t);
      const uint16_t *a = As + ((wave & 1) * 16 + (lane & 15)) * kGradLd + 8 * (lane >> 4);
      const uint16_t *b = Bs + ((wave >> 1) * 16 + (lane & 15)) * kGradLd + 8 * (lane >> 4);
#pragma unroll
      for (uint32_t c = 0; c < kGradK / 64; ++c) {
        if (c && rows - (s0 + j) * kGradK < kGradK) break;  // the last 64 rows
        acc = mfma_bf16(*(const u32x4 *)(a + 64 * c), *(const u32x4 *)(b + 64 * c), acc);
        acc = mfma_bf16(*(const u32x4 *)(a + 64 * c + 32), *(const u32x4 *)(b + 64 * c + 32), acc);
      }
    }
  }
  return acc;
}

// Sum over rows of X's columns c0 .. + 63 (weighted by s when set), to the first
// 64 threads: chunks of 256 rows, each summed in order by a wave, four chunks
// staged at a time so that the ordered sum waits on LDS and not once per row on
// memory; the chunks' sums added in order.
__device__ inline float col_sums(uint64_t rows, const uint16_t *__restrict__ X, uint32_t ld,
                                 const float *__restrict__ s, uint32_t c0, uint16_t *smem) {
  constexpr uint32_t kStage = kColChunks * kColRows, kLoads = kStage / 32;
  float *ss = reinterpret_cast<float *>(smem + kStage * 64), *part = ss + kStage;
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float total = 0.f;
  for (uint64_t r0 = 0; r0 < rows; r0 += kStage) {
    u32x4 v[kLoads];
#pragma unroll
    for (uint32_t i = 0; i < kLoads; ++i) {
      const uint64_t r = r0 + (tid >> 3) + 32 * i;
      v[i] = *(const u32x4 *)(X + (r < rows ? r : rows - 1) * ld + c0 + 8 * (tid & 7));
    }
#pragma unroll
    for (uint32_t i = 0; i < kStage / kGradThreads; ++i) {
      const uint64_t r = r0 + tid + kGradThreads * i;
      ss[tid + kGradThreads * i] = s && r < rows ? s[r] : 1.f;
    }
#pragma unroll
    for (uint32_t i = 0; i < kLoads; ++i) *(u32x4 *)(smem + ((tid >> 3) + 32 * i) * 64 + 8 * (tid & 7)) = v[i];
    __syncthreads();
    const uint64_t first = r0 + wave * kColRows;
    if (first < rows) {
      const uint32_t nr = (uint32_t)(rows - first < kColRows ? rows - first : kColRows);
      const uint16_t *x = smem + wave * kColRows * 64 + lane;
      const float *w = ss + wave * kColRows;
      float acc = 0.f;
#pragma unroll 16
      for (uint32_t r = 0; r < nr; ++r) acc = __builtin_fmaf(w[r], bf2f(x[r * 64]), acc);
      part[tid] = acc;
    }
    __syncthreads();
    if (tid < 64)
      for (uint32_t w = 0; w < kColChunks && r0 + w * kColRows < rows; ++w) total += part[w * 64 + lane];
  }
  return total;
}

// sum of x[0..rows) (fixed-order tree over 256 strided partial sums)
__device__ inline float scalar_sum(const float *__restrict__ x, uint64_t rows, uint16_t *smem) {
  float *red = reinterpret_cast<float *>(smem);
  float acc = 0.f;
  for (uint64_t i = threadIdx.x; i < rows; i += 256) acc += x[i];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (uint32_t w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  return red[0];
}

constexpr uint32_t kTileLds = 2 * 64 * kGradLd * 2;  // bytes of a tile's two buffers
constexpr uint32_t kGradLds = kColChunks * (kColRows * (64 * 2 + 4) + 64 * 4);
static_assert(kGradLds >= kTileLds && kGradLds <= 160 * 1024, "LDS of train_grads_kernel");

__global__ __launch_bounds__(kGradThreads) void train_grads_kernel(const TrainGrads g, const TrainParams P,
                                                                   const TrainAdam A) {
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t T = P.H / 32, TF = P.F / 32, CG = P.H / 64;
  // this workgroup's sums; of them this thread's: n parameters i0, i0 + ld, ...
  uint32_t b = blockIdx.x, n = 0, ld = 0, c0 = 0, m0 = 0, layer = 0;
  uint64_t i0 = 0;
  const bool cols = b < 4 * CG, scalar = !cols && b < 4 * CG + 2;
  if (cols) {
    layer = b / CG;  // 0: the head's weights, then the biases from the last layer's
    c0 = 64 * (b % CG);
    i0 = (layer == 0 ? P.off_w4 : layer == 1 ? P.off_b3 : layer == 2 ? P.off_b2 : P.off_b1) + c0 + lane;
    n = wave == 0;
  } else if (scalar) {
    layer = b - 4 * CG;  // 0: the head's bias, 1: the loss
    i0 = P.off_b4;
    n = layer == 0 && tid == 0;
  } else {
    b -= 4 * CG + 2;
    layer = b < T * T ? 2 : b < 2 * T * T ? 1 : 0;
    b -= (2 - layer) * T * T;
    const uint32_t nt = layer ? T : TF;
    m0 = 32 * (b / nt);
    c0 = 32 * (b % nt);
    ld = layer ? P.H : P.F;
    i0 = (layer == 2 ? P.off_w3 : layer == 1 ? P.off_w2 : 0) +
         (uint64_t)(m0 + (wave & 1) * 16 + 4 * (lane >> 4)) * ld + c0 + (wave >> 1) * 16 + (lane & 15);
    n = 4;
  }
  float4v p, m, v, gr{};  // (inactive ones read i0's)
#pragma unroll
  for (uint32_t r = 0; r < 4; ++r) {
    const uint64_t i = i0 + (uint64_t)(r < n ? r : 0) * ld;
    p[r] = P.p[i];
    m[r] = P.m[i];
    v[r] = P.v[i];
  }
  if (cols) {
    gr[0] = col_sums(g.rows, layer == 0 ? g.h3 : layer == 1 ? g.d3 : layer == 2 ? g.d2 : g.d1, P.H,
                     layer == 0 ? g.dy : nullptr, c0, smem);
  } else if (scalar) {
    gr[0] = scalar_sum(layer ? g.sq : g.dy, g.rows, smem);
    if (layer && tid == 0) *g.loss = gr[0];
  } else {
    gr = grad_tile(g.rows, layer == 2 ? g.d3 : layer == 1 ? g.d2 : g.d1, P.H,
                   layer == 2 ? g.h2 : layer == 1 ? g.h1 : g.xb, ld, m0, c0, smem);
  }
#pragma unroll 1
  for (uint32_t r = 0; r < n; ++r) {
    auto at = [r](const float4v &x) { return r == 0 ? x[0] : r == 1 ? x[1] : r == 2 ? x[2] : x[3]; };
    param_step(P, A, i0 + (uint64_t)r * ld, at(p), at(m), at(v), at(gr));
  }
}

__global__ void train_copies_kernel(const TrainParams P) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < P.n) store_copies(P, i, P.p[i]);
}

}  // namespace

static bool train_shape(uint32_t F, uint32_t H) { return F % 64 == 0 && H % 64 == 0 && F && H && F <= 256 && H <= 256; }

hipError_t launch_train_rows(const TrainRows &g, hipStream_t s) {
  if (!train_shape(g.F, g.H) || g.rows == 0 || g.rows % 64 || g.rows / kRows > 0x7FFFFFFFull)
    return hipErrorInvalidValue;
  const size_t lds = (size_t)kRows * ((g.F + kPad) + 6 * (g.H + kPad)) * sizeof(uint16_t) + 4 * kMaxWidth * sizeof(float);
  const dim3 grid((unsigned)(g.rows / kRows)), block(kRowThreads);
#define CCUT_ROWS(FF, HH) \
  case FF + HH / 64: hipLaunchKernelGGL((train_rows_kernel<FF, HH>), grid, block, lds, s, g); break;
#define CCUT_ROWS_F(FF) CCUT_ROWS(FF, 64) CCUT_ROWS(FF, 128) CCUT_ROWS(FF, 192) CCUT_ROWS(FF, 256)
  switch (g.F + g.H / 64) {
    CCUT_ROWS_F(64)
    CCUT_ROWS_F(128)
    CCUT_ROWS_F(192)
    CCUT_ROWS_F(256)
    default: return hipErrorInvalidValue;
  }
#undef CCUT_ROWS_F
#undef CCUT_ROWS
  return hipGetLastError();
}

hipError_t launch_train_grads(const TrainGrads &g, const TrainParams &P, const TrainAdam &A, hipStream_t s) {
  if (!train_shape(P.F, P.H) || g.rows == 0 || g.rows % 64) return hipErrorInvalidValue;
  const uint32_t T = P.H / 32, TF = P.F / 32;
  hipError_t e = hipFuncSetAttribute((const void *)train_grads_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)kGradLds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(train_grads_kernel, dim3(4 * (P.H / 64) + 2 + 2 * T * T + T * TF), dim3(kGradThreads), kGradLds, s,
                     g, P, A);
  return hipGetLastError();
}

hipError_t launch_train_copies(const TrainParams &P, hipStream_t s) {
  hipLaunchKernelGGL(train_copies_kernel, dim3((unsigned)((P.n + 255) / 256)), dim3(256), 0, s, P);
  return hipGetLastError();
}

}  // namespace ccut
