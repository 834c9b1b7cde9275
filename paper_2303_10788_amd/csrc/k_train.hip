// Training of the term network (F -> H -> H -> H -> 1, ReLU): one step is
// three launches.
//
// * train_rows_kernel: everything that is local to a row of the batch.  A
//   workgroup of eight waves takes 16 rows: it gathers them, runs the three
//   layers and the head, forms the loss terms and carries the gradient back
//   to every layer's pre-activations, the activations staying in LDS.
// * train_grads_kernel: the sums over the batch, all independent of each
//   other: 32 x 32 tiles of the three weight gradients, the column sums of
//   the bias gradients and of the head's weights (chunks of 256 rows), and
//   the two scalar sums.
// * train_update_kernel: the chunks of the column sums added in order, Adam,
//   and the bf16 copies of the new weights.
//
// A step of 1024 rows is bound by the dependent chain of small products, not
// by their arithmetic (1 GFLOP) nor by memory (2 MB): one 16-row workgroup
// runs five products of at most 256 x 256 weights after one another.  So rows
// are split finely (64 workgroups at 1024 rows; 32 rows a workgroup would
// leave more of the chip idle), each wave's weights of the next product are
// loaded before the epilogue and the barrier of the current one, and the
// weights are kept a second time in the order the lanes read them (16 bytes a
// lane, 1 KB a wave and load: rows of a row-major weight would be fetched in
// 32-byte pieces).  The ordered sums over 1024 rows (32 dependent products of a
// weight gradient's element, 256 dependent additions of a column-sum chunk) are
// staged through LDS ahead of their use, and no sum is split further: every
// result has the same bits as one launch per operation gave.  Measured at 1024
// rows, F 64, H 256: 35 us a step, against 411 us for 27 launches per step with
// a memory access per row and column in the column sums (58 us each) and
// 64 x 64 tiles for the weight gradients (16 workgroups, 35 us each).
#include "bf16.hpp"
#include "common.hpp"

namespace ccut {

namespace {

constexpr uint32_t kRows = 16, kRowThreads = 512, kRowWaves = kRowThreads / 64;
constexpr uint32_t kPad = 8;       // row padding of the LDS tiles (bf16)
constexpr uint32_t kMaxChunks = 8; // 32-wide pieces of the inner index (at most 256)
constexpr uint32_t kWaveTiles = 2; // 16-wide column tiles of a wave (at most 256 columns over 8 waves)

// A wave's share of one layer's weights: columns 16 (wave + 8 t) .. + 15.
struct WaveWeights {
  u32x4 w[kWaveTiles][kMaxChunks];
};

__device__ inline void load_weights(WaveWeights &B, const uint16_t *__restrict__ packed, uint32_t N, uint32_t K,
                                    uint32_t wave, uint32_t lane) {
  const uint32_t nc = K >> 5;
#pragma unroll
  for (uint32_t t = 0; t < kWaveTiles; ++t) {
    const uint32_t nt = wave + kRowWaves * t;
    const u32x4 *src = reinterpret_cast<const u32x4 *>(packed) + (size_t)nt * nc * 64 + lane;
#pragma unroll
    for (uint32_t c = 0; c < kMaxChunks; ++c)
      if (nt * 16 < N && c < nc) B.w[t][c] = src[c * 64];
  }
}

// acc[t] = rows (16 x K in LDS, row stride lda) times the wave's columns, the
// inner index ascending in steps of 32.
__device__ inline void row_products(const uint16_t *A, uint32_t lda, const WaveWeights &B, uint32_t N, uint32_t K,
                                    uint32_t wave, uint32_t lane, float4v (&acc)[kWaveTiles]) {
  const uint32_t nc = K >> 5;
#pragma unroll
  for (uint32_t t = 0; t < kWaveTiles; ++t) acc[t] = float4v{0.f, 0.f, 0.f, 0.f};
  const uint16_t *a = A + (lane & 15) * lda + 8 * (lane >> 4);
#pragma unroll
  for (uint32_t c = 0; c < kMaxChunks; ++c) {
    if (c >= nc) break;
    const u32x4 av = *(const u32x4 *)(a + 32 * c);
#pragma unroll
    for (uint32_t t = 0; t < kWaveTiles; ++t)
      if ((wave + kRowWaves * t) * 16 < N) acc[t] = mfma_bf16(av, B.w[t][c], acc[t]);
  }
}

// LDS tile [16][ld] to rows r0 .. r0 + 15 of a global [rows][width] array.
__device__ inline void store_rows(const uint16_t *tile, uint32_t ld, uint32_t width, uint64_t r0,
                                  uint16_t *__restrict__ out) {
  const uint32_t per = width / 8;
  for (uint32_t i = threadIdx.x; i < kRows * per; i += kRowThreads) {
    const uint32_t m = i / per, c = (i % per) * 8;
    *(u32x4 *)(out + (r0 + m) * width + c) = *(const u32x4 *)(tile + m * ld + c);
  }
}

__global__ __launch_bounds__(kRowThreads) void train_rows_kernel(const TrainRows g) {
  extern __shared__ __attribute__((aligned(16))) uint16_t tr_smem[];
  const uint32_t F = g.F, H = g.H, ldx = F + kPad, ld = H + kPad;
  uint16_t *xs = tr_smem, *a1 = xs + kRows * ldx, *a2 = a1 + kRows * ld, *a3 = a2 + kRows * ld, *dz = a3 + kRows * ld;
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t r0 = (uint64_t)blockIdx.x * kRows;
  WaveWeights B;
  load_weights(B, g.w1, H, F, wave, lane);
  // the rows: data row philox(i, step) mod n, or row i itself; 32 lanes a row
  const uint32_t m = tid >> 5, l = tid & 31;
  uint64_t src = r0 + m;
  if (g.gather) {
    const U4 o = philox10((uint32_t)(r0 + m), g.step, 0x4D4C5000u, 0u, (uint32_t)g.seed, (uint32_t)(g.seed >> 32));
    src = (((uint64_t)o.w[1] << 32) | o.w[0]) % g.n;
  }
  const float target = g.t[src];
  if (g.xf) {  // fp32 rows, rounded here
    for (uint32_t c = l; c < F; c += 32) xs[m * ldx + c] = f2bf(g.xf[src * F + c]);
  } else if (((uintptr_t)g.x & 15) == 0) {
    for (uint32_t c = l * 8; c < F; c += 256) *(u32x4 *)(xs + m * ldx + c) = *(const u32x4 *)(g.x + src * F + c);
  } else {  // a view whose rows are not 16-byte aligned
    for (uint32_t c = l; c < F; c += 32) xs[m * ldx + c] = g.x[src * F + c];
  }
  __syncthreads();
  store_rows(xs, ldx, F, r0, g.xb);
  float4v acc[kWaveTiles];
  // a layer: products, the next product's weights on their way, epilogue
  auto relu = [&](const float *__restrict__ bias, uint16_t *out) {
#pragma unroll
    for (uint32_t t = 0; t < kWaveTiles; ++t) {
      const uint32_t n = (wave + kRowWaves * t) * 16 + (lane & 15);
      if (n >= H) continue;
      const float b = bias[n];
#pragma unroll
      for (uint32_t r = 0; r < 4; ++r) out[(4 * (lane >> 4) + r) * ld + n] = f2bf(fmaxf(acc[t][r] + b, 0.f));
    }
    __syncthreads();
  };
  row_products(xs, ldx, B, H, F, wave, lane, acc);
  load_weights(B, g.w2, H, H, wave, lane);
  relu(g.b1, a1);
  row_products(a1, ld, B, H, H, wave, lane, acc);
  load_weights(B, g.w3, H, H, wave, lane);
  relu(g.b2, a2);
  row_products(a2, ld, B, H, H, wave, lane, acc);
  load_weights(B, g.w3t, H, H, wave, lane);
  relu(g.b3, a3);
  // head: 32 lanes per row, eight consecutive elements per lane, butterfly;
  // loss term and gradient at the last layer's pre-activations
  {
    float s = 0.f;
    if (l * 8 < H) {
#pragma unroll
      for (uint32_t e = 0; e < 8; ++e) s += bf2f(a3[m * ld + l * 8 + e]) * bf2f(g.w4[l * 8 + e]);
    }
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) s += __shfl_xor(s, o, 32);
    const float y = s + g.b4[0];
    const float r = y - target;
    const float d = r * g.inv_b2;
    if (l == 0) {
      g.dy[r0 + m] = d;
      g.sq[r0 + m] = r * r;
    }
    for (uint32_t n = l; n < H; n += 32)
      dz[m * ld + n] = f2bf(bf2f(a3[m * ld + n]) > 0.f ? d * bf2f(g.w4[n]) : 0.f);
  }
  __syncthreads();
  store_rows(a1, ld, H, r0, g.h1);
  store_rows(a2, ld, H, r0, g.h2);
  store_rows(a3, ld, H, r0, g.h3);
  store_rows(dz, ld, H, r0, g.d3);
  // gradient through the ReLU of the layer below (its outputs in `act`)
  auto mask = [&](const uint16_t *act, uint16_t *out) {
#pragma unroll
    for (uint32_t t = 0; t < kWaveTiles; ++t) {
      const uint32_t n = (wave + kRowWaves * t) * 16 + (lane & 15);
      if (n >= H) continue;
#pragma unroll
      for (uint32_t r = 0; r < 4; ++r) {
        const uint32_t i = (4 * (lane >> 4) + r) * ld + n;
        out[i] = f2bf(bf2f(act[i]) > 0.f ? acc[t][r] : 0.f);
      }
    }
    __syncthreads();
  };
  row_products(dz, ld, B, H, H, wave, lane, acc);
  load_weights(B, g.w2t, H, H, wave, lane);
  __syncthreads();  // a3 (stored) and dz (read) are free
  mask(a2, a3);
  store_rows(a3, ld, H, r0, g.d2);
  row_products(a3, ld, B, H, H, wave, lane, acc);
  mask(a1, dz);
  store_rows(dz, ld, H, r0, g.d1);
}

// ------------------------------------------------------- sums over the batch

constexpr uint32_t kGradThreads = 256;
constexpr uint32_t kGradK = 128;              // rows staged at a time
constexpr uint32_t kGradLd = kGradK + 8;      // padded LDS stride (bf16)
constexpr uint32_t kColRows = kColChunkRows;  // rows of a column-sum chunk

// 128 rows by 32 columns of a row-major [rows][width] array, as columns of
// consecutive rows: thread t (of 128) holds rows 4 (t / 4) .. + 3, columns
// 8 (t % 4) .. + 7.
struct GradRegs {
  u32x4 v[4];
};
__device__ inline void grad_load(GradRegs &R, const uint16_t *__restrict__ src, uint32_t width, uint64_t r0,
                                 uint64_t rows, uint32_t c0, uint32_t t) {
#pragma unroll
  for (uint32_t i = 0; i < 4; ++i) {
    const uint64_t r = r0 + 4 * (t >> 2) + i;
    if (r < rows) R.v[i] = *(const u32x4 *)(src + r * width + c0 + 8 * (t & 3));
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

// dW[m][n] = sum over rows of D[row][m] X[row][n], one 32 x 32 tile per
// workgroup, one 16 x 16 block per wave, rows ascending in steps of 32.  Bound
// by the chain of `rows` / 32 dependent products; the next 128 rows are loaded
// while the current ones are summed.
__device__ void grad_tile(const TrainGrads &g, const uint16_t *__restrict__ D, const uint16_t *__restrict__ X,
                          uint32_t in, uint32_t m0, uint32_t n0, float *__restrict__ out, uint16_t *smem) {
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t half = tid >> 7, t = tid & 127;
  const uint16_t *src = half ? X : D;
  const uint32_t width = half ? in : g.H, c0 = half ? n0 : m0;
  const uint64_t rows = g.rows;
  GradRegs R;
  grad_load(R, src, width, 0, rows, c0, t);
  float4v acc = float4v{0.f, 0.f, 0.f, 0.f};
  uint32_t buf = 0;
  for (uint64_t k0 = 0; k0 < rows; k0 += kGradK, buf ^= 1) {
    uint16_t *As = smem + buf * 64 * kGradLd, *Bs = As + 32 * kGradLd;
    grad_store(R, half ? Bs : As, t);
    __syncthreads();  // (two buffers: the other one's readers passed this barrier's predecessor)
    if (k0 + kGradK < rows) grad_load(R, src, width, k0 + kGradK, rows, c0, t);
    const uint16_t *a = As + ((wave & 1) * 16 + (lane & 15)) * kGradLd + 8 * (lane >> 4);
    const uint16_t *b = Bs + ((wave >> 1) * 16 + (lane & 15)) * kGradLd + 8 * (lane >> 4);
    if (rows - k0 >= kGradK) {
#pragma unroll
      for (uint32_t c = 0; c < kGradK / 32; ++c)
        acc = mfma_bf16(*(const u32x4 *)(a + 32 * c), *(const u32x4 *)(b + 32 * c), acc);
    } else {  // the last 64 rows
#pragma unroll
      for (uint32_t c = 0; c < 2; ++c)
        acc = mfma_bf16(*(const u32x4 *)(a + 32 * c), *(const u32x4 *)(b + 32 * c), acc);
    }
  }
#pragma unroll
  for (uint32_t r = 0; r < 4; ++r)
    out[(size_t)(m0 + (wave & 1) * 16 + 4 * (lane >> 4) + r) * in + n0 + (wave >> 1) * 16 + (lane & 15)] = acc[r];
}

// Column sums of 64 columns over one chunk of 256 rows, rows in order
// (weighted by s when set): the chunk is staged whole, so the ordered sum
// waits on LDS and not once per row on memory.
__device__ void col_chunk(const TrainGrads &g, const uint16_t *__restrict__ X, const float *__restrict__ s,
                          uint64_t chunk, uint32_t c0, float *__restrict__ part, uint16_t *smem) {
  float *ss = reinterpret_cast<float *>(smem + kColRows * 64);
  const uint32_t tid = threadIdx.x;
  const uint64_t r0 = chunk * kColRows;
  const uint32_t nr = (uint32_t)(g.rows - r0 < kColRows ? g.rows - r0 : kColRows);
  u32x4 v[8];
#pragma unroll
  for (uint32_t i = 0; i < 8; ++i) {
    const uint32_t r = (tid >> 3) + 32 * i;
    if (r < nr) v[i] = *(const u32x4 *)(X + (r0 + r) * g.H + c0 + 8 * (tid & 7));
  }
  if (tid < nr) ss[tid] = s ? s[r0 + tid] : 1.f;
#pragma unroll
  for (uint32_t i = 0; i < 8; ++i) {
    const uint32_t r = (tid >> 3) + 32 * i;
    if (r < nr) *(u32x4 *)(smem + r * 64 + 8 * (tid & 7)) = v[i];
  }
  __syncthreads();
  if (tid >= 64) return;
  float acc = 0.f;
#pragma unroll 16
  for (uint32_t r = 0; r < nr; ++r) acc += ss[r] * bf2f(smem[r * 64 + tid]);
  part[chunk * g.H + c0 + tid] = acc;
}

// *out = sum of x[0..rows) (fixed-order tree over 256 strided partial sums)
__device__ void scalar_sum(const float *__restrict__ x, uint64_t rows, float *__restrict__ out, uint16_t *smem) {
  float *red = reinterpret_cast<float *>(smem);
  float acc = 0.f;
  for (uint64_t i = threadIdx.x; i < rows; i += 256) acc += x[i];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (uint32_t w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = red[0];
}

constexpr uint32_t kGradLds = 2 * 64 * kGradLd * 2;  // bytes of a tile's two buffers
static_assert(kGradLds >= kColRows * 64 * 2 + kColRows * 4, "a column-sum chunk and its weights");

__global__ __launch_bounds__(kGradThreads) void train_grads_kernel(const TrainGrads g) {
  __shared__ __attribute__((aligned(16))) uint16_t smem[kGradLds / 2];
  const uint32_t T = g.H / 32, TF = g.F / 32, CG = g.H / 64;
  uint64_t b = blockIdx.x;
  // the weight gradients first: theirs is the longest chain
  if (b < (uint64_t)T * T) return grad_tile(g, g.d3, g.h2, g.H, 32 * (uint32_t)(b / T), 32 * (uint32_t)(b % T), g.gw3, smem);
  b -= (uint64_t)T * T;
  if (b < (uint64_t)T * T) return grad_tile(g, g.d2, g.h1, g.H, 32 * (uint32_t)(b / T), 32 * (uint32_t)(b % T), g.gw2, smem);
  b -= (uint64_t)T * T;
  if (b < (uint64_t)T * TF) return grad_tile(g, g.d1, g.xb, g.F, 32 * (uint32_t)(b / TF), 32 * (uint32_t)(b % TF), g.gw1, smem);
  b -= (uint64_t)T * TF;
  if (b < 2) return scalar_sum(b ? g.sq : g.dy, g.rows, b ? g.loss : g.gb4, smem);
  b -= 2;
  const uint64_t chunks = (g.rows + kColRows - 1) / kColRows, per = chunks * CG;
  const uint32_t kind = (uint32_t)(b / per);
  const uint64_t chunk = (b % per) / CG;
  const uint32_t c0 = 64 * (uint32_t)(b % CG);
  const uint16_t *X = kind == 0 ? g.h3 : kind == 1 ? g.d3 : kind == 2 ? g.d2 : g.d1;
  col_chunk(g, X, kind == 0 ? g.dy : nullptr, chunk, c0, g.part + (size_t)kind * chunks * g.H, smem);
}

// ------------------------------------------------------------------ update

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

// The gradient of parameter i: of a bias or of the head's weights, the chunks
// of its column sum in order.
__device__ inline float gradient(const TrainParams &P, uint64_t i, uint64_t chunks) {
  uint32_t kind, n;
  if (i >= P.off_w4 && i < P.off_b4) {
    kind = 0;
    n = (uint32_t)(i - P.off_w4);
  } else if (i >= P.off_b3 && i < P.off_w4) {
    kind = 1;
    n = (uint32_t)(i - P.off_b3);
  } else if (i >= P.off_b2 && i < P.off_w3) {
    kind = 2;
    n = (uint32_t)(i - P.off_b2);
  } else if (i >= P.off_b1 && i < P.off_w2) {
    kind = 3;
    n = (uint32_t)(i - P.off_b1);
  } else {
    return P.g[i];
  }
  const float *part = P.part + (size_t)kind * chunks * P.H + n;
  float acc = 0.f;
  for (uint64_t c = 0; c < chunks; ++c) acc += part[c * P.H];
  return acc;
}

__global__ void train_gradients_kernel(const TrainParams P, uint64_t chunks) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < P.n) P.g[i] = gradient(P, i, chunks);
}

// Adam (Kingma & Ba) on the flat fp32 parameters; c1 = 1 - b1^t,
// c2 = 1 - b2^t.
__global__ void train_update_kernel(const TrainParams P, uint64_t chunks, float lr, float b1, float b2, float c1,
                                    float c2, float eps) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= P.n) return;
  const float gi = gradient(P, i, chunks);
  const float mi = b1 * P.m[i] + (1.f - b1) * gi;
  const float vi = b2 * P.v[i] + (1.f - b2) * gi * gi;
  P.m[i] = mi;
  P.v[i] = vi;
  const float np = P.p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  P.p[i] = np;
  store_copies(P, i, np);
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
  const size_t lds = (size_t)kRows * ((g.F + kPad) + 4 * (g.H + kPad)) * sizeof(uint16_t);
  hipLaunchKernelGGL(train_rows_kernel, dim3((unsigned)(g.rows / kRows)), dim3(kRowThreads), lds, s, g);
  return hipGetLastError();
}

hipError_t launch_train_grads(const TrainGrads &g, hipStream_t s) {
  if (!train_shape(g.F, g.H) || g.rows == 0 || g.rows % 64) return hipErrorInvalidValue;
  const uint64_t T = g.H / 32, TF = g.F / 32;
  const uint64_t grid = 2 * T * T + T * TF + 2 + 4 * train_chunks(g.rows) * (g.H / 64);
  if (grid > 0x7FFFFFFFull) return hipErrorInvalidValue;
  hipLaunchKernelGGL(train_grads_kernel, dim3((unsigned)grid), dim3(kGradThreads), 0, s, g);
  return hipGetLastError();
}

hipError_t launch_train_gradients(const TrainParams &P, uint64_t rows, hipStream_t s) {
  hipLaunchKernelGGL(train_gradients_kernel, dim3((unsigned)((P.n + 255) / 256)), dim3(256), 0, s, P,
                     train_chunks(rows));
  return hipGetLastError();
}

hipError_t launch_train_update(const TrainParams &P, uint64_t rows, float lr, float b1, float b2, float c1, float c2,
                               float eps, hipStream_t s) {
  hipLaunchKernelGGL(train_update_kernel, dim3((unsigned)((P.n + 255) / 256)), dim3(256), 0, s, P, train_chunks(rows),
                     lr, b1, b2, c1, c2, eps);
  return hipGetLastError();
}

hipError_t launch_train_copies(const TrainParams &P, hipStream_t s) {
  hipLaunchKernelGGL(train_copies_kernel, dim3((unsigned)((P.n + 255) / 256)), dim3(256), 0, s, P);
  return hipGetLastError();
}

}  // namespace ccut
