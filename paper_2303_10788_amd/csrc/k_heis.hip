// Exact Pauli-basis tensors of Clifford fragments in the Heisenberg picture
// (the Clifford-specific cutting optimisation the paper outlines in Sec. IX:
// Clifford expectations are -1, 0 or +1 and most Pauli terms vanish).
//
// For a Clifford fragment U with quantum inputs (prepared as the operator
// P_in), circuit inputs |0> and a measured set, the Pauli-basis entry is
//   tau[S; P_out, P_in] = Tr[(Z_S (x) Q_out) U rho_in U^dag]
//                       = Tr[O rho_in],   O = U^dag (Z_S (x) Q_out) U,
// and with O = (-1)^s sigma_1 (x) ... (x) sigma_m:
//   Tr[O rho_in] = (-1)^s 2^#in [sigma|inputs == P_in] [sigma|circuit inputs in {I, Z}].
// The marginal tensor is T[b; P] = 2^-r sum_S (-1)^{b.S} tau[S; P] (the
// projector onto outcome b is 2^-r sum_S (-1)^{b.S} Z_S), a Walsh-Hadamard
// transform over subsets S of the r requested outputs.  No variant is
// enumerated: only the r requested Z's and the X, Z of each quantum output
// are carried back through the fragment once.
#include <algorithm>

#include "common.hpp"
#include "pauli.hpp"

namespace ccut {

namespace {

// Shared pass of many fragments' rows: the descriptor array in the global
// address space, read through a reference.
typedef __attribute__((address_space(1))) const FragDev g_FragDevH;

// The row pass bit-sliced: column q of the x (z) parts holds bit q of
// 64 rows per word, so a gate reads and writes only its qubits' column
// words and applies its rule to 64 rows with a few 64-bit operations.  The
// stream comes in layers of ops on disjoint qubits.  Lane l works on row
// word w = l mod RWp (RWp = RW rounded up to a power of two) and, within a
// layer, on op l / RWp of each group of 64 / RWp ops, so a layer costs one
// round trip through LDS instead of one per gate.  Each lane XORs the sign
// changes of its ops into one private word (XOR commutes, and an op reads
// the columns as they are before it: earlier layers are complete and its
// own layer never touches its qubits); one reduction over the lanes of each
// row word adds them up at the end.
constexpr uint32_t kSlicedRows = 1024;
constexpr uint32_t kOpStage = 1024;  // op words staged in LDS (a layer has at most 512)
constexpr uint32_t kLayStage = 256;  // layer offsets staged in LDS

// Fill dst[0, CAP) from src[0, n) (zeros past n) with all loads of a lane
// issued before its first store, so the copy costs one memory latency
// rather than one per word (one wave).
template <uint32_t CAP>
__device__ inline void stage_words(uint32_t *dst, const uint32_t *src, uint32_t n, uint32_t lane) {
  constexpr uint32_t K = (CAP + 63) / 64;
  uint32_t t[K];
#pragma unroll
  for (uint32_t k = 0; k < K; ++k) {
    const uint32_t i = lane + 64 * k;
    t[k] = i < n && i < CAP ? src[i] : 0u;
  }
#pragma unroll
  for (uint32_t k = 0; k < K; ++k)
    if (lane + 64 * k < CAP) dst[lane + 64 * k] = t[k];
}

// kCarryWaves waves per workgroup: a layer's ops are spread over all lanes and
// the waves meet at a barrier after each layer (a lane reads columns other
// waves wrote in the previous layer); wave 0 stages op words and layer
// offsets and transposes rows in and out, and the lanes' sign shares are
// XOR-reduced within each wave, then across the waves through LDS.
constexpr uint32_t kCarryWaves = 4;
template <class D>
__device__ void rows_sliced_body(const D &F, uint32_t W, const uint64_t *__restrict__ in, uint64_t *__restrict__ out,
                                 uint32_t n_rows, uint64_t *cols) {
  constexpr uint32_t NW = kCarryWaves, T = 64 * NW;
  const uint32_t m = F.m;
  const uint32_t RW = (n_rows + 63) / 64;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  uint32_t lg = 0;
  while ((1u << lg) < RW) ++lg;
  const uint32_t RWp = 1u << lg, w = tid & (RWp - 1), o = tid >> lg, per = T >> lg;
  uint64_t *Xc = cols, *Zc = cols + (size_t)m * RW;
  uint32_t *sops = reinterpret_cast<uint32_t *>(Zc + (size_t)m * RW);
  const uint32_t RS = 2 * W + 1;  // row stride in words
  uint64_t sg = 0;  // this lane's share of sign word w
  if (wave == 0) {
    // transpose in, 64 rows at a time: lane l loads row 64 iw + l whole,
    // and column word (q, iw) is the ballot of bit q over the lanes
    for (uint32_t iw = 0; iw < RW; ++iw) {
      const uint32_t r = 64 * iw + lane;
      const bool ok = r < n_rows;
      const uint64_t *row = in + (size_t)(ok ? r : 0) * RS;
      uint64_t xr[8], zr[8];
#pragma unroll
      for (uint32_t k = 0; k < 8; ++k) {
        xr[k] = ok && k < W ? row[k] : 0ull;
        zr[k] = ok && k < W ? row[W + k] : 0ull;
      }
      const uint64_t sw = __ballot(ok && (row[2 * W] & 1ull));
      if (lane == iw) sg = sw;  // lane iw starts with sign word iw
#pragma unroll
      for (uint32_t k = 0; k < 8; ++k) {
        if (k >= W) break;
        const uint32_t nq = 64 * k < m ? min(64u, m - 64 * k) : 0u;
        for (uint32_t i = 0; i < nq; ++i) {
          const uint64_t cx = __ballot((xr[k] >> i) & 1ull), cz = __ballot((zr[k] >> i) & 1ull);
          if (lane == i) {
            Xc[(size_t)(64 * k + i) * RW + iw] = cx;
            Zc[(size_t)(64 * k + i) * RW + iw] = cz;
          }
        }
      }
    }
  }
  const bool live = w < RW;
  __syncthreads();
  // Layer offsets are staged in LDS too (without offsets every op is a
  // layer of its own).  One layer of lookahead: the next layer's end offset
  // and this lane's first op word of the next layer are read before the
  // current layer's column traffic, so only the column reads wait on LDS.
  // Op words are restaged when the next layer (at most 512 ops) might not
  // lie inside the staged window.
  uint32_t *slay = sops + kOpStage;
  const uint32_t *lay = F.layers;
  const uint32_t n_layers = lay ? F.n_layers : F.n_ops;
  uint32_t stage0 = 0;
  if (wave == 0) stage_words<kOpStage>(sops, F.ops, F.n_ops, lane);
  uint32_t s0 = 0;
  for (uint32_t L0 = 0; L0 < n_layers; L0 += kLayStage) {
    const uint32_t nl = min(kLayStage, n_layers - L0);
    if (wave == 0) {
      if (lay) {
        stage_words<kLayStage + 1>(slay, lay + L0, nl + 1, lane);
      } else {
        for (uint32_t i = lane; i <= nl; i += 64) slay[i] = L0 + i;
      }
    }
    __syncthreads();  // the staged words (and, the first time, the op window) are in place
    uint32_t v_s1 = slay[1];
    uint32_t v_wd = sops[s0 + o - stage0];  // this lane's first op word of the current layer
    for (uint32_t L = 0; L < nl; ++L) {
      const uint32_t s1 = __builtin_amdgcn_readfirstlane(v_s1);
      const uint32_t wd0 = v_wd;
      const bool keep = s1 + 512 <= stage0 + kOpStage;  // the next layer is inside the window
      uint32_t v_s1n = 0, v_wdn = 0;
      if (L + 2 <= nl) v_s1n = slay[L + 2];
      if (keep) v_wdn = sops[s1 + o - stage0];
      for (uint32_t c0 = s0 + o; c0 < s1; c0 += per) {
        if (!live) continue;
        const uint32_t wd = c0 == s0 + o ? wd0 : sops[c0 - stage0];
        const uint32_t kind = op_kind(wd), a = op_q0(wd), b = op_q1(wd);
        uint64_t *xa = Xc + (size_t)a * RW + w, *za = Zc + (size_t)a * RW + w;
        if (kind == G_CX || kind == G_CZ) {
          uint64_t *xb = Xc + (size_t)b * RW + w, *zb = Zc + (size_t)b * RW + w;
          const uint64_t x1 = *xa, z1 = *za, x2 = *xb, z2 = *zb;
          if (kind == G_CX) {
            sg ^= x1 & z2 & ~(x2 ^ z1);
            *xb = x2 ^ x1;
            *za = z1 ^ z2;
          } else {
            sg ^= x1 & x2 & (z1 ^ z2);
            *za = z1 ^ x2;
            *zb = z2 ^ x1;
          }
        } else {
          const C1Map g = c1_decode(b);
          const uint64_t x = *xa, z = *za;
          sg ^= (x & (0ull - g.al)) ^ (z & (0ull - g.be)) ^ (x & z & (0ull - g.ga));
          *xa = (x & (0ull - g.m00)) ^ (z & (0ull - g.m01));
          *za = (x & (0ull - g.m10)) ^ (z & (0ull - g.m11));
        }
      }
      asm volatile("" ::: "memory");
      __syncthreads();  // every wave is done with this layer's columns (and op words)
      if (!keep) {  // restage from the next layer's start (in issue order after this layer's reads)
        stage0 = s1;
        if (wave == 0) stage_words<kOpStage>(sops, F.ops + s1, F.n_ops - s1, lane);
        __syncthreads();
        v_wdn = sops[o];
      }
      s0 = s1;
      v_s1 = v_s1n;
      v_wd = v_wdn;
    }
    __syncthreads();  // every wave has read this stage's layer offsets
  }
  // sign word w: XOR of the shares of every lane on row word w (lane w of
  // wave 0 ends with it)
  for (uint32_t off = RWp; off < 64; off <<= 1) sg ^= __shfl_xor(sg, off);
  __syncthreads();
  uint64_t *red = reinterpret_cast<uint64_t *>(sops);  // the op window is no longer read
  if (lane < RWp) red[wave * 64 + lane] = sg;
  __syncthreads();
  if (wave == 0 && lane < RWp)
    for (uint32_t v = 1; v < NW; ++v) sg ^= red[v * 64 + lane];
  if (wave != 0) return;
  // transpose out, 64 rows at a time: lane l gathers row 64 rw + l from the
  // column words (each read is the same address for every lane)
  for (uint32_t rw = 0; rw < RW; ++rw) {
    const uint32_t r = 64 * rw + lane;
    for (uint32_t wq = 0; wq < W; ++wq) {
      const uint32_t nq = 64 * wq < m ? min(64u, m - 64 * wq) : 0u;
      uint64_t xw = 0, zw = 0;
#pragma unroll 8
      for (uint32_t i = 0; i < nq; ++i) {
        const size_t c = (size_t)(64 * wq + i) * RW + rw;
        xw |= ((Xc[c] >> lane) & 1ull) << i;
        zw |= ((Zc[c] >> lane) & 1ull) << i;
      }
      if (r < n_rows) {
        out[(size_t)r * RS + wq] = xw;
        out[(size_t)r * RS + W + wq] = zw;
      }
    }
  }
  for (uint32_t rw = 0; rw < RW; ++rw) {
    const uint64_t word = __shfl(sg, rw);
    const uint32_t r = 64 * rw + lane;
    if (r < n_rows) out[(size_t)r * RS + 2 * W] = (word >> lane) & 1ull;
  }
}

// Block x carries rows [1024 x, 1024 x + 1024) (rows are independent).
__global__ __launch_bounds__(64 * kCarryWaves) void rows_sliced_kernel(const FragDev F, uint32_t W,
                                                                       const uint64_t *__restrict__ in,
                                                                       uint64_t *__restrict__ out, uint32_t n_rows) {
  extern __shared__ uint64_t cols[];
  const uint32_t r0 = blockIdx.x * kSlicedRows;
  const size_t RS = 2 * W + 1;
  rows_sliced_body(F, W, in + r0 * RS, out + r0 * RS, min(kSlicedRows, n_rows - r0), cols);
}

// The stream jobs of a batch: block x carries job x's rows.
__global__ __launch_bounds__(64 * kCarryWaves) void sliced_batch_kernel(const FragDev *__restrict__ descs,
                                                                        const CarryJob *__restrict__ jobs,
                                                                        const uint64_t *__restrict__ in,
                                                                        uint64_t *__restrict__ out) {
  extern __shared__ uint64_t cols[];
  const CarryJob &J = jobs[blockIdx.x];
  const g_FragDevH &F = ((const g_FragDevH *)descs)[J.desc];
  rows_sliced_body(F, J.W, in + J.in_off, out + J.out_off, J.n_rows, cols);
}

// One bit of a program word as a mask (0 or all ones).
__device__ inline uint64_t word_mask(uint32_t w, uint32_t bit) {
  return (uint64_t)(int64_t)((int32_t)(w << (31 - bit)) >> 31);
}

// The carry-back with qubits in lanes: lane q of the workgroup holds qubit
// q's x and z bits of 64 rows in registers for the whole program, so a step
// is a few dozen logical operations per lane and one exchange with the
// partner lane: within a wave (up to 64 qubits) a lane exchange, else one LDS
// write, a barrier and one LDS read (two buffers in turn, so one barrier a
// step is enough).  Every lane runs the same instructions whatever its gate.
// Bound by that chain of steps: the program's words are fetched kCarryAhead
// chunks ahead, one-qubit runs cost no step of their own, and 64 rows to a
// workgroup keep the workgroups independent.  The loop is unrolled by one
// chunk only: a launch runs few iterations, and its instructions come cold.
// Signs: each lane collects its share of the 64 rows' sign bits, XORed over
// the lanes at the end.  Measured on MI355X against the layered stream below
// (LDS columns, a divergent round trip per gate kind and layer, one workgroup
// for all rows): 24 qubits 25 -> 11 us, 156 qubits and 160 rows 114 -> 14 us,
// 394 qubits 90 -> 17 us, a 256-circuit batch 65 -> 21 us; unrolled by 16
// steps the first two took 13 and 17 us.
constexpr uint32_t kCarryAhead = 4;
template <bool MULTI, class D>
__device__ void carry_lanes_body(const D &F, uint32_t W, const uint64_t *__restrict__ in, uint64_t *__restrict__ out,
                                 uint32_t n_rows, ulonglong2 *ex) {
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, mp = blockDim.x;
  const uint32_t own = carry_waves(F.m);  // waves that hold qubits (a batch's blocks may have more)
  const uint32_t RS = 2 * W + 1;
  const uint32_t n_chunks = F.n_steps / kCarryChunk, stride = 64 * own;
  const bool mine = wave < own;
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 *prog = reinterpret_cast<const u32x4 *>(F.lanes) + tid;
  u32x4 queue[kCarryAhead];
#pragma unroll
  for (uint32_t i = 0; i < kCarryAhead; ++i)
    queue[i] = mine && i < n_chunks ? prog[(size_t)i * stride] : u32x4{0u, 0u, 0u, 0u};
  // lane r reads row r's words of this wave's qubits; transposed, lane q
  // holds qubit q's bits over the rows
  uint64_t x = 0, z = 0, sg = 0;
  const bool row = lane < n_rows;
  if (mine && row) {
    x = in[(size_t)lane * RS + wave];
    z = in[(size_t)lane * RS + W + wave];
  }
  const uint64_t s0 = __ballot(wave == 0 && row && (in[(size_t)lane * RS + 2 * W] & 1ull));
  if (tid == 0) sg = s0;
  x = transpose64(x, lane);
  z = transpose64(z, lane);
  uint32_t buf = 0;
#pragma unroll 1
  for (uint32_t c = 0; c < n_chunks; ++c) {
    const u32x4 cur = queue[0];
#pragma unroll
    for (uint32_t i = 0; i + 1 < kCarryAhead; ++i) queue[i] = queue[i + 1];
    if (mine && c + kCarryAhead < n_chunks) queue[kCarryAhead - 1] = prog[(size_t)(c + kCarryAhead) * stride];
#pragma unroll
    for (uint32_t i = 0; i < kCarryChunk; ++i) {
      const uint32_t w = cur[i];
      {  // the one-qubit map (c1_decode; the diagonal is stored inverted)
        const uint64_t i00 = word_mask(w, 0), m01 = word_mask(w, 1), m10 = word_mask(w, 2), i11 = word_mask(w, 3);
        sg ^= (x & word_mask(w, 4)) ^ (z & word_mask(w, 5)) ^ (x & z & word_mask(w, 6));
        const uint64_t x1 = (x & ~i00) ^ (z & m01);
        z = (z & ~i11) ^ (x & m10);
        x = x1;
      }
      uint64_t px, pz;
      if (MULTI) {
        ulonglong2 *e = ex + buf * mp;
        e[tid] = make_ulonglong2(x, z);
        __syncthreads();
        const ulonglong2 p = *reinterpret_cast<const ulonglong2 *>(reinterpret_cast<const char *>(e) + (w >> 16));
        px = p.x;
        pz = p.y;
        buf ^= 1;
      } else {
        const int addr = (int)(w >> 18);  // four bytes a lane
        const uint32_t x0 = __builtin_amdgcn_ds_bpermute(addr, (int)(uint32_t)x);
        const uint32_t x1 = __builtin_amdgcn_ds_bpermute(addr, (int)(uint32_t)(x >> 32));
        const uint32_t z0 = __builtin_amdgcn_ds_bpermute(addr, (int)(uint32_t)z);
        const uint32_t z1 = __builtin_amdgcn_ds_bpermute(addr, (int)(uint32_t)(z >> 32));
        px = (uint64_t)x1 << 32 | x0;
        pz = (uint64_t)z1 << 32 | z0;
      }
      // CX (control 1, target 2): sign x1 z2 ~(x2 ^ z1), x2 ^= x1, z1 ^= z2;
      // CZ: sign x1 x2 (z1 ^ z2), z1 ^= x2, z2 ^= x1
      const uint64_t mc = word_mask(w, 7), mt = word_mask(w, 8), mz = word_mask(w, 9), ml = word_mask(w, 10);
      sg ^= x & ((pz & ~(px ^ z) & mc) ^ (px & (z ^ pz) & ml));
      x ^= px & mt;
      z ^= (pz & mc) ^ (px & mz);
    }
  }
  x = transpose64(x, lane);
  z = transpose64(z, lane);
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) sg ^= __shfl_xor((unsigned long long)sg, off);
  if (MULTI) {
    __syncthreads();  // the last exchange is read
    if (lane == 0) ex[wave].x = sg;
    __syncthreads();
    sg = 0;
    for (uint32_t v = 0; v < mp / 64; ++v) sg ^= ex[v].x;
  }
  if (!row) return;
  if (mine) {
    out[(size_t)lane * RS + wave] = x;
    out[(size_t)lane * RS + W + wave] = z;
  }
  if (wave == 0) {
    for (uint32_t w = own; w < W; ++w) out[(size_t)lane * RS + w] = out[(size_t)lane * RS + W + w] = 0;
    out[(size_t)lane * RS + 2 * W] = (sg >> lane) & 1ull;
  }
}

// Block x carries rows [64 x, 64 x + 64).
template <bool MULTI>
__global__ __launch_bounds__(MULTI ? 512 : 64) void carry_lanes_kernel(const FragDev F, uint32_t W,
                                                                       const uint64_t *__restrict__ in,
                                                                       uint64_t *__restrict__ out, uint32_t n_rows) {
  __shared__ ulonglong2 ex[MULTI ? 2 * 512 : 1];
  const uint32_t r0 = blockIdx.x * 64;
  const size_t RS = 2 * W + 1;
  carry_lanes_body<MULTI>(F, W, in + r0 * RS, out + r0 * RS, min(64u, n_rows - r0), ex);
}

// Block x carries job x's rows (at most 64).
template <bool MULTI>
__global__ __launch_bounds__(MULTI ? 512 : 64) void carry_batch_kernel(const FragDev *__restrict__ descs,
                                                                       const CarryJob *__restrict__ jobs,
                                                                       const uint64_t *__restrict__ in,
                                                                       uint64_t *__restrict__ out) {
  __shared__ ulonglong2 ex[MULTI ? 2 * 512 : 1];
  const CarryJob &J = jobs[blockIdx.x];
  const g_FragDevH &F = ((const g_FragDevH *)descs)[J.desc];
  carry_lanes_body<MULTI>(F, J.W, in + J.in_off, out + J.out_off, J.n_rows, ex);
}

struct HeisArgs {
  uint32_t m, W, n_axes, n_in, n_out, r;
  uint32_t axis_side[kMaxAxes];
  uint32_t axis_local[kMaxAxes];
  uint64_t cin_mask[8];  // local qubits that are circuit inputs
  uint32_t n_str;        // Z-string mode: number of string rows (0 = marginal mode)
};

// One thread per (S or string, P_out combination).  rows: for the marginal
// mode the r requested Z images followed by (X_c, Z_c) images per output;
// for the string mode n_str string images followed by the output images.
// tau[p_f][col] (zero-filled by the caller) receives the single nonzero
// entry of this (col, P_out) if the circuit-input condition holds.
template <int W>
__global__ void tau_kernel(const HeisArgs A, const uint64_t *__restrict__ rows, double *__restrict__ tau,
                           uint64_t ncols) {
  const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint64_t n_pout = 1ull << (2 * A.n_out);
  if (t >= ncols * n_pout) return;
  const uint64_t col = t % ncols;
  const uint64_t pc = t / ncols;
  const uint32_t RW = 2 * W + 1;
  PAcc<W> acc;
  pclear(acc);
  uint32_t out_base;
  if (A.n_str == 0) {
    for (uint32_t j = 0; j < A.r; ++j)
      if ((col >> j) & 1ull) pmul<W>(acc, rows + (size_t)j * RW);
    out_base = A.r;
  } else {
    pmul<W>(acc, rows + (size_t)col * RW);
    out_base = A.n_str;
  }
  // output Paulis, in output-axis order
  uint32_t oc = 0;
  uint64_t pf = 0;
  for (uint32_t j = 0; j < A.n_axes; ++j) {
    if (A.axis_side[j] != 0) continue;
    const uint32_t P = (uint32_t)((pc >> (2 * oc)) & 3ull);  // I, X, Y, Z
    pmul_out<W>(acc, P, rows + (size_t)(out_base + 2 * oc) * RW);
    pf |= (uint64_t)P << (2 * j);
    ++oc;
  }
  // circuit inputs must carry I or Z
#pragma unroll
  for (int w = 0; w < W; ++w)
    if (acc.x[w] & A.cin_mask[w]) return;
  for (uint32_t j = 0; j < A.n_axes; ++j)
    if (A.axis_side[j] == 1) pf |= (uint64_t)pdigit<W>(acc, A.axis_local[j]) << (2 * j);
  tau[pf * ncols + col] = ldexp(psign<W>(acc) ? -1.0 : 1.0, (int)A.n_in);
}

// T[row][b] = 2^-r sum_S (-1)^{b.S} tau[row][S]: in-place WHT per row in LDS.
constexpr int kWht = 256;
__global__ __launch_bounds__(kWht) void subset_wht_kernel(double *__restrict__ data, uint32_t r) {
  extern __shared__ double w[];
  const uint32_t n = 1u << r;
  double *row = data + (uint64_t)blockIdx.x * n;
  for (uint32_t i = threadIdx.x; i < n; i += kWht) w[i] = row[i];
  __syncthreads();
  for (uint32_t s = 0; s < r; ++s) {
    for (uint32_t k = threadIdx.x; k < n / 2; k += kWht) {
      const uint32_t i0 = ((k >> s) << (s + 1)) | (k & ((1u << s) - 1)), i1 = i0 | (1u << s);
      const double a = w[i0], b = w[i1];
      w[i0] = a + b;
      w[i1] = a - b;
    }
    __syncthreads();
  }
  for (uint32_t i = threadIdx.x; i < n; i += kWht) row[i] = ldexp(w[i], -(int)r);
}

// The same for rows of at most 64 entries: one wave per row, entry l in
// lane l, the butterflies through lane exchanges (the same additions and
// subtractions in the same order as the LDS version), four rows per
// workgroup, coalesced row reads and writes.
__global__ __launch_bounds__(256) void subset_wht_wave_kernel(double *__restrict__ data, uint32_t r, uint64_t nrows) {
  const uint64_t row = (uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= nrows) return;  // whole waves leave together
  const uint32_t l = threadIdx.x & 63, n = 1u << r;
  double v = l < n ? data[row * n + l] : 0.0;
  for (uint32_t s = 0; s < r; ++s) {
    const double p = __shfl_xor(v, 1 << s);
    v = ((l >> s) & 1u) ? p - v : v + p;  // the pair (a, b) becomes (a + b, a - b)
  }
  if (l < n) data[row * n + l] = ldexp(v, -(int)r);
}

__global__ void fill_zero_kernel(double *p, uint64_t n) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    p[i] = 0.0;
}

// A small fragment's whole tensor in one launch: workgroup P_out carries the
// rows back itself (one wave, rows left in LDS), places its 4^n_in x 2^r
// entries in an LDS tile, transforms the tile's rows over S (the additions
// of the kernels above in the same order) and writes them out.  All of it is
// latency: carry, clearing, entries and transform took 5 + 1 + 2 + 1 us as
// launches of their own at 16 entries an output Pauli (8 qubits), 7 + 2 + 5 +
// 3 us at 64 x 256 (17 qubits), with the gaps between them on top.  With one
// stream for the call the waited marginals went from 71 to 53 us and from 64
// to 43 us on MI355X.
__global__ __launch_bounds__(256) void heis_tile_kernel(const FragDev F, const HeisArgs A,
                                                        const uint64_t *__restrict__ in, uint32_t n_rows,
                                                        double *__restrict__ T) {
  __shared__ double tile[kHeisTile];
  __shared__ uint64_t rows[kHeisTileRows * 3];
  const uint32_t n = 1u << A.r, total = n << (2 * A.n_in), pc = blockIdx.x;
  for (uint32_t i = threadIdx.x; i < total; i += 256) tile[i] = 0.0;
  if (threadIdx.x < 64) carry_lanes_body<false>(F, 1, in, rows, n_rows, nullptr);
  __syncthreads();
  for (uint32_t col = threadIdx.x; col < n; col += 256) {
    PAcc<1> acc;
    pclear(acc);
    for (uint32_t j = 0; j < A.r; ++j)
      if ((col >> j) & 1u) pmul<1>(acc, rows + 3 * j);
    for (uint32_t oc = 0; oc < A.n_out; ++oc) pmul_out<1>(acc, (pc >> (2 * oc)) & 3u, rows + 3 * (A.r + 2 * oc));
    if (acc.x[0] & A.cin_mask[0]) continue;
    uint32_t pin = 0, ic = 0;
    for (uint32_t j = 0; j < A.n_axes; ++j)
      if (A.axis_side[j] == 1) pin |= pdigit<1>(acc, A.axis_local[j]) << (2 * ic++);
    tile[(pin << A.r) | col] = ldexp(psign<1>(acc) ? -1.0 : 1.0, (int)A.n_in);
  }
  __syncthreads();
  for (uint32_t s = 0; s < A.r; ++s) {
    for (uint32_t k = threadIdx.x; k < total / 2; k += 256) {
      const uint32_t i0 = ((k >> s) << (s + 1)) | (k & ((1u << s) - 1)), i1 = i0 | (1u << s);
      const double a = tile[i0], b = tile[i1];
      tile[i0] = a + b;
      tile[i1] = a - b;
    }
    __syncthreads();
  }
  for (uint32_t i = threadIdx.x; i < total; i += 256) {
    uint64_t pf = 0;
    uint32_t po = pc, pi = i >> A.r;
    for (uint32_t j = 0; j < A.n_axes; ++j) {
      uint32_t &d = A.axis_side[j] == 1 ? pi : po;
      pf |= (uint64_t)(d & 3u) << (2 * j);
      d >>= 2;
    }
    T[(pf << A.r) | (i & (n - 1))] = ldexp(tile[i], -(int)A.r);
  }
}

HeisArgs heis_args(const FragDev &F, uint32_t W, uint32_t n_in, uint32_t n_out, uint32_t r, uint32_t n_str,
                   const uint64_t *cin_mask) {
  HeisArgs A{};
  A.m = F.m;
  A.W = W;
  A.n_axes = F.n_axes;
  A.n_in = n_in;
  A.n_out = n_out;
  A.r = r;
  A.n_str = n_str;
  for (uint32_t j = 0; j < F.n_axes; ++j) {
    A.axis_side[j] = F.axis_side[j];
    A.axis_local[j] = F.axis_local[j];
  }
  for (uint32_t w = 0; w < 8; ++w) A.cin_mask[w] = w < W ? cin_mask[w] : 0;
  return A;
}

template <int W>
hipError_t run_w(const HeisArgs &A, const uint64_t *rows, double *tau, uint64_t ncols, hipStream_t s) {
  hipError_t e;
  const uint64_t total_tau = ncols << (2 * A.n_axes);
  hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)std::min<uint64_t>((total_tau + 255) / 256, 65536)), dim3(256),
                     0, s, tau, total_tau);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const uint64_t nt = ncols << (2 * A.n_out);
  hipLaunchKernelGGL((tau_kernel<W>), dim3((unsigned)((nt + 255) / 256)), dim3(256), 0, s, A, rows, tau, ncols);
  return hipGetLastError();
}

}  // namespace

// rows: carried-back Pauli rows [n_rows][2W+1] with W = words(m) rounded up
// to {1, 2, 4, 8}.  Marginal mode (n_str == 0): rows are
// r requested Z's then (X_c, Z_c) per output axis; tau is [4^n_axes][2^r] and
// is turned into T[p_f][b] in place.  String mode: rows are n_str strings then
// the output pairs; tau is [4^n_axes][n_str] = t_f[p_f][string].
size_t rows_sliced_lds(uint32_t m, uint32_t n_rows) {
  return (size_t)2 * m * ((n_rows + 63) / 64) * 8 + (kOpStage + kLayStage + 1) * 4;
}

hipError_t launch_rows(const FragDev &F, uint32_t W, const uint64_t *in, uint64_t *out, uint32_t n_rows,
                       hipStream_t s) {
  if (n_rows == 0) return hipSuccess;
  if (!in || (W != 1 && W != 2 && W != 4 && W != 8) || F.m > 64 * W) return hipErrorInvalidValue;
  // a lane program wherever the plan built one: it stands for every stream but
  // those of more than 64 MB of program (a word per qubit and step, against
  // one per gate), which the layered kernel takes
  if (F.lanes) {
    if (F.n_steps % kCarryChunk) return hipErrorInvalidValue;
    const dim3 grid((n_rows + 63) / 64), block(64 * carry_waves(F.m));
    if (F.m <= 64)
      hipLaunchKernelGGL(carry_lanes_kernel<false>, grid, block, 0, s, F, W, in, out, n_rows);
    else
      hipLaunchKernelGGL(carry_lanes_kernel<true>, grid, block, 0, s, F, W, in, out, n_rows);
    return hipGetLastError();
  }
  const size_t lds = rows_sliced_lds(F.m, std::min(n_rows, kSlicedRows));
  if (lds > 160 * 1024) return hipErrorInvalidValue;
  hipError_t e = hipFuncSetAttribute((const void *)rows_sliced_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(rows_sliced_kernel, dim3((n_rows + kSlicedRows - 1) / kSlicedRows), dim3(64 * kCarryWaves), lds, s,
                     F, W, in, out, n_rows);
  return hipGetLastError();
}

hipError_t launch_carry_batch(const FragDev *descs, const CarryJob *jobs, uint32_t n_lanes, uint32_t waves,
                              uint32_t n_stream, uint32_t max_m, uint32_t max_rows, const uint64_t *in, uint64_t *out,
                              hipStream_t s) {
  if (n_lanes) {
    if (waves == 0 || waves > 8) return hipErrorInvalidValue;
    if (waves == 1)
      hipLaunchKernelGGL(carry_batch_kernel<false>, dim3(n_lanes), dim3(64), 0, s, descs, jobs, in, out);
    else
      hipLaunchKernelGGL(carry_batch_kernel<true>, dim3(n_lanes), dim3(64 * waves), 0, s, descs, jobs, in, out);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (n_stream == 0) return hipSuccess;
  if (max_rows > kSlicedRows) return hipErrorInvalidValue;
  const size_t lds = rows_sliced_lds(max_m, max_rows);
  if (lds > 160 * 1024) return hipErrorInvalidValue;
  hipError_t e = hipFuncSetAttribute((const void *)sliced_batch_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(sliced_batch_kernel, dim3(n_stream), dim3(64 * kCarryWaves), lds, s, descs, jobs + n_lanes, in,
                     out);
  return hipGetLastError();
}

hipError_t launch_heisenberg(const FragDev &F, uint32_t W, uint32_t n_in, uint32_t n_out, uint32_t r,
                             uint32_t n_str, const uint64_t *cin_mask, const uint64_t *rows, double *tau,
                             hipStream_t s) {
  const HeisArgs A = heis_args(F, W, n_in, n_out, r, n_str, cin_mask);
  const uint64_t ncols = n_str ? n_str : (1ull << r);
  hipError_t e;
  switch (W) {
    case 1: e = run_w<1>(A, rows, tau, ncols, s); break;
    case 2: e = run_w<2>(A, rows, tau, ncols, s); break;
    case 4: e = run_w<4>(A, rows, tau, ncols, s); break;
    case 8: e = run_w<8>(A, rows, tau, ncols, s); break;
    default: return hipErrorInvalidValue;
  }
  if (e != hipSuccess || n_str) return e;
  const uint64_t nrows = 1ull << (2 * F.n_axes);
  if (r == 0) return hipSuccess;
  if (r <= 6) {
    for (uint64_t r0 = 0; r0 < nrows; r0 += (1ull << 32)) {
      const uint64_t cnt = std::min<uint64_t>(nrows - r0, 1ull << 32);
      hipLaunchKernelGGL(subset_wht_wave_kernel, dim3((unsigned)((cnt + 3) / 4)), dim3(256), 0, s, tau + (r0 << r), r,
                         cnt);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
  }
  for (uint64_t r0 = 0; r0 < nrows; r0 += (1ull << 30)) {
    const uint64_t cnt = std::min<uint64_t>(nrows - r0, 1ull << 30);
    hipLaunchKernelGGL(subset_wht_kernel, dim3((unsigned)cnt), dim3(kWht), (size_t(1) << r) * 8, s,
                       tau + (r0 << r), r);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_heis_tile(const FragDev &F, uint32_t n_in, uint32_t n_out, uint32_t r, const uint64_t *cin_mask,
                            const uint64_t *in, uint32_t n_rows, double *T, hipStream_t s) {
  if (!F.lanes || F.n_steps % kCarryChunk || !in || n_rows != r + 2 * n_out || n_in + n_out != F.n_axes ||
      !heis_one_launch(F.m, F.n_steps, n_in, n_out, r))
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(heis_tile_kernel, dim3(1u << (2 * n_out)), dim3(256), 0, s, F,
                     heis_args(F, 1, n_in, n_out, r, 0, cin_mask), in, n_rows, T);
  return hipGetLastError();
}

}  // namespace ccut
