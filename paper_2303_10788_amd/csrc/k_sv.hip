// Non-Clifford fragment variants on a dense fp64 state vector (the paper's
// exact backend for non-Clifford fragments, Sec. V-B).
//
// Variants of a fragment share everything but their preparations and their
// final basis rotations.  The fragment is linear in its input state, and
// |+> = (|0> + |1>)/sqrt2, |+i> = (|0> + i|1>)/sqrt2.  So it is run only on
// the 2^n_in computational-basis inputs (evolve pass, final states to HBM),
// and every variant's amplitudes are combinations of those states over the
// cut axes (combine pass): an input axis combines the states of its two
// inputs, an output axis the two halves of its qubit.
//
// The gate program is a list of three-qubit unitaries (the host fuses the
// gates greedily, build_sv_program): one step multiplies a real 16 x 16
// matrix (8 basis states, real and imaginary parts) with the state seen as
// 16 x 2^(m-3), on the fp64 matrix cores.  Rows of a step's operand: the 8
// states of its three qubits' bits (b0 b1 b2), real parts 0-7, imaginary
// parts 8-15; columns: the other qubits' bits.  v_mfma_f64_16x16x4_f64 takes
// B[k][col] from lane 16 k + col and leaves D[row][col] in lane
// 16 (row % 4) + col, register row / 4, so with k = 4 chunk + lane / 16 a
// lane holds the same two amplitudes (b2 = 0, 1) before and after the
// product: it reads them from LDS as two 16-byte words and writes them back
// to the same place, and one barrier a step is all the waves need.
//
// A run is bound by the chain of steps: per step an LDS round trip, four
// dependent products (64 cycles each) per tile of 128 amplitudes and the
// barrier; from 11 qubits on by the matrix cores (2048 cycles a step at 12).
// Fusing three qubits a step is what shortens the chain: gates applied one at
// a time to amplitudes in registers took 163 steps of 0.5 us for a 10-qubit
// fragment, the 38 fused ones 0.68 us each.  (Four qubits a step would double
// the products for a quarter fewer steps.)  Measured on MI355X, evolve pass:
// 10 qubits 80 -> 26 us, 7 qubits 24 -> 7 us; both passes of a 256-circuit
// batch 1905 -> 770 us of kernel time over its three streams.
#include "common.hpp"

// No implicit contraction: every fused multiply-add is written out, so the
// single-fragment and the batched kernel (the same body inlined in
// different code) round identically.
#pragma clang fp contract(off)

namespace ccut {

namespace {

struct __attribute__((aligned(16))) C2 {
  double re, im;
};
typedef double double4v __attribute__((ext_vector_type(4)));
typedef double double2v __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <class T>
__device__ inline const T *uniform_ptr(const T *p) {
  const uint64_t u = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u), hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
  return (const T *)(((uint64_t)hi << 32) | lo);
}

// LDS slot of amplitude i: bits 4-7 and 8-11 folded onto the lowest four, so
// lanes that differ in four bits of different residues mod 4 (the host picks
// them so where it can) fall on different banks.
__device__ inline uint32_t sv_slot(uint32_t i) { return i ^ ((i >> 4) & 15u) ^ ((i >> 8) & 15u); }

constexpr uint32_t kSvAhead = 2;  // steps whose matrices are on their way (4: 98 registers, one workgroup a CU)

// Runs the program on computational-basis input blk.  blockDim.x =
// 64 sv_waves(m).
template <class D>
__device__ __attribute__((always_inline)) void sv_evolve(D &F, uint32_t blk, C2 *S, C2 *__restrict__ states) {
  const uint32_t m = F.m, n_steps = F.n_ops;
  const uint32_t tid = threadIdx.x, lane = tid & 63, BS = blockDim.x;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t mm = m < 3 ? 3 : m, N = 1u << mm;  // fewer than three qubits: idle ones added above
  const bool multi = BS > 64;
  // this lane's matrix elements A[row lane % 16][k = 4 c + lane / 16], c < 4,
  // and its LDS offsets, loaded kSvAhead steps ahead
  typedef __attribute__((address_space(1))) const double2v g_double2;
  typedef __attribute__((address_space(1))) const u32x4 g_u32x4;
  const g_double2 *mats = (const g_double2 *)uniform_ptr(F.mats) + 2 * lane;
  const g_u32x4 *words = (const g_u32x4 *)uniform_ptr(F.ops) + lane;
  double2v qa[kSvAhead], qb[kSvAhead];
  u32x4 qw[kSvAhead];
#pragma unroll
  for (uint32_t i = 0; i < kSvAhead; ++i) {
    qa[i] = qb[i] = double2v{0.0, 0.0};
    qw[i] = u32x4{0u, 0u, 0u, 0u};
    if (i < n_steps) {
      qw[i] = words[(size_t)i * 64];
      qa[i] = mats[(size_t)i * 128];
      qb[i] = mats[(size_t)i * 128 + 1];
    }
  }
  uint32_t start = 0, n_in = 0;
  for (uint32_t j = 0; j < F.n_axes; ++j)
    if (F.axis_side[j] == 1) start |= ((blk >> n_in++) & 1u) << F.axis_local[j];
  for (uint32_t i = tid; i < N; i += BS) S[sv_slot(i)] = C2{i == start ? 1.0 : 0.0, 0.0};
  const uint32_t wb0 = wave & 1u ? 0xFFFFu : 0u, wb1 = wave & 2u ? ~0u : 0u, wb2 = wave & 4u ? 0xFFFFu : 0u,
                 wb3 = wave & 8u ? ~0u : 0u;
  const bool live = (lane & 15u) < (1u << (mm - 3 < 4 ? mm - 3 : 4));  // fewer than 16 columns: lanes idle
  const uint32_t n_tiles = mm > 7 ? 1u << (mm - 7) : 1u, waves = BS >> 6;
  const bool two = n_tiles > waves;  // 12 qubits: two tiles a wave
  char *Sb = reinterpret_cast<char *>(S);
  auto tile = [&](const double2v A01, const double2v A23, uint32_t off, uint32_t breg) __attribute__((always_inline)) {
    C2 x0{0.0, 0.0}, x1 = x0;
    if (live) {
      x0 = *reinterpret_cast<C2 *>(Sb + off);
      x1 = *reinterpret_cast<C2 *>(Sb + (off ^ breg));
    }
    double4v d{0.0, 0.0, 0.0, 0.0};
    d = __builtin_amdgcn_mfma_f64_16x16x4f64(A01.x, x0.re, d, 0, 0, 0);
    d = __builtin_amdgcn_mfma_f64_16x16x4f64(A01.y, x1.re, d, 0, 0, 0);
    d = __builtin_amdgcn_mfma_f64_16x16x4f64(A23.x, x0.im, d, 0, 0, 0);
    d = __builtin_amdgcn_mfma_f64_16x16x4f64(A23.y, x1.im, d, 0, 0, 0);
    if (live) {
      *reinterpret_cast<C2 *>(Sb + off) = C2{d[0], d[2]};
      *reinterpret_cast<C2 *>(Sb + (off ^ breg)) = C2{d[1], d[3]};
    }
  };
  auto step = [&](const double2v A01, const double2v A23, const u32x4 w) __attribute__((always_inline)) {
    // the lane's offset within tile 0, the register bit's, and tile bits 0-4's
    const uint32_t breg = w.x >> 16;
    const uint32_t off = (w.x & 0xFFFFu) ^ (w.y & wb0) ^ ((w.y & wb1) >> 16) ^ (w.z & wb2) ^ ((w.z & wb3) >> 16);
    if (multi) {
      __syncthreads();  // the previous step is written
    } else {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    tile(A01, A23, off, breg);
    if (two) tile(A01, A23, off ^ w.w, breg);
  };
#pragma unroll 1
  for (uint32_t s0 = 0; s0 < n_steps; s0 += kSvAhead) {
#pragma unroll
    for (uint32_t i = 0; i < kSvAhead; ++i) {
      const uint32_t s = s0 + i;
      if (s >= n_steps) break;
      const double2v A01 = qa[i], A23 = qb[i];
      const u32x4 w = qw[i];
      if (s + kSvAhead < n_steps) {
        qw[i] = words[(size_t)(s + kSvAhead) * 64];
        qa[i] = mats[(size_t)(s + kSvAhead) * 128];
        qb[i] = mats[(size_t)(s + kSvAhead) * 128 + 1];
      }
      step(A01, A23, w);
    }
  }
  __syncthreads();
  const uint32_t n_amp = 1u << m;
  C2 *dst = states + (size_t)blk * n_amp;
  for (uint32_t i = tid; i < n_amp; i += BS) dst[i] = S[sv_slot(i)];
}

// Combine pass.  Along every cut axis two values (an input's two states, an
// output qubit's two amplitudes) give up to six: 0: a, 1: b, 2: a + b,
// 3: a - b, 4: a - ib, 5: a + ib (2 to 5 without their factor 1/sqrt2: the
// probability takes 1/2 for each, exactly).  An input's preparations 0, 1, +,
// +i are values 0, 1, 2, 5; an output's outcomes in X are 2, 3, in Y 4, 5, in
// Z 0, 1.  A wave takes one choice of values along the axes beyond the first
// two (unit / x blocks) and, per lane, one outcome x of the requested qubits
// and a share of the unmeasured qubits' configurations; it reads the 2^L
// amplitudes of its configuration along the first L <= 4 axes at once (the
// axes beyond four summed in as they are read), reduces them to the first two
// axes and adds up all 36 probabilities in registers, so a state is read
// 4^-2 (inputs) or 6^-2 (outputs) as often as there are variants.  The lanes
// that share an outcome add up in a fixed order; with few outcomes (four lanes
// or more each) the 36 sums are spread over the wave.  Bound by fp64 adds and
// the loads from L2.  Measured for the 11- and 12-qubit fragments of a
// 256-circuit batch: 277 -> 118 us against one workgroup per variant (state
// combined and rotated in LDS, a barrier per rotation and unmeasured qubit); for
// 10 qubits, two outputs and no requested qubit 7 us (30 to 38 where one lane
// added up all 36), with 6 to 8 requested ones 5 us.
__device__ inline C2 sv_value(C2 a, C2 b, uint32_t k) {
  switch (k) {
    case 0: return a;
    case 1: return b;
    case 2: return C2{a.re + b.re, a.im + b.im};
    case 3: return C2{a.re - b.re, a.im - b.im};
    case 4: return C2{a.re + b.im, a.im - b.re};
    default: return C2{a.re - b.im, a.im + b.re};
  }
}
// choice d of an axis (input: preparation; output: 2 basis + outcome) -> value
__device__ inline uint32_t sv_kind(bool input, uint32_t d) {
  return input ? (d == 3 ? 5u : d) : (d < 4 ? d + 2 : d - 4);
}
// both squares rounded: (x, y) and (y, x) have the same probability, so values
// that are zero by such a symmetry come out as zero
__device__ inline double sv_prob(C2 a) { return a.re * a.re + a.im * a.im; }

// lds: 36 rows of kSvRow doubles, the wave's sums on their way out (one short loop
// stores them all: written out 36 times, the stores took as long to fetch as
// the rest of a small call to run)
// A walk is a serial chain of loads, and few outcomes make few units: the waves
// of a unit take equal shares of the configurations that a lane walks through
// (sv_share_bits: at most eight waves, a lone one for walks of up to eight, which
// a second wave's sums through LDS would not shorten), and add their sums up
// pairwise in a fixed order.  Calls on 12 qubits with one requested: four inputs
// 248 -> 155 us, three 129 -> 73, four outputs 80 -> 52; 11 qubits, three inputs
// 100 -> 66.
constexpr uint32_t kSvRow = 65;    // (64 lanes, padded: lanes that read different rows meet different banks)
constexpr uint32_t kSvSpread = 2;  // see the end of sv_combine
constexpr uint32_t kSvShareBits = 3;
__host__ __device__ inline uint32_t sv_lane_bits(uint32_t r, uint32_t nu) {  // of configurations, beside the outcome's
  const uint32_t lr = r < 6 ? r : 6;
  return nu < 6 - lr ? nu : 6 - lr;
}
__host__ __device__ inline uint32_t sv_share_bits(uint32_t r, uint32_t nu) {
  const uint32_t walk = nu - sv_lane_bits(r, nu);
  return walk <= 3 ? 0 : walk - 3 < kSvShareBits ? walk - 3 : kSvShareBits;
}
template <int L, class D>
__device__ __attribute__((always_inline)) void sv_combine(D &F, double *__restrict__ dist, uint32_t unit,
                                                          const C2 *__restrict__ states, double *lds) {
  const uint32_t n_axes = F.n_axes, nm = F.n_meas, ins = F.in_axes, rmask = F.req_mask, umask = F.rest_mask;
  const uint32_t lane = threadIdx.x & 63, share = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t r = __popc(rmask), nu = __popc(umask);
  const uint32_t lr = r < 6 ? r : 6, lu = sv_lane_bits(r, nu);  // lane bits: outcome, configuration
  const uint32_t sb = sv_share_bits(r, nu);
  const uint32_t xb = r - lr;
  uint32_t group = unit >> xb;
  // this lane's amplitude index and outcome, bit by bit over the qubits
  uint32_t base = 0, out = 0, uhi = umask;  // uhi: configurations walked through one after another
  {
    uint32_t x = (lane & ((1u << lr) - 1)) | (unit & ((1u << xb) - 1)) << lr, u = lane >> lr, pos = 0;
    const uint32_t mmask = ~umask;
    uint32_t left = lu;
#pragma unroll 1
    for (uint32_t q = 0, all = rmask | umask; all >> q; ++q) {
      if (rmask >> q & 1u) {
        base |= (x & 1u) << q;
        out |= (x & 1u) << pos;
        x >>= 1;
      } else if ((umask >> q & 1u) && left) {
        base |= (u & 1u) << q;
        u >>= 1;
        --left;
        uhi &= ~(1u << q);
      }
      pos += mmask >> q & 1u;
    }
  }
  for (uint32_t i = sb; i-- > 0;) {  // the share: the highest of the bits walked through
    const uint32_t q = 31u - (uint32_t)__builtin_clz(uhi);
    base |= (share >> i & 1u) << q;
    uhi &= ~(1u << q);
  }
  const bool live = lane < 1u << (lr + lu);
  // choices along the axes beyond the first two (three bits each)
  uint64_t kinds = 0;
  uint32_t v = 0;
  int halves = (int)F.sv_halves;
#pragma unroll 1
  for (uint32_t j = 2; j < n_axes; ++j) {
    const bool in = ins >> j & 1u;
    const uint32_t n = in ? 4u : 6u, d = group % n, k = sv_kind(in, d);
    group /= n;
    kinds |= (uint64_t)k << (3 * j);
    halves += k >= 2;
    v += (in ? d : d >> 1) * F.axis_stride[j];
    if (!in && (d & 1u)) out |= F.axis_obit[j];
  }
  double acc[L > 1 ? 6 : 1][L > 0 ? 6 : 1];
#pragma unroll
  for (int i = 0; i < (L > 1 ? 6 : 1); ++i)
#pragma unroll
    for (int j = 0; j < (L > 0 ? 6 : 1); ++j) acc[i][j] = 0.0;
  typedef __attribute__((address_space(1))) const double2v g_double2;
  const g_double2 *src = (const g_double2 *)states + base;
  uint32_t corner[1 << L];  // offsets of the first L axes' corners
#pragma unroll
  for (int l = 0; l < (1 << L); ++l) {
    corner[l] = 0;
#pragma unroll
    for (int j = 0; j < L; ++j) corner[l] += l >> j & 1 ? F.axis_dist[j] : 0u;
  }
  constexpr bool kPrefetch = L < 4;  // (16 amplitudes twice would halve the waves)
  auto load = [&](double2v(&t)[1 << L], uint32_t off) __attribute__((always_inline)) {
#pragma unroll
    for (int l = 0; l < (1 << L); ++l) t[l] = live ? src[off + corner[l]] : double2v{0.0, 0.0};
  };
  double2v nxt[1 << L];
  if (kPrefetch && n_axes <= 4) load(nxt, 0);
  uint32_t uc = 0;
#pragma unroll 1
  do {  // the configurations of uhi, ascending
    C2 A[1 << L];
    const uint32_t un = (uc - uhi) & uhi;
    if (n_axes <= 4) {
      if constexpr (kPrefetch) {
#pragma unroll
        for (int l = 0; l < (1 << L); ++l) A[l] = C2{nxt[l].x, nxt[l].y};
        if (un) load(nxt, un);
      } else {
        double2v t[1 << L];
        load(t, uc);
#pragma unroll
        for (int l = 0; l < (1 << L); ++l) A[l] = C2{t[l].x, t[l].y};
      }
    } else {
#pragma unroll
      for (int l = 0; l < (1 << L); ++l) A[l] = C2{0.0, 0.0};
#pragma unroll 1
      for (uint32_t h = 0; h < 1u << (n_axes - 4); ++h) {
        // the choice's coefficient of this corner of the upper axes: 0, or i^ph
        uint32_t off = uc, ph = 0;
        bool in = true;
        for (uint32_t j = 4; j < n_axes; ++j) {
          const uint32_t hb = h >> (j - 4) & 1u, k = kinds >> (3 * j) & 7u;
          if (hb) off += F.axis_dist[j];
          if (k < 2) in &= hb == k;
          if (hb) ph += k == 3 ? 2u : k == 4 ? 3u : k == 5 ? 1u : 0u;
        }
        if (!in) continue;
        ph &= 3u;
        double2v t[1 << L];
        load(t, off);
#pragma unroll
        for (int l = 0; l < (1 << L); ++l) {
          A[l].re += ph == 0 ? t[l].x : ph == 1 ? -t[l].y : ph == 2 ? -t[l].x : t[l].y;
          A[l].im += ph == 0 ? t[l].y : ph == 1 ? t[l].x : ph == 2 ? -t[l].y : -t[l].x;
        }
      }
    }
    if constexpr (L > 3) {
#pragma unroll
      for (int l = 0; l < 8; ++l) A[l] = sv_value(A[l], A[l + 8], kinds >> 9 & 7u);
    }
    if constexpr (L > 2) {
#pragma unroll
      for (int l = 0; l < 4; ++l) A[l] = sv_value(A[l], A[l + 4], kinds >> 6 & 7u);
    }
    if constexpr (L == 0) {
      acc[0][0] += sv_prob(A[0]);
    } else {
#pragma unroll
      for (uint32_t k1 = 0; k1 < (L > 1 ? 6 : 1); ++k1) {
        C2 a = A[0], b = A[1];
        if constexpr (L > 1) {
          if ((ins >> 1 & 1u) && (k1 == 3 || k1 == 4)) continue;
          a = sv_value(A[0], A[2], k1);
          b = sv_value(A[1], A[3], k1);
        }
#pragma unroll
        for (uint32_t k0 = 0; k0 < 6; ++k0) {
          if ((ins & 1u) && (k0 == 3 || k0 == 4)) continue;
          acc[k1][k0] += sv_prob(sv_value(a, b, k0));
        }
      }
    }
    uc = un;
  } while (uc);
  constexpr uint32_t n1 = L > 1 ? 6 : 1, n0 = L > 0 ? 6 : 1;
  for (uint32_t h = 1u << sb >> 1; h; h >>= 1) {  // the upper half of the waves hands its sums to the lower half
    double *to = lds + (share & (h - 1)) * (36 * kSvRow) + lane;
    if (share >= h && share < 2 * h) {
#pragma unroll
      for (uint32_t k = 0; k < n1 * n0; ++k) to[k * kSvRow] = acc[k / n0][k % n0];
    }
    __syncthreads();
    if (share < h) {
#pragma unroll
      for (uint32_t k = 0; k < n1 * n0; ++k) acc[k / n0][k % n0] += to[k * kSvRow];
    }
    __syncthreads();
  }
  if (share) return;
#pragma unroll
  for (uint32_t k1 = 0; k1 < n1; ++k1)
#pragma unroll
    for (uint32_t k0 = 0; k0 < n0; ++k0) lds[(k1 * n0 + k0) * kSvRow + lane] = acc[k1][k0];
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __attribute__((address_space(1))) double *o = (__attribute__((address_space(1))) double *)dist;
  const bool in0 = ins & 1u, in1 = ins >> 1 & 1u;
  const uint32_t e1 = L > 1 ? (in1 ? 4u : 6u) : 1u, e0 = L > 0 ? (in0 ? 4u : 6u) : 1u;
  const uint32_t st0 = L > 0 ? F.axis_stride[0] : 0u, st1 = L > 1 ? F.axis_stride[1] : 0u;
  const uint32_t ob0 = L > 0 ? F.axis_obit[0] : 0u, ob1 = L > 1 ? F.axis_obit[1] : 0u;
  if (lu >= kSvSpread) {
    // few outcomes of many lanes each: the choices along the two axes go to
    // the lanes too, each summing the lanes that share its outcome in order (the
    // same sums as below; from four lanes to an outcome on, as with two the
    // sums below take one more read each)
    const double *src = lds + (lane & ((1u << lr) - 1));
#pragma unroll 1
    for (uint32_t d = lane >> lr; d < e1 * e0; d += 64u >> lr) {
      const uint32_t d1 = d / e0, d0 = d - d1 * e0;
      const uint32_t k1 = L > 1 ? sv_kind(in1, d1) : 0u, k0 = L > 0 ? sv_kind(in0, d0) : 0u;
      const double *row = src + (k1 * n0 + k0) * kSvRow;
      double p = row[0];
#pragma unroll 8
      for (uint32_t t = 1; t < 1u << lu; ++t) p += row[t << lr];
      const uint32_t vv = v + (in1 ? d1 : d1 >> 1) * st1 + (in0 ? d0 : d0 >> 1) * st0;
      const uint32_t oo = out | (d1 & 1u ? ob1 : 0u) | (d0 & 1u ? ob0 : 0u);
      o[((size_t)vv << nm) + oo] = ldexp(p, -(halves + (k1 >= 2) + (k0 >= 2)));
    }
    return;
  }
  if (lane >= 1u << lr) return;
#pragma unroll 1
  for (uint32_t d1 = 0; d1 < e1; ++d1) {
    uint32_t v1 = v, o1 = out, k1 = 0;
    int h1 = halves;
    if (L > 1) {
      k1 = sv_kind(in1, d1);
      h1 += k1 >= 2;
      v1 += (in1 ? d1 : d1 >> 1) * st1;
      o1 |= d1 & 1u ? ob1 : 0u;  // (0 for an input)
    }
    const double *src1 = lds + k1 * n0 * kSvRow + lane;
    double p[n0];
#pragma unroll
    for (uint32_t d0 = 0; d0 < n0; ++d0) p[d0] = src1[(L > 0 ? sv_kind(in0, d0) : 0u) * kSvRow];
    for (uint32_t t = 1; t < 1u << lu; ++t)  // the lanes that share the outcome, in order
#pragma unroll
      for (uint32_t d0 = 0; d0 < n0; ++d0) p[d0] += src1[(L > 0 ? sv_kind(in0, d0) : 0u) * kSvRow + (t << lr)];
#pragma unroll
    for (uint32_t d0 = 0; d0 < n0; ++d0) {
      if (d0 >= e0) continue;
      const uint32_t vv = v1 + (in0 ? d0 : d0 >> 1) * st0, oo = o1 | (d0 & 1u ? ob0 : 0u);
      o[((size_t)vv << nm) + oo] = ldexp(p[d0], -(h1 + (L > 0 && sv_kind(in0, d0) >= 2 ? 1 : 0)));
    }
  }
}

template <class D>
__device__ __attribute__((always_inline)) void sv_combine_any(D &F, double *__restrict__ dist, uint32_t unit,
                                                              const C2 *__restrict__ states, double *lds) {
  switch (F.n_axes) {
    case 0: sv_combine<0>(F, dist, unit, states, lds); break;
    case 1: sv_combine<1>(F, dist, unit, states, lds); break;
    case 2: sv_combine<2>(F, dist, unit, states, lds); break;
    case 3: sv_combine<3>(F, dist, unit, states, lds); break;
    default: sv_combine<4>(F, dist, unit, states, lds); break;
  }
}

// Descriptors in constant memory: fields read with a uniform index are scalar loads.
typedef __attribute__((address_space(4))) const FragDev c_FragDev;
__device__ inline c_FragDev &const_desc(const FragDev *descs, uint32_t i) {
  return ((c_FragDev *)(uintptr_t)descs)[i];
}

// two workgroups of 16 waves to a compute unit
__global__ __launch_bounds__(1024, 8) void sv_evolve_kernel(const FragDev F, C2 *__restrict__ states) {
  extern __shared__ C2 smem[];
  sv_evolve(F, blockIdx.x, smem, states);
}

// One unit a workgroup, 2^sv_share_bits waves.
__global__ __launch_bounds__(64 << kSvShareBits) void sv_combine_kernel(const FragDev F, double *__restrict__ dist,
                                                                        const C2 *__restrict__ states) {
  extern __shared__ double lds[];
  sv_combine_any(F, dist, blockIdx.x, states, lds);
}

// Many fragments of one shape: workgroup x belongs to the job holding x.
__device__ inline const SvJob &sv_job(const SvJob *__restrict__ jobs, uint32_t n_jobs) {
  uint32_t lo = 0, hi = n_jobs;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) / 2;
    if (jobs[mid].wg0 <= blockIdx.x) lo = mid;
    else hi = mid;
  }
  return jobs[__builtin_amdgcn_readfirstlane(lo)];
}

__global__ __launch_bounds__(1024, 8) void sv_evolve_batch_kernel(const FragDev *__restrict__ descs,
                                                                  const SvJob *__restrict__ jobs, uint32_t n_jobs) {
  extern __shared__ C2 smem[];
  // the job's fields are workgroup-uniform: keep them in scalar registers
  const SvJob &J = sv_job(jobs, n_jobs);
  const uint32_t desc = __builtin_amdgcn_readfirstlane(J.desc);
  const uint32_t blk = __builtin_amdgcn_readfirstlane((uint32_t)(blockIdx.x - J.wg0));
  sv_evolve(const_desc(descs, desc), blk, smem, reinterpret_cast<C2 *>(const_cast<double *>(uniform_ptr(J.states))));
}

__global__ __launch_bounds__(64 << kSvShareBits) void sv_combine_batch_kernel(const FragDev *__restrict__ descs,
                                                                              const SvJob *__restrict__ jobs,
                                                                              uint32_t n_jobs) {
  extern __shared__ double lds[];
  const SvJob &J = sv_job(jobs, n_jobs);
  const uint32_t desc = __builtin_amdgcn_readfirstlane(J.desc);
  const uint32_t unit = __builtin_amdgcn_readfirstlane((uint32_t)(blockIdx.x - J.wg0));
  sv_combine_any(const_desc(descs, desc), const_cast<double *>(uniform_ptr(J.dist)), unit,
                 reinterpret_cast<const C2 *>(uniform_ptr(J.states)), lds);
}

}  // namespace

uint32_t sv_inputs(const FragDev &h) {
  uint32_t n_in = 0;
  for (uint32_t j = 0; j < h.n_axes; ++j) n_in += h.axis_side[j] == 1;
  return n_in;
}

size_t sv_states_bytes(const FragDev &h) { return ((size_t)1 << (sv_inputs(h) + h.m)) * sizeof(C2); }

// Units of the combine pass: blocks of 64 outcomes of the requested qubits
// times the choices along the axes beyond the first two.
static uint64_t combine_units(const FragDev &h) {
  const uint32_t n_in = sv_inputs(h), n_out = h.n_axes - n_in, r = h.n_meas - n_out;
  uint64_t u = r > 6 ? 1ull << (r - 6) : 1ull;
  for (uint32_t j = 2; j < h.n_axes; ++j) u *= h.axis_side[j] == 1 ? 4 : 6;
  return u;
}

// Workgroups of a pass, with their threads and LDS bytes: evolve (one workgroup
// per computational-basis input, its state in LDS) or combine (one per unit).
SvShape sv_pass_shape(const FragDev &h, bool combine) {
  SvShape S;
  if (!combine) {
    S.n_wg = 1ull << sv_inputs(h);
    S.threads = 64 * sv_waves(h.m);
    S.lds = ((size_t)1 << (h.m < 3 ? 3 : h.m)) * sizeof(C2);
  } else {
    const uint32_t sb = sv_share_bits(__builtin_popcount(h.req_mask), __builtin_popcount(h.rest_mask));
    S.n_wg = combine_units(h);
    S.threads = 64u << sb;
    S.lds = (sb > 1 ? 1u << (sb - 1) : 1u) * (36 * kSvRow * sizeof(double));
  }
  return S;
}

static hipError_t set_lds(const void *kernel, const SvShape &S) {
  if (S.lds > 160 * 1024 || S.n_wg > 0x7FFFFFFFull || S.threads == 0 || S.threads > 1024) return hipErrorInvalidValue;
  if (S.lds <= 64 * 1024) return hipSuccess;  // (what every launch may ask for)
  return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)S.lds);
}

hipError_t launch_sv_batch(const FragDev *descs, const SvJob *jobs, uint32_t n_jobs, const SvShape &S, bool combine,
                           hipStream_t s) {
  if (n_jobs == 0) return hipSuccess;
  const hipError_t e = set_lds(combine ? (const void *)sv_combine_batch_kernel : (const void *)sv_evolve_batch_kernel, S);
  if (e != hipSuccess) return e;
  if (combine)
    hipLaunchKernelGGL(sv_combine_batch_kernel, dim3((unsigned)S.n_wg), dim3(S.threads), S.lds, s, descs, jobs, n_jobs);
  else
    hipLaunchKernelGGL(sv_evolve_batch_kernel, dim3((unsigned)S.n_wg), dim3(S.threads), S.lds, s, descs, jobs, n_jobs);
  return hipGetLastError();
}

hipError_t launch_sv(const FragDev &h, double *dist, void *states, hipStream_t s) {
  if (h.m == 0 || h.m > (uint32_t)kMaxNcQubits || h.n_meas > h.m || !states) return hipErrorInvalidValue;
  SvShape S = sv_pass_shape(h, false);
  hipError_t e = set_lds((const void *)sv_evolve_kernel, S);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(sv_evolve_kernel, dim3((unsigned)S.n_wg), dim3(S.threads), S.lds, s, h, static_cast<C2 *>(states));
  if ((e = hipGetLastError()) != hipSuccess) return e;
  S = sv_pass_shape(h, true);
  if ((e = set_lds((const void *)sv_combine_kernel, S)) != hipSuccess) return e;
  hipLaunchKernelGGL(sv_combine_kernel, dim3((unsigned)S.n_wg), dim3(S.threads), S.lds, s, h, dist,
                     static_cast<const C2 *>(states));
  return hipGetLastError();
}

}  // namespace ccut
