// Host-side planning (see plan.hpp).  Fragments follow the paper's cutter
// output (Sec. V-A): disjoint subcircuits after cutting; roles of fragment
// inputs and outputs follow Sec. V-B.
#include "plan.hpp"

#include <algorithm>
#include <cmath>
#include <complex>
#include <cstdint>
#include <cstring>
#include <map>
#include <numeric>
#include <set>
#include <utility>

#include "../../include/ccut.h"

namespace ccut {

namespace {

bool is_two_qubit(uint32_t k) { return k == G_CX || k == G_CZ; }
bool is_clifford(uint32_t k) { return k <= G_CZ; }

struct DSU {
  std::vector<uint32_t> p;
  explicit DSU(size_t n) : p(n) { std::iota(p.begin(), p.end(), 0u); }
  uint32_t find(uint32_t a) {
    while (p[a] != a) {
      p[a] = p[p[a]];
      a = p[a];
    }
    return a;
  }
  void unite(uint32_t a, uint32_t b) {
    a = find(a);
    b = find(b);
    if (a != b) p[a] = b;
  }
};

using cplx = std::complex<double>;
struct M2 {
  cplx a, b, c, d;  // [[a, b], [c, d]]
};
M2 mul(const M2 &L, const M2 &R) {  // L * R
  return {L.a * R.a + L.b * R.c, L.a * R.b + L.b * R.d, L.c * R.a + L.d * R.c, L.c * R.b + L.d * R.d};
}
M2 gate_matrix(uint32_t kind, double theta) {
  const double r = 1.0 / std::sqrt(2.0);
  const cplx i(0, 1);
  switch (kind) {
    case G_H: return {r, r, r, -r};
    case G_S: return {1, 0, 0, i};
    case G_SDG: return {1, 0, 0, -i};
    case G_X: return {0, 1, 1, 0};
    case G_Y: return {0, -i, i, 0};
    case G_Z: return {1, 0, 0, -1};
    case G_T: return {1, 0, 0, std::polar(1.0, M_PI / 4)};
    case G_TDG: return {1, 0, 0, std::polar(1.0, -M_PI / 4)};
    case G_RZ: return {1, 0, 0, std::polar(1.0, theta)};
    default: return {1, 0, 0, 1};
  }
}

// Fuse every run of one-qubit gates on a qubit (up to the next two-qubit
// gate touching it) into one matrix; runs on different qubits commute with
// the two-qubit gates that do not touch them, so emitting a run just before
// the first two-qubit gate on its qubit preserves the circuit.  A run that
// is diagonal so far also commutes with a CZ on its qubit and with a CX it
// controls, so it continues past them.  Diagonal gates that end a qubit which
// goes into no cut change no outcome (it is measured in Z or summed over) and
// are left out: a T there would only round amplitudes of equal magnitude
// differently.  (An angle that is no number is not left out: what it makes of
// the outcomes is no number either.)
void fuse_one_qubit_runs(Fragment &F) {
  const uint32_t m = F.m();
  std::vector<char> end(m, 1), skip(F.op_words.size(), 0);
  for (const Axis &a : F.axes)
    if (a.side == 0) end[a.local] = 0;
  for (size_t g = F.op_words.size(); g-- > 0;) {
    const uint32_t k = op_kind(F.op_words[g]), q = op_q0(F.op_words[g]);
    if (is_two_qubit(k)) {
      end[q] = end[op_q1(F.op_words[g])] = 0;
    } else {
      const M2 M = gate_matrix(k, F.op_theta[g]);
      end[q] = end[q] && M.b == 0.0 && M.c == 0.0 && std::isfinite(M.d.real()) && std::isfinite(M.d.imag());
      skip[g] = end[q];
    }
  }
  std::vector<M2> pend(m, M2{1, 0, 0, 1});
  std::vector<char> has(m, 0), rz(m, 0);  // rz: an RZ is in the run
  auto flush = [&](uint32_t q) {
    if (!has[q]) return;
    const M2 &M = pend[q];
    F.sv_words.push_back(pack_op(G_U2, q, 0));
    F.sv_rz.push_back(rz[q]);
    const cplx e[4] = {M.a, M.b, M.c, M.d};
    for (auto &z : e) {
      F.sv_mats.push_back(z.real());
      F.sv_mats.push_back(z.imag());
    }
    pend[q] = M2{1, 0, 0, 1};
    has[q] = rz[q] = 0;
  };
  for (size_t g = 0; g < F.op_words.size(); ++g) {
    const uint32_t w = F.op_words[g], k = op_kind(w), a = op_q0(w), b = op_q1(w);
    if (skip[g]) continue;
    if (is_two_qubit(k)) {
      // a diagonal run commutes with a CZ on its qubit and with a CX it
      // controls, so it stays pending and merges with the next run
      auto diag = [&](uint32_t q) { return pend[q].b == 0.0 && pend[q].c == 0.0; };
      if (!(diag(a) && (k == G_CZ || k == G_CX))) flush(a);
      if (!(diag(b) && k == G_CZ)) flush(b);
      F.sv_words.push_back(w);
      F.sv_rz.push_back(0);
      for (int t = 0; t < 8; ++t) F.sv_mats.push_back(0.0);
    } else {
      pend[a] = mul(gate_matrix(k, F.op_theta[g]), pend[a]);
      has[a] = 1;
      rz[a] |= k == G_RZ;
    }
  }
  for (size_t g = 0; g < skip.size(); ++g)  // a run left out as a whole still counts as one (ccut_fragment_ops)
    if (skip[g] && !has[op_q0(F.op_words[g])]) has[op_q0(F.op_words[g])] = 2;
  F.sv_left_out = 0;
  for (uint32_t q = 0; q < m; ++q)
    if (has[q] == 2) {
      ++F.sv_left_out;
      has[q] = 0;
    }
  if (F.sv_left_out && F.sv_words.empty() && std::count(has.begin(), has.end(), 1) == 0) {
    --F.sv_left_out;  // a program has a step: one of them as the identity
    has[0] = 1;
  }
  for (uint32_t q = 0; q < m; ++q) flush(q);
}

// The state-vector program: the fused stream cut into three-qubit unitaries.
// A block starts at the first op not yet taken and takes, in order, every
// later op on its three qubits that no skipped op comes before on any of its
// qubits (an op is skipped when it leaves the block's qubits; ops on disjoint
// qubits commute).  Its first two qubits are the starting op's (a one-qubit
// op's partner in its next two-qubit gate), the third is the one that lets it
// take most ops.
struct SvBlock {
  uint32_t q[3];
  std::vector<size_t> ops;
};

void sv_blocks(const Fragment &F, uint32_t mm, std::vector<SvBlock> &blocks) {
  const size_t n = F.sv_words.size();
  std::vector<uint32_t> mask(n);
  std::vector<std::vector<size_t>> on(mm);  // each qubit's ops in order
  std::vector<size_t> head(mm, 0);          // of them taken: always the first ones
  for (size_t g = 0; g < n; ++g) {
    const uint32_t w = F.sv_words[g];
    mask[g] = 1u << op_q0(w) | (is_two_qubit(op_kind(w)) ? 1u << op_q1(w) : 0u);
    for (uint32_t r = mask[g]; r; r &= r - 1) on[__builtin_ctz(r)].push_back(g);
  }
  // the ops on `set` that a block may take, in order; only ops that touch a
  // qubit of it which is not blocked yet are looked at
  auto scan = [&](uint32_t set, std::vector<size_t> *take) {
    size_t at[32], count = 0;
    for (uint32_t r = set; r; r &= r - 1) at[__builtin_ctz(r)] = head[__builtin_ctz(r)];
    for (uint32_t open = set;;) {
      size_t g = n;
      for (uint32_t r = open; r; r &= r - 1) {
        const uint32_t q = __builtin_ctz(r);
        if (at[q] < on[q].size()) g = std::min(g, on[q][at[q]]);
      }
      if (g == n) return count;
      if (!(mask[g] & ~open)) {
        ++count;
        if (take) take->push_back(g);
        for (uint32_t r = mask[g]; r; r &= r - 1) ++at[__builtin_ctz(r)];
      } else {
        open &= ~mask[g];
      }
    }
  };
  std::vector<char> done(n, 0);
  for (size_t g0 = 0; g0 < n; ++g0) {
    if (done[g0]) continue;
    uint32_t pair = mask[g0];
    if (__builtin_popcount(pair) == 1) {
      const uint32_t q = __builtin_ctz(pair);
      for (size_t i = head[q]; i < on[q].size() && __builtin_popcount(pair) == 1; ++i) pair |= mask[on[q][i]];
    }
    for (uint32_t q = 0; __builtin_popcount(pair) < 2; ++q) pair |= 1u << q;
    uint32_t best = 0;
    size_t most = 0;
    for (uint32_t q = 0; q < mm; ++q) {
      if (pair >> q & 1u) continue;
      const size_t c = scan(pair | 1u << q, nullptr);
      if (c > most) {
        most = c;
        best = q;
      }
    }
    const uint32_t set = pair | 1u << best;
    SvBlock B;
    for (uint32_t q = 0, i = 0; q < mm; ++q)
      if (set >> q & 1u) B.q[i++] = q;
    scan(set, &B.ops);
    for (size_t g : B.ops) {
      done[g] = 1;
      for (uint32_t r = mask[g]; r; r &= r - 1) ++head[__builtin_ctz(r)];
    }
    blocks.push_back(std::move(B));
  }
}

// The block's 8 x 8 unitary, bit i of a basis index = qubit q[i].
void sv_block_matrix(const Fragment &F, const SvBlock &B, cplx (&U)[8][8]) {
  for (uint32_t i = 0; i < 8; ++i)
    for (uint32_t j = 0; j < 8; ++j) U[i][j] = i == j ? 1.0 : 0.0;
  auto local = [&](uint32_t q) { return 1u << (q == B.q[0] ? 0 : q == B.q[1] ? 1 : 2); };
  for (size_t g : B.ops) {
    const uint32_t w = F.sv_words[g], k = op_kind(w), a = local(op_q0(w));
    if (k == G_U2) {
      const double *e = &F.sv_mats[8 * g];
      const cplx m00(e[0], e[1]), m01(e[2], e[3]), m10(e[4], e[5]), m11(e[6], e[7]);
      for (uint32_t i = 0; i < 8; ++i) {
        if (i & a) continue;
        for (uint32_t j = 0; j < 8; ++j) {
          const cplx x = U[i][j], y = U[i | a][j];
          U[i][j] = m00 * x + m01 * y;
          U[i | a][j] = m10 * x + m11 * y;
        }
      }
    } else {
      const uint32_t b = local(op_q1(w));
      for (uint32_t i = 0; i < 8; ++i) {
        if (!(i & a) || (i & b)) continue;
        for (uint32_t j = 0; j < 8; ++j) {
          if (k == G_CX)
            std::swap(U[i][j], U[i | b][j]);
          else
            U[i | b][j] = -U[i | b][j];
        }
      }
    }
  }
}

// Puts the matrix of a block of Clifford gates and T, times sqrt2 if the result
// says so, on its exact values where these are of the form (a + b / sqrt2) / 64
// with whole a, b (found from the product of the gates, which is within 2e-14
// of them), of the two scalings the one with fewer entries of b.  Whole
// multiples of powers of two keep the products of a step exact, so amplitudes
// that cancel cancel to zero rather than to a rounding residue.  The angle of an
// RZ is the caller's, however close to a multiple of pi / 4 (or no number at
// all): a block that holds one stays as it is.
bool sv_exact_matrix(cplx (&U)[8][8]) {
  const double r = 0.70710678118654752440, tol = 64.0 * 2e-14;
  struct Value {
    double u, out[2];  // a magnitude, its exact value as it is and times sqrt2
    bool root[2];
  };
  Value seen[16];  // a block has a few magnitudes; one with more is not of this form
  uint32_t n_seen = 0, roots[2] = {};
  uint8_t at[128];
  const double *flat = reinterpret_cast<const double *>(U);
  for (uint32_t i = 0; i < 128; ++i) {
    const double u = std::fabs(flat[i]);
    uint32_t k = 0;
    while (k < n_seen && std::fabs(seen[k].u - u) > 2e-14) ++k;
    if (k == n_seen) {
      if (n_seen == 16) return false;
      Value &x = seen[n_seen++];
      x.u = u;
      for (int odd = 0; odd < 2; ++odd) {
        const double v = 64.0 * u * (odd ? 2.0 * r : 1.0);
        bool found = false;
        for (int t = 0; t <= 192 && !found; ++t) {  // no root, roots alone, then both
          double a = 0.0, b = 0.0;
          if (t == 1) b = std::floor(v / r + 0.5);
          if (t >= 2) b = t & 1 ? -(t / 2) : t / 2;
          if (t != 1) a = std::floor(v - b * r + 0.5);
          if (std::fabs(v - (a + b * r)) > tol) continue;
          found = true;
          x.out[odd] = (double)((a + b * 0.70710678118654752440084436210485L) / 64.0L);
          x.root[odd] = b != 0.0;
        }
        if (!found) return false;
      }
    }
    at[i] = (uint8_t)k;
  }
  for (uint32_t e = 0; e < 64; ++e)  // entries; column 0 (where a run starts) decides a draw
    for (int odd = 0; odd < 2; ++odd)
      roots[odd] += seen[at[2 * e]].root[odd] || seen[at[2 * e + 1]].root[odd] ? (e % 8 == 0 ? 65u : 64u) : 0u;
  const bool odd = roots[1] < roots[0];
  double *to = reinterpret_cast<double *>(U);
  for (uint32_t i = 0; i < 128; ++i) to[i] = std::copysign(seen[at[i]].out[odd], flat[i]);
  return odd;
}

// Per step four words and four doubles a lane (sv_prog, sv_prog_mats).  Words:
// LDS byte offsets (16 bits each) of the lane's index bits and of the register
// bit, then of tile bits 0-1, 2-3 and 4.  Doubles: lane l's matrix elements
// A[l % 16][4 c + l / 16], c < 4.  The block's qubits are lane bits 4 and 5 and
// the register; the other qubits fill lane bits 0-3 (residues 0, 1, 2, 3 mod 4
// where they can: different LDS banks), then the tile.
void build_sv_program(Fragment &F) {
  const uint32_t m = F.m(), mm = std::max(m, 3u);
  std::vector<SvBlock> blocks;
  sv_blocks(F, mm, blocks);
  F.sv_halves = 0;
  F.sv_prog.reserve(256 * blocks.size());
  F.sv_prog_mats.reserve(256 * blocks.size());
  auto slot = [](uint32_t p) { return ((1u << p) | (p >= 4 ? 1u << (p & 3u) : 0u)) * 16u; };  // p < 12: sv_slot(2^p)
  for (const SvBlock &B : blocks) {
    std::vector<uint32_t> rest;
    for (uint32_t q = 0; q < mm; ++q)
      if (q != B.q[0] && q != B.q[1] && q != B.q[2]) rest.push_back(q);
    std::vector<uint32_t> cols;
    for (uint32_t r = 0; r < 4 && !rest.empty(); ++r) {
      size_t at = 0;
      for (size_t i = 0; i < rest.size(); ++i)
        if ((rest[i] & 3u) == r) {
          at = i;
          break;
        }
      cols.push_back(rest[at]);
      rest.erase(rest.begin() + (long)at);
    }
    uint32_t off[12] = {};  // lane 0-5, register, tile 0-4
    for (size_t i = 0; i < cols.size(); ++i) off[i] = slot(cols[i]);
    off[4] = slot(B.q[0]);
    off[5] = slot(B.q[1]);
    off[6] = slot(B.q[2]);
    for (size_t i = 0; i < rest.size(); ++i) off[7 + i] = slot(rest[i]);
    for (uint32_t l = 0; l < 64; ++l) {
      uint32_t o = 0;
      for (uint32_t j = 0; j < 6; ++j) o ^= l >> j & 1u ? off[j] : 0u;
      F.sv_prog.insert(F.sv_prog.end(), {o | off[6] << 16, off[7] | off[8] << 16, off[9] | off[10] << 16, off[11]});
    }
    cplx U[8][8];
    sv_block_matrix(F, B, U);
    // every second factor sqrt2 takes the one before it out with 1/2; one
    // that is left halves the probabilities (sv_combine)
    const bool rz = std::any_of(B.ops.begin(), B.ops.end(), [&](size_t g) { return F.sv_rz[g] != 0; });
    const bool odd = !rz && sv_exact_matrix(U);
    const double half = odd && F.sv_halves ? 0.5 : 1.0;
    F.sv_halves ^= odd;
    for (uint32_t l = 0; l < 64; ++l)
      for (uint32_t c = 0; c < 4; ++c) {
        const uint32_t row = l % 16, k = 4 * c + l / 16;
        const cplx u = half * U[row & 7u][k & 7u];
        F.sv_prog_mats.push_back(row < 8 ? (k < 8 ? u.real() : -u.imag()) : (k < 8 ? u.imag() : u.real()));
      }
  }
}

// Order a Clifford stream by ASAP layer: op g goes one layer after the
// latest earlier op on any of its qubits, so each layer acts on disjoint
// qubits and per-qubit order is kept (ops on disjoint qubits commute).
void layer_stream(std::vector<uint32_t> &words, std::vector<uint32_t> &starts, uint32_t m) {
  std::vector<int32_t> qlayer(m, -1);
  std::vector<uint32_t> lay(words.size());
  uint32_t nl = 0;
  for (size_t g = 0; g < words.size(); ++g) {
    const uint32_t w = words[g], k = op_kind(w), a = op_q0(w);
    const uint32_t b = (k == G_CX || k == G_CZ) ? op_q1(w) : a;
    const int32_t L = std::max(qlayer[a], qlayer[b]) + 1;
    lay[g] = (uint32_t)L;
    qlayer[a] = qlayer[b] = L;
    nl = std::max(nl, (uint32_t)L + 1);
  }
  starts.assign(nl + 1, 0);
  for (uint32_t L : lay) starts[L + 1]++;
  for (uint32_t L = 0; L < nl; ++L) starts[L + 1] += starts[L];
  std::vector<uint32_t> pos(starts.begin(), starts.end() - 1), out(words.size());
  for (size_t g = 0; g < words.size(); ++g) out[pos[lay[g]]++] = words[g];
  words.swap(out);
}

// The carry-back stream as a lane program: step s holds one word per qubit,
// a two-qubit gate at the first step after both its qubits' earlier gates, a
// one-qubit run merged into the word of the gate it precedes (or in a step of
// its own after the last one).  Steps are padded to a multiple of 4, qubits
// to whole waves.  False (and no program) where it would take more than
// kLaneWordsMax words: deep streams that keep few qubits busy at a time.
bool lane_program(const std::vector<uint32_t> &stream, uint32_t m, std::vector<uint32_t> &prog) {
  const uint64_t mp = 64 * carry_waves(m);
  std::vector<uint64_t> next(m, 0);
  std::vector<uint32_t> run(m, 0u);  // pending one-qubit map
  auto put = [&](uint64_t s, uint32_t q, uint32_t word) {
    const uint64_t need = (s / kCarryChunk + 1) * kCarryChunk * mp;
    if (need > kLaneWordsMax) return false;
    if (prog.size() < need) prog.resize(need, 0u);
    prog[(s / kCarryChunk * mp + q) * kCarryChunk + s % kCarryChunk] = word;
    return true;
  };
  for (const uint32_t w : stream) {
    const uint32_t k = op_kind(w), a = op_q0(w), b = op_q1(w);
    if (!is_two_qubit(k)) {
      run[a] = c1_then(run[a], b);
      continue;
    }
    const uint64_t s = std::max(next[a], next[b]);
    const uint32_t ra = k == G_CX ? kCarryControl : kCarryCz | kCarryLead, rb = k == G_CX ? kCarryTarget : kCarryCz;
    if (!put(s, a, carry_word(run[a], ra, b)) || !put(s, b, carry_word(run[b], rb, a))) {
      prog.clear();
      return false;
    }
    run[a] = run[b] = 0u;
    next[a] = next[b] = s + 1;
  }
  for (uint32_t q = 0; q < m; ++q)
    if (run[q] && !put(next[q], q, carry_word(run[q], 0, q))) {
      prog.clear();
      return false;
    }
  return true;
}

// Fuse every run of one-qubit Cliffords on a qubit into one G_C1 word,
// emitted just before the next two-qubit gate on that qubit (or at the
// end): the forward stream (gate counts) and, from the same runs, the
// reversed stream of inverse gates for the Heisenberg carry-back.
void fuse_clifford_runs(Fragment &F) {
  const uint32_t m = F.m();
  std::vector<uint32_t> fwd(m, 0u), inv(m, 0u);
  std::vector<char> has(m, 0);
  std::vector<uint32_t> back;  // built forward, reversed at the end
  auto flush = [&](uint32_t q) {
    if (!has[q]) return;
    F.cl_words.push_back(pack_op(G_C1, q, fwd[q]));
    back.push_back(pack_op(G_C1, q, inv[q]));
    fwd[q] = inv[q] = 0u;
    has[q] = 0;
  };
  for (size_t g = 0; g < F.op_words.size(); ++g) {
    const uint32_t w = F.op_words[g], k = op_kind(w), a = op_q0(w), b = op_q1(w);
    if (is_two_qubit(k)) {
      flush(a);
      flush(b);
      F.cl_words.push_back(w);
      back.push_back(w);  // CX and CZ are their own inverses
    } else {
      const uint32_t kinv = k == G_S ? (uint32_t)G_SDG : k == G_SDG ? (uint32_t)G_S : k;
      fwd[a] = c1_then(fwd[a], c1_of_gate(k));
      inv[a] = c1_then(c1_of_gate(kinv), inv[a]);  // the inverse run applies the last gate's inverse first
      has[a] = 1;
    }
  }
  for (uint32_t q = 0; q < m; ++q) flush(q);
  std::reverse(back.begin(), back.end());
  if (m <= 512 && lane_program(back, m, F.cl_lanes)) return;
  F.cl_back = std::move(back);
  layer_stream(F.cl_back, F.cl_back_layers, m);
}

}  // namespace

int build_plan(uint32_t n, const HostOp *ops, size_t n_ops, const uint32_t *cut_q,
               const uint32_t *cut_after, size_t k, uint32_t max_nc, uint32_t max_cuts,
               PlanData &out, std::string &err) {
  if (n == 0 || n >= 16384) {
    err = "n_qubits must be in [1, 16383]";
    return CCUT_E_INVALID;
  }
  for (size_t i = 0; i < n_ops; ++i) {
    const HostOp &o = ops[i];
    if (o.kind > G_RZ) {
      err = "op " + std::to_string(i) + ": unknown gate kind";
      return CCUT_E_INVALID;
    }
    if (o.q0 >= n) {
      err = "op " + std::to_string(i) + ": qubit out of range";
      return CCUT_E_INVALID;
    }
    if (is_two_qubit(o.kind) && (o.q1 >= n || o.q1 == o.q0)) {
      err = "op " + std::to_string(i) + ": bad two-qubit operands";
      return CCUT_E_INVALID;
    }
  }
  std::set<std::pair<uint32_t, uint32_t>> seen;
  for (size_t c = 0; c < k; ++c) {
    if (cut_q[c] >= n || cut_after[c] >= n_ops) {
      err = "cut " + std::to_string(c) + ": out of range";
      return CCUT_E_INVALID;
    }
    const HostOp &o = ops[cut_after[c]];
    bool on = o.q0 == cut_q[c] || (is_two_qubit(o.kind) && o.q1 == cut_q[c]);
    if (!on) {
      err = "cut " + std::to_string(c) + ": op " + std::to_string(cut_after[c]) +
            " does not act on qubit " + std::to_string(cut_q[c]);
      return CCUT_E_INVALID;
    }
    if (!seen.insert({cut_q[c], cut_after[c]}).second) {
      err = "cut " + std::to_string(c) + ": duplicate";
      return CCUT_E_INVALID;
    }
  }
  if (k > max_cuts) {
    err = "k = " + std::to_string(k) + " cuts exceeds max_cuts = " + std::to_string(max_cuts);
    return CCUT_E_TOO_MANY_CUTS;
  }
  // position of each op along each of its wires
  std::vector<uint32_t> wire_len(n, 0);
  std::vector<uint32_t> pos0(n_ops), pos1(n_ops, 0);
  for (size_t i = 0; i < n_ops; ++i) {
    pos0[i] = wire_len[ops[i].q0]++;
    if (is_two_qubit(ops[i].kind)) pos1[i] = wire_len[ops[i].q1]++;
  }
  // cuts on each wire sorted by position; cut c separates segment s and s+1
  std::vector<std::vector<std::pair<uint32_t, uint32_t>>> wire_cuts(n);
  for (size_t c = 0; c < k; ++c) {
    const HostOp &o = ops[cut_after[c]];
    uint32_t p = (o.q0 == cut_q[c]) ? pos0[cut_after[c]] : pos1[cut_after[c]];
    wire_cuts[cut_q[c]].push_back({p, (uint32_t)c});
  }
  std::vector<uint32_t> seg_base(n + 1, 0);
  for (uint32_t q = 0; q < n; ++q) {
    std::sort(wire_cuts[q].begin(), wire_cuts[q].end());
    seg_base[q + 1] = seg_base[q] + (uint32_t)wire_cuts[q].size() + 1;
  }
  std::vector<uint32_t> cut_wire(k), cut_seg(k);
  for (uint32_t q = 0; q < n; ++q)
    for (size_t s = 0; s < wire_cuts[q].size(); ++s) {
      cut_wire[wire_cuts[q][s].second] = q;
      cut_seg[wire_cuts[q][s].second] = (uint32_t)s;
    }
  auto seg_of = [&](uint32_t q, uint32_t p) -> uint32_t {
    // segment index = number of cuts on the wire strictly before position p
    uint32_t s = 0;
    for (auto &wc : wire_cuts[q])
      if (wc.first < p) ++s;
    return s;
  };
  const uint32_t n_segs = seg_base[n];
  std::vector<uint32_t> op_seg0(n_ops), op_seg1(n_ops, 0);
  DSU dsu(n_segs);
  for (size_t i = 0; i < n_ops; ++i) {
    op_seg0[i] = seg_base[ops[i].q0] + seg_of(ops[i].q0, pos0[i]);
    if (is_two_qubit(ops[i].kind)) {
      op_seg1[i] = seg_base[ops[i].q1] + seg_of(ops[i].q1, pos1[i]);
      dsu.unite(op_seg0[i], op_seg1[i]);
    }
  }
  // components, ordered by their smallest (wire, segment), i.e. smallest global segment id
  std::map<uint32_t, std::vector<uint32_t>> comps;
  for (uint32_t s = 0; s < n_segs; ++s) comps[dsu.find(s)].push_back(s);
  std::vector<std::vector<uint32_t>> groups;
  for (auto &kv : comps) groups.push_back(kv.second);
  std::sort(groups.begin(), groups.end(),
            [](const std::vector<uint32_t> &a, const std::vector<uint32_t> &b) { return a[0] < b[0]; });
  if (groups.size() > 255) {
    err = "more than 255 fragments";
    return CCUT_E_UNSUPPORTED;
  }
  std::vector<uint32_t> seg_wire(n_segs), seg_idx(n_segs);
  for (uint32_t q = 0; q < n; ++q)
    for (uint32_t s = seg_base[q]; s < seg_base[q + 1]; ++s) {
      seg_wire[s] = q;
      seg_idx[s] = s - seg_base[q];
    }
  std::vector<int32_t> seg_frag(n_segs), seg_local(n_segs);
  out = PlanData();
  out.n = n;
  out.k = (uint32_t)k;
  out.frags.resize(groups.size());
  for (size_t fi = 0; fi < groups.size(); ++fi) {
    Fragment &F = out.frags[fi];
    F.index = (uint32_t)fi;
    F.out_local.assign(n, -1);
    for (size_t j = 0; j < groups[fi].size(); ++j) {
      uint32_t s = groups[fi][j];  // ascending global id = ascending (wire, segment)
      seg_frag[s] = (int32_t)fi;
      seg_local[s] = (int32_t)j;
      F.wires.push_back(seg_wire[s]);
      F.segs.push_back(seg_idx[s]);
      if (s + 1 == seg_base[seg_wire[s] + 1]) F.out_local[seg_wire[s]] = (int32_t)j;
    }
  }
  for (size_t i = 0; i < n_ops; ++i) {
    Fragment &F = out.frags[seg_frag[op_seg0[i]]];
    uint32_t l0 = (uint32_t)seg_local[op_seg0[i]];
    uint32_t l1 = is_two_qubit(ops[i].kind) ? (uint32_t)seg_local[op_seg1[i]] : 0u;
    F.op_words.push_back(pack_op(ops[i].kind, l0, l1));
    F.op_theta.push_back(ops[i].theta);
    if (!is_clifford(ops[i].kind)) F.clifford = false;
  }
  for (size_t c = 0; c < k; ++c) {
    uint32_t up = seg_base[cut_wire[c]] + cut_seg[c];
    uint32_t down = up + 1;
    Fragment &Fu = out.frags[seg_frag[up]];
    Fu.axes.push_back({(uint32_t)c, 0u, (uint32_t)seg_local[up]});
    Fragment &Fd = out.frags[seg_frag[down]];
    Fd.axes.push_back({(uint32_t)c, 1u, (uint32_t)seg_local[down]});
  }
  for (Fragment &F : out.frags) {
    std::stable_sort(F.axes.begin(), F.axes.end(), [](const Axis &a, const Axis &b) {
      return a.cut != b.cut ? a.cut < b.cut : a.side < b.side;
    });
    if (F.axes.size() > (size_t)kMaxAxes) {
      err = "fragment " + std::to_string(F.index) + " has more than 16 cut axes";
      return CCUT_E_UNSUPPORTED;
    }
    uint64_t nv = 1;
    for (const Axis &a : F.axes) nv *= a.radix();
    if (nv > 0xFFFFFFFFull) {
      err = "fragment " + std::to_string(F.index) + " has more than 2^32 variants";
      return CCUT_E_UNSUPPORTED;
    }
    F.n_variants = nv;
    if (!F.clifford) {
      fuse_one_qubit_runs(F);
      if (F.m() <= (uint32_t)kMaxNcQubits) build_sv_program(F);
    } else {
      fuse_clifford_runs(F);
    }
    if (!F.clifford && F.m() > max_nc) {
      err = "non-Clifford fragment " + std::to_string(F.index) + " has " + std::to_string(F.m()) +
            " qubits > max_nc_qubits = " + std::to_string(max_nc);
      return CCUT_E_NC_TOO_WIDE;
    }
  }
  return CCUT_OK;
}

static FragRequest finish_request(const Fragment &f, std::vector<uint32_t> wanted_local,
                                  std::vector<uint32_t> wanted_user) {
  FragRequest r;
  std::set<uint32_t> meas(wanted_local.begin(), wanted_local.end());
  for (const Axis &a : f.axes)
    if (a.side == 0) meas.insert(a.local);
  r.meas.assign(meas.begin(), meas.end());
  std::map<uint32_t, uint32_t> pos;
  for (size_t j = 0; j < r.meas.size(); ++j) pos[r.meas[j]] = (uint32_t)j;
  std::vector<std::pair<uint32_t, uint32_t>> req;
  for (size_t i = 0; i < wanted_local.size(); ++i) req.push_back({pos[wanted_local[i]], wanted_user[i]});
  std::sort(req.begin(), req.end());
  for (auto &p : req) {
    r.req_pos.push_back(p.first);
    r.req_user.push_back(p.second);
  }
  for (const Axis &a : f.axes) r.axis_outpos.push_back(a.side == 0 ? (int32_t)pos[a.local] : -1);
  return r;
}

FragRequest marginal_request(const Fragment &f, const uint32_t *qubits, uint32_t nq) {
  std::vector<uint32_t> wl, wu;
  for (uint32_t i = 0; i < nq; ++i) {
    int32_t l = f.out_local[qubits[i]];
    if (l >= 0) {
      wl.push_back((uint32_t)l);
      wu.push_back(i);
    }
  }
  return finish_request(f, wl, wu);
}

FragRequest zstring_request(const Fragment &f, const std::vector<uint64_t> &anymask) {
  std::vector<uint32_t> wl, wu;
  for (uint32_t q = 0; q < (uint32_t)f.out_local.size(); ++q) {
    if (f.out_local[q] >= 0 && ((anymask[q >> 6] >> (q & 63)) & 1ull)) {
      wl.push_back((uint32_t)f.out_local[q]);
      wu.push_back(q);  // for Z strings the "user bit" is the circuit qubit
    }
  }
  return finish_request(f, wl, wu);
}

FragDev make_frag_dev(const Fragment &f, const FragRequest &r, uint64_t vid_base) {
  FragDev d{};
  d.m = f.m();
  d.n_ops = f.clifford ? 0u : (uint32_t)(f.sv_prog.size() / 256);
  d.n_axes = (uint32_t)f.axes.size();
  d.n_meas = (uint32_t)r.meas.size();
  d.n_req = (uint32_t)r.req_pos.size();
  d.clifford = f.clifford ? 1u : 0u;
  d.n_variants = f.n_variants;
  d.vid_base = vid_base;
  for (size_t j = 0; j < f.axes.size(); ++j) {
    d.axis_side[j] = f.axes[j].side;
    d.axis_local[j] = f.axes[j].local;
    d.axis_radix[j] = f.axes[j].radix();
    d.axis_cut[j] = f.axes[j].cut;
  }
  for (size_t j = 0; j < r.meas.size() && j < (size_t)kMaxMeas; ++j) d.meas[j] = (uint16_t)r.meas[j];
  if (!f.clifford && d.m <= (uint32_t)kMaxNcQubits) {
    uint32_t n_in = 0, stride = 1, outs = 0;
    for (size_t j = 0; j < f.axes.size(); ++j) {
      const Axis &a = f.axes[j];
      d.axis_stride[j] = stride;
      stride *= a.radix();
      if (a.side == 1) {
        d.in_axes |= 1u << j;
        d.axis_dist[j] = 1u << (d.m + n_in++);
      } else {
        d.axis_dist[j] = 1u << a.local;
        d.axis_obit[j] = 1u << r.axis_outpos[j];
        outs |= 1u << a.local;
      }
    }
    for (uint32_t q : r.meas) d.req_mask |= 1u << q;
    d.req_mask &= ~outs;
    d.rest_mask = ((1u << d.m) - 1) & ~(d.req_mask | outs);
  }
  return d;
}

}  // namespace ccut
