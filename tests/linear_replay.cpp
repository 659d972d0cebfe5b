// Replays the linear schedules of the generated kernels (linear_plan.h) on the
// CPU in double precision: every instruction on a full state held at its
// physical index, exchanges through their LDS slots, streaming passes through
// their address columns.  Compared with the circuit's primitives (CNOTs
// included) applied one by one: the measured <Z> and the probabilities of the
// forward, the adjoint walking a copy of the final state back through every saved
// state, and its gradients per slot (unit chain-rule factors).  Constant Paulis,
// which the tables' frame carries, and the heads' gradients are left to the tests
// on a GPU.  Prints one line per circuit; exits non-zero on a mismatch.
#include <cmath>
#include <complex>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <random>

#include "vqc.h"
#include "vqc_internal.h"

using namespace vqc;
using C = std::complex<double>;
using State = std::vector<C>;

namespace {

int fail(const char* what, int n, int seed) {
  std::printf("FAIL %s n=%d seed=%d\n", what, n, seed);
  return 1;
}

uint32_t odd(uint32_t v) { return (uint32_t)__builtin_parity(v); }

// exp(-i th/2 P) on the pairs (y, y ^ x) with the sign of parity(z & y)
void rotate(State& s, int op, uint32_t x, uint32_t z, double th) {
  const double c = std::cos(th / 2), s0 = std::sin(th / 2);
  for (uint32_t y = 0; y < s.size(); ++y) {
    const double sn = op == OP_RX && odd(z & y) ? -s0 : s0;
    if (op == OP_RZ) {
      s[y] *= C(c, odd(z & y) ? sn : -sn);
      continue;
    }
    const uint32_t v = y ^ x;
    if (op == OP_RX ? v < y : odd(z & y)) continue;
    const C a = s[y], b = s[v];
    if (op == OP_RX) {
      s[y] = c * a - C(0, sn) * b;
      s[v] = c * b - C(0, sn) * a;
    } else {
      s[y] = c * a - sn * b;
      s[v] = sn * a + c * b;
    }
  }
}

void sign_flip(State& s, uint32_t z, uint32_t z2) {
  for (uint32_t y = 0; y < s.size(); ++y)
    if (odd(z & y) & odd(z2 & y)) s[y] = -s[y];
}

uint32_t xor_cols(const std::vector<uint32_t>& cols, int off, uint32_t bits) {
  uint32_t o = 0;
  for (int p = 0; bits >> p; ++p)
    if ((bits >> p) & 1u) o ^= cols[off + p];
  return o;
}

bool exchange(State& s, const Plan& p, int off) {
  const uint32_t K = 1u << p.k;
  std::vector<uint32_t> at(K, ~0u);
  for (uint32_t y = 0; y < K; ++y) {
    const uint32_t slot = xor_cols(p.cols, off, y);
    if (slot >= K || at[slot] != ~0u) return false;
    at[slot] = y;
  }
  State t(s.size());
  for (uint32_t y = 0; y < K; ++y) {
    const uint32_t slot = xor_cols(p.cols, off + p.k, y);
    if (slot >= K) return false;
    for (uint32_t g = 0; g < s.size(); g += K) t[g | y] = s[g | at[slot]];
  }
  s.swap(t);
  // 32 consecutive lanes on 32 banks, both ways (5 thread bits above the registers)
  const int R = p.path == VQC_PATH_RESIDENT ? p.R : p.Rf;
  for (int side = 0; side < 2; ++side) {
    uint32_t seen = 0;
    for (uint32_t l = 0; l < 32; ++l)
      seen |= 1u << (xor_cols(p.cols, off + side * p.k, l << R) & 31u);
    if (seen != 0xffffffffu) return false;
  }
  return true;
}

// Im <l| P |a>, P the Pauli of a rotation: its gradient at the gate's output
double im_pauli(const State& l, const State& a, int op, uint32_t x, uint32_t z) {
  const bool y_kind = op == OP_RY;
  C v = 0;
  for (uint32_t y = 0; y < a.size(); ++y) {
    // P |y> = (-1)^parity(z & y) |y ^ x>, times i for RY (Y = i X Z)
    const C t = std::conj(l[y ^ x]) * a[y];
    v += odd(z & y) ? -t : t;
  }
  return (y_kind ? C(0, 1) * v : v).imag();
}

// grad: per gradient accumulator (LinIns::slot) the sum of its rotations' gradients
bool run(State& a, State* l, const Plan& p, const std::vector<LinIns>& ins, int off, int n_ins,
         const std::vector<double>& th, bool bwd, int R, std::vector<double>* grad = nullptr) {
  for (int i = off; i < off + n_ins; ++i) {
    const LinIns& e = ins[i];
    if (grad && e.op != OP_EXCHANGE && e.slot >= 0) {
      if (e.slot >= (int)grad->size()) return false;
      const double g = im_pauli(*l, a, e.op, e.x, e.z);
      (*grad)[e.slot] += e.neg ? -g : g;
    }
    if (e.op == OP_EXCHANGE) {
      if (!e.lam && !exchange(a, p, e.arg)) return false;
      if (l && !exchange(*l, p, e.arg)) return false;
      continue;
    }
    for (State* s : {&a, l}) {
      if (!s) continue;
      if (e.op != OP_RZ && (e.x == 0 || e.x >> R)) return false;
      if (e.op != OP_RZ && odd(e.z & e.x) != (e.op == OP_RY)) return false;
      rotate(*s, e.op, e.x, e.z, bwd != e.neg ? -th[e.arg] : th[e.arg]);
    }
  }
  return true;
}

// address of physical index y: columns per thread bit, register bit, tile bit
std::vector<uint32_t> addresses(const Plan& p, int off, int R) {
  std::vector<uint32_t> a(1u << p.nq);
  const int t = p.k - R;
  for (uint32_t y = 0; y < a.size(); ++y) {
    uint32_t o = 0;
    for (int b = 0; b < p.nq; ++b)
      if ((y >> b) & 1u) o ^= p.cols[off + (b < R ? t + b : b < p.k ? b - R : b)];
    a[y] = o;
  }
  return a;
}

double diff(const State& a, const State& b) {
  double d = 0;
  for (size_t i = 0; i < a.size(); ++i) d = std::max(d, std::abs(a[i] - b[i]));
  return d;
}

void apply_prim(State& s, const Prim& g, const std::vector<double>& th) {
  if (g.kind == P_CNOT) {
    for (uint32_t y = 0; y < s.size(); ++y)
      if (((y >> g.q0) & 1u) && !((y >> g.q1) & 1u)) std::swap(s[y], s[y | 1u << g.q1]);
  } else if (g.kind == P_CZ) {
    sign_flip(s, 1u << g.q0, 1u << g.q1);
  } else {
    rotate(s, g.kind == P_RX ? OP_RX : g.kind == P_RY ? OP_RY : OP_RZ,
           g.kind == P_RZ ? 0u : 1u << g.q0, g.kind == P_RX ? 0u : 1u << g.q0, th[g.occ]);
  }
}

std::vector<double> expectations(const State& s, const std::vector<uint32_t>& rows) {
  std::vector<double> e;
  for (uint32_t r : rows) {
    double v = 0;
    for (uint32_t y = 0; y < s.size(); ++y) v += odd(r & y) ? -std::norm(s[y]) : std::norm(s[y]);
    e.push_back(v);
  }
  return e;
}

// The measured Z-strings' sum with the cotangent, applied to a state.
State observed(const State& s, const std::vector<uint32_t>& rows, const std::vector<double>& cot) {
  State l(s);
  for (uint32_t y = 0; y < s.size(); ++y) {
    double v = 0;
    for (size_t q = 0; q < rows.size(); ++q) v += odd(rows[q] & y) ? -cot[q] : cot[q];
    l[y] *= v;
  }
  return l;
}

double worst(const std::vector<double>& a, const std::vector<double>& b) {
  double d = a.size() == b.size() ? 0 : 1;
  for (size_t i = 0; i < a.size() && i < b.size(); ++i) d = std::max(d, std::fabs(a[i] - b[i]));
  return d;
}

// The probabilities' way out of the last pass: a tile stores at least 16 consecutive
// floats of a 128-byte line itself (lo: its logical addresses), or they are stored
// at its own addresses (out) and put in order by tiles whose waves read and write
// 64 consecutive floats and hit every LDS bank.
bool probability_stores(const Plan& p, const std::vector<uint32_t>& lo,
                        const std::vector<uint32_t>& out, const State& a, const State& ref) {
  std::map<uint32_t, int> line;
  for (uint32_t y = 0; y < 1u << p.k; ++y) ++line[lo[y] >> 5];
  const ProbOrder& o = p.order;
  if (!o.on) return line.begin()->second >= 16;
  if (line.begin()->second >= 16) return false;
  std::vector<double> raw(a.size()), got(a.size(), -1);
  for (uint32_t y = 0; y < a.size(); ++y) raw[out[y]] = std::norm(a[y]);
  const int K = kOrderBits, R = kOrderRegs;
  for (uint32_t g = 0; g < a.size() >> K; ++g) {
    std::vector<double> lds(1u << K, -1);
    for (int side = 0; side < 2; ++side)
      for (uint32_t y = 0; y < 1u << K; ++y) {
        const uint32_t i = y | g << K;
        const uint32_t at = xor_cols(side ? o.dst_col : o.src_col, 0, i);
        const uint32_t slot = xor_cols(side ? o.rd : o.wr, 0, y);
        if (slot >> K || at >= a.size()) return false;
        if (side) {
          if (got[at] >= 0 || lds[slot] < 0) return false;
          got[at] = lds[slot];
        } else {
          if (lds[slot] >= 0) return false;
          lds[slot] = raw[at];
        }
      }
  }
  for (const auto* c : {&o.src_col, &o.dst_col}) {
    uint32_t all = 0;
    for (int i = 0; i < 6; ++i) all |= (*c)[R + i] == 1u << i ? 1u << i : 0u;
    if (all != 63u) return false;
  }
  for (const auto* c : {&o.wr, &o.rd}) {
    uint32_t banks = 0;
    for (uint32_t l = 0; l < 32; ++l) banks |= 1u << (xor_cols(*c, R, l) & 31u);
    if (banks != ~0u) return false;
  }
  double d = 0;
  for (size_t x = 0; x < got.size(); ++x) d = std::max(d, std::fabs(got[x] - std::norm(ref[x])));
  return d <= 1e-10;
}

// Entanglers before the random gates, which leave the later rotations few or no
// directions along single qubits: every pair in order, the last qubit with all
// others both ways, random CNOTs, SWAPs and CZs; the last three again after a
// layer of rotations (a product head).
enum Prefix { kNone, kPairs, kHub, kNetwork, kHeadHub, kHeadNetwork, kHeadPairs };

void add_prefix(std::vector<HostOp>& ops, int prefix, int n, std::mt19937& rng) {
  auto gate = [&](int kind, int a, int b) {
    HostOp o{};
    o.kind = kind;
    o.w[0] = a;
    o.w[1] = b;
    o.src[0] = VQC_SRC_PARAM;
    o.mul[0] = 1.f;
    ops.push_back(o);
  };
  if (prefix >= kHeadHub)
    for (int q = 0; q < n; ++q) gate(VQC_RY, q, 0);
  if (prefix == kPairs || prefix == kHeadPairs)
    for (int i = 0; i < n; ++i)
      for (int j = i + 1; j < n; ++j) gate(VQC_CNOT, i, j);
  if (prefix == kHub || prefix == kHeadHub) {
    for (int a = 0; a + 1 < n; ++a) gate(VQC_CNOT, n - 1, a);
    for (int a = 0; a + 1 < n; ++a) gate(VQC_CNOT, a, n - 1);
  }
  if (prefix == kNetwork || prefix == kHeadNetwork)
    for (int i = 40 + (int)(rng() % 41u); i > 0; --i) {
      const int a = (int)(rng() % (unsigned)n), b = (a + 1 + (int)(rng() % (unsigned)(n - 1))) % n;
      const int r = (int)(rng() % 10u);
      gate(r < 8 ? VQC_CNOT : r < 9 ? VQC_SWAP : VQC_CZ, a, b);
    }
}

// Every kind of plan of one random circuit: resident (with and without the
// heads' rotations) or streaming (the same).
int check(int n, int seed, int gates, int tile, int rb, int prefix) {
  std::mt19937 rng(seed);
  auto pick = [&](int m) { return (int)(rng() % (unsigned)m); };
  std::vector<HostOp> ops;
  const int P = std::max(gates, 1);
  const int style = seed % 4;  // how many entanglers
  add_prefix(ops, prefix, n, rng);
  for (int i = 0; i < gates; ++i) {
    HostOp o{};
    for (int j = 0; j < 3; ++j) {
      o.src[j] = pick(8) == 0 ? VQC_SRC_CONST : VQC_SRC_PARAM;
      o.idx[j] = pick(P);
      o.val[j] = o.src[j] == VQC_SRC_CONST ? 0.3f : 0.f;
      o.mul[j] = 1.f;
    }
    const int r = pick(10);
    o.kind = style == 3 ? pick(kNumGateKinds)
             : r < 2 + 2 * style ? (pick(4) ? VQC_CNOT : VQC_CZ)
             : r < 8 ? pick(3) : VQC_ROT;
    o.w[0] = pick(n);
    do o.w[1] = pick(n); while (o.w[1] == o.w[0]);
    do o.w[2] = pick(n); while (o.w[2] == o.w[0] || o.w[2] == o.w[1]);
    ops.push_back(o);
  }
  Plan full;
  std::string msg;
  const int path = n >= 14 ? VQC_PATH_STREAM : VQC_PATH_RESIDENT;
  if (build_plan(ops, n, P, 0, path, rb, full, msg, true, tile)) return fail(msg.c_str(), n, seed);
  if (!full.linear) return fail("no linear schedule", n, seed);
  std::vector<double> th(full.occ_src.size());
  for (double& t : th) t = std::uniform_real_distribution<double>(-3, 3)(rng);
  // constant Paulis do not run (the tables' frame carries them): as identities
  // they are absent from both sides here
  for (size_t k = 0; k < th.size(); ++k)
    if (full.occ_src[k] == VQC_SRC_CONST &&
        std::min(std::fabs(full.occ_cs[2 * k]), std::fabs(full.occ_cs[2 * k + 1])) < 1e-15f)
      th[k] = 0;
  for (int step = 0; step < 2; ++step) {
    Plan p = full;
    if (step && path == VQC_PATH_STREAM) {
      const int rc = build_step_plan(full, p, msg);
      if (rc == 1) continue;
      if (rc) return fail(msg.c_str(), n, seed);
    }
    // the state the forward starts from: |0...0>, or the heads' product
    State ref(1u << n);
    ref[0] = 1;
    std::vector<char> in_head(th.size(), 0);
    for (const auto& hq : full.head)
      for (const Prim& g : hq) in_head[g.occ] = 1;
    if (step)
      for (const Prim& g : full.prims)
        if (g.occ >= 0 && in_head[g.occ]) apply_prim(ref, g, th);
    const State begin = ref;
    for (const Prim& g : full.prims)
      if (!(step && g.occ >= 0 && in_head[g.occ])) apply_prim(ref, g, th);
    for (const Prim& g : full.tail) apply_prim(ref, g, th);
    std::vector<uint32_t> bits;
    for (int q = 0; q < n; ++q) bits.push_back(1u << q);
    const std::vector<double> E = expectations(ref, bits);
    // every slot's gradient (unit chain-rule factors), the circuit walked back gate
    // by gate
    std::vector<double> cot, want_g(P, 0), got_g(P, 0);
    for (int q = 0; q < n; ++q) cot.push_back(std::cos(1.0 + 2.0 * q));
    {
      State a = ref, l = observed(ref, bits, cot);
      auto back = [&](const Prim& g) {
        const bool rot = g.kind != P_CNOT && g.kind != P_CZ;
        if (rot && full.occ_slot[g.occ] >= 0)
          want_g[full.occ_slot[g.occ]] += im_pauli(
              l, a, g.kind == P_RX ? OP_RX : g.kind == P_RY ? OP_RY : OP_RZ,
              g.kind == P_RZ ? 0u : 1u << g.q0, g.kind == P_RX ? 0u : 1u << g.q0);
        std::vector<double> inv;
        if (rot) inv.assign(th.size(), -th[g.occ]);
        apply_prim(a, g, inv);
        apply_prim(l, g, inv);
      };
      for (size_t i = full.tail.size(); i-- > 0;) back(full.tail[i]);
      for (size_t i = full.prims.size(); i-- > 0;) {
        const Prim& g = full.prims[i];
        if (!(step && g.occ >= 0 && in_head[g.occ])) back(g);
      }
    }
    auto to_tile = [&](const State& s, int map_off) {  // logical order -> a unit basis
      State t(s.size());
      for (uint32_t x = 0; x < s.size(); ++x) {
        uint32_t y = 0;
        for (int q = 0; q < n; ++q)
          if ((x >> q) & 1u) y |= 1u << p.maps[map_off + q];
        t[y] = s[x];
      }
      return t;
    };
    if (path == VQC_PATH_RESIDENT) {
      const LinSchedule& L = step ? p.lin_step : p.lin;
      State a = to_tile(begin, L.start_off);
      if (!run(a, nullptr, p, L.f, 0, (int)L.f.size(), th, false, p.R))
        return fail("forward instruction", n, seed);
      if (worst(expectations(a, L.zrow), E) > 1e-10) return fail("<Z>", n, seed);
      double d = 0;
      for (uint32_t y = 0; y < a.size(); ++y)
        d = std::max(d, std::fabs(std::norm(a[y]) - std::norm(ref[xor_cols(L.lcol, 0, y)])));
      if (d > 1e-10) return fail("probabilities", n, seed);
      State ag = a, lg = observed(a, L.zrow, cot);
      if (!run(ag, &lg, p, L.b, 0, (int)L.b.size(), th, true, p.R, &got_g))
        return fail("adjoint instruction", n, seed);
      if (worst(got_g, want_g) > 1e-9) return fail("gradients", n, seed);
      State l = a;
      if (!run(a, &l, p, L.b, 0, (int)L.b.size(), th, true, p.R))
        return fail("adjoint instruction", n, seed);
      const State want = step ? to_tile(begin, L.bwd_end_off) : begin;
      if (diff(l, want) > 1e-10 && (step || std::abs(l[0] - begin[0]) > 1e-10))
        return fail("adjoint end", n, seed);
      continue;
    }
    std::vector<State> ck;
    State a;
    for (size_t i = 0; i < p.fpass.size(); ++i) {
      const PassPlan& pp = p.fpass[i];
      if (i == 0) {
        a = to_tile(begin, pp.start_off);
        const std::vector<uint32_t> ad = addresses(p, pp.io_off, p.Rf);
        for (uint32_t y = 0; y < a.size(); ++y)
          if (std::abs(a[y] - begin[ad[y]]) > 0) return fail("start columns", n, seed);
      } else {
        const std::vector<uint32_t> ad = addresses(p, pp.io_off, p.Rf);
        for (uint32_t y = 0; y < a.size(); ++y) a[y] = ck.back()[ad[y]];
      }
      for (int off : {pp.io_off, pp.io_out_off}) {
        uint32_t seen = 0;
        for (int b = 0; b < p.k; ++b) {
          const uint32_t c = p.cols[off + b];
          if (!c || (c & (c - 1u)) || (seen & c)) return fail("local columns", n, seed);
          seen |= c;
        }
      }
      if (!run(a, nullptr, p, p.lin.f, pp.ins_off, pp.n_ins, th, false, p.Rf))
        return fail("forward instruction", n, seed);
      const std::vector<uint32_t> out = addresses(p, pp.io_out_off, p.Rf);
      State m(a.size());
      for (uint32_t y = 0; y < a.size(); ++y) m[out[y]] = a[y];
      ck.push_back(m);
      if (i + 1 == p.fpass.size()) {
        if (worst(expectations(a, p.lin.zrow), E) > 1e-10) return fail("<Z>", n, seed);
        const std::vector<uint32_t> lo = addresses(p, pp.io_lout_off, p.Rf);
        double d = 0;
        for (uint32_t y = 0; y < a.size(); ++y)
          d = std::max(d, std::fabs(std::norm(a[y]) - std::norm(ref[lo[y]])));
        if (d > 1e-10) return fail("probabilities", n, seed);
        if (!probability_stores(p, lo, out, a, ref)) return fail("probability stores", n, seed);
      }
    }
    State lm = ck.back(), gm(lm.size());
    std::vector<char> added(P, 0);
    for (size_t j = 0; j < p.bpass.size(); ++j) {
      const PassPlan& pp = p.bpass[j];
      const size_t i = p.fpass.size() - 1 - j;
      const std::vector<uint32_t> in = addresses(p, pp.io_off, p.Rb);
      State l(a.size());
      for (uint32_t y = 0; y < a.size(); ++y) {
        a[y] = ck[i][in[y]];
        l[y] = lm[in[y]];
      }
      if (j == 0 && worst(expectations(a, p.lin.zrow_b), E) > 1e-10)
        return fail("adjoint <Z> rows", n, seed);
      {
        State ag = a, lg(a.size());
        if (j == 0) lg = observed(a, p.lin.zrow_b, cot);
        else
          for (uint32_t y = 0; y < a.size(); ++y) lg[y] = gm[in[y]];
        std::vector<double> part(pp.n_slots, 0);
        if (!run(ag, &lg, p, p.lin.b, pp.ins_off, pp.n_ins, th, true, p.Rb, &part))
          return fail("adjoint instruction", n, seed);
        for (int i2 = 0; i2 < pp.n_slots; ++i2) {
          const int s = p.pslots[pp.slots_off + i2], slot = s < 0 ? ~s : s;
          // complemented: the first pass to add to the slot, which stores
          if (slot >= P || (s < 0) != !added[slot]) return fail("slot order", n, seed);
          added[slot] = 1;
          got_g[slot] += part[i2];
        }
        if (i > 0) {
          const std::vector<uint32_t> out = addresses(p, pp.io_out_off, p.Rb);
          for (uint32_t y = 0; y < a.size(); ++y) gm[out[y]] = lg[y];
        } else if (worst(got_g, want_g) > 1e-9) {
          return fail("gradients", n, seed);
        }
      }
      if (!run(a, &l, p, p.lin.b, pp.ins_off, pp.n_ins, th, true, p.Rb))
        return fail("adjoint instruction", n, seed);
      if (i > 0) {
        const std::vector<uint32_t> out = addresses(p, pp.io_out_off, p.Rb);
        for (uint32_t y = 0; y < a.size(); ++y) lm[out[y]] = l[y];
        if (diff(lm, ck[i - 1]) > 1e-10) return fail("adjoint pass output", n, seed);
      } else if (step ? diff(l, to_tile(begin, pp.end_off)) > 1e-10
                      : std::abs(l[0] - 1.0) > 1e-10) {
        return fail("adjoint end", n, seed);
      }
    }
    // no more passes, hence saved states, than with the CNOTs as gates
    if (2 * p.fpass.size() > full.gate_passes) return fail("more passes", n, seed);
    std::printf("n=%d seed=%d step=%d passes=%zu\n", n, seed, step, p.fpass.size());
  }
  return 0;
}

}  // namespace

int main(int argc, char** argv) {
  const int n = std::atoi(argv[1]), first = std::atoi(argv[2]), count = std::atoi(argv[3]);
  const int gates = std::atoi(argv[4]), tile = std::atoi(argv[5]), rb = std::atoi(argv[6]);
  const int prefix = argc > 7 ? std::atoi(argv[7]) : kNone;
  for (int s = first; s < first + count; ++s)
    if (check(n, s, gates, tile, rb, prefix)) return 1;
  std::printf("ok\n");
  return 0;
}
