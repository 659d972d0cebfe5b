// linear_plan.h -- schedules of the generated kernels that hold one sample per
// workgroup (part of planner.cpp).
//
// Entanglers as a change of basis.  A CNOT permutes basis states linearly over
// GF(2), so it need not run: the state is kept as if no CNOT had been applied,
// and every later gate is the Pauli rotation that the CNOTs before it turn it
// into.  In these fixed coordinates y in GF(2)^n qubit q's X acts as y -> y ^ v_q
// and its Z reads parity(w_q & y); CNOT(c, t) maps v_c ^= v_t, w_t ^= w_c.  A CZ
// does not run either: it is the sign of a product of two parities, every output
// is diagonal, so it only matters to the later RX and RY, whose Pauli T_x Z_z (T_x
// |y> = |y ^ x>) it takes to T_x Z_z', z' = z ^ (w_b x) w_a ^ (w_a x) w_b, times
// the sign of (w_a x)(w_b x).  A rotation is then a pair (x, z) and a sign: RX and
// RY pair y with y ^ x under the sign of parity(z & y), RZ is diagonal, and two
// gates commute when their symplectic product is even, which lets more gates
// pass a waiting one than disjoint qubits do.  Constant rotations by pi are
// Paulis, which the tangent form's frame carries anyway: they do not run.
//
// A layout of the register tile is any basis of GF(2)^n: physical bit p moves
// along vector b[p].  A gate runs where its x lies in the span of the register
// bits' vectors; an exchange changes the local basis by any invertible map for
// the price of a permutation.  A streaming pass holds a k-dimensional subspace
// and the states between two passes are stored in a basis in which both
// passes' subspaces are spanned by address bits.  Measured on one box against
// the schedules that run the CNOTs: see emit_linear (jit.cpp).

// An echelon basis of a subspace, by leading bit.
struct Span {
  uint32_t row[32];
  int dim = 0;
  Span() { std::memset(row, 0, sizeof row); }
  uint32_t residue(uint32_t v) const {
    for (uint32_t todo = v; todo;) {
      const int b = 31 - __builtin_clz(todo);
      if (row[b]) v ^= row[b];
      todo = b ? v & ((1u << b) - 1u) : 0u;
    }
    return v;
  }
  bool holds(uint32_t v) const { return residue(v) == 0; }
  bool add(uint32_t v) {
    v = residue(v);
    if (!v) return false;
    row[31 - __builtin_clz(v)] = v;
    ++dim;
    return true;
  }
};

uint32_t odd(uint32_t v) { return (uint32_t)__builtin_parity(v); }

// Whether a constant rotation is a Pauli or the identity (up to a phase) to
// the last bit of its (cos, sin) pair.
bool constant_pauli(const Plan& plan, int occ) {
  return plan.occ_src[occ] == VQC_SRC_CONST &&
         std::min(std::fabs(plan.occ_cs[2 * occ]), std::fabs(plan.occ_cs[2 * occ + 1])) < 1e-15f;
}

// Whether the generated kernels' tables are sure to fit in LDS after `base`
// bytes (they then use the tangent form and its frame).
bool tables_fit(const Plan& plan, size_t base) {
  const size_t nocc = plan.occ_src.size();
  return base + nocc / 8 + 2 * nocc * 4 + (size_t)plan.n * 4 + 128 <= (size_t)kLdsBytes;
}

// The circuit's gates (those of `skip` left out), and the rows of every
// measured qubit's Z after the whole circuit, the folded trailing entanglers
// included.  tangent: constant Paulis are left to the frame.
std::vector<LinGate> linear_gates(const Plan& plan, const std::vector<char>* skip,
                                  std::vector<uint32_t>& wfull, bool tangent) {
  uint32_t v[kMaxQubits], w[kMaxQubits];
  for (int q = 0; q < kMaxQubits; ++q) v[q] = w[q] = 1u << q;
  std::vector<LinGate> g;
  std::vector<std::pair<uint32_t, uint32_t>> cz;
  for (const Prim& p : plan.prims) {
    switch (p.kind) {
      case P_CNOT:
        v[p.q0] ^= v[p.q1];
        w[p.q1] ^= w[p.q0];
        break;
      case P_CZ: cz.push_back({w[p.q0], w[p.q1]}); break;
      default: {
        if ((skip && (*skip)[p.occ]) || (tangent && constant_pauli(plan, p.occ))) break;
        LinGate e{p.kind, p.kind == P_RZ ? 0u : v[p.q0], p.kind == P_RX ? 0u : w[p.q0], p.occ, false,
                  p.kind == P_RZ && plan.occ_src[p.occ] != VQC_SRC_CONST};
        for (const auto& c : cz) {
          const uint32_t a = odd(c.first & e.x), b = odd(c.second & e.x);
          e.z ^= (b ? c.first : 0u) ^ (a ? c.second : 0u);
          e.neg ^= (a & b) != 0u;
        }
        g.push_back(e);
      }
    }
  }
  for (const Prim& p : plan.tail)
    if (p.kind == P_CNOT) w[p.q1] ^= w[p.q0];
  wfull.assign(w, w + plan.n);
  return g;
}

// Which gates a scan may take: all; all but the held diagonals; diagonals only.
enum ScanMode { kTakeAll, kTakeEager, kTakeDiagonal };

// occ_slot: at most `cap` gradient slots per streaming pass (its accumulators
// in LDS).
struct ScanLimits {
  int cap = INT_MAX;
  const std::vector<int32_t>* occ_slot = nullptr;
  size_t window = SIZE_MAX;  // gates looked at
};

// Scans over the gates of one list.  Which earlier gates a gate anticommutes with is
// formed once per list, as bits (anti; the angle table in LDS bounds a list to
// kLdsBytes / 8 gates, 52 MB), and what a direction leaves outside a span once per
// span: the many scans that compare candidate directions then cost a few
// instructions per gate.  Planning one circuit on the host, ms, with both formed in
// every scan and this way: 12 qubits strongly entangling of 6 layers 12 -> 4.5, of 100
// layers 300 -> 103; 13-qubit HEA of 6 layers 10 -> 4; 20-qubit ring of 8 layers and
// its step 32 -> 10, 20 qubits strongly entangling of 4 layers 13 -> 5, of 100 layers
// 670 -> 190; 10 qubits with 4000 random gates 570 -> 205.
class Scanner {
 public:
  explicit Scanner(const std::vector<LinGate>& gates)
      : g(gates), words((int)(gates.size() + 63) / 64), res(gates.size()),
        res_of(gates.size(), 0) {
    anti.assign((size_t)words * gates.size(), 0);
    wait.assign(words, 0);
    std::vector<uint64_t> cx((size_t)words * 32, 0), cz((size_t)words * 32, 0);
    for (size_t i = 0; i < gates.size(); ++i) {
      uint64_t* row = anti.data() + i * words;
      const int end = (int)(i / 64) + 1;
      auto add = [&](const std::vector<uint64_t>& c, uint32_t bits) {
        for (; bits; bits &= bits - 1u) {
          const uint64_t* col = c.data() + (size_t)__builtin_ctz(bits) * words;
          for (int w = 0; w < end; ++w) row[w] ^= col[w];
        }
      };
      add(cx, gates[i].z);
      add(cz, gates[i].x);
      const uint64_t bit = 1ull << (i % 64);
      for (uint32_t m = gates[i].x; m; m &= m - 1u)
        cx[(size_t)__builtin_ctz(m) * words + i / 64] |= bit;
      for (uint32_t m = gates[i].z; m; m &= m - 1u)
        cz[(size_t)__builtin_ctz(m) * words + i / 64] |= bit;
    }
  }

  // The span the following scans' gates move in.
  void span(const Span& s) {
    S = s;
    ++span_no;
  }

  // Walks the gates `pos` in order and takes every one that commutes with all
  // gates left waiting before it, may run (mode, slot cap) and moves along a
  // vector of the span, or along `extra` (a residue outside it, 0: none) and one.
  // Returns how many of those taken are not diagonal.  cand: the directions
  // outside the span of gates that nothing else stops, one per coset.
  int scan(const std::vector<int>& pos, uint32_t extra, ScanMode mode, const ScanLimits& cap,
           std::vector<int>* took, std::vector<uint32_t>* cand) {
    constexpr size_t kMaxCand = 16;
    constexpr int kGiveUp = 128;  // gates stopped in a row: those after them stay for a later scan
    const int lo = pos.empty() ? 0 : pos[0] / 64;
    int cleared = lo;  // words [lo, cleared) of wait are this scan's
    int stopped = 0, count = 0, n_slots = 0;
    ++scan_no;
    uint32_t cosets[kMaxCand];
    const size_t end = std::min(pos.size(), cap.window);
    for (size_t j = 0; j < end && stopped < kGiveUp; ++j) {
      const int i = pos[j];
      const LinGate& e = g[i];
      for (; cleared <= i / 64; ++cleared) wait[cleared] = 0;
      const uint64_t* row = anti.data() + (size_t)i * words;
      bool stop = false;
      for (int w = lo; w <= i / 64 && !stop; ++w) stop = (row[w] & wait[w]) != 0;
      if (!stop) stop = mode == kTakeEager ? e.held : mode == kTakeDiagonal ? e.x != 0u : false;
      if (!stop) {
        if (res_of[i] != span_no) {
          res[i] = S.residue(e.x);
          res_of[i] = span_no;
        }
        const uint32_t r = res[i];
        const bool holds = !r || r == extra;
        if (cap.occ_slot && e.occ >= 0) {
          const int s = (*cap.occ_slot)[e.occ];
          if (s >= 0 && !seen(s)) {
            if (n_slots >= cap.cap) {
              stop = true;
            } else if (holds) {
              slot_scan[s] = scan_no;
              ++n_slots;
            }
          }
        }
        if (!stop && holds) {
          stopped = 0;
          if (took) took->push_back(i);
          if (e.x) ++count;
          continue;
        }
        if (!stop && cand && cand->size() < kMaxCand &&
            std::find(cosets, cosets + cand->size(), r) == cosets + cand->size()) {
          cosets[cand->size()] = r;
          cand->push_back(e.x);
        }
      }
      ++stopped;
      wait[i / 64] |= 1ull << (i % 64);
    }
    return count;
  }

  int scan(const std::vector<int>& pos, const Span& s, ScanMode mode, const ScanLimits& cap,
           std::vector<int>* took, std::vector<uint32_t>* cand) {
    span(s);
    return scan(pos, 0u, mode, cap, took, cand);
  }

  const std::vector<LinGate>& g;

 private:
  bool seen(int slot) {
    if ((size_t)slot >= slot_scan.size()) slot_scan.resize((size_t)slot + 1, 0);
    return slot_scan[slot] == scan_no;
  }
  int words;
  std::vector<uint64_t> anti, wait;
  Span S;
  std::vector<uint32_t> res;
  std::vector<unsigned> res_of, slot_scan;
  unsigned span_no = 0, scan_no = 0;
};

// Up to `dims` independent directions that let a scan take the most gates:
// grown one at a time, by the count each candidate gives (ties: the earlier
// gate's), or in circuit order; the better of the two.
std::vector<uint32_t> choose_directions(Scanner& g, const std::vector<int>& pos, int dims,
                                        ScanMode mode, const ScanLimits& cap) {
  std::vector<uint32_t> best;
  int best_count = -1;
  for (int look = 1; look >= 0; --look) {
    Span S;
    std::vector<uint32_t> dirs;
    std::vector<uint32_t> cand;
    while ((int)dirs.size() < dims) {
      cand.clear();
      g.scan(pos, S, mode, cap, nullptr, &cand);
      if (cand.empty()) break;
      size_t pick = 0;
      if (look && cand.size() > 1) {
        int most = -1;
        for (size_t c = 0; c < cand.size(); ++c) {
          const int n = g.scan(pos, S.residue(cand[c]), mode, cap, nullptr, nullptr);
          if (n > most) {
            most = n;
            pick = c;
          }
        }
      }
      S.add(cand[pick]);
      dirs.push_back(cand[pick]);
    }
    const int n = g.scan(pos, S, mode, cap, nullptr, nullptr);
    if (n > best_count) {
      best_count = n;
      best = dirs;
    }
  }
  return best;
}

// The gates of `pos` without those taken (in the order of pos).
void drop_taken(std::vector<int>& pos, const std::vector<int>& took) {
  if (took.empty()) return;
  size_t t = 0, to = 0, at = 0;
  for (; t < took.size(); ++at) {
    if (pos[at] == took[t]) ++t;
    else pos[to++] = pos[at];
  }
  pos.erase(pos.begin() + to, pos.begin() + at);
}

std::vector<int> every_gate(const std::vector<LinGate>& g) {
  std::vector<int> pos(g.size());
  for (size_t i = 0; i < g.size(); ++i) pos[i] = (int)i;
  return pos;
}

// A basis of GF(2)^n: physical bit (or address bit) p moves along b[p].
struct Basis {
  int n = 0;
  uint32_t b[kMaxQubits] = {0};
  uint32_t inv[kMaxQubits] = {0};  // coordinate p of v is parity(inv[p] & v)
  bool invert() {
    uint32_t m[kMaxQubits], id[kMaxQubits];
    for (int i = 0; i < n; ++i) {
      m[i] = 0;
      for (int p = 0; p < n; ++p) m[i] |= ((b[p] >> i) & 1u) << p;
      id[i] = 1u << i;
    }
    for (int p = 0; p < n; ++p) {
      int r = p;
      while (r < n && !((m[r] >> p) & 1u)) ++r;
      if (r == n) return false;
      std::swap(m[r], m[p]);
      std::swap(id[r], id[p]);
      for (int i = 0; i < n; ++i)
        if (i != p && ((m[i] >> p) & 1u)) {
          m[i] ^= m[p];
          id[i] ^= id[p];
        }
    }
    for (int p = 0; p < n; ++p) inv[p] = id[p];
    return true;
  }
  uint32_t coord(uint32_t v) const {
    uint32_t c = 0;
    for (int p = 0; p < n; ++p) c |= odd(inv[p] & v) << p;
    return c;
  }
  uint32_t row(uint32_t z) const {  // parity mask over the bits of a parity of coordinates
    uint32_t m = 0;
    for (int p = 0; p < n; ++p) m |= odd(z & b[p]) << p;
    return m;
  }
  bool same(const Basis& o) const { return std::memcmp(b, o.b, sizeof(uint32_t) * n) == 0; }
  bool unit() const {
    for (int p = 0; p < n; ++p)
      if (b[p] & (b[p] - 1u)) return false;
    return true;
  }
};

// Exchange tables from basis A to basis B of the same k-dimensional local
// space.  The LDS slot of an amplitude is a linear function lam of its
// position; its bank bits are independent on the lane bits' span of A and on
// that of B, so that 32 consecutive lanes hit 32 banks both when writing and
// when reading: on the intersection of the spans the bank bits are shared, and
// each further vector of B's span takes the bank bit of one of A's.  The rest
// of lam numbers the bank bits' kernel.
int emit_linear_exchange(const Basis& A, const Basis& B, int k, int R,
                         std::vector<uint32_t>& cols) {
  const int lb = std::min(kBankBits, k - R);
  // B's vectors in A's coordinates
  uint32_t in_a[kMaxQubits];
  for (int p = 0; p < k; ++p) in_a[p] = A.coord(B.b[p]);
  const uint32_t lanes = ((1u << lb) - 1u) << R;
  // UB = span of in_a[R .. R + lb): vectors reduced outside A's lane bits
  std::vector<std::pair<uint32_t, uint32_t>> out;  // (reduced outside part, vector)
  std::vector<uint32_t> both, rest;                // UB within UA; UB's others
  for (int i = 0; i < lb; ++i) {
    uint32_t v = in_a[R + i], o = v & ~lanes;
    for (const auto& e : out)
      if (o & (e.first & (0u - e.first))) {
        o ^= e.first;
        v ^= e.second;
      }
    if (o) {
      for (auto& e : out)
        if (e.first & (o & (0u - o))) {
          e.first ^= o;
          e.second ^= v;
        }
      out.push_back({o, v});
    } else {
      both.push_back(v);
    }
  }
  for (const auto& e : out) rest.push_back(e.second);
  // a basis of the local space: both | part of UA | rest | others, with lam of each
  Basis full;
  full.n = k;
  uint32_t lam[kMaxQubits] = {0};
  Span s;
  int at = 0, bank = 0, high = lb;
  for (uint32_t v : both) {
    s.add(v);
    lam[at] = 1u << bank++;
    full.b[at++] = v;
  }
  const int shared = bank;
  for (int i = 0; i < lb; ++i)
    if (s.add(1u << (R + i))) {
      lam[at] = 1u << bank++;
      full.b[at++] = 1u << (R + i);
    }
  int j = shared;
  for (uint32_t v : rest)
    if (s.add(v)) {
      lam[at] = 1u << j++ | 1u << high++;
      full.b[at++] = v;
    }
  for (int p = 0; p < k; ++p)
    if (s.add(1u << p)) {
      lam[at] = 1u << high++;
      full.b[at++] = 1u << p;
    }
  full.invert();
  auto slot = [&](uint32_t v) {
    const uint32_t c = full.coord(v);
    uint32_t o = 0;
    for (int p = 0; p < k; ++p)
      if ((c >> p) & 1u) o ^= lam[p];
    return o;
  };
  const int off = (int)cols.size();
  for (int p = 0; p < k; ++p) cols.push_back(slot(1u << p));
  for (int p = 0; p < k; ++p) cols.push_back(slot(in_a[p]));
  // where each physical bit's vector goes (the generated kernels swap register
  // bits with lane bits without LDS); k when it is not a vector of B
  for (int p = 0; p < k; ++p) {
    uint32_t d = (uint32_t)k;
    for (int q = 0; q < k; ++q)
      if (B.b[q] == A.b[p]) d = (uint32_t)q;
    cols.push_back(d);
  }
  return off;
}

// The basis after an exchange that brings `dirs` onto the register bits:
// vectors already on a register bit or a thread bit stay where they can, and
// the register vectors that leave take the thread bits that came free.
Basis exchanged(const Basis& A, const std::vector<uint32_t>& dirs, int k, int R) {
  Span want, used;
  for (uint32_t d : dirs) want.add(d);
  Basis B = A;
  std::vector<char> kept(R, 0);
  int open = R;
  for (int r = 0; r < R; ++r)
    if (want.holds(A.b[r])) {
      used.add(A.b[r]);
      kept[r] = 1;
      --open;
    }
  std::vector<uint32_t> in;
  for (uint32_t d : dirs)
    if (used.add(d)) in.push_back(d);
  for (int r = 0; r < R && (int)in.size() < open; ++r)
    if (!kept[r] && used.add(A.b[r])) {
      kept[r] = 1;
      --open;
    }
  size_t next = 0;
  for (int r = 0; r < R; ++r)
    if (!kept[r]) B.b[r] = in[next++];
  std::vector<int> free_bits;
  for (int p = R; p < k; ++p)
    if (!used.add(A.b[p])) free_bits.push_back(p);
  next = 0;
  for (int r = 0; r < R; ++r)
    if (!kept[r] && used.add(A.b[r])) B.b[free_bits[next++]] = A.b[r];
  B.invert();
  return B;
}

struct LinearSweep {
  std::vector<LinIns> ins;
  std::vector<uint32_t> cols;  // exchange tables, offsets relative to this vector
  int exchanges = 0;
  double cost = 0.0;
  Basis end;
};

void linear_exchange(LinearSweep& s, const Basis& to, int k, int R, bool lam) {
  LinIns e;
  e.op = OP_EXCHANGE;
  e.arg = emit_linear_exchange(s.end, to, k, R, s.cols);
  e.lam = lam;
  s.ins.push_back(e);
  ++s.exchanges;
  s.end = to;
}

// One register-level sweep over the scanner's gates from basis `start`.  Variable RZs
// wait until at least `flush_at` other gates on the present register bits wait for
// them (or nothing else can run): a run of diagonals costs about as much as one of
// them, an exchange more.  The cost is an instruction count per wave:
// per exchange and state the LDS accesses and addresses of 2^R amplitudes, per
// run of diagonals the cheaper of gate by gate and one product.
LinearSweep linear_sweep(Scanner& scanner, const Basis& start, int k, int R, bool bwd,
                         int flush_at) {
  const std::vector<LinGate>& g = scanner.g;
  LinearSweep s;
  s.end = start;
  const double N = 1 << R, states = bwd ? 2.0 : 1.0;
  const ScanLimits none;
  ScanLimits near;  // an exchange runs about ten gates: those close by decide
  near.window = 64;
  std::vector<int> pos = every_gate(g);
  auto emit_gates = [&](const std::vector<int>& took) {
    for (int i : took) {
      const LinGate& e = g[i];
      LinIns n;
      n.op = e.kind == P_RX ? OP_RX : e.kind == P_RY ? OP_RY : OP_RZ;
      n.x = s.end.coord(e.x);
      n.z = s.end.row(e.z);
      n.neg = e.neg;
      n.arg = e.occ;
      s.ins.push_back(n);
    }
    std::vector<int> sorted(took);
    std::sort(sorted.begin(), sorted.end());
    drop_taken(pos, sorted);
  };
  bool fresh = false;  // an exchange and nothing since
  while (!pos.empty()) {
    Span S;
    for (int r = 0; r < R; ++r) S.add(s.end.b[r]);
    std::vector<int> took;
    scanner.scan(pos, S, kTakeEager, none, &took, nullptr);
    if (!took.empty()) {
      emit_gates(took);
      fresh = false;
    }
    if (pos.empty()) break;
    const int ready = scanner.scan(pos, S, kTakeAll, none, nullptr, nullptr);
    std::vector<uint32_t> dirs;
    bool flush = ready >= flush_at || (fresh && ready > 0);
    if (!flush) {
      dirs = choose_directions(scanner, pos, R, flush_at == INT_MAX ? kTakeEager : kTakeAll, near);
      flush = true;
      for (uint32_t d : dirs) flush = flush && S.holds(d);
    }
    if (flush) {
      std::vector<int> diag, fixed, rz;  // (all commute)
      scanner.scan(pos, S, kTakeDiagonal, none, &diag, nullptr);
      if (diag.empty()) {  // only gates off the register bits are left to run
        dirs = choose_directions(scanner, pos, R, kTakeAll, none);
        if (dirs.empty()) break;
      } else {
        int held = 0;
        for (int i : diag) {
          (g[i].held ? rz : fixed).push_back(i);
          if (g[i].held) ++held;
        }
        s.cost += std::min(held * states * (bwd ? 3.0 : 2.0) * N,
                           states * 4 * N + (bwd ? 3 * N : 0.0) + 60 + 3 * held);
        fixed.insert(fixed.end(), rz.begin(), rz.end());
        emit_gates(fixed);
        fresh = false;
        continue;
      }
    }
    const Basis to = exchanged(s.end, dirs, k, R);
    if (to.same(s.end)) break;  // internal failure: best_sweep counts the gates
    linear_exchange(s, to, k, R, false);
    s.cost += states * (6 * N + 30);
    fresh = true;
  }
  return s;
}

// The cheapest of the sweeps over a few thresholds (they differ only where an RZ
// waits); false when a gate never ran.  No threshold wins everywhere (step of 12 qubits, 6 strongly entangling
// layers: 493, 495 and 500 us with 1, 3 and none, 481 us with the choice; 14
// qubits re-uploading: 9.81, 9.61, 9.51 and 9.55 ms).
bool best_sweep(const std::vector<LinGate>& g, const Basis& start, int k, int R, bool bwd,
                LinearSweep& best) {
  best.cost = -1.0;
  Scanner scanner(g);
  const bool held = std::any_of(g.begin(), g.end(), [](const LinGate& e) { return e.held; });
  for (int flush_at : {1, 3, INT_MAX}) {
    if (best.cost >= 0.0 && !held) break;
    LinearSweep s = linear_sweep(scanner, start, k, R, bwd, flush_at);
    size_t gates = 0;
    for (const LinIns& n : s.ins) gates += n.op != OP_EXCHANGE;
    if (gates != g.size()) return false;
    if (best.cost < 0.0 || s.cost < best.cost) best = std::move(s);
  }
  return true;
}

// Appends a sweep's instructions (and its exchange tables) to a schedule.
template <typename SlotFn>
void append_sweep(const LinearSweep& s, std::vector<LinIns>& out, std::vector<uint32_t>& cols,
                  SlotFn slot_of) {
  const int base = (int)cols.size();
  cols.insert(cols.end(), s.cols.begin(), s.cols.end());
  for (LinIns n : s.ins) {
    if (n.op == OP_EXCHANGE) n.arg += base;
    else n.slot = slot_of(n.arg);
    out.push_back(n);
  }
}

int append_basis_map(const Basis& B, std::vector<uint8_t>& maps) {
  const int off = (int)maps.size();
  for (int q = 0; q < B.n; ++q) {
    uint8_t at = 0;
    for (int p = 0; p < B.n; ++p)
      if (B.b[p] == 1u << q) at = (uint8_t)p;
    maps.push_back(at);
  }
  return off;
}

// Logical directions (one qubit each) for the register bits of a sweep's start:
// those that let the first scan take the most gates; ties and the rest by first
// use, `allowed` the qubits to choose from.
std::vector<uint32_t> start_qubits(const std::vector<LinGate>& g, int nq, int R, uint32_t allowed) {
  const std::vector<int> pos = every_gate(g);
  std::vector<int> first(nq, INT_MAX);
  for (size_t i = 0; i < g.size(); ++i)
    for (int q = 0; q < nq; ++q)
      if (((g[i].x >> q) & 1u) && first[q] == INT_MAX) first[q] = (int)i;
  Scanner scanner(g);
  const ScanLimits none;
  Span S;
  std::vector<uint32_t> dirs;
  uint32_t used = 0;
  while ((int)dirs.size() < R) {
    int best = -1, most = -1;
    scanner.span(S);
    for (int q = 0; q < nq; ++q) {
      if (!((allowed >> q) & 1u) || ((used >> q) & 1u)) continue;
      const int n = scanner.scan(pos, S.residue(1u << q), kTakeAll, none, nullptr, nullptr);
      if (n > most || (n == most && first[q] < first[best])) {
        most = n;
        best = q;
      }
    }
    used |= 1u << best;
    S.add(1u << best);
    dirs.push_back(1u << best);
  }
  return dirs;
}

// A unit basis near B: units stay, other bits take the qubits left over.
Basis unit_basis(const Basis& B, int k) {
  Basis U = B;
  uint32_t have = 0;
  for (int p = 0; p < B.n; ++p)
    if (!(B.b[p] & (B.b[p] - 1u))) have |= B.b[p];
  uint32_t space = 0;
  for (int p = 0; p < k; ++p) space |= B.b[p];
  for (int p = 0; p < k; ++p)
    if (B.b[p] & (B.b[p] - 1u)) {
      const uint32_t left = space & ~have;
      U.b[p] = left & (0u - left);
      have |= U.b[p];
    }
  U.invert();
  return U;
}

// Both sweeps of a resident circuit (the gates of `skip` left out: the product
// head, whose adjoint ends in a unit basis).
int plan_linear_resident(Plan& plan, const std::vector<char>* skip, LinSchedule& out,
                         std::string& msg) {
  const int nq = plan.nq, k = plan.k, R = plan.R;
  std::vector<uint32_t> wfull;
  const std::vector<LinGate> g =
      linear_gates(plan, skip, wfull, tables_fit(plan, std::max(plan.lds_step, plan.lds_bwd)));
  Basis start;
  start.n = nq;
  const std::vector<uint32_t> regs = start_qubits(g, nq, R, (1u << nq) - 1u);
  uint32_t used = 0;
  for (int r = 0; r < R; ++r) used |= start.b[r] = regs[r];
  int p = R;
  for (int q = 0; q < nq; ++q)
    if (!((used >> q) & 1u)) start.b[p++] = 1u << q;
  start.invert();
  LinearSweep f, b;
  const std::vector<LinGate> rev(g.rbegin(), g.rend());
  if (!best_sweep(g, start, k, R, false, f) || !best_sweep(rev, f.end, k, R, true, b)) {
    msg = "internal: a gate was not scheduled";
    return VQC_ERR_UNSUPPORTED;
  }
  if (skip && !b.end.unit()) linear_exchange(b, unit_basis(b.end, k), k, R, true);
  auto slot_of = [&](int occ) { return plan.occ_slot[occ]; };
  append_sweep(f, out.f, plan.cols, slot_of);
  append_sweep(b, out.b, plan.cols, slot_of);
  out.start_off = append_basis_map(start, plan.maps);
  out.bwd_end_off = append_basis_map(b.end, plan.maps);
  for (int q = 0; q < plan.n; ++q) out.zrow.push_back(f.end.row(wfull[q]));
  for (int i = 0; i < k; ++i) {
    uint32_t c = 0;
    for (int q = 0; q < plan.n; ++q) c |= odd(wfull[q] & f.end.b[i]) << q;
    out.lcol.push_back(c);
  }
  return 0;
}

// ---------------------------------------------------------------- streaming
// Pass partition: the first pass's local space is spanned by k qubits (it
// starts from |0...0>, a product state or a caller's state in logical order),
// found by dropping one qubit at a time; every later pass grows its space
// along the directions that let it run the most gates.  Rotations after a CNOT
// ring need no qubit of the ring on chip but their own direction, so that a
// pass runs two to three layers of a 16-qubit ring circuit on 12 dimensions
// (5 passes per direction instead of the 10 that run the CNOTs as gates).
bool partition_linear(const std::vector<LinGate>& all, int nq, int k, const ScanLimits& cap,
                      std::vector<LinearPass>& passes) {
  std::vector<int> pos = every_gate(all);
  Scanner scanner(all);
  do {
    LinearPass lp;
    Span S;
    if (passes.empty()) {
      std::vector<int> first(nq, INT_MAX);
      for (size_t i = 0; i < all.size(); ++i)
        for (int q = 0; q < nq; ++q)
          if (((all[i].x >> q) & 1u) && first[q] == INT_MAX) first[q] = (int)i;
      uint32_t in = (1u << nq) - 1u;
      auto span_of = [&](uint32_t m) {
        Span s;
        for (int q = 0; q < nq; ++q)
          if ((m >> q) & 1u) s.add(1u << q);
        return s;
      };
      for (int drop = 0; drop < nq - k; ++drop) {
        int best = -1, most = -1;
        for (int q = 0; q < nq; ++q) {
          if (!((in >> q) & 1u)) continue;
          const int n = scanner.scan(pos, span_of(in & ~(1u << q)), kTakeAll, cap, nullptr,
                                     nullptr);
          if (n > most || (n == most && first[q] >= first[best])) {
            most = n;
            best = q;
          }
        }
        in &= ~(1u << best);
      }
      S = span_of(in);
      for (int q = 0; q < nq; ++q)
        if ((in >> q) & 1u) lp.V.push_back(1u << q);
    } else {
      for (uint32_t d : choose_directions(scanner, pos, k, kTakeAll, cap))
        if (S.add(d)) lp.V.push_back(d);
      for (uint32_t v : passes.back().V)  // shared with the pass before: longer runs of addresses
        if (S.dim < k && S.add(v)) lp.V.push_back(v);
      for (int q = 0; q < nq && S.dim < k; ++q)
        if (S.add(1u << q)) lp.V.push_back(1u << q);
    }
    std::vector<int> took;
    scanner.scan(pos, S, kTakeAll, cap, &took, nullptr);
    if (took.empty() && !pos.empty() && !passes.empty()) return false;
    for (int i : took) lp.g.push_back(all[i]);
    drop_taken(pos, took);
    passes.push_back(std::move(lp));
  } while (!pos.empty());
  return true;
}

// The passes of the schedule that runs the CNOTs as gates, as linear passes: each
// one's local space is spanned by its local qubits' directions at its start, in
// which it runs at least the same gates.  Rarely these are fewer than the greedy
// ones, and a training call keeps a state per pass: the fewer are taken, so that no
// call needs more workspace than with the CNOTs as gates.  A group that runs no
// rotation needs no pass: its CNOTs are in v.  But the first pass starts in
// logical order, in a local space spanned by qubits, so when the first that runs
// rotations has another one the first group stays as a pass of no gates.  False
// when the slot cap leaves gates over or there is no gate.
bool partition_like_gates(const Plan& plan, const std::vector<LinGate>& all, const ScanLimits& cap,
                          std::vector<LinearPass>& passes) {
  std::vector<StreamGroup> groups;
  std::string msg;
  if (partition_stream(plan.prims, plan.nq, plan.ng, groups, msg) < 0) return false;
  uint32_t v[kMaxQubits];
  for (int q = 0; q < kMaxQubits; ++q) v[q] = 1u << q;
  std::vector<int> pos = every_gate(all);
  Scanner scanner(all);
  for (const StreamGroup& grp : groups) {
    LinearPass lp;
    Span S;
    uint32_t qubits = 0;
    for (int q = 0; q < plan.nq; ++q)
      if (!((grp.glob >> q) & 1u) && S.add(v[q])) {
        lp.V.push_back(v[q]);
        qubits |= v[q];
      }
    std::vector<int> took;
    scanner.scan(pos, S, kTakeAll, cap, &took, nullptr);
    for (int i : took) lp.g.push_back(all[i]);
    drop_taken(pos, took);
    if (!took.empty()) {
      if (passes.empty() && __builtin_popcount(qubits) != plan.k) {
        LinearPass start;
        for (int q = 0; q < plan.nq; ++q)
          if (!((groups[0].glob >> q) & 1u)) start.V.push_back(1u << q);
        passes.push_back(std::move(start));
      }
      passes.push_back(std::move(lp));
    }
    for (const Prim& p : grp.prims)
      if (p.kind == P_CNOT) v[p.q0] ^= v[p.q1];
  }
  return pos.empty() && !passes.empty();
}

// The memory layout between a pass with local space V and one with local space
// W: a basis over the address bits in which both are spanned by address bits.
// Their intersection takes the low bits (consecutive lanes then touch
// consecutive addresses on both sides), and where it can be the directions the
// passes want on their register bits there (dV, dW) are basis vectors.
Basis boundary_basis(const std::vector<uint32_t>& V, const std::vector<uint32_t>& W,
                     const std::vector<uint32_t>& dV, const std::vector<uint32_t>& dW, int nq) {
  Span sV;
  for (uint32_t v : V) sV.add(v);
  std::vector<uint32_t> inter;
  {
    std::vector<std::pair<uint32_t, uint32_t>> rows;  // (residue mod V, vector of W)
    for (uint32_t w : W) {
      uint32_t r = sV.residue(w), c = w;
      for (const auto& e : rows)
        if (r & (1u << (31 - __builtin_clz(e.first)))) {
          r ^= e.first;
          c ^= e.second;
        }
      if (!r) inter.push_back(c);
      else {
        rows.push_back({r, c});
        std::sort(rows.begin(), rows.end(),
                  [](const std::pair<uint32_t, uint32_t>& a,
                     const std::pair<uint32_t, uint32_t>& b) { return a.first > b.first; });
      }
    }
  }
  Span sI;
  for (uint32_t v : inter) sI.add(v);
  // extensions of the intersection to V and to W, the wanted directions first
  Span low;  // wanted directions (or what they leave) inside the intersection
  std::vector<uint32_t> low_want;
  auto extend = [&](const std::vector<uint32_t>& space, const std::vector<uint32_t>& want) {
    Span t = sI;
    std::vector<uint32_t> ext;
    for (uint32_t d : want) {
      if (t.add(d)) {
        ext.push_back(d);
        continue;
      }
      for (uint32_t s = 0; s < (1u << ext.size()); ++s) {
        uint32_t c = d;
        for (size_t j = 0; j < ext.size(); ++j)
          if ((s >> j) & 1u) c ^= ext[j];
        if (sI.holds(c)) {
          if (low.add(c)) low_want.push_back(c);
          break;
        }
      }
    }
    for (uint32_t v : space)
      if (t.add(v)) ext.push_back(v);
    return ext;
  };
  const std::vector<uint32_t> extV = extend(V, dV), extW = extend(W, dW);
  Basis M;
  M.n = nq;
  int at = 0;
  Span s = low;
  for (uint32_t v : inter)
    if (s.add(v)) M.b[at++] = v;
  for (uint32_t v : low_want) M.b[at++] = v;
  Span all;
  for (int i = 0; i < at; ++i) all.add(M.b[i]);
  auto put = [&](uint32_t v) {
    if (at < nq && all.add(v)) M.b[at++] = v;
  };
  for (uint32_t v : extV) put(v);
  for (uint32_t v : extW) put(v);
  for (int q = 0; q < nq; ++q) put(1u << q);
  M.invert();
  return M;
}

// A pass's tile basis at a boundary: its register bits get the wanted
// directions that are vectors of the layout M (then its highest address bits),
// its thread bits the other local vectors by ascending address, and the tile
// index the qubits that complete its space.
bool tile_basis(const Basis& M, const std::vector<uint32_t>& V, const std::vector<uint32_t>& want,
                int k, int R, Basis& B) {
  Span s;
  for (uint32_t v : V) s.add(v);
  std::vector<uint32_t> local;
  for (int a = 0; a < M.n; ++a)
    if (s.holds(M.b[a])) local.push_back(M.b[a]);
  if ((int)local.size() != k) return false;
  std::vector<uint32_t> regs;
  for (uint32_t d : want)
    if ((int)regs.size() < R && std::find(regs.begin(), regs.end(), d) == regs.end() &&
        std::find(local.begin(), local.end(), d) != local.end())
      regs.push_back(d);
  for (size_t i = local.size(); i-- > 0 && (int)regs.size() < R;)
    if (std::find(regs.begin(), regs.end(), local[i]) == regs.end()) regs.push_back(local[i]);
  B = Basis();
  B.n = M.n;
  int at = 0;
  for (uint32_t v : regs) B.b[at++] = v;
  for (uint32_t v : local)
    if (std::find(regs.begin(), regs.end(), v) == regs.end()) B.b[at++] = v;
  for (int q = 0; q < M.n; ++q)
    if (s.add(1u << q)) B.b[at++] = 1u << q;
  return at == M.n && B.invert();
}

// The k + ng address columns of a tile in basis B under layout M: thread bits,
// register bits, then the tile index bits.  The local columns are single bits
// (M is a basis of the local space); a tile index bit's may be any.
void push_linear_io(const Basis& B, const Basis& M, int k, int R, std::vector<uint32_t>& cols) {
  for (int p = R; p < k; ++p) cols.push_back(M.coord(B.b[p]));
  for (int p = 0; p < R; ++p) cols.push_back(M.coord(B.b[p]));
  for (int p = k; p < B.n; ++p) cols.push_back(M.coord(B.b[p]));
}

// The probabilities' way into logical order from the last pass's layout M: its
// address bits' images (rows of the measured Z-strings) give the destination.  A
// tile of the last pass covers the 128-byte lines of the destination in runs of
// 2^c floats, c of the 5 lowest bits; from c = 4 on the pass stores them itself,
// below they go through order_kernel, where the times on both sides stand, in calls
// large enough to repay its launch (about 3 us): from 2^20 amplitudes, at c = 3 from
// 2^23.  Time that they add, us, stored by the pass and ordered: c = 0, 2^20 9.0, 7.6;
// c = 1, 2^21 13.5, 9.9; c = 2, 2^17.6 5.3, 5.4 and 2^20 9.3, 7.1; c = 3, 2^22 5.1, 6.7
// (20 qubits) and 21, 13 (14 qubits), 2^25 102, 92 and 140, 62.
bool order_probs(const Basis& M, const std::vector<uint32_t>& wfull, const std::vector<uint32_t>& V,
                 ProbOrder& out) {
  constexpr int kLineBits = 5, k = kOrderBits, R = kOrderRegs;
  Basis img;  // the image of each address bit
  img.n = M.n;
  for (int a = 0; a < M.n; ++a)
    for (int q = 0; q < M.n; ++q) img.b[a] |= odd(wfull[q] & M.b[a]) << q;
  if (!img.invert()) return false;
  auto image = [&](uint32_t v) {
    uint32_t o = 0;
    for (int q = 0; q < M.n; ++q) o |= odd(wfull[q] & v) << q;
    return o;
  };
  Span lines;
  for (uint32_t v : V) lines.add(image(v) >> kLineBits);
  const int c = (int)V.size() - lines.dim;
  out = ProbOrder();
  if (c >= 4) return true;
  out.from = int64_t(1) << (c < 3 ? 20 : 23);
  // in address coordinates: 64 consecutive addresses, the directions of 64
  // consecutive destinations, further addresses up to a tile's dimension
  Basis A, B;
  A.n = B.n = M.n;
  Span s;
  std::vector<uint32_t> local;
  auto take = [&](uint32_t v) {
    if ((int)local.size() < k && s.add(v)) local.push_back(v);
  };
  for (int i = 0; i < 6; ++i) take(1u << i);
  for (int i = 0; i < 6; ++i) take(img.coord(1u << i));
  for (int a = 6; a < M.n; ++a) take(1u << a);
  auto place = [&](Basis& T, const std::vector<uint32_t>& v) {  // v: its lanes first
    for (int i = 0; i < k; ++i) T.b[i < k - R ? R + i : i - (k - R)] = v[i];
  };
  place(A, local);
  std::vector<uint32_t> lanes;
  Span t;
  for (int i = 0; i < 6; ++i)
    if (t.add(img.coord(1u << i))) lanes.push_back(img.coord(1u << i));
  for (uint32_t v : local)
    if (t.add(v)) lanes.push_back(v);
  place(B, lanes);
  int at = k;
  for (int a = 0; a < M.n; ++a)
    if (s.add(1u << a)) {
      A.b[at] = B.b[at] = 1u << a;
      ++at;
    }
  if (at != M.n || !A.invert() || !B.invert()) return false;
  std::vector<uint32_t> cols;
  emit_linear_exchange(A, B, k, R, cols);
  out.wr.assign(cols.begin(), cols.begin() + k);
  out.rd.assign(cols.begin() + k, cols.begin() + 2 * k);
  for (int p = 0; p < M.n; ++p) {
    uint32_t d = 0;
    for (int a = 0; a < M.n; ++a)
      if ((B.b[p] >> a) & 1u) d ^= img.b[a];
    out.src_col.push_back(A.b[p]);
    out.dst_col.push_back(d);
  }
  out.on = true;
  return true;
}

// A streaming circuit's gates (the table kernel holds all entries, a pass at most
// the slots' accumulators).
std::vector<LinGate> stream_gates(const Plan& plan, std::vector<uint32_t>& wfull) {
  const size_t acc = (size_t)plan.slot_cap * ((1u << (plan.k - plan.Rb)) / 64u) * 4;
  return linear_gates(plan, nullptr, wfull,
                      tables_fit(plan, plan.occ_src.size() * 8) &&
                          tables_fit(plan, plan.lds_fwd + acc + 16));
}

int plan_linear_stream(Plan& plan, std::string& msg) {
  const int nq = plan.nq, k = plan.k;
  std::vector<uint32_t> wfull;
  const std::vector<LinGate> all = stream_gates(plan, wfull);
  const ScanLimits cap{plan.slot_cap, &plan.occ_slot};
  std::vector<LinearPass> ps;
  auto internal = [&](const char* what) {
    msg = std::string("internal: ") + what;
    return VQC_ERR_UNSUPPORTED;
  };
  ps.swap(plan.parts);  // from the choice of the tile size
  if (ps.empty() && !partition_linear(all, nq, k, cap, ps))
    return internal("streaming pass made no progress");
  if (2 * ps.size() + 4 > plan.gate_passes) {  // not clearly fewer
    std::vector<LinearPass> like;
    if (partition_like_gates(plan, all, cap, like) && like.size() < ps.size()) ps.swap(like);
  }
  const size_t nf = ps.size();
  plan.cols.clear();
  plan.maps.clear();
  plan.pslots.clear();
  plan.fpass.clear();
  plan.bpass.clear();
  plan.max_pass_slots = 0;
  plan.lin = LinSchedule();
  std::set<int32_t> seen_f, seen_b;  // slots of the passes before
  auto finish = [&](PassPlan& pp, const LinearSweep& s, std::vector<LinIns>& out, const Basis& in,
                    const Basis& in_layout, const Basis& out_layout) {
    std::map<int, int> local_slot;
    std::vector<int32_t> slots;
    std::set<int32_t>& before = &out == &plan.lin.f ? seen_f : seen_b;
    auto slot_of = [&](int occ) -> int {
      const int sl = plan.occ_slot[occ];
      if (sl < 0) return -1;
      auto it = local_slot.find(sl);
      if (it != local_slot.end()) return it->second;
      local_slot[sl] = (int)slots.size();
      // complemented: no earlier pass adds to the slot
      slots.push_back(before.insert(sl).second ? ~sl : sl);
      return (int)slots.size() - 1;
    };
    const int R = &out == &plan.lin.f ? plan.Rf : plan.Rb;
    pp.ins_off = (int)out.size();
    append_sweep(s, out, plan.cols, slot_of);
    pp.n_ins = (int)out.size() - pp.ins_off;
    pp.start_off = append_basis_map(in, plan.maps);
    pp.end_off = append_basis_map(s.end, plan.maps);
    pp.io_off = pp.io_lin_off = (int)plan.cols.size();
    push_linear_io(in, in_layout, k, R, plan.cols);
    pp.io_out_off = (int)plan.cols.size();
    push_linear_io(s.end, out_layout, k, R, plan.cols);
    pp.io_lout_off = (int)plan.cols.size();
    for (int i = 0; i < nq; ++i) {
      const int p = i < k - R ? R + i : i < k ? i - (k - R) : i;
      uint32_t c = 0;
      for (int q = 0; q < plan.n; ++q) c |= odd(wfull[q] & s.end.b[p]) << q;
      plan.cols.push_back(c);
    }
    pp.slots_off = (int)plan.pslots.size();
    pp.n_slots = (int)slots.size();
    plan.pslots.insert(plan.pslots.end(), slots.begin(), slots.end());
    plan.max_pass_slots = std::max(plan.max_pass_slots, pp.n_slots);
  };
  const ScanLimits none;
  auto first_directions = [&](const std::vector<LinGate>& g, int R) {
    Scanner scanner(g);
    return choose_directions(scanner, every_gate(g), R, kTakeAll, none);
  };
  // layout[i]: what pass i reads; layout[i + 1]: what it writes
  std::vector<Basis> layout(nf + 1), starts(nf), stores(nf);
  layout[0].n = nq;
  for (int q = 0; q < nq; ++q) layout[0].b[q] = 1u << q;
  layout[0].invert();
  uint32_t space0 = 0;
  for (uint32_t v : ps[0].V) space0 |= v;
  std::vector<uint32_t> want = start_qubits(ps[0].g, nq, plan.Rf, space0);
  std::vector<std::vector<uint32_t>> want_in(nf), want_out(nf);
  for (size_t i = 0; i < nf; ++i) {
    want_in[i] = want;
    if (!tile_basis(layout[i], ps[i].V, want, k, plan.Rf, starts[i]))
      return internal("tile basis");
    LinearSweep s;
    if (!best_sweep(ps[i].g, starts[i], k, plan.Rf, false, s))
      return internal("a gate was not scheduled");
    const std::vector<uint32_t> last(s.end.b, s.end.b + plan.Rf);
    want_out[i] = last;
    if (i + 1 < nf) {
      want = first_directions(ps[i + 1].g, plan.Rf);
      layout[i + 1] = boundary_basis(ps[i].V, ps[i + 1].V, last, want, nq);
      if (!tile_basis(layout[i + 1], ps[i].V, last, k, plan.Rf, stores[i]))
        return internal("tile basis");
      if (!stores[i].same(s.end)) linear_exchange(s, stores[i], k, plan.Rf, false);
    } else {
      // only its own mirror reads the last output: any basis of its space does
      layout[nf].n = nq;
      int at = 0;
      for (int p = plan.Rf; p < k; ++p) layout[nf].b[at++] = s.end.b[p];
      for (int p = 0; p < plan.Rf; ++p) layout[nf].b[at++] = s.end.b[p];
      for (int p = k; p < nq; ++p) layout[nf].b[at++] = s.end.b[p];
      layout[nf].invert();
      stores[i] = s.end;
      for (int q = 0; q < plan.n; ++q) plan.lin.zrow.push_back(s.end.row(wfull[q]));
      if (!order_probs(layout[nf], wfull, ps[i].V, plan.order))
        return internal("order of the probabilities");
    }
    PassPlan pp;
    if (i == 0) pp.flags |= PF_INIT;
    if (i + 1 == nf) pp.flags |= PF_ZPART;
    finish(pp, s, plan.lin.f, starts[i], layout[i], layout[i + 1]);
    plan.fpass.push_back(pp);
  }
  // the adjoint: each pass mirrored, from the layout its forward pass wrote to
  // the one it read
  for (size_t j = 0; j < nf; ++j) {
    const size_t i = nf - 1 - j;
    Basis in;
    if (!tile_basis(layout[i + 1], ps[i].V, want_out[i], k, plan.Rb, in))
      return internal("tile basis");
    if (j == 0)
      for (int q = 0; q < plan.n; ++q) plan.lin.zrow_b.push_back(in.row(wfull[q]));
    const std::vector<LinGate> rev(ps[i].g.rbegin(), ps[i].g.rend());
    LinearSweep s;
    if (!best_sweep(rev, in, k, plan.Rb, true, s)) return internal("a gate was not scheduled");
    if (i > 0 || plan.product_head) {
      Basis to;
      if (!tile_basis(layout[i], ps[i].V, want_in[i], k, plan.Rb, to))
        return internal("tile basis");
      if (!to.same(s.end) && (i > 0 || !s.end.unit()))
        linear_exchange(s, to, k, plan.Rb, true);
    }
    PassPlan pp;
    if (j == 0) pp.flags |= PF_MAKE_LAMBDA;
    if (i == 0) pp.flags |= PF_LAST_ADJ;
    finish(pp, s, plan.lin.b, in, layout[i + 1], i > 0 ? layout[i] : layout[0]);
    plan.bpass.push_back(pp);
  }
  return 0;
}
