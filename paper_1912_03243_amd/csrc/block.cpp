// Planning of register-resident tile programs (block_ops.hpp): the circuit's
// gates rewritten as rotations and phases, and every tile pass turned into
// stages of register, lane and wave bits with their ops.  Pure C++.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <exception>
#include <system_error>
#include <thread>

#include "absorb.hpp"
#include "juqcs_internal.hpp"

namespace juqcs {

namespace {

using R = BlkReal;
using C = cplx<R>;

C widen(cplx<double> a) { return C{a.re, a.im}; }
C mul(C a, C b) { return C{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }
// a *= b, where b is 1 most of the time
void join(C* a, const C& b) {
  if (b.re != 1 || b.im != 0) *a = mul(*a, b);
}
// (the exponents of the wider type leave room for the squares)
R norm2(C a) { return a.re * a.re + a.im * a.im; }
// a conj(b) f
C times(C a, C b, R f) { return C{(a.re * b.re + a.im * b.im) * f, (a.im * b.re - a.re * b.im) * f}; }
C div(C a, C b) { return times(a, b, 1 / norm2(b)); }
bool zero(C a) { return a.re == 0 && a.im == 0; }
// Equal up to what an FP64 value of that size cannot tell apart.
bool equal(C a, R re) { return std::fabs(a.re - re) <= 0x1p-58L && std::fabs(a.im) <= 0x1p-58L; }
bool one(C a) { return equal(a, 1); }
bool minus_one(C a) { return equal(a, -1); }
// Neither a nor 1 / a comes near FP64's range.
bool ranged(C a) {
  const R m = std::max(std::fabs(a.re), std::fabs(a.im));
  return m >= 1e-300 && m <= 1e300;
}

// Collects the single-qubit gates of each qubit until a gate that does not
// commute with them, then emits them as one gate.
struct Rewriter {
  R tol;
  bool keep;  // phases of 1 too, so that the gates' kinds do not depend on their values
  std::vector<BlkGate>* out;
  struct Open {
    bool any = false;
    double share = 0.5;  // of the norm, in the set half, as far as is known
    C m[4];
  };
  std::vector<Open> open;

  void single(int q, const cplx<double>* u) {
    Open& w = open[q];
    if (!w.any) {
      w.any = true;
      for (int i = 0; i < 4; ++i) w.m[i] = widen(u[i]);
      return;
    }
    if (zero(w.m[1]) && zero(w.m[2])) {  // a diagonal that an earlier gate left
      const C x = w.m[0], y = w.m[3];
      for (int i = 0; i < 4; ++i) {
        const C z = widen(u[i]);
        w.m[i] = i & 1 ? mul(z, y) : x.re == 1 && x.im == 0 ? z : mul(z, x);
      }
      return;
    }
    C r[4];
    for (int i = 0; i < 2; ++i)
      for (int j = 0; j < 2; ++j) {
        const C x = mul(widen(u[2 * i]), w.m[j]), y = mul(widen(u[2 * i + 1]), w.m[2 + j]);
        r[2 * i + j] = C{x.re + y.re, x.im + y.im};
      }
    for (int i = 0; i < 4; ++i) w.m[i] = r[i];
  }

  void push_phase(int q, C lam, C ph) {
    if (!keep && one(ph) && one(lam)) return;
    BlkGate g;
    g.kind = BlkGate::PHASE1;
    g.q[0] = q;
    g.ph = ph;
    g.lam = lam;
    out->push_back(g);
  }

  // The rotation form needs b c / (a d) real and negative (t^2 is its size).
  // Turns the entries until it is, the small ones most: by angles in
  // proportion to 1 / |entry|^2, the least change of the matrix (n2: |a|^2,
  // |b|^2, ..).  False where an entry would change by more than the root of
  // miss2.  (A pair of zeros has the form.)
  static bool fit(C* m, const R* n2, R miss2) {
    if ((zero(m[1]) && zero(m[2])) || (zero(m[0]) && zero(m[3]))) return true;
    const C ad = mul(m[0], m[3]), bc = mul(m[1], m[2]);
    const R re = -(bc.re * ad.re + bc.im * ad.im), im = bc.re * ad.im - bc.im * ad.re;
    if (!(re > 0)) return false;
    if (im == 0) return true;
    // weights 1 / n2, over their sum, without a division each
    const R ad2 = n2[0] * n2[3], bc2 = n2[1] * n2[2];
    const R w[4] = {n2[3] * bc2, n2[2] * ad2, n2[1] * ad2, n2[0] * bc2};
    const R off = im / (re * (w[0] + w[1] + w[2] + w[3]));
    for (int i = 0; i < 4; ++i)
      if (!(off * off * w[i] * w[i] * n2[i] <= miss2)) return false;
    for (int i = 0; i < 4; ++i) {
      const R turn = i == 0 || i == 3 ? off * w[i] : -off * w[i];
      m[i] = C{m[i].re - turn * m[i].im, m[i].im + turn * m[i].re};
    }
    return true;
  }

  // Emits what is open on qubit q.  all = false: a diagonal may stay open
  // (the next gate on q commutes with diagonals).
  void flush(int q, bool all) {
    Open& w = open[q];
    if (!w.any) return;
    C m[4] = {w.m[0], w.m[1], w.m[2], w.m[3]};
    R n2[4];
    for (int i = 0; i < 4; ++i) n2[i] = norm2(m[i]);
    const R miss2 = tol * tol * std::max(std::max(n2[0], n2[1]), std::max(n2[2], n2[3]));
    if (zero(m[1]) && zero(m[2])) {
      if (!all) return;
      w.any = false;
      const C ph = zero(m[0]) ? C{0, 0} : div(m[3], m[0]);
      if (ranged(m[0]) && ranged(ph)) push_phase(q, m[0], ph);
      else dense(q, w.m);
      return;
    }
    // diag(lam, mu) R diag(1, p) with R = [[1, -t], [t, 1]] (|a d| >= |b c|) or
    // [[t, -1], [1, t]]
    BlkGate g;
    g.kind = BlkGate::ROT;
    g.q[0] = q;
    const R ad2 = n2[0] * n2[3], bc2 = n2[1] * n2[2];
    g.formb = bc2 > ad2;
    if (fit(m, n2, miss2)) {
      // (one division for two quotients: they are slow in this type)
      C rest;
      if (!g.formb) {  // mu = c / t, p = d / mu, rest = mu / a
        g.t = std::sqrt(std::sqrt(bc2 / ad2));
        g.lam = m[0];
        const R ta2 = g.t * norm2(m[0]), c2 = norm2(m[2]), f = 1 / (ta2 * c2);
        g.ph = times(m[3], m[2], g.t * ta2 * f);
        rest = times(m[2], m[0], c2 * f);
      } else if (zero(m[0])) {
        g.lam = m[2];
        g.ph = times(C{-m[1].re, -m[1].im}, m[2], 1 / norm2(m[2]));
        rest = C{1, 0};
      } else {  // lam = a / t, p = -b / lam, rest = c / lam
        g.t = std::sqrt(std::sqrt(ad2 / bc2));
        const R a2 = norm2(m[0]), f = 1 / (g.t * a2), h = g.t * g.t * f;
        g.lam = C{m[0].re * a2 * f, m[0].im * a2 * f};
        g.ph = times(C{-m[1].re, -m[1].im}, m[0], h);
        rest = times(m[2], m[0], h);
      }
      if (ranged(g.lam) && ranged(g.ph) && ranged(rest)) {
        g.share = w.share;
        w.share = moved(w.share, n2);
        out->push_back(g);
        w.m[0] = C{1, 0};
        w.m[1] = w.m[2] = C{0, 0};
        w.m[3] = rest;
        w.any = keep || !one(rest);
        if (all && w.any) {
          w.any = false;
          push_phase(q, C{1, 0}, rest);
        }
        return;
      }
    }
    w.any = false;
    w.share = moved(w.share, n2);
    dense(q, w.m);
  }

  // The share after a matrix with entries of sizes squared n2: a column's where
  // the qubit was in |0> or |1>.  (Gates that are diagonal on the qubit keep it,
  // so the second rotation finds this share whatever has entangled the qubit.)
  static double moved(double share, const R* n2) {
    if (share != 0.0 && share != 1.0) return 0.5;
    const R a = n2[share == 0.0 ? 0 : 1], b = n2[share == 0.0 ? 2 : 3];
    return a + b > 0 ? (double)(b / (a + b)) : 0.5;
  }

  void dense(int q, const C* m) {
    BlkGate g;
    g.kind = BlkGate::DENSE;
    g.q[0] = q;
    for (int i = 0; i < 4; ++i) g.m[i] = m[i];
    out->push_back(g);
  }
};

}  // namespace

bool block_gates(int n, const std::vector<Gate>& gates, double tol, std::vector<BlkGate>* out, bool keep,
                 const std::vector<int>* order, const uint64_t* basis) {
  const size_t count = order ? order->size() : gates.size();
  out->clear();
  out->reserve(count + n);
  Rewriter rw;
  rw.tol = tol;
  rw.keep = keep;
  rw.out = out;
  rw.open.resize(n);
  if (basis)
    for (int q = 0; q < n; ++q) rw.open[q].share = (double)((*basis >> q) & 1);
  for (size_t k = 0; k < count; ++k) {
    const Gate& g = gates[order ? (*order)[k] : k];
    if (g.nq == 1) {
      rw.single(g.q[0], g.m);
      continue;
    }
    const cplx<double>* m = g.m;  // index b_q0 + 2 b_q1
    const auto zero = [](cplx<double> a) { return a.re == 0.0 && a.im == 0.0; };
    const auto one = [](cplx<double> a) { return a.re == 1.0 && a.im == 0.0; };
    BlkGate b;
    b.q[0] = g.q[0];
    b.q[1] = g.q[1];
    bool diag = one(m[0]) && one(m[5]) && one(m[10]), cnot = one(m[0]) && one(m[10]) && one(m[7]) && one(m[13]);
    for (int i = 0; i < 16; ++i) {
      if (i != 0 && i != 5 && i != 10 && i != 15 && !zero(m[i])) diag = false;
      if (i != 0 && i != 10 && i != 7 && i != 13 && !zero(m[i])) cnot = false;
    }
    if (diag && ranged(widen(m[15]))) {
      b.kind = BlkGate::CPHASE;
      b.ph = widen(m[15]);
      rw.flush(b.q[0], false);
      rw.flush(b.q[1], false);
    } else if (cnot) {
      b.kind = BlkGate::CNOT;
      rw.flush(b.q[0], false);
      rw.flush(b.q[1], true);
      const double c = rw.open[b.q[0]].share;
      double& t = rw.open[b.q[1]].share;
      t = c == 0.0 ? t : c == 1.0 ? 1.0 - t : 0.5;
    } else {
      bool swap = one(m[0]) && one(m[6]) && one(m[9]) && one(m[15]);
      for (int i = 0; i < 16; ++i)
        if (i != 0 && i != 6 && i != 9 && i != 15 && !zero(m[i])) swap = false;
      if (!swap) return false;
      rw.flush(b.q[0], true);
      rw.flush(b.q[1], true);
      std::swap(rw.open[b.q[0]].share, rw.open[b.q[1]].share);
      b.kind = BlkGate::CNOT;
      out->push_back(b);
      std::swap(b.q[0], b.q[1]);
      out->push_back(b);
      std::swap(b.q[0], b.q[1]);
    }
    out->push_back(b);
  }
  for (int q = 0; q < n; ++q) rw.flush(q, true);
  return true;
}

uint64_t block_shape(const std::vector<BlkGate>& gates) {
  uint64_t h = 1469598103934665603ull;
  for (const BlkGate& g : gates) {
    const uint64_t v = (uint64_t)g.kind | (uint64_t)(uint8_t)g.q[0] << 8 | (uint64_t)(uint8_t)g.q[1] << 16 |
                       (uint64_t)g.formb << 24 | (uint64_t)one(g.ph) << 25 | (uint64_t)minus_one(g.ph) << 26 |
                       (uint64_t)one(g.lam) << 27;
    h = (h ^ v) * 1099511628211ull;
    h ^= h >> 29;
  }
  return h;
}

namespace {

// A gate of one pass on tile-local bits (q < 64) or, for controls and
// controlled phases, bits of the tile number (q - 64).
struct Local {
  const BlkGate* g;
  int q[2];
};

bool outside(int q) { return q >= 64; }
uint32_t bit(int q) { return outside(q) ? 0u : 1u << q; }

bool moves(const Local& l) { return l.g->kind != BlkGate::PHASE1 && l.g->kind != BlkGate::CPHASE; }

// Gates (in order) that a stage with register bits P can apply: every target
// a register bit, at least one bit of a controlled phase, and no earlier
// gate left behind that does not commute.  Diagonal gates and controls
// commute with each other.
AbsorbMask stage_mask(const Local& l) {
  AbsorbMask m;
  const uint32_t a = bit(l.q[0]);
  switch (l.g->kind) {
    case BlkGate::ROT:
    case BlkGate::DENSE:
      m.full = a;
      break;
    case BlkGate::PHASE1:
      m.diag = a;
      break;
    case BlkGate::CPHASE:
      m.diag = a | bit(l.q[1]);
      break;
    default:  // CNOT
      m.full = bit(l.q[1]);
      m.diag = a;
  }
  m.weight = moves(l) ? 4 : 1;
  return m;
}


// The gates of a pass that no stage has taken, in order: those of left, then all
// from next on.  A stage looks at few of them, its register bits are blocked
// soon; bits that gates rarely act on are not, so it stops after kWindow in a
// row that it does not take.  Planning takes time in proportion to the gates
// then (50,000 mixed gates on one tile 40 ms; 4.5 s when every stage went
// through all).
struct Rest {
  static constexpr size_t kWindow = 512;
  std::vector<AbsorbMask> masks;  // of every gate of the pass
  // from each gate on: bits with a non-diagonal gate, those of CNOT targets, and
  // the bits that gates act on other than diagonally
  std::vector<uint32_t> nondiag, target, full;
  std::vector<int> left;
  size_t next = 0;
  uint64_t weight = 0;
  explicit Rest(const std::vector<Local>& gs)
      : masks(gs.size()), nondiag(gs.size() + 1), target(gs.size() + 1), full(gs.size() + 1) {
    for (size_t i = gs.size(); i-- > 0;) {
      const Local& l = gs[i];
      const bool cnot = l.g->kind == BlkGate::CNOT;
      masks[i] = stage_mask(l);
      nondiag[i] = nondiag[i + 1] | (moves(l) ? bit(l.q[cnot ? 1 : 0]) : 0u);
      target[i] = target[i + 1] | (cnot ? bit(l.q[1]) : 0u);
      full[i] = full[i + 1] | (uint32_t)masks[i].full;
      weight += masks[i].weight;
    }
  }
  bool empty() const { return left.empty() && next == masks.size(); }
  // Goes on to the gates from next on for as long as one of kWindow in a row is
  // taken; those before the last one taken that are not go to keep.
  template <typename Take>
  void go_on(Take take, std::vector<int>* keep) {
    for (size_t i = next; i < masks.size() && i - next <= kWindow; ++i) {
      const int t = take((int)i);  // 1: taken; -1: no gate from here on can be
      if (t < 0) return;
      if (t == 0) continue;
      while (next < i) keep->push_back((int)next++);
      ++next;
    }
  }
};

// Controlled phases with one register bit that no later gate of the stage
// takes over are left for a stage where one does, if there is one: there
// they cost a sign per thread, here a sweep over half of the registers.
// later: bits with a non-diagonal gate after those of keep.
void leave_for_later(const std::vector<Local>& gs, uint32_t P, uint32_t later, std::vector<int>* take,
                     std::vector<int>* keep) {
  for (int i : *keep)
    if (moves(gs[i])) later |= bit(gs[i].q[gs[i].g->kind == BlkGate::CNOT ? 1 : 0]);
  uint32_t now = 0;    // register bits with a rotation further on in this stage
  std::vector<int> stay, left;
  for (size_t k = take->size(); k-- > 0;) {
    const Local& l = gs[(*take)[k]];
    const uint32_t t = moves(l) ? bit(l.q[l.g->kind == BlkGate::CNOT ? 1 : 0]) : 0u;
    now |= t;
    const uint32_t m = bit(l.q[0]) | bit(l.q[1] < 0 ? 64 : l.q[1]);
    const bool single = l.g->kind == BlkGate::CPHASE && (m & P & ((m & P) - 1)) == 0;
    (single && !(m & now) && (m & later) ? left : stay).push_back((*take)[k]);
  }
  if (stay.empty()) return;
  take->assign(stay.rbegin(), stay.rend());
  keep->insert(keep->end(), left.begin(), left.end());
  std::sort(keep->begin(), keep->end());
}

// Register bits for the next stage: greedily the bit that lets the most
// through, among the bits of allowed (at least K of them), besides those of
// fixed.  got: what they let through.
uint32_t pick_regs(const std::vector<AbsorbMask>& left, const Rest& rest, int tb, int K, uint32_t allowed,
                   uint64_t* got, uint32_t fixed = 0) {
  uint32_t P = fixed;
  AbsorbSearch search(left, rest.masks.data() + rest.next, rest.masks.size() - rest.next, P,
                      Rest::kWindow);
  for (int k = __builtin_popcount(fixed); k < K; ++k) {
    uint64_t sets[32], w[32];
    int which[32], count = 0;
    for (int b = 0; b < tb; ++b)
      if (((allowed & ~P) >> b) & 1) {
        which[count] = b;
        sets[count++] = P | 1u << b;
      }
    search.weights(sets, count, w);
    P |= 1u << which[std::max_element(w, w + count) - w];
    search.grow(P);
  }
  *got = search.taken();
  return P;
}

enum EKind { E_ROT, E_DENSE, E_SWAP, E_PHASE, E_PAIR, E_NEG, E_SIGNS, E_SCALE };

struct EOp {  // an op of a stage before it is put into layers
  EKind kind = E_ROT;
  int J = 0;            // ROT, DENSE, SWAP, NEG: register bit
  uint32_t cm = 0;      // SWAP, PHASE, PAIR, SIGNS: register bits
  uint32_t tmask = 0;   // tile-local bits (thread bits of the stage)
  uint64_t gmask = 0;
  C ph{1, 0};
  R t = 0;
  std::vector<C> m;     // DENSE: the matrix
  C lam{1, 0};
  double share = 0.5;   // ROT: of the norm, in the set half
  struct Col {          // phase where an outer bit is set
    C ph;
    int q;
  };
  std::vector<Col> col;
  bool plain() const { return !tmask && !gmask && col.empty(); }
};

struct StagePlan {
  uint32_t regs = 0;
  std::vector<std::pair<int, int>> lin;  // CNOTs (control, target) done by the exchange before the stage
  C scal{1, 0};  // scalar factors of the stage's gates that no op carries
  std::vector<EOp> ops;
  int reg[8], thr[kBlkThrBits];
};

// What a pass carries from stage to stage per tile bit: whether the bit is
// stored complemented, and a phase of its (stored) set half still to apply.
struct Frame {
  uint32_t flip = 0;
  C pend[32];
  C outer[64];  // the same for bits of the tile number
  Frame() {
    for (C& z : pend) z = C{1, 0};
    for (C& z : outer) z = C{1, 0};
  }
  bool flipped(int q) const { return !outside(q) && ((flip >> q) & 1); }
};

// CNOTs that no later gate of the stage waits for are left to the exchange
// that follows: there they only change the addresses.
void leave_cnots(const std::vector<Local>& gs, std::vector<int>* take, std::vector<int>* keep) {
  uint32_t any = 0, full = 0;  // bits that later gates of the stage act on (full: not diagonally)
  std::vector<int> stay, left;
  for (size_t k = take->size(); k-- > 0;) {
    const int i = (*take)[k];
    const Local& l = gs[i];
    const uint32_t a = bit(l.q[0]), b = l.q[1] < 0 ? 0u : bit(l.q[1]);
    if (l.g->kind == BlkGate::CNOT) {
      if (!outside(l.q[0]) && !(b & any) && !(a & full)) {
        left.push_back(i);
        continue;
      }
      full |= b;
    } else if (moves(l)) {
      full |= a;
    }
    any |= a | b;
    stay.push_back(i);
  }
  take->assign(stay.rbegin(), stay.rend());
  keep->insert(keep->end(), left.begin(), left.end());
  std::sort(keep->begin(), keep->end());
}

// Takes the CNOTs between tile bits that no gate left behind comes before.
void take_linear(const std::vector<Local>& gs, Frame& fr, Rest* rest, std::vector<std::pair<int, int>>* lin) {
  uint32_t any = 0, full = 0;
  std::vector<int> keep;
  const auto take = [&](int i) {
    const Local& l = gs[i];
    const uint32_t a = bit(l.q[0]), b = l.q[1] < 0 ? 0u : bit(l.q[1]);
    if (l.g->kind == BlkGate::CNOT && !outside(l.q[0]) && !(b & any) && !(a & full) && one(fr.pend[l.q[1]])) {
      lin->push_back({l.q[0], l.q[1]});
      if (fr.flipped(l.q[0])) fr.flip ^= b;  // a flipped control also flips the target
      rest->weight -= rest->masks[i].weight;
      return true;
    }
    any |= a | b;
    if (l.g->kind == BlkGate::CNOT) full |= b;
    else if (moves(l)) full |= a;
    return false;
  };
  for (int i : rest->left)
    if (!take(i)) keep.push_back(i);
  rest->go_on([&](int i) { return !(rest->target[i] & ~any) ? -1 : take(i) ? 1 : 0; }, &keep);
  rest->left.swap(keep);
}

// Emits the ops of a stage for its gates in order.
struct Emitter {
  const std::vector<Local>& gs;
  Frame& fr;
  StagePlan& st;
  int K;
  int jof_[64];
  // what waits for each register bit's next op, on the stored set half: a
  // phase, sign masks, and phases that depend on an outer bit
  struct Wait {
    C ph{1, 0};
    uint32_t tmask = 0;
    uint64_t gmask = 0;
    std::vector<EOp::Col> col;
    bool outer() const { return tmask || gmask || !col.empty(); }
  };
  std::vector<Wait> wait;

  Emitter(const std::vector<Local>& g, Frame& f, StagePlan& s, int k) : gs(g), fr(f), st(s), K(k), wait(k) {
    for (int& j : jof_) j = -1;
    for (int j = 0; j < K; ++j) {
      jof_[s.reg[j]] = j;
      wait[j].ph = f.pend[s.reg[j]];
      f.pend[s.reg[j]] = C{1, 0};
    }
  }
  int jof(int q) const { return outside(q) ? -1 : jof_[q]; }

  void take_wait(EOp& e, int j) {
    Wait& w = wait[j];
    join(&e.ph, w.ph);
    e.tmask = w.tmask;
    e.gmask = w.gmask;
    e.col = std::move(w.col);
    w = Wait();
  }
  void settle(int j) {  // applies what waits for j now
    Wait& w = wait[j];
    if (!w.outer() && one(w.ph)) return;
    EOp e;
    e.J = j;
    e.kind = w.col.empty() && one(w.ph) ? E_NEG : E_ROT;  // a phase alone: t = 0
    take_wait(e, j);
    st.ops.push_back(std::move(e));
  }
  // phase of the set half of bit q (as stored)
  void phase_on(int q, C p) {
    const int j = jof(q);
    if (outside(q)) fr.outer[q - 64] = mul(fr.outer[q - 64], p);
    else if (j >= 0) wait[j].ph = mul(wait[j].ph, p);
    else fr.pend[q] = mul(fr.pend[q], p);
  }

  void gate(const Local& l) {
    const BlkGate& g = *l.g;
    const int q0 = l.q[0], q1 = l.q[1], j = jof(q0);
    const bool f0 = fr.flipped(q0);
    const auto inv = [](C p) { return div(C{1, 0}, p); };
    EOp e;
    e.J = j;
    switch (g.kind) {
      case BlkGate::ROT:
        // on a flipped bit diag(1, p) is p diag(1, 1 / p) and t changes sign;
        // the second form is [[1, t], [-t, 1]] after a flip
        e.kind = E_ROT;
        e.lam = g.lam;
        e.ph = f0 ? inv(g.ph) : g.ph;
        e.share = f0 ? 1.0 - g.share : g.share;
        e.t = f0 ? -g.t : g.t;
        if (f0) e.lam = mul(e.lam, g.ph);
        if (g.formb) {
          e.ph = C{-e.ph.re, -e.ph.im};
          if (f0) e.lam = C{-e.lam.re, -e.lam.im};
          fr.flip ^= 1u << q0;
        }
        take_wait(e, j);
        st.ops.push_back(std::move(e));
        break;
      case BlkGate::DENSE: {
        if (wait[j].outer()) settle(j);
        const C p = wait[j].ph;  // a plain phase joins the matrix's second column
        wait[j] = Wait();
        e.kind = E_DENSE;
        if (f0) e.m = {g.m[3], mul(g.m[2], p), g.m[1], mul(g.m[0], p)};
        else e.m = {g.m[0], mul(g.m[1], p), g.m[2], mul(g.m[3], p)};
        st.ops.push_back(std::move(e));
        break;
      }
      case BlkGate::PHASE1:
        st.scal = mul(st.scal, g.lam);
        if (f0) st.scal = mul(st.scal, g.ph);
        phase_on(q0, f0 ? inv(g.ph) : g.ph);
        break;
      case BlkGate::CPHASE: {
        // phi (f0 + s0 b0) (f1 + s1 b1) with f = 1, s = -1 on a flipped bit
        const bool f1 = fr.flipped(q1);
        const C p = g.ph, ip = f0 || f1 ? inv(p) : p;
        if (f0 && f1) st.scal = mul(st.scal, p);
        if (f0) phase_on(q1, f1 ? ip : p);
        if (f1) phase_on(q0, f0 ? ip : p);
        const C pp = f0 != f1 ? ip : p;
        const bool neg = minus_one(pp);
        const int j1 = jof(q1);
        if (j >= 0 && j1 >= 0) {
          e.kind = neg ? E_PAIR : E_PHASE;
          e.cm = (1u << j) | (1u << j1);
          if (!neg) e.ph = pp;
          st.ops.push_back(std::move(e));
          break;
        }
        const int other = j >= 0 ? q1 : q0;
        Wait& w = wait[j >= 0 ? j : j1];
        if (!neg) w.col.push_back({pp, other});
        else if (outside(other)) w.gmask ^= uint64_t(1) << (other - 64);
        else w.tmask ^= 1u << other;
        break;
      }
      default: {  // CNOT; a flipped control also flips the target
        const int jt = jof(q1);
        settle(jt);
        e.kind = E_SWAP;
        e.J = jt;
        if (j >= 0) e.cm = 1u << j;
        else if (outside(q0)) e.gmask = uint64_t(1) << (q0 - 64);
        else e.tmask = 1u << q0;
        st.ops.push_back(std::move(e));
        if (f0) fr.flip ^= 1u << q1;
        break;
      }
    }
  }

  void finish() {
    for (int j = 0; j < K; ++j) {
      if (!wait[j].outer()) {  // a plain phase can wait for a later stage
        fr.pend[st.reg[j]] = wait[j].ph;
        wait[j].ph = C{1, 0};
      }
      settle(j);
    }
  }
};

// Applies the phases that a pass's stages left pending, at its end.
void settle_frame(Frame& fr, StagePlan& st, int tb, int K) {
  EOp s;
  s.kind = E_SIGNS;
  std::vector<EOp> rest;
  for (int b = 0; b < tb; ++b) {
    const C p = fr.pend[b];
    if (one(p)) continue;
    int j = -1;
    for (int i = 0; i < K; ++i)
      if (st.reg[i] == b) j = i;
    if (minus_one(p)) {
      if (j >= 0) s.cm |= 1u << j;
      else s.tmask |= 1u << b;
    } else {
      EOp e;
      e.kind = j >= 0 ? E_ROT : E_PHASE;
      if (j >= 0) {
        e.J = j;
        e.ph = p;
      } else {
        e.col.push_back({p, b});
      }
      // phases of thread bits share one op
      if (j < 0 && !rest.empty() && rest.back().kind == E_PHASE) rest.back().col.push_back({p, b});
      else rest.push_back(std::move(e));
    }
  }
  EOp outer;
  outer.kind = E_PHASE;
  for (int b = 0; b < 64; ++b) {
    const C p = fr.outer[b];
    if (one(p)) continue;
    if (minus_one(p)) s.gmask |= uint64_t(1) << b;
    else outer.col.push_back({p, 64 + b});
  }
  if (!outer.col.empty()) rest.push_back(std::move(outer));
  if (s.cm || s.tmask || s.gmask) st.ops.push_back(std::move(s));
  for (EOp& e : rest) st.ops.push_back(std::move(e));
}

R rounded(R x, bool fp64) { return fp64 ? (R)(double)x : (R)(float)(double)x; }

// Rounds the phases and tangents of the ops to the state's precision.  What the
// rounding multiplies a half (or quarter) of the state by is divided out of the
// whole on average, with the scalars of the pass: left to itself, each rounding
// changes the norm and turns that part of the state.  (The first rotations after
// a basis state find other shares of it in that half, which the gates tell.)
void round_phases(std::vector<StagePlan>& st, bool fp64) {
  for (StagePlan& s : st)
    for (EOp& e : s.ops) {
      const auto phase = [&](C* p, double share) {
        const C r{rounded(p->re, fp64), rounded(p->im, fp64)};
        const double x = (double)(p->re - r.re), y = (double)(p->im - r.im);  // far below r: to first order
        const double u = (double)r.re, v = (double)r.im, f = share / (u * u + v * v);
        if ((x == 0.0 && y == 0.0) || !std::isfinite(f)) return;
        e.lam = mul(e.lam, C{1 + (R)((x * u + y * v) * f), (R)((y * u - x * v) * f)});
        *p = r;
      };
      if (e.kind != E_ROT && e.kind != E_PHASE) continue;
      const double share = e.kind == E_ROT ? e.share : 1.0 / (1 << __builtin_popcount(e.cm));
      phase(&e.ph, share);
      for (EOp::Col& c : e.col) phase(&c.ph, share / 2);
      if (e.kind == E_ROT) {
        const R t = rounded(e.t, fp64);
        if (t != e.t) {
          const double u = (double)t;
          const R f = 1 + (R)((double)(e.t - t) * u / (1.0 + u * u));
          e.lam = C{e.lam.re * f, e.lam.im * f};
          e.t = t;
        }
      }
    }
}

// Scalar parts of the pass's gates: their product goes into the matrix of a
// rotation without outer signs or phases, as a dense 2x2, or (none there) into
// an op of its own.  On the way it is kept within 2^+-20 of what the registers
// hold (a rotation [[1, -t], [t, 1]] enlarges them by up to sqrt(2)); where
// every rotation has outer signs or phases, an op of its own does that from
// 2^+-24 on: a scalar left over a pass of 300 such rotations would round to
// zero in FP32.
void place_scalars(std::vector<StagePlan>& st) {
  C run{1, 0};
  int at_stage = -1, at_op = 0;  // the last op that can carry a scalar
  auto carry = [](EOp* e, C s) {
    if (e->kind == E_SCALE) {
      e->ph = mul(e->ph, s);
    } else if (e->kind == E_ROT) {
      e->kind = E_DENSE;
      e->m = {s, mul(s, C{-e->t * e->ph.re, -e->t * e->ph.im}), C{s.re * e->t, s.im * e->t}, mul(s, e->ph)};
    } else {
      for (C& z : e->m) z = mul(s, z);
    }
  };
  for (size_t i = 0; i < st.size(); ++i) {
    std::vector<EOp>& ops = st[i].ops;
    join(&run, st[i].scal);
    for (size_t k = 0; k < ops.size(); ++k) {
      join(&run, ops[k].lam);
      const double a = (double)norm2(run);
      if ((ops[k].kind == E_ROT && ops[k].plain()) || ops[k].kind == E_DENSE) {
        at_stage = (int)i;
        at_op = (int)k;
        if (a <= 0x1p40 && a >= 0x1p-40) continue;
        carry(&ops[k], run);
      } else {
        if (a <= 0x1p48 && a >= 0x1p-48) continue;
        EOp e;
        e.kind = E_SCALE;
        e.ph = run;
        ops.insert(ops.begin() + (std::ptrdiff_t)++k, std::move(e));
        at_stage = (int)i;
        at_op = (int)k;
      }
      run = C{1, 0};
    }
  }
  if (one(run)) return;
  if (at_stage < 0) {
    EOp e;
    e.kind = E_SCALE;
    at_stage = (int)st.size() - 1;
    at_op = (int)st.back().ops.size();
    st.back().ops.push_back(std::move(e));
  }
  carry(&st[at_stage].ops[at_op], run);
}

// Puts a stage's ops into layers and appends them to the plan as device
// stages: misc ops, then an even number of layers (sign changes, then one
// rotation per register bit at most); misc ops in between start another
// device stage of the same layout.
void emit_layers(const StagePlan& p, int nthr, BlkStage base, BlkPlan* plan) {
  const auto tmask_of = [&](uint32_t m) {
    uint32_t t = 0;
    for (int i = 0; i < nthr; ++i)
      if ((m >> p.thr[i]) & 1) t |= 1u << i;
    return t;
  };
  struct Layer {
    BlkLayer<double> y{};
    BlkMore more{};
    std::vector<const EOp*> misc;
    std::vector<EOp::Col> col[kBlkRegs];
    uint32_t sgn = 0;  // register bits in a sign change
  };
  const auto push_op = [&](uint32_t kind, uint32_t tm, uint64_t gm, const double* c, int n) {
    BlkOp o{};
    o.kind = kind;
    o.tmask = tm;
    o.gmask = gm;
    plan->ops.push_back(o);
    for (int i = 0; i < 8; ++i) plan->ocoef.push_back(i < n ? c[i] : 0.0);
    return (int)plan->ops.size() - 1;
  };
  const auto push_cols = [&](const std::vector<EOp::Col>& col, int32_t* c0, int32_t* c1) {
    *c0 = (int32_t)plan->ops.size();
    for (const EOp::Col& c : col) {
      const double v[2] = {(double)c.ph.re, (double)c.ph.im};
      push_op(0, outside(c.q) ? 0u : tmask_of(1u << c.q), outside(c.q) ? uint64_t(1) << (c.q - 64) : 0, v, 2);
    }
    *c1 = (int32_t)plan->ops.size();
  };
  const auto start = [&](Layer& cur) {  // misc ops of a device stage
    std::vector<std::pair<int32_t, int32_t>> cols;
    for (const EOp* e : cur.misc) {
      std::pair<int32_t, int32_t> c{0, 0};
      if (!e->col.empty()) push_cols(e->col, &c.first, &c.second);
      cols.push_back(c);
    }
    base.misc_begin = (int32_t)plan->ops.size();
    for (size_t i = 0; i < cur.misc.size(); ++i) {
      const EOp& e = *cur.misc[i];
      double c[8] = {(double)e.ph.re, (double)e.ph.im, 0, 0, 0, 0, 0, 0};
      uint32_t kind = 0;
      int lo = 0, hi = 0;  // register control bits
      if (e.cm) {
        lo = __builtin_ctz(e.cm);
        hi = 31 - __builtin_clz(e.cm);
      }
      if (e.kind == E_DENSE) {
        kind = blk_dense(e.J);
        for (int k = 0; k < 4; ++k) c[2 * k] = (double)e.m[k].re, c[2 * k + 1] = (double)e.m[k].im;
      } else if (e.kind == E_SWAP) {
        kind = blk_swap(e.J, e.cm ? lo : e.J);
      } else if (e.kind == E_SIGNS) {
        kind = blk_signs(e.cm);
      } else {
        kind = e.cm ? blk_phase(lo, hi) : blk_phase();
      }
      const int o = push_op(kind, tmask_of(e.tmask), e.gmask, c, 8);
      plan->ops[o].col_begin = cols[i].first;
      plan->ops[o].col_end = cols[i].second;
    }
    base.misc_end = (int32_t)plan->ops.size();
    base.layer_begin = (int32_t)plan->layers.size();
  };
  const auto push_layer = [&](Layer& cur) {
    for (int j = 0; j < kBlkRegs; ++j)
      if (!cur.col[j].empty()) push_cols(cur.col[j], &cur.more.col_begin[j], &cur.more.col_end[j]);
    plan->layers.push_back(cur.y);
    plan->more.push_back(cur.more);
  };
  const auto finish = [&]() {
    if ((plan->layers.size() - base.layer_begin) % 2) {
      plan->layers.push_back(BlkLayer<double>{});
      plan->more.push_back(BlkMore{});
    }
    base.layer_end = (int32_t)plan->layers.size();
    plan->stages.push_back(base);
    base.exchange = BLK_STAY;
  };
  // every op goes to the first layer that it may: level[j] is the first one
  // whose rotation of bit j comes after everything placed on j so far
  std::vector<Layer> ly;
  int level[kBlkRegs] = {};
  const auto at = [&](int l) -> Layer& {
    if ((int)ly.size() <= l) ly.resize(l + 1);
    return ly[l];
  };
  const auto masks = [&](Layer& y, const EOp& e) {
    y.y.tmask[e.J] = tmask_of(e.tmask);
    y.more.gmask[e.J] = e.gmask;
    if (e.gmask) y.y.flags |= BLK_GMASK << e.J;
  };
  for (const EOp& e : p.ops) {
    const uint32_t jb = 1u << e.J;
    const uint32_t u = e.kind == E_ROT || e.kind == E_NEG || e.kind == E_DENSE ? jb
                       : e.kind == E_SWAP ? jb | e.cm
                       : e.kind == E_SCALE ? (1u << kBlkRegs) - 1 : e.cm;
    int l = 0;
    for (int j = 0; j < kBlkRegs; ++j)
      if ((u >> j) & 1) l = std::max(l, level[j]);
    // misc ops run first in their layer: not after a sign change on their bits
    const bool moves = e.kind == E_DENSE || e.kind == E_SWAP;
    if (moves && (int)ly.size() > l && (ly[l].sgn & u)) ++l;
    if (e.kind == E_NEG && (int)ly.size() > l && (ly[l].y.flags & (BLK_NEG << e.J))) ++l;
    if (e.kind == E_ROT && (int)ly.size() > l && (ly[l].y.flags & (BLK_NEG << e.J))) ++l;
    Layer& y = at(l);
    switch (e.kind) {
      case E_ROT:
        y.y.flags |= BLK_ROT << e.J;
        if (e.tmask || e.gmask) {
          y.y.flags |= BLK_OUTER << e.J;
          masks(y, e);
        }
        if (!e.col.empty()) {
          y.y.flags |= (BLK_OUTER | BLK_COL) << e.J;
          y.col[e.J] = e.col;
        }
        y.y.c[3 * e.J] = (double)e.ph.re;
        y.y.c[3 * e.J + 1] = (double)e.ph.im;
        y.y.c[3 * e.J + 2] = (double)e.t;
        break;
      case E_PAIR:
        {
          int i = 0;
          while (!((e.cm >> i) & 1)) ++i;
          int j = i + 1;
          while (!((e.cm >> j) & 1)) ++j;
          y.y.pairs ^= 1 << pair_bit(i, j);
        }
        y.sgn |= e.cm;
        break;
      case E_NEG:
        y.y.flags |= BLK_NEG << e.J;
        masks(y, e);
        y.sgn |= jb;
        break;
      default: y.misc.push_back(&e); break;
    }
    for (int j = 0; j < kBlkRegs; ++j)
      if ((u >> j) & 1) level[j] = std::max(level[j], e.kind == E_ROT ? l + 1 : l);
  }
  if (ly.empty()) ly.resize(1);
  for (size_t l = 0; l < ly.size(); ++l) {
    if (l > 0 && !ly[l].misc.empty()) finish();
    if (l == 0 || !ly[l].misc.empty()) start(ly[l]);
    if (ly[l].y.flags || ly[l].y.pairs) push_layer(ly[l]);
  }
  finish();
}

// LDS slot (8 bytes) of tile element e: the higher bits folded onto the five
// that pick the bank, so that lanes that step by large powers of two spread
// over the banks.  Linear over XOR.
int slot(int e) { return e ^ (((e >> 5) ^ (e >> 10)) & 31); }
constexpr int kSlotBytes = 8;

}  // namespace

void plan_block_pass(const TileGeom& tg, const std::vector<const BlkGate*>& gates,
                     const std::vector<std::array<int, 2>>& at_bits, bool fp64, int low, BlkPlan* plan, int codes) {
  const int tb = tg.b, K = kBlkRegs, nthr = tb - K, lanes = std::min(6, nthr), waves = nthr - lanes;
  // tile-local bit of a physical bit, or 64 + its bit in the tile number
  int local_of[64];
  int tau = 0;
  for (int p = 0; p < tg.n; ++p) {
    local_of[p] = -1;
    if (p < tg.L) local_of[p] = p;
    for (int j = 0; j < tg.H; ++j)
      if (tg.hbits[j] == p) local_of[p] = tg.L + j;
    if (local_of[p] < 0) local_of[p] = 64 + tau++;
  }
  std::vector<Local> gs;
  gs.reserve(gates.size());
  for (size_t i = 0; i < gates.size(); ++i) {
    Local l;
    l.g = gates[i];
    for (int j = 0; j < 2; ++j) l.q[j] = at_bits[i][j] < 0 ? -1 : local_of[at_bits[i][j]];
    gs.push_back(l);
  }
  // destination bit of each local bit (relabel swaps); the low bits of the
  // source order must be lane bits as the tile is read, those of the
  // destination order as it is written
  int dest[64];
  for (int b = 0; b < tb; ++b) dest[b] = b;
  for (int i = 0; i < tg.nswap; ++i) std::swap(dest[tg.swap_a[i]], dest[tg.swap_b[i]]);
  // (two-byte amplitudes: those above the three of a 16-byte group of codes,
  // which are register bits then, up to the scale block's last)
  const int vec = codes > 0 ? 3 : 0;
  low = codes > 0 ? std::max(codes, 6) : std::min(low, lanes);
  const uint32_t all = (1u << tb) - 1, vec_src = (1u << vec) - 1, low_src = ((1u << low) - 1) & ~vec_src;
  uint32_t low_dst = 0, vec_dst = 0;
  for (int b = 0; b < tb; ++b) {
    if (dest[b] < vec) vec_dst |= 1u << b;
    else if (dest[b] < low) low_dst |= 1u << b;
  }
  const auto writes = [&](uint32_t regs) { return !(regs & low_dst) && (regs & vec_dst) == vec_dst; };
  // register bits in ascending order, those of a group of codes first as they
  // are read (first stage) and written
  const auto order_regs = [&](uint32_t regs, bool first, StagePlan* s) {
    int k = 0;
    s->regs = regs;
    if (!first && writes(regs))
      for (int d = 0; d < vec; ++d)
        for (int b = 0; b < tb; ++b)
          if (dest[b] == d) s->reg[k++] = b;
    for (int b = 0; b < tb; ++b)
      if ((regs >> b) & 1 && std::find(s->reg, s->reg + k, b) == s->reg + k) s->reg[k++] = b;
  };
  // A stage that is both the first and the last has to lay out a scale block
  // as it is read and as it is written.
  bool block_same = true;
  for (int b = 0; b < codes; ++b) block_same = block_same && dest[b] == b;
  std::vector<StagePlan> st;
  Frame fr;
  std::vector<std::pair<int, int>> lin;
  bool stuck = false;  // the last stage and exchange took nothing
  Rest rest(gs);
  do {
    std::vector<AbsorbMask> rm;
    uint64_t got = 0, need = vec_dst | rest.full[rest.next];
    for (int i : rest.left) {
      rm.push_back(rest.masks[i]);
      need |= rm.back().full;
    }
    const uint32_t first = st.empty() ? low_src : 0u;
    uint32_t P = pick_regs(rm, rest, tb, K, all & ~first, &got, st.empty() ? vec_src : 0u);
    // a last stage that needs no further exchange, if one finishes the pass
    if (!writes(P) && !st.empty() && !(need & low_dst) && __builtin_popcountll(need) <= K) {
      const uint32_t P2 = pick_regs(rm, rest, tb, K, all & ~low_dst, &got, vec_dst);
      if (got == rest.weight) P = P2;
    }
    StagePlan s;
    s.regs = P;
    std::vector<int> take, keep;
    Absorb ab(P);
    for (size_t k = 0; k < rm.size(); ++k) (ab.take(rm[k]) ? take : keep).push_back(rest.left[k]);
    rest.go_on(
        [&](int i) {
          if (ab.done()) return -1;
          if (!ab.take(rest.masks[i])) return 0;
          take.push_back(i);
          return 1;
        },
        &keep);
    leave_for_later(gs, P, rest.nondiag[rest.next], &take, &keep);
    // (a CNOT onto a bit with a phase pending cannot wait for an exchange)
    if (!stuck) leave_cnots(gs, &take, &keep);
    stuck = take.empty();
    order_regs(P, st.empty(), &s);
    s.ops.reserve(take.size() + K);
    Emitter em(gs, fr, s, K);
    for (int i : take) {
      em.gate(gs[i]);
      rest.weight -= rest.masks[i].weight;
    }
    em.finish();
    s.lin.swap(lin);
    st.push_back(std::move(s));
    rest.left.swap(keep);
    take_linear(gs, fr, &rest, &lin);
    stuck = stuck && lin.empty();
  } while (!rest.empty());
  // stage at which a bit is next a register bit (or must be a lane)
  auto next_use = [&](int b, size_t from) {
    for (size_t s = from; s < st.size(); ++s)
      if (((st[s].regs >> b) & 1) || (s + 1 == st.size() && ((low_dst >> b) & 1))) return (int)s;
    return (int)st.size() + 1;
  };
  // the tile is written from lanes that hold the destination's low bits
  if (!writes(st.back().regs) || (st.size() == 1 && (low_src != low_dst || !block_same)) || !lin.empty()) {
    StagePlan s;
    s.lin.swap(lin);
    // bits that stay where they are first, then the highest
    uint32_t regs = vec_dst;
    int k = vec;
    for (int pass = 0; pass < 2; ++pass)
      for (int b = tb - 1; b >= 0 && k < K; --b) {
        if (((low_dst | regs) >> b) & 1) continue;
        if (pass == 0 && !((st.back().regs >> b) & 1)) continue;
        regs |= 1u << b;
        ++k;
      }
    if (vec > 0) {
      order_regs(regs, false, &s);
    } else {
      s.regs = regs;
      k = 0;
      for (int pass = 0; pass < 2; ++pass)
        for (int b = tb - 1; b >= 0; --b)
          if ((regs >> b) & 1 && (int)((st.back().regs >> b) & 1) == 1 - pass) s.reg[k++] = b;
    }
    st.push_back(std::move(s));
  }
  settle_frame(fr, st.back(), tb, K);
  round_phases(st, fp64);
  place_scalars(st);
  // thread bits: wave bits kept from stage to stage while they can be, else
  // those that are needed again last; lane bits in an order whose LDS access
  // phases (8 lanes of 16 bytes, 16 of 8) reach distinct bank slots
  std::vector<int> wv;
  constexpr int phase = 4;
  // at[s][b]: where (in which of the first stage's elements' slots) the tile
  // element 1 << b of stage s lies: the CNOTs done by the exchanges so far,
  // linear over XOR; from[s][b]: the same in the elements of the stage before
  struct Map {
    int e[kBlkRegs + kBlkThrBits];
  };
  std::vector<Map> at(st.size()), from(st.size());
  for (int b = 0; b < tb; ++b) at[0].e[b] = 1 << b;
  for (size_t s = 0; s < st.size(); ++s) {
    StagePlan& p = st[s];
    if (s > 0)
      for (int b = 0; b < tb; ++b) {
        int x = 1 << b, y = 0;
        for (size_t i = p.lin.size(); i-- > 0;)
          if ((x >> p.lin[i].first) & 1) x ^= 1 << p.lin[i].second;
        for (int c = 0; c < tb; ++c)
          if ((x >> c) & 1) y ^= at[s - 1].e[c];
        from[s].e[b] = x;
        at[s].e[b] = y;
      }
    const bool f = s == 0, l = s + 1 == st.size();
    const uint32_t no = p.regs | (f ? low_src : 0u) | (l ? low_dst : 0u);
    bool keep = !f;
    for (int b : wv) keep = keep && !((no >> b) & 1);
    if (!keep) {
      std::vector<int> cand;
      for (int b = 0; b < tb; ++b)
        if (!((no >> b) & 1)) cand.push_back(b);
      std::stable_sort(cand.begin(), cand.end(), [&](int x, int y) { return next_use(x, s + 1) > next_use(y, s + 1); });
      wv.assign(cand.begin(), cand.begin() + waves);
      std::sort(wv.begin(), wv.end());
    }
    std::vector<int> ln;
    uint32_t used = p.regs;
    for (int b : wv) used |= 1u << b;
    int span = 1;
    auto dir = [&](int b) { return slot(at[s].e[b]) & ((1 << phase) - 1); };
    auto put = [&](int b) {
      int g = span;
      for (int u = 0; u < (1 << phase); ++u)
        if ((span >> u) & 1) g |= 1 << (u ^ dir(b));
      span = g;
      ln.push_back(b);
      used |= 1u << b;
    };
    if (f || l) {
      // (the bits of a scale block are the lowest lane bits, in any order)
      for (int pass = vec > 0 ? 0 : 1; pass < 2; ++pass)
        for (int d = 0; d < (pass == 0 ? codes : low); ++d)
          for (int b = 0; b < tb; ++b)
            if ((f ? b : dest[b]) == d && !((used >> b) & 1) && (pass == 1 || !((span >> dir(b)) & 1))) put(b);
    }
    for (int pass = 0; pass < 2; ++pass)
      for (int b = 0; b < tb; ++b) {
        if ((used >> b) & 1 || (int)ln.size() >= lanes) continue;
        if (pass == 0 && ((span >> dir(b)) & 1)) continue;
        put(b);
      }
    for (int i = 0; i < lanes; ++i) p.thr[i] = ln[i];
    for (int i = 0; i < waves; ++i) p.thr[lanes + i] = wv[i];
  }
  // serialise
  BlkPass out{};
  BlkGeom& g = out.g;
  g.n = tg.n;
  g.b = tb;
  g.L = tg.L;
  g.H = tg.H;
  g.block_bits = tg.block_bits;
  for (int j = 0; j < tg.H; ++j) g.hbits[j] = tg.hbits[j];
  auto phys = [&](int b) { return (int32_t)(b < tg.L ? b : tg.hbits[b - tg.L]); };
  for (int i = 0; i < nthr; ++i) {
    g.ld_thr[i] = phys(st.front().thr[i]);
    g.st_thr[i] = phys(dest[st.back().thr[i]]);
  }
  for (int j = 0; j < K; ++j) {
    g.ld_reg[j] = phys(st.front().reg[j]);
    g.st_reg[j] = phys(dest[st.back().reg[j]]);
  }
  // Whether every wave's elements of stage b lie in slots of its own elements of
  // stage a.  in: the element of a in whose slot each element 1 << e of b lies.
  auto same_slots = [&](const StagePlan& a, const StagePlan& b, const Map& in) {
    for (int i = lanes; i < nthr; ++i)
      for (int e = 0; e < tb; ++e)
        if (((in.e[e] >> a.thr[i]) & 1) != (e == b.thr[i])) return false;
    return true;
  };
  // A tile's first exchange writes the first stage's slots, which other waves
  // may still read in the last exchange of the tile before unless they are
  // the wave's own there.
  g.tile_sync = st.size() > 1 && !same_slots(st.front(), st.back(), at.back());
  for (int b = 0; b < tb; ++b)
    if ((fr.flip >> b) & 1) g.st_flip |= uint64_t(1) << phys(dest[b]);
  out.stage_begin = (int32_t)plan->stages.size();
  for (size_t s = 0; s < st.size(); ++s) {
    const StagePlan& p = st[s];
    BlkStage x{};
    x.exchange = s > 0 && !same_slots(st[s - 1], p, from[s]) ? BLK_CROSS : BLK_WAVE;
    for (int j = 0; j < K; ++j) x.row[j] = slot(at[s].e[p.reg[j]]) * kSlotBytes;
    for (int i = 0; i < nthr; ++i) x.thr[i] = slot(at[s].e[p.thr[i]]) * kSlotBytes;
    emit_layers(p, nthr, x, plan);
  }
  plan->passes.push_back(out);
  plan->passes.back().g.nst = (int32_t)plan->stages.size() - out.stage_begin;
}

namespace {

template <typename T>
void put_reals(const BlkPlan& plan, const BlkLayout& l, char* h) {
  auto* y = (BlkLayer<T>*)(h + l.o_layers);
  for (size_t i = 0; i < plan.layers.size(); ++i) {
    const BlkLayer<double>& x = plan.layers[i];
    y[i].flags = x.flags;
    y[i].pairs = x.pairs;
    for (int j = 0; j < kBlkRegs; ++j) y[i].tmask[j] = x.tmask[j];
    for (int j = 0; j < 3 * kBlkRegs; ++j) y[i].c[j] = (T)x.c[j];
  }
  T* c = (T*)(h + l.o_ocoef);
  for (size_t i = 0; i < plan.ocoef.size(); ++i) c[i] = (T)plan.ocoef[i];
}

}  // namespace

BlkLayout block_layout(const BlkSizes& z, bool fp64) {
  const auto up = [](size_t x) { return (x + 255) & ~size_t(255); };
  BlkLayout l;
  l.o_geoms = up(z.stages * sizeof(BlkStage));
  l.o_layers = up(l.o_geoms + z.passes * sizeof(BlkPass));
  // two more layers: the kernels read up to two records ahead
  l.o_more = up(l.o_layers + (z.layers + 2) * (fp64 ? sizeof(BlkLayer<double>) : sizeof(BlkLayer<float>)));
  l.o_ops = up(l.o_more + z.layers * sizeof(BlkMore));
  l.o_ocoef = up(l.o_ops + z.ops * sizeof(BlkOp));
  l.total = up(l.o_ocoef + 8 * z.ops * (fp64 ? sizeof(double) : sizeof(float)));
  return l;
}

BlkLayout block_image(const BlkPlan& plan, bool fp64, char* h) {
  const BlkLayout l = block_layout(BlkSizes(plan), fp64);
  const auto put = [&](size_t o, const void* p, size_t n) {
    if (n) std::memcpy(h + o, p, n);
  };
  put(0, plan.stages.data(), plan.stages.size() * sizeof(BlkStage));
  put(l.o_geoms, plan.passes.data(), plan.passes.size() * sizeof(BlkPass));
  put(l.o_more, plan.more.data(), plan.more.size() * sizeof(BlkMore));
  put(l.o_ops, plan.ops.data(), plan.ops.size() * sizeof(BlkOp));
  if (fp64) put_reals<double>(plan, l, h);
  else put_reals<float>(plan, l, h);
  return l;
}

namespace {

// Modelled duration (ms) of a plan on 2^30 amplitudes, from passes measured
// on MI355X: HBM time of a pass, and on chip a rotation, a layer, an exchange
// and the tile's own load and store; the two overlap to about two thirds.
double plan_ms(const BlkPlan& p, bool fp64) {
  const double mem = fp64 ? 6.2 : 3.1, half = fp64 ? 1.0 : 0.6;
  double total = 0.0;
  for (const BlkPass& ps : p.passes) {
    double c = 0.8;
    for (int s = 0; s < ps.g.nst; ++s) {
      const BlkStage& st = p.stages[ps.stage_begin + s];
      if (s > 0 && st.exchange != BLK_STAY) c += 0.45;
      c += 0.2 * (st.misc_end - st.misc_begin) + 0.05 * (st.layer_end - st.layer_begin);
      for (int l = st.layer_begin; l < st.layer_end; ++l)
        for (int j = 0; j < kBlkRegs; ++j)
          if (p.layers[l].flags & (BLK_ROT << j)) c += 0.135;
    }
    c *= half;
    total += std::max(c, mem) + 0.35 * std::min(c, mem);
  }
  return total;
}

// Whether every op's coefficients can be held in the state's precision: the
// largest of an op's neither overflows nor vanishes, nor comes near it (the
// amplitudes take the ops one by one).  Matrices far from unitary ones may not
// be; the fused passes multiply them in FP64 first.
bool in_range(const BlkPlan& p, bool fp64) {
  const double most = fp64 ? 0x1p500 : 0x1p60, most2 = most * most;
  const auto ok = [&](double x, double y) {
    const double n = x * x + y * y;
    return n >= 1.0 / most2 && n <= most2;
  };
  for (const BlkLayer<double>& y : p.layers)
    for (int j = 0; j < kBlkRegs; ++j)
      if ((y.flags & (BLK_ROT << j)) && !(ok(y.c[3 * j], y.c[3 * j + 1]) && std::isfinite(y.c[3 * j + 2])))
        return false;
  for (size_t o = 0; o < p.ops.size(); ++o) {
    const uint32_t kind = p.ops[o].kind;
    const double* c = &p.ocoef[8 * o];
    if ((kind == 0 || (kind & (blk_phase() * 127))) && !ok(c[0], c[1])) return false;
    if (kind & (blk_dense(0) * 15)) {
      double m = 0.0;
      for (int i = 0; i < 8; ++i) {
        if (!std::isfinite(c[i])) return false;
        m = std::max(m, std::fabs(c[i]));
      }
      if (!ok(m, 0.0)) return false;
    }
  }
  return true;
}

}  // namespace

// The qubits of the gates alone, for the tile selection.  strict: a gate is
// in a tile only when all of its qubits are; else (more gates per pass, but
// greedier) controlled phases need one and CNOTs their target in the tile,
// and gates that are diagonal on a qubit pass each other.
void block_schedule(int n, int L, int b, const std::vector<BlkGate>& bg, int max_take, bool relabel, bool strict,
                    BlkSchedule* out) {
  std::vector<Gate>& shape = out->shape;
  shape.assign(bg.size(), Gate{});
  for (size_t i = 0; i < bg.size(); ++i) {
    const BlkGate::Kind k = bg[i].kind;
    shape[i].nq = k == BlkGate::CPHASE || k == BlkGate::CNOT ? 2 : 1;
    shape[i].q[0] = bg[i].q[0];
    shape[i].q[1] = bg[i].q[1];
    shape[i].diag_on = strict ? 0 : k == BlkGate::CPHASE ? 3 : k == BlkGate::CNOT || k == BlkGate::PHASE1 ? 1 : 0;
  }
  out->kinds.clear();
  for (const BlkGate& g : bg) out->kinds.push_back(g.kind);
  out->low = std::min(L, n);
  if (relabel) {
    select_tiles_relabel(n, L, b, 0, shape, &out->sched, max_take);
  } else {
    select_tiles(n, L, b, 0, shape, &out->sched, max_take);
    out->sched.final_pos.resize(n);
    for (int q = 0; q < n; ++q) out->sched.final_pos[q] = q;
  }
  if (out->sched.passes.empty()) {  // no gates: one pass that writes the state as it is
    TilePass p{};
    p.g.n = n;
    p.g.b = p.g.L = std::min(n, b);
    out->sched.passes.push_back(p);
    out->sched.taken.emplace_back();
  }
}

bool block_build(const BlkSchedule& bs, const std::vector<BlkGate>& bg, bool fp64, BlkPlan* plan) {
  if (bs.kinds.size() != bg.size() || bs.sched.gates != (int64_t)bg.size()) return false;
  for (size_t i = 0; i < bg.size(); ++i)
    if (bs.kinds[i] != bg[i].kind || bs.shape[i].q[0] != bg[i].q[0] || bs.shape[i].q[1] != bg[i].q[1]) return false;
  const TileSchedule& sched = bs.sched;
  const std::vector<Gate>& src = sched.tgates.empty() ? bs.shape : sched.tgates;
  for (size_t i = 0; i < sched.passes.size(); ++i) {
    std::vector<const BlkGate*> mine;
    std::vector<std::array<int, 2>> at;
    mine.reserve(sched.taken[i].size());
    at.reserve(sched.taken[i].size());
    for (int t : sched.taken[i]) {
      mine.push_back(&bg[sched.tsrc.empty() ? t : sched.tsrc[t]]);
      at.push_back({src[t].q[0], src[t].nq > 1 ? src[t].q[1] : -1});
    }
    plan_block_pass(sched.passes[i].g, mine, at, fp64, std::min(bs.low, fp64 ? 5 : 6), plan);
  }
  return in_range(*plan, fp64);
}

bool block_tile_plan(const TilePlan& tp, int block_bits, BlkPlan* plan) {
  for (const TilePass& ps : tp.passes) {
    // a pass's gates in the order that its ops apply them
    std::vector<int> order;
    for (int o = ps.op_begin; o < ps.op_begin + ps.op_count; ++o)
      order.insert(order.end(), tp.op_gates[o].begin(), tp.op_gates[o].end());
    std::vector<BlkGate> bg;
    if (!block_gates(ps.g.n, tp.src, block_tol(false), &bg, false, &order)) return false;
    std::vector<const BlkGate*> mine;
    std::vector<std::array<int, 2>> at;
    for (const BlkGate& g : bg) {
      mine.push_back(&g);
      at.push_back({g.q[0], g.kind == BlkGate::CPHASE || g.kind == BlkGate::CNOT ? g.q[1] : -1});
    }
    plan_block_pass(ps.g, mine, at, false, 0, plan, block_bits);
  }
  return in_range(*plan, false);
}

void append_plan(const BlkPlan& p, BlkPlan* all) {
  const int s0 = (int)all->stages.size(), l0 = (int)all->layers.size(), o0 = (int)all->ops.size();
  for (BlkPass x : p.passes) {
    x.stage_begin += s0;
    all->passes.push_back(x);
  }
  for (BlkStage x : p.stages) {
    x.layer_begin += l0;
    x.layer_end += l0;
    x.misc_begin += o0;
    x.misc_end += o0;
    all->stages.push_back(x);
  }
  all->layers.insert(all->layers.end(), p.layers.begin(), p.layers.end());
  for (BlkMore x : p.more) {
    for (int j = 0; j < kBlkRegs; ++j) {
      x.col_begin[j] += o0;
      x.col_end[j] += o0;
    }
    all->more.push_back(x);
  }
  for (BlkOp x : p.ops) {
    x.col_begin += o0;
    x.col_end += o0;
    all->ops.push_back(x);
  }
  all->ocoef.insert(all->ocoef.end(), p.ocoef.begin(), p.ocoef.end());
}

bool plan_block(int n, int L, int b, const std::vector<Gate>& gates, bool fp64, int max_take, bool relabel,
                BlkPlan* plan, std::vector<int>* final_pos, const uint64_t* basis) {
  *plan = BlkPlan();
  std::vector<BlkGate> bg;
  if (!block_gates(n, gates, block_tol(fp64), &bg, false, nullptr, basis)) return false;
  // Both selections where a run takes far longer than planning (2^24
  // amplitudes or more), side by side, and the better by plan_ms; else the
  // second alone.
  const int ways = n >= 24 ? 2 : 1;
  BlkPlan cand[2];
  BlkSchedule bs[2];
  std::exception_ptr error[2];
  const auto way = [&](int strict) {
    try {
      block_schedule(n, L, b, bg, max_take, relabel, strict != 0, &bs[strict]);
      if (!block_build(bs[strict], bg, fp64, &cand[strict])) cand[strict] = BlkPlan();
    } catch (...) {
      error[strict] = std::current_exception();
    }
  };
  std::thread other;
  if (ways > 1) {
    try {
      other = std::thread(way, 1);
    } catch (const std::system_error&) {  // no thread to be had
      way(1);
    }
  }
  way(0);
  if (other.joinable()) other.join();
  double best = 0.0;
  for (int strict = 0; strict < ways; ++strict) {
    if (error[strict]) std::rethrow_exception(error[strict]);
    if (cand[strict].passes.empty()) continue;
    const double ms = plan_ms(cand[strict], fp64);
    if (plan->passes.empty() || ms < best) {
      best = ms;
      *plan = std::move(cand[strict]);
      *final_pos = bs[strict].sched.final_pos;
    }
  }
  return !plan->passes.empty();
}

}  // namespace juqcs
