// Runs register-resident tile programs on the host, the way their kernels do:
// every thread's registers, the exchanges through LDS slots, the layers in
// order, in the state's precision.  It also looks for accesses of LDS that
// nothing orders: two waves at one slot, one of them writing, between two
// barriers of the workgroup, over two tiles in a row.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "juqcs_internal.hpp"

namespace juqcs {
void set_error(const std::string&) {}
}  // namespace juqcs

using namespace juqcs;

namespace {

struct Report {
  int64_t passes = 0;    // passes of the plan (0: the fused passes are taken)
  int64_t races = 0;     // unordered accesses of a slot
  int64_t misplaced = 0; // amplitudes written twice or never
  int64_t blocks = 0;    // scale blocks whose amplitudes do not lie in neighbouring lanes
  double least = 0, most = 0;  // size of the smallest and the largest op (largest coefficient of each)
  int64_t layers = 0, misc = 0, stages = 0;
};

// Slots of an LDS tile: who touched them since the last barrier.
struct Slots {
  std::vector<int> wave, epoch;
  std::vector<char> shared, written;
  int now = 0;
  int64_t races = 0;
  explicit Slots(size_t n) : wave(n, -1), epoch(n, -1), shared(n), written(n) {}
  void touch(size_t s, int w, bool write) {
    if (epoch[s] != now) {
      epoch[s] = now;
      wave[s] = w;
      shared[s] = 0;
      written[s] = write;
      return;
    }
    if (wave[s] != w) shared[s] = 1;
    written[s] |= write;
    if (shared[s] && written[s]) ++races;
  }
  void barrier() { ++now; }
};

int thread_offset(const BlkStage& s, int nthr, int tid) {
  int o = 0;
  for (int i = 0; i < nthr; ++i)
    if ((tid >> i) & 1) o ^= s.thr[i];
  return o / 8;
}
int reg_offset(const BlkStage& s, int r) {
  int o = 0;
  for (int j = 0; j < kBlkRegs; ++j)
    if ((r >> j) & 1) o ^= s.row[j];
  return o / 8;
}

void exchange_slots(const BlkStage& a, const BlkStage& b, int nthr, bool fp64, Slots* sl) {
  const auto all = [&](const BlkStage& s, bool write) {
    for (int t = 0; t < 1 << nthr; ++t)
      for (int r = 0; r < 1 << kBlkRegs; ++r) sl->touch(thread_offset(s, nthr, t) ^ reg_offset(s, r), t >> 6, write);
  };
  const auto sync = [&] {
    if (b.exchange == BLK_CROSS) sl->barrier();
  };
  for (int part = 0; part < (fp64 ? 2 : 1); ++part) {  // one component at a time
    if (part > 0) sync();
    all(a, true);
    sync();
    all(b, false);
  }
}

template <typename T>
struct Tile {
  struct Amp {
    T x, y;
  };
  const BlkPlan& p;
  const BlkPass& ps;
  int nthr;
  std::vector<Amp> a;  // 2^kBlkRegs per thread
  Tile(const BlkPlan& plan, const BlkPass& pass)
      : p(plan), ps(pass), nthr(pass.g.b - kBlkRegs), a(size_t(1) << pass.g.b) {}

  static void mul(Amp& v, T C, T S) {
    const T x = v.x;
    v.x = std::fma(-S, v.y, C * x);
    v.y = std::fma(S, x, C * v.y);
  }
  void collect(int c0, int c1, uint32_t tid, uint64_t tau, T* C, T* S) const {
    for (int o = c0; o < c1; ++o) {
      const BlkOp& q = p.ops[o];
      if ((tid & q.tmask) != q.tmask || (tau & q.gmask) != q.gmask) continue;
      const T u = (T)p.ocoef[8 * o], v = (T)p.ocoef[8 * o + 1], x = *C, y = *S;
      *C = std::fma(-v, y, u * x);
      *S = std::fma(v, x, u * y);
    }
  }
  static bool odd(uint32_t x, uint64_t y) { return (__builtin_popcount(x) + __builtin_popcountll(y)) & 1; }

  void misc(const BlkOp& o, const double* c64, uint32_t tid, uint64_t tau, Amp* v) const {
    T c[8];
    for (int i = 0; i < 8; ++i) c[i] = (T)c64[i];
    const bool on = (tid & o.tmask) == o.tmask && (tau & o.gmask) == o.gmask;
    for (int r = 0; r < 1 << kBlkRegs; ++r)
      for (int j = 0; j < kBlkRegs; ++j) {
        if ((r >> j) & 1) continue;
        Amp &u = v[r], &w = v[r | 1 << j];
        if (o.kind & blk_dense(j)) {
          const Amp x = u, y = w;
          u.x = std::fma(-c[3], y.y, std::fma(c[2], y.x, std::fma(-c[1], x.y, c[0] * x.x)));
          u.y = std::fma(c[3], y.x, std::fma(c[2], y.y, std::fma(c[1], x.x, c[0] * x.y)));
          w.x = std::fma(-c[7], y.y, std::fma(c[6], y.x, std::fma(-c[5], x.y, c[4] * x.x)));
          w.y = std::fma(c[7], y.x, std::fma(c[6], y.y, std::fma(c[5], x.x, c[4] * x.y)));
        }
        for (int i = 0; i < kBlkRegs; ++i)
          if ((o.kind & blk_swap(j, i)) && (i == j ? on : (r >> i) & 1)) std::swap(u, w);
      }
    if (o.kind & blk_signs(0))
      for (int r = 0; r < 1 << kBlkRegs; ++r)
        if (odd((tid & o.tmask), tau & o.gmask) != odd(r & (o.kind >> 28), 0)) v[r] = Amp{-v[r].x, -v[r].y};
    if (o.kind & (blk_phase() * 127)) {
      T C = c[0], S = c[1];
      collect(o.col_begin, o.col_end, tid, tau, &C, &S);
      int m = 0;
      for (int i = 0; i < kBlkRegs; ++i)
        for (int j = i + 1; j < kBlkRegs; ++j)
          if (o.kind & blk_phase(i, j)) m = 1 << i | 1 << j;
      for (int r = 0; r < 1 << kBlkRegs; ++r)
        if ((r & m) == m) mul(v[r], C, S);
    }
  }
  void layer(const BlkLayer<double>& y, const BlkMore& more, uint32_t tid, uint64_t tau, Amp* v) const {
    const auto sign = [&](int j) {
      return odd(tid & y.tmask[j], y.flags & (BLK_GMASK << j) ? tau & more.gmask[j] : 0);
    };
    for (int i = 0; i < kBlkRegs; ++i)
      for (int j = i + 1; j < kBlkRegs; ++j)
        if (y.pairs & (1 << pair_bit(i, j)))
          for (int r = 0; r < 1 << kBlkRegs; ++r)
            if (((r >> i) & (r >> j)) & 1) v[r] = Amp{-v[r].x, -v[r].y};
    for (int j = 0; j < kBlkRegs; ++j)
      if ((y.flags & (BLK_NEG << j)) && sign(j))
        for (int r = 0; r < 1 << kBlkRegs; ++r)
          if ((r >> j) & 1) v[r] = Amp{-v[r].x, -v[r].y};
    for (int j = 0; j < kBlkRegs; ++j) {
      if (!(y.flags & (BLK_ROT << j))) continue;
      T C = (T)y.c[3 * j], S = (T)y.c[3 * j + 1];
      const T t = (T)y.c[3 * j + 2];
      if (y.flags & (BLK_OUTER << j)) {
        if (y.flags & (BLK_COL << j)) collect(more.col_begin[j], more.col_end[j], tid, tau, &C, &S);
        if (sign(j)) C = -C, S = -S;
      }
      for (int r = 0; r < 1 << kBlkRegs; ++r) {
        if ((r >> j) & 1) continue;
        Amp &u = v[r], &w = v[r | 1 << j];
        mul(w, C, S);
        const Amp z = w;
        w = Amp{std::fma(t, u.x, z.x), std::fma(t, u.y, z.y)};
        u = Amp{std::fma(-t, z.x, u.x), std::fma(-t, z.y, u.y)};
      }
    }
  }

  void stages(uint64_t tau) {
    std::vector<Amp> sh(a.size());
    for (int s = 0; s < ps.g.nst; ++s) {
      const BlkStage& st = p.stages[ps.stage_begin + s];
      if (s > 0 && st.exchange != BLK_STAY) {
        const BlkStage& from = p.stages[ps.stage_begin + s - 1];
        for (size_t e = 0; e < a.size(); ++e)
          sh[thread_offset(from, nthr, (int)(e >> kBlkRegs)) ^ reg_offset(from, (int)(e & 15))] = a[e];
        for (size_t e = 0; e < a.size(); ++e)
          a[e] = sh[thread_offset(st, nthr, (int)(e >> kBlkRegs)) ^ reg_offset(st, (int)(e & 15))];
      }
      for (int t = 0; t < 1 << nthr; ++t) {
        Amp* v = &a[(size_t)t << kBlkRegs];
        for (int o = st.misc_begin; o < st.misc_end; ++o) misc(p.ops[o], &p.ocoef[8 * o], t, tau, v);
        for (int l = st.layer_begin; l < st.layer_end; ++l) layer(p.layers[l], p.more[l], t, tau, v);
      }
    }
  }
};

uint64_t place(uint32_t x, int n, const int32_t* pos) {
  uint64_t o = 0;
  for (int i = 0; i < n; ++i) o |= (uint64_t)((x >> i) & 1) << pos[i];
  return o;
}

template <typename T>
void run_plan(const BlkPlan& p, int codes, std::vector<cplx<double>>* state, Report* rep) {
  typedef typename Tile<T>::Amp Amp;
  std::vector<Amp> psi(state->size()), out(state->size());
  for (size_t i = 0; i < psi.size(); ++i) psi[i] = Amp{(T)(*state)[i].re, (T)(*state)[i].im};
  for (const BlkPass& ps : p.passes) {
    const BlkGeom& g = ps.g;
    Tile<T> tile(p, ps);
    const int nthr = tile.nthr;
    std::vector<char> seen(psi.size());
    for (uint64_t tau = 0; tau < (uint64_t)psi.size() >> g.b; ++tau) {
      uint64_t base = tau << g.L;
      for (int j = 0; j < g.H; ++j) base = insert_zero(base, g.hbits[j]);
      for (size_t e = 0; e < tile.a.size(); ++e)
        tile.a[e] = psi[base + (place(e >> kBlkRegs, nthr, g.ld_thr) | place(e & 15, kBlkRegs, g.ld_reg))];
      tile.stages(tau);
      for (size_t e = 0; e < tile.a.size(); ++e) {
        const uint64_t at =
            base + ((place(e >> kBlkRegs, nthr, g.st_thr) | place(e & 15, kBlkRegs, g.st_reg)) ^ g.st_flip);
        out[at] = tile.a[e];
        rep->misplaced += seen[at];
        seen[at] = 1;
      }
    }
    psi.swap(out);
    // the amplitudes of a scale block lie in lanes that differ in the lowest bits
    if (codes > 0)
      for (int side = 0; side < 2; ++side) {
        const int32_t *thr = side ? g.st_thr : g.ld_thr, *reg = side ? g.st_reg : g.ld_reg;
        int lanes = 0;
        for (int i = 0; i < codes - 3; ++i) lanes |= 1 << thr[i];
        if (reg[0] != 0 || reg[1] != 1 || reg[2] != 2 || (side && lanes != (1 << codes) - 8)) ++rep->blocks;
      }
    // two tiles of the pass, one after the other
    Slots sl(size_t(1) << g.b);
    for (int k = 0; k < 2; ++k) {
      for (int s = 1; s < g.nst; ++s)
        if (p.stages[ps.stage_begin + s].exchange != BLK_STAY)
          exchange_slots(p.stages[ps.stage_begin + s - 1], p.stages[ps.stage_begin + s], nthr, sizeof(T) == 8, &sl);
      if (g.tile_sync) sl.barrier();
    }
    rep->races += sl.races;
  }
  for (size_t i = 0; i < psi.size(); ++i) (*state)[i] = cplx<double>{(double)psi[i].x, (double)psi[i].y};
}

void sizes(const BlkPlan& p, bool fp64, Report* rep) {
  rep->least = INFINITY;
  const auto op = [&](double x) {
    if (!fp64) x = (float)x;
    if (std::isnan(x)) x = INFINITY;
    rep->least = std::min(rep->least, x);
    rep->most = std::max(rep->most, x);
  };
  for (const BlkLayer<double>& y : p.layers)
    for (int j = 0; j < kBlkRegs; ++j)
      if (y.flags & (BLK_ROT << j)) op(std::hypot(y.c[3 * j], y.c[3 * j + 1]));
  for (size_t o = 0; o < p.ops.size(); ++o) {
    if ((p.ops[o].kind & (blk_phase() * 127)) || p.ops[o].kind == 0)
      op(std::hypot(p.ocoef[8 * o], p.ocoef[8 * o + 1]));
    if (p.ops[o].kind & 15) {
      double m = 0;
      for (int i = 0; i < 8; ++i) m = std::max(m, std::fabs(p.ocoef[8 * o + i]));
      op(m);
    }
  }
  rep->passes = (int64_t)p.passes.size();
  rep->stages = (int64_t)p.stages.size();
  rep->layers = (int64_t)p.layers.size();
  for (const BlkStage& s : p.stages) rep->misc += s.misc_end - s.misc_begin;
}

}  // namespace

// Plans a circuit with the given tile geometry and runs the plan on psi (2^n
// complex numbers; qubit q on bit q before and after).  block_bits > 0: the
// passes of a two-byte state, without its codes; basis: the basis state that psi
// is (null: unknown); psi null: the plan alone.
// Returns 0, or 1 where the plan is left to the fused passes.
extern "C" int run_program(int n, const juqcs_gate* gates, int64_t count, int fp64, int low, int tile, int pass_gates,
                           int relabel, int block_bits, const uint64_t* basis, double* psi, Report* rep) {
  *rep = Report();
  std::vector<Gate> gs(count);
  std::string err;
  for (int64_t i = 0; i < count; ++i)
    if (!decode_gate(gates[i], n, &gs[i], &err)) return 2;
  BlkPlan plan;
  std::vector<int> moved;
  const int L = std::min(low, n);
  if (block_bits > 0) {
    TilePlan tp;
    plan_tiles(n, L, tile, block_bits, gs, &tp, 3, 0, pass_gates, 0, relabel >= 0, &moved);
    if (!block_tile_plan(tp, block_bits, &plan)) return 1;
  } else if (!plan_block(n, L, tile, gs, fp64 != 0, pass_gates, relabel >= 0, &plan, &moved, basis)) {
    return 1;
  }
  sizes(plan, fp64 != 0, rep);
  if (!psi) return 0;
  std::vector<cplx<double>> v(size_t(1) << n);
  std::memcpy(v.data(), psi, v.size() * sizeof v[0]);
  if (fp64) run_plan<double>(plan, block_bits, &v, rep);
  else run_plan<float>(plan, block_bits, &v, rep);
  if (relabel < 0 || moved.empty()) {
    std::memcpy(psi, v.data(), v.size() * sizeof v[0]);
    return 0;
  }
  for (size_t i = 0; i < v.size(); ++i) {
    size_t at = 0;
    for (int q = 0; q < n; ++q) at |= ((i >> q) & 1) << moved[q];
    psi[2 * i] = v[at].re;
    psi[2 * i + 1] = v[at].im;
  }
  return 0;
}
