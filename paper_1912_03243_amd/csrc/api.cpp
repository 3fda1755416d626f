// C-ABI entry points of libjuqcs_gpu (declared in include/juqcs_gpu.h).
// Host-side validation, the logical->physical qubit map, workspace handling,
// and dispatch to the kernels and the planner.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "juqcs_internal.hpp"

namespace juqcs {

namespace {
thread_local std::string g_last_error;
}

void set_error(const std::string& msg) { g_last_error = msg; }

}  // namespace juqcs

using namespace juqcs;

namespace {

constexpr size_t kWorkBytes = size_t(32) << 20;  // 32 MiB library workspace
constexpr size_t kPartialOff = 0;                // 16 KiB of FP64 partials
constexpr size_t kResultOff = 64 << 10;          // small results (norm, Pauli sums)
constexpr size_t kRingOff = 128 << 10;           // programs, matrices, indices
constexpr int kDefaultBlockBits = 8;

using C = cplx<double>;

juqcs_status fail(juqcs_status st, const std::string& msg) {
  set_error(msg);
  return st;
}

juqcs_status hip_fail(hipError_t e, const char* where) {
  set_error(std::string(where) + ": " + hipGetErrorString(e));
  return JUQCS_ERR_HIP;
}

size_t amp_size(juqcs_dtype dt) { return dt == JUQCS_C128 ? 16 : dt == JUQCS_C64 ? 8 : 2; }

bool finite8(const double* u, int count) {
  for (int i = 0; i < count; ++i)
    if (!std::isfinite(u[i])) return false;
  return true;
}

}  // namespace

struct juqcs_state {
  int n;
  juqcs_dtype dt;
  int B;
  void* amps;
  void* scales;
  char* work;
  size_t work_bytes;
  hipStream_t stream;
  // FP64 complex factor of the whole state: the logical state is gf times
  // the stored amplitudes (phases and scalar weights are absorbed here
  // instead of passes over the data)
  C gf{1.0, 0.0};
  double size = 1.0;  // product of the factors of juqcs_scale since the last init
  bool fresh = false;  // no gate since juqcs_state_init put it into a basis state
  uint64_t basis = 0;  // that basis state
  int phys[64];  // logical qubit -> physical bit
  size_t ring;   // next free offset inside the ring
  // per-pass timing of juqcs_run_circuit when profiling (else empty)
  bool profiling = false;
  std::vector<hipEvent_t> ev;
  double bytes = 0.0;      // algorithmic bytes of the passes launched by the call
  double mma_flops = 0.0;  // flops of the fused blocks launched by the call
};

namespace {

// Pass timing: an event pair around every pass launch on the state's stream.
void prof_begin(juqcs_state* st) {
  if (!st->profiling) return;
  hipEvent_t e;
  if (hipEventCreate(&e) == hipSuccess) {
    (void)hipEventRecord(e, st->stream);
    st->ev.push_back(e);
  }
}
void prof_end(juqcs_state* st) { prof_begin(st); }

double prof_collect(juqcs_state* st) {
  double total = 0.0;
  if (!st->ev.empty()) (void)hipEventSynchronize(st->ev.back());
  for (size_t i = 0; i + 1 < st->ev.size(); i += 2) {
    float ms = 0.0f;
    if (hipEventElapsedTime(&ms, st->ev[i], st->ev[i + 1]) == hipSuccess) total += ms;
  }
  for (hipEvent_t e : st->ev) (void)hipEventDestroy(e);
  st->ev.clear();
  return total;
}

double full_pass_bytes(const juqcs_state* st) {
  const double count = std::ldexp(1.0, st->n);
  double b = 2.0 * count * (double)(st->dt == JUQCS_C128 ? 16 : st->dt == JUQCS_C64 ? 8 : 2);
  if (st->dt == JUQCS_ENC2) b += 2.0 * 4.0 * std::ldexp(1.0, st->n - st->B);
  return b;
}

// Stream-ordered ring allocation inside the workspace: later kernels on the
// same stream only start after earlier ones finish, so reusing ring space is
// safe for work issued on the handle's stream.
char* ring_alloc(juqcs_state* st, size_t bytes) {
  bytes = (bytes + 255) & ~size_t(255);
  if (kRingOff + bytes > st->work_bytes) return nullptr;
  if (st->ring + bytes > st->work_bytes) st->ring = kRingOff;
  char* p = st->work + st->ring;
  st->ring += bytes;
  return p;
}

juqcs_status upload(juqcs_state* st, const void* host, size_t bytes, char** dev) {
  *dev = ring_alloc(st, bytes);
  if (!*dev) return fail(JUQCS_ERR_SIZE, "workspace too small for upload");
  hipError_t e = hipMemcpyAsync(*dev, host, bytes, hipMemcpyHostToDevice, st->stream);
  if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync");
  return JUQCS_OK;
}

juqcs_status check_state(const juqcs_state* st) {
  if (!st) return fail(JUQCS_ERR_ARG, "null state handle");
  return JUQCS_OK;
}

juqcs_status check_qubit(const juqcs_state* st, int q) {
  if (q < 0 || q >= st->n) return fail(JUQCS_ERR_QUBIT, "qubit out of range");
  return JUQCS_OK;
}

bool is_diag2(const C u[4]) {
  return u[1].re == 0.0 && u[1].im == 0.0 && u[2].re == 0.0 && u[2].im == 0.0;
}
bool is_one(C z) { return z.re == 1.0 && z.im == 0.0; }

template <typename T>
void convert(const std::vector<C>& in, std::vector<cplx<T>>* out) {
  out->resize(in.size());
  for (size_t i = 0; i < in.size(); ++i) (*out)[i] = {(T)in[i].re, (T)in[i].im};
}

// Runs a tile plan: upload ops + matrices once, then launch every pass.
juqcs_status run_tile_plan(juqcs_state* st, const TilePlan& plan) {
  if (plan.passes.empty()) return JUQCS_OK;
  const size_t ops_bytes = plan.ops.size() * sizeof(TileOp);
  std::vector<char> buf;
  size_t mats_off = (ops_bytes + 255) & ~size_t(255);
  std::vector<TileOp> ops = plan.ops;
  if (st->dt == JUQCS_C128) {
    // 8x8 ops of pipelined passes in three-product form, appended
    std::vector<C> mats = plan.mats;
    for (const TilePass& p : plan.passes) {
      if (!tile_pipelined(st->dt, p.g, p.op_count)) continue;
      for (int o = p.op_begin; o < p.op_begin + p.op_count; ++o) {
        TileOp& op = ops[o];
        if (op.kind != TOP_DENSE3) continue;
        const C* m = plan.mats.data() + op.moff;
        std::vector<double> g(192);
        for (int r = 0; r < 8; ++r)
          for (int c = 0; c < 8; ++c) {
            const C z = m[8 * r + c];
            g[24 * r + c] = z.re;
            g[24 * r + 8 + c] = z.re + z.im;
            g[24 * r + 16 + c] = z.im - z.re;
          }
        op.kind = TOP_DENSE3G;
        op.moff = (int64_t)mats.size();
        for (int i = 0; i < 96; ++i) mats.push_back({g[2 * i], g[2 * i + 1]});
      }
    }
    buf.resize(mats_off + mats.size() * sizeof(C));
    std::memcpy(buf.data() + mats_off, mats.data(), mats.size() * sizeof(C));
  } else {
    std::vector<cplx<float>> m;
    convert(plan.mats, &m);
    buf.resize(mats_off + m.size() * sizeof(cplx<float>));
    std::memcpy(buf.data() + mats_off, m.data(), m.size() * sizeof(cplx<float>));
  }
  std::memcpy(buf.data(), ops.data(), ops_bytes);
  char* dev = nullptr;
  juqcs_status rc = upload(st, buf.data(), buf.size(), &dev);
  if (rc != JUQCS_OK) return rc;
  const TileOp* d_ops = (const TileOp*)dev;
  const void* d_mats = dev + mats_off;
  for (const TilePass& p : plan.passes) {
    prof_begin(st);
    hipError_t e = launch_tile(st->dt, st->amps, st->scales, p.g, d_ops + p.op_begin,
                               p.op_count, d_mats, st->stream);
    prof_end(st);
    if (e != hipSuccess) return hip_fail(e, "tile pass launch");
    st->bytes += full_pass_bytes(st);
  }
  return JUQCS_OK;
}

// Whether a register-resident plan fits the workspace's ring at once (fused
// plans of very many controlled phases are smaller).
bool fits_ring(const juqcs_state* st, const BlkPlan& plan) {
  const size_t bytes = block_layout(BlkSizes(plan), st->dt == JUQCS_C128).total;
  return kRingOff + ((bytes + 255) & ~size_t(255)) <= st->work_bytes;
}

// Runs a register-resident plan: one upload, then every pass.
juqcs_status run_block_plan(juqcs_state* st, const BlkPlan& plan) {
  if (plan.passes.empty()) return JUQCS_OK;
  const bool fp64 = st->dt == JUQCS_C128;
  const BlkLayout lay = block_layout(BlkSizes(plan), fp64);
  std::vector<char> buf(lay.total, 0);
  block_image(plan, fp64, buf.data());
  char* dev = nullptr;
  if (juqcs_status rc = upload(st, buf.data(), buf.size(), &dev)) return rc;
  const BlkDev bd = block_device(lay, dev);
  for (size_t i = 0; i < plan.passes.size(); ++i) {
    prof_begin(st);
    hipError_t e = launch_block(st->dt, st->amps, st->scales, plan.passes[i], (const BlkPass*)(dev + lay.o_geoms) + i, bd,
                                st->stream);
    prof_end(st);
    if (e != hipSuccess) return hip_fail(e, "tile pass launch");
    st->bytes += full_pass_bytes(st);
  }
  return JUQCS_OK;
}

// Defaults measured on MI355X for layered circuits (2^b-amplitude tiles,
// chunks of 2^L contiguous amplitudes).
void default_tile_bits(juqcs_dtype dt, int B, int* L, int* b) {
  if (dt == JUQCS_C128) {
    *b = 13;
    *L = 5;
  } else if (dt == JUQCS_C64) {
    *b = 13;
    *L = 7;
  } else {
    *b = 13;
    *L = std::max(B, 7);
  }
}

// Modelled duration (ms) of a tile plan on MI355X: a pass costs the longer of
// its HBM traffic and its on-chip ops (the pipelined kernels overlap the
// two).  Per-pass and per-op figures are measured durations per 2^30
// amplitudes with the fixed-size kernels.
double tile_plan_ms(const TilePlan& p, juqcs_dtype dt, int n) {
  struct Costs {
    double mem, dense1, dense2, diag2, dense3, dense4;
  };
  static constexpr Costs kC128{7.9, 0.50, 0.70, 0.45, 1.33, 4.0};
  static constexpr Costs kC64{4.0, 0.34, 0.56, 0.40, 1.20, 3.0};
  static constexpr Costs kEnc2{4.8, 0.34, 0.56, 0.40, 1.20, 3.0};
  const Costs& c = dt == JUQCS_C128 ? kC128 : dt == JUQCS_C64 ? kC64 : kEnc2;
  double total = 0.0;
  for (const TilePass& ps : p.passes) {
    double ops = 0.0;
    for (int o = 0; o < ps.op_count; ++o) {
      switch (p.ops[ps.op_begin + o].kind) {
        case TOP_DENSE1: ops += c.dense1; break;
        case TOP_DENSE2: ops += c.dense2; break;
        case TOP_DIAG2:
        case TOP_PERM: ops += c.diag2; break;
        case TOP_DENSE3: ops += c.dense3; break;
        default: ops += c.dense4; break;
      }
    }
    total += std::max(c.mem, ops);
  }
  return total * std::ldexp(1.0, n - 30);
}

// pass_gates: > 0 caps the gates per pass, -1 lifts the cap, 0 is the
// planner's choice: no cap for register-resident passes of C128 and C64 (ms on
// 31 qubits, 16 brick layers in C64: 157.2 without, 152.4 at 140 gates, 157.7
// at 100, 171.8 at 60; 28 qubits 17.6, 17.9, 18.4, 20.8; 30 qubits, 20 layers
// in C128 153.3, 154.5, 160.5, 177.8; random pairs and mixed gates within 3%
// down to 80; the cost model does not tell these apart: it would take 100) and
// for C128; for other C64 passes and ENC2 the cap that the cost model prefers.
// relabel >= 0: plans may move qubits onto the low physical bits between
// passes (the layout st->phys follows); -1: the data stay where they are
// (explicit layout moves rely on that).
juqcs_status tile_gates(juqcs_state* st, const std::vector<Gate>& gates, int L, int b,
                        int64_t* passes, int kin = 0, int pass_gates = -1, int relabel = -1) {
  const int maxb = tile_max_bits(st->dt);
  {  // each of the two defaults on its own
    int dL = 0, db = 0;
    default_tile_bits(st->dt, st->B, &dL, &db);
    if (b <= 0) b = db;
    if (L <= 0) L = std::min(dL, b);
  }
  if (b > maxb) return fail(JUQCS_ERR_ARG, "tile_bits above the LDS limit");
  if (L > b) return fail(JUQCS_ERR_ARG, "low_bits > tile_bits");
  if (b - L > kMaxGather) return fail(JUQCS_ERR_ARG, "too many gathered tile bits");
  if (st->dt == JUQCS_ENC2 && L < st->B) L = st->B;
  if (st->dt == JUQCS_ENC2 && b < L + 2) b = std::min(maxb, L + 2);  // room for two gathered qubits
  if (st->n > b && b - L < 2)
    return fail(JUQCS_ERR_ARG, "a tile needs at least two gathered bits (tile_bits >= low_bits + 2)");
  // No fusion width asked for.  Register-resident passes hold up to 2^24 times
  // an amplitude on the way, so states scaled up to near the end of their range
  // take the fused ones.
  const bool block = kin <= 0 && st->size <= (st->dt == JUQCS_C128 ? 0x1p990 : 0x1p100);
  if (kin <= 0) kin = 3;
  if (kin > 4) return fail(JUQCS_ERR_ARG, "in-pass fusion width must be 1..4");
  if (pass_gates < -1) return fail(JUQCS_ERR_ARG, "pass_gates must be >= -1");
  if (relabel < -1 || relabel > 1) return fail(JUQCS_ERR_ARG, "relabel must be -1, 0 or 1");
  if (gates.empty()) {  // (a register-resident plan of no gates writes the state as it is)
    if (passes) *passes = 0;
    return JUQCS_OK;
  }
  const bool fresh = st->fresh;
  st->fresh = false;
  const int cap = tile_mat_cap(st->dt, std::min(b, st->n));
  const int mcap = tile_mma_cap(st->dt, std::min(b, st->n));
  const int l = std::min(L, st->n);
  const bool rl = relabel >= 0;
  std::vector<int> moved;  // moved[p]: physical bit that the qubit at bit p ends on
  if (block && block_sized(st->dt, std::min(b, st->n))) {
    BlkPlan bp;
    if (plan_block(st->n, l, b, gates, st->dt == JUQCS_C128, std::max(pass_gates, 0), rl, &bp, &moved,
                   fresh ? &st->basis : nullptr) &&
        fits_ring(st, bp)) {
      if (passes) *passes = (int64_t)bp.passes.size();
      if (juqcs_status rc = run_block_plan(st, bp)) return rc;
      if (rl)
        for (int q = 0; q < st->n; ++q) st->phys[q] = moved[st->phys[q]];
      return JUQCS_OK;
    }
  }
  TilePlan plan;
  if (pass_gates != 0 || st->dt == JUQCS_C128) {
    plan_tiles(st->n, l, b, st->B, gates, &plan, kin, cap, std::max(pass_gates, 0), mcap, rl, &moved);
  } else {
    double best = 0.0;
    for (int take : {0, 90, 60, 40}) {
      if (take > 0 && (int64_t)gates.size() <= take) continue;  // same as no cap
      TilePlan cand;
      std::vector<int> mv;
      plan_tiles(st->n, l, b, st->B, gates, &cand, kin, cap, take, mcap, rl, &mv);
      const double ms = tile_plan_ms(cand, st->dt, st->n);
      if (plan.passes.empty() || ms < best) {
        best = ms;
        plan = std::move(cand);
        moved = std::move(mv);
      }
    }
  }
  if (plan.gates != (int64_t)gates.size())
    return fail(JUQCS_ERR_UNSUPPORTED, "a gate does not fit any tile of this geometry");
  if (passes) *passes = (int64_t)plan.passes.size();
  BlkPlan bp;
  const bool codes = block && st->dt == JUQCS_ENC2 && block_codes_sized(st->B, std::min(b, st->n)) &&
                     block_tile_plan(plan, st->B, &bp) && fits_ring(st, bp);
  if (juqcs_status rc = codes ? run_block_plan(st, bp) : run_tile_plan(st, plan)) return rc;
  if (rl)
    for (int q = 0; q < st->n; ++q) st->phys[q] = moved[st->phys[q]];
  return JUQCS_OK;
}

// Gate on physical qubits.
Gate make_gate1(int t, const C u[4]) {
  Gate g{};
  g.nq = 1;
  g.q[0] = t;
  g.q[1] = -1;
  for (int i = 0; i < 4; ++i) g.m[i] = u[i];
  g.diag = is_diag2(u);
  return g;
}

// Fraction of the state a per-gate pass reads and writes when the given
// physical bits must be 1: the per-gate kernels move whole runs of 1 KiB,
// so only bits at or above a run (64 C128 / 128 C64 amplitudes) select.
double touched(const juqcs_state* st, uint64_t mask) {
  const int rb = st->dt == JUQCS_C128 ? 6 : 7;
  double f = 1.0;
  for (int q = rb; q < 64; ++q)
    if ((mask >> q) & 1) f *= 0.5;
  return f;
}

juqcs_status apply_gate_plain(juqcs_state* st, const Gate& g0) {
  hipError_t e = hipSuccess;
  st->fresh = false;
  Gate g = g0;
  if (g.nq == 1 && g.diag && !is_one(g.m[0]) && (g.m[0].re != 0.0 || g.m[0].im != 0.0)) {
    // diag(a, b) = a diag(1, b / a): the factor a goes into the state's FP64
    // global factor, and only the half with the target bit set is touched
    const C a = g.m[0], b = g.m[3];
    const double den = a.re * a.re + a.im * a.im;
    g.m[0] = C{1.0, 0.0};
    g.m[3] = C{(b.re * a.re + b.im * a.im) / den, (b.im * a.re - b.re * a.im) / den};
    st->gf = cmul(st->gf, a);
  }
  if (st->dt == JUQCS_ENC2) {
    if (g.nq == 1 && g.diag && is_one(g.m[0]) && is_one(g.m[3])) return JUQCS_OK;
    std::vector<Gate> one{g};
    return tile_gates(st, one, 0, 0, nullptr);
  }
  const double full = full_pass_bytes(st);
  prof_begin(st);
  if (g.nq == 1) {
    const C* u = g.m;
    const C d1 = u[3];
    if (g.diag && is_one(u[0])) {
      if (is_one(d1)) {
        prof_end(st);
        return JUQCS_OK;  // identity (up to the global factor)
      }
      e = launch_diag(st->dt, st->amps, st->n, uint64_t(1) << g.q[0], d1, st->stream);
      st->bytes += touched(st, uint64_t(1) << g.q[0]) * full;
    } else {
      e = launch_1q(st->dt, st->amps, st->n, g.q[0], -1, u, st->stream);
      st->bytes += full;
    }
  } else {
    // controlled-U form: identity where bit q0 is clear?
    const C* m = g.m;
    bool ctrl = true;  // rows/cols with b_q0 = 0 are identity (index r = b_q0 + 2 b_q1)
    for (int r = 0; r < 4; ++r)
      for (int c = 0; c < 4; ++c) {
        const bool r0 = (r & 1) == 0, c0 = (c & 1) == 0;
        if (r0 || c0) {
          const C want = (r == c) ? C{1, 0} : C{0, 0};
          if (m[r * 4 + c].re != want.re || m[r * 4 + c].im != want.im) ctrl = false;
        }
      }
    if (ctrl) {
      const C u[4] = {m[1 * 4 + 1], m[1 * 4 + 3], m[3 * 4 + 1], m[3 * 4 + 3]};
      if (is_diag2(u) && is_one(u[0])) {
        if (is_one(u[3])) {
          prof_end(st);
          return JUQCS_OK;
        }
        const uint64_t mask = (uint64_t(1) << g.q[0]) | (uint64_t(1) << g.q[1]);
        e = launch_diag(st->dt, st->amps, st->n, mask, u[3], st->stream);
        st->bytes += touched(st, mask) * full;
      } else {
        e = launch_1q(st->dt, st->amps, st->n, g.q[1], g.q[0], u, st->stream);
        st->bytes += touched(st, uint64_t(1) << g.q[0]) * full;
      }
    } else {
      e = launch_2q(st->dt, st->amps, st->n, g.q[0], g.q[1], m, st->stream);
      st->bytes += full;
    }
  }
  prof_end(st);
  if (e != hipSuccess) return hip_fail(e, "gate launch");
  return JUQCS_OK;
}

// Real embedding of a complex K x K matrix, padded to R = max(16, 2K), stored
// transposed (At[col * R + row]), interleaved rows (row 2r+p = part p of r).
template <typename T>
std::vector<T> embed_real(const C* m, int K) {
  const int R = std::max(16, 2 * K);
  std::vector<T> at((size_t)R * R, T(0));
  for (int r = 0; r < K; ++r)
    for (int c = 0; c < K; ++c) {
      const C z = m[r * K + c];
      // rows (2r, 2r+1), cols (2c, 2c+1): [[re, -im], [im, re]]
      at[(size_t)(2 * c) * R + 2 * r] = (T)z.re;
      at[(size_t)(2 * c + 1) * R + 2 * r] = (T)(-z.im);
      at[(size_t)(2 * c) * R + 2 * r + 1] = (T)z.im;
      at[(size_t)(2 * c + 1) * R + 2 * r + 1] = (T)z.re;
    }
  return at;
}

juqcs_status apply_fused_phys(juqcs_state* st, int k, const int* targets, const C* m,
                              juqcs_mma mode) {
  st->fresh = false;
  if (mode == JUQCS_MMA_AUTO) mode = st->dt == JUQCS_C128 ? JUQCS_MMA_FP64 : JUQCS_MMA_FP32;
  if (st->dt == JUQCS_C128 && mode != JUQCS_MMA_FP64)
    return fail(JUQCS_ERR_DTYPE, "C128 states use FP64 matrix cores");
  if (st->dt == JUQCS_C64 && mode == JUQCS_MMA_FP64)
    return fail(JUQCS_ERR_DTYPE, "C64 states use FP32/BF16 matrix cores");
  const int K = 1 << k;
  char* dev = nullptr;
  juqcs_status rc;
  if (mode == JUQCS_MMA_FP64) {
    std::vector<double> at = embed_real<double>(m, K);
    rc = upload(st, at.data(), at.size() * sizeof(double), &dev);
  } else {
    std::vector<float> at = embed_real<float>(m, K);
    rc = upload(st, at.data(), at.size() * sizeof(float), &dev);
  }
  if (rc != JUQCS_OK) return rc;
  prof_begin(st);
  hipError_t e = launch_fused(st->dt, st->amps, st->n, k, targets, dev, mode, st->stream);
  prof_end(st);
  if (e != hipSuccess) return hip_fail(e, "fused launch");
  st->bytes += full_pass_bytes(st);
  st->mma_flops += 8.0 * (double)K * std::ldexp(1.0, st->n);
  return JUQCS_OK;
}

juqcs_status decode_all(juqcs_state* st, const juqcs_gate* gates, size_t count,
                        std::vector<Gate>* out) {
  out->resize(count);
  std::string err;
  for (size_t i = 0; i < count; ++i) {
    if (!decode_gate(gates[i], st->n, &(*out)[i], &err)) {
      const bool numeric = err.find("non-finite") != std::string::npos;
      const bool qubit = err.find("qubit") != std::string::npos;
      return fail(numeric ? JUQCS_ERR_NUMERIC : qubit ? JUQCS_ERR_QUBIT : JUQCS_ERR_ARG,
                  "gate " + std::to_string(i) + ": " + err);
    }
    Gate& g = (*out)[i];
    for (int j = 0; j < g.nq; ++j) g.q[j] = st->phys[g.q[j]];
  }
  return JUQCS_OK;
}

juqcs_status sync(juqcs_state* st) {
  hipError_t e = hipStreamSynchronize(st->stream);
  if (e != hipSuccess) return hip_fail(e, "stream synchronize");
  e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "device");
  return JUQCS_OK;
}

// Physical data move: SWAP gates on physical bit pairs, run as tile passes.
juqcs_status move_layout(juqcs_state* st, const int* target) {
  std::vector<int> cur(st->phys, st->phys + st->n);
  std::vector<Gate> swaps;
  // where[p] = logical qubit currently at physical bit p
  std::vector<int> where(st->n);
  for (int q = 0; q < st->n; ++q) where[cur[q]] = q;
  for (int q = 0; q < st->n; ++q) {
    const int from = cur[q], to = target[q];
    if (from == to) continue;
    Gate g{};
    g.nq = 2;
    g.q[0] = from;
    g.q[1] = to;
    for (int i = 0; i < 16; ++i) g.m[i] = C{0, 0};
    g.m[0] = g.m[1 * 4 + 2] = g.m[2 * 4 + 1] = g.m[15] = C{1, 0};  // SWAP
    g.diag = false;
    swaps.push_back(g);
    const int other = where[to];
    cur[other] = from;
    where[from] = other;
    cur[q] = to;
    where[to] = q;
  }
  if (!swaps.empty()) {
    juqcs_status rc = tile_gates(st, swaps, 0, 0, nullptr);
    if (rc != JUQCS_OK) return rc;
  }
  for (int q = 0; q < st->n; ++q) st->phys[q] = target[q];
  return JUQCS_OK;
}

juqcs_status run_planned(juqcs_state* st, const std::vector<Gate>& g, int mode,
                         juqcs_plan_opts* o);

// ---------------------------------------------------------------- tuning --
// Circuit structure key: FNV-1a over n, the amplitude type, the ENC2 block
// bits and every gate's op and qubits.
uint64_t structure_key(const juqcs_state* st, const juqcs_gate* gates, size_t count) {
  uint64_t h = 1469598103934665603ull;
  auto mix = [&](int64_t v) {
    for (int i = 0; i < 8; ++i) {
      h ^= (uint64_t)((v >> (8 * i)) & 0xff);
      h *= 1099511628211ull;
    }
  };
  mix(st->n);
  mix(st->dt);
  mix(st->B);
  for (size_t i = 0; i < count; ++i) {
    mix(gates[i].op);
    mix(gates[i].q0);
    mix(gates[i].q1);
  }
  return h;
}

struct TuneEntry {
  juqcs_tune_result r;
  int n = 0, dtype = 0;
};
std::mutex g_tune_mu;
std::map<uint64_t, TuneEntry> g_tune;

bool tuned_options(uint64_t key, juqcs_plan_opts* o) {
  std::lock_guard<std::mutex> lock(g_tune_mu);
  auto it = g_tune.find(key);
  if (it == g_tune.end()) return false;
  const juqcs_plan_opts& t = it->second.r.opts;
  o->mode = t.mode;
  o->fuse_k = t.fuse_k;
  o->mma = t.mma;
  o->tile_bits = t.tile_bits;
  o->low_bits = t.low_bits;
  o->pass_gates = t.pass_gates;
  o->relabel = t.relabel;
  return true;
}

}  // namespace

extern "C" {

const char* juqcs_last_error(void) { return juqcs::g_last_error.c_str(); }

const char* juqcs_version(void) { return "juqcs_gpu 0.1 (gfx950)"; }

juqcs_status juqcs_state_bytes(int n, juqcs_dtype dt, int block_bits, size_t* amp_bytes,
                               size_t* scale_bytes, size_t* work_bytes) {
  if (n < 1 || n > 40) return fail(JUQCS_ERR_ARG, "n must be in [1, 40]");
  if (dt != JUQCS_C128 && dt != JUQCS_C64 && dt != JUQCS_ENC2)
    return fail(JUQCS_ERR_DTYPE, "unknown dtype");
  int B = block_bits == 0 ? kDefaultBlockBits : block_bits;
  if (dt == JUQCS_ENC2) {
    if (B < 3 || B > 12) return fail(JUQCS_ERR_ARG, "block_bits must be in [3, 12]");
    if (n < B) return fail(JUQCS_ERR_ARG, "ENC2 needs n >= block_bits");
  }
  const uint64_t count = uint64_t(1) << n;
  if (amp_bytes) *amp_bytes = (size_t)(count * amp_size(dt));
  if (scale_bytes) *scale_bytes = dt == JUQCS_ENC2 ? (size_t)(4 * (count >> B)) : 0;
  if (work_bytes) *work_bytes = kWorkBytes;
  return JUQCS_OK;
}

juqcs_status juqcs_state_create(juqcs_state** out, int n, juqcs_dtype dt, int block_bits,
                                void* d_amps, size_t amp_bytes, void* d_scales,
                                size_t scale_bytes, void* d_work, size_t work_bytes,
                                void* hip_stream) {
  if (!out) return fail(JUQCS_ERR_ARG, "null output pointer");
  *out = nullptr;
  size_t need_a = 0, need_s = 0, need_w = 0;
  juqcs_status rc = juqcs_state_bytes(n, dt, block_bits, &need_a, &need_s, &need_w);
  if (rc != JUQCS_OK) return rc;
  if (!d_amps) return fail(JUQCS_ERR_ARG, "null amplitude buffer");
  if (((uintptr_t)d_amps & 15) != 0) return fail(JUQCS_ERR_ARG, "amplitudes not 16-byte aligned");
  if (amp_bytes < need_a) return fail(JUQCS_ERR_SIZE, "amplitude buffer too small");
  if (dt == JUQCS_ENC2) {
    if (!d_scales) return fail(JUQCS_ERR_ARG, "null scale buffer");
    if (scale_bytes < need_s) return fail(JUQCS_ERR_SIZE, "scale buffer too small");
  }
  if (!d_work) return fail(JUQCS_ERR_ARG, "null workspace (juqcs_state_bytes gives its size)");
  if (((uintptr_t)d_work & 255) != 0) return fail(JUQCS_ERR_ARG, "workspace not 256-byte aligned");
  if (work_bytes < need_w) return fail(JUQCS_ERR_SIZE, "workspace too small");
  juqcs_state* st = new juqcs_state();
  st->n = n;
  st->dt = dt;
  st->B = dt == JUQCS_ENC2 ? (block_bits == 0 ? kDefaultBlockBits : block_bits) : 0;
  st->amps = d_amps;
  st->scales = d_scales;
  st->stream = (hipStream_t)hip_stream;
  st->work = (char*)d_work;
  st->work_bytes = work_bytes;
  st->ring = kRingOff;
  for (int q = 0; q < 64; ++q) st->phys[q] = q;
  *out = st;
  return JUQCS_OK;
}

juqcs_status juqcs_state_destroy(juqcs_state* st) {
  if (!st) return JUQCS_OK;
  delete st;
  return JUQCS_OK;
}

juqcs_status juqcs_state_set_stream(juqcs_state* st, void* hip_stream) {
  if (check_state(st)) return JUQCS_ERR_ARG;
  st->stream = (hipStream_t)hip_stream;
  return JUQCS_OK;
}

juqcs_status juqcs_state_init(juqcs_state* st, uint64_t basis_index) {
  if (check_state(st)) return JUQCS_ERR_ARG;
  if (st->n < 64 && (basis_index >> st->n) != 0) return fail(JUQCS_ERR_ARG, "basis index >= 2^n");
  for (int q = 0; q < 64; ++q) st->phys[q] = q;
  st->gf = C{1.0, 0.0};
  st->size = 1.0;
  st->fresh = true;
  st->basis = basis_index;
  hipError_t e = launch_init(st->dt, st->amps, st->scales, st->n, st->B, basis_index, st->stream);
  if (e != hipSuccess) return hip_fail(e, "init launch");
  return JUQCS_OK;
}

juqcs_status juqcs_apply_1q(juqcs_state* st, int t, const double u[8]) {
  if (check_state(st)) return JUQCS_ERR_ARG;
  if (!u) return fail(JUQCS_ERR_ARG, "null matrix");
  if (juqcs_status rc = check_qubit(st, t)) return rc;
  if (!finite8(u, 8)) return fail(JUQCS_ERR_NUMERIC, "non-finite matrix entry");
  const C m[4] = {{u[0], u[1]}, {u[2], u[3]}, {u[4], u[5]}, {u[6], u[7]}};
  return apply_gate_plain(st, make_gate1(st->phys[t], m));
}

juqcs_status juqcs_apply_controlled(juqcs_state* st, int c, int t, const double u[8]) {
  if (check_state(st)) return JUQCS_ERR_ARG;
  if (!u) return fail(JUQCS_ERR_ARG, "null matrix");
  if (juqcs_status rc = check_qubit(st, c)) return rc;
  if (juqcs_status rc = check_qubit(st, t)) return rc;
  if (c == t) return fail(JUQCS_ERR_QUBIT, "control equals target");
  if (!finite8(u, 8)) return fail(JUQCS_ERR_NUMERIC, "non-finite matrix entry");
  Gate g{};
  g.nq = 2;
  g.q[0] = st->phys[c];
  g.q[1] = st->phys[t];
  for (int i = 0; i < 16; ++i) g.m[i] = C{0, 0};
  g.m[0] = g.m[2 * 4 + 2] = C{1, 0};  // index b_c + 2 b_t: control clear -> identity
  g.m[1 * 4 + 1] = C{u[0], u[1]};
  g.m[1 * 4 + 3] = C{u[2], u[3]};
  g.m[3 * 4 + 1] = C{u[4], u[5]};
  g.m[3 * 4 + 3] = C{u[6], u[7]};
  g.diag = false;
  return apply_gate_plain(st, g);
}

juqcs_status juqcs_apply_2q(juqcs_state* st, int q0, int q1, const double m[32]) {
  if (check_state(st)) return JUQCS_ERR_ARG;
  if (!m) return fail(JUQCS_ERR_ARG, "null matrix");
  if (juqcs_status rc = check_qubit(st, q0)) return rc;
  if (juqcs_status rc = check_qubit(st, q1)) return rc;
  if (q0 == q1) return fail(JUQCS_ERR_QUBIT, "repeated qubit");
  if (!finite8(m, 32)) return fail(JUQCS_ERR_NUMERIC, "non-finite matrix entry");
  Gate g{};
  g.nq = 2;
  g.q[0] = st->phys[q0];
  g.q[1] = st->phys[q1];
  for (int i = 0; i < 16; ++i) g.m[i] = C{m[2 * i], m[2 * i + 1]};
  g.diag = false;
  return apply_gate_plain(st, g);
}

juqcs_status juqcs_apply_fused_k(juqcs_state* st, int k, const int* targets, const double* m,
                                 juqcs_mma mode) {
  if (check_state(st)) return JUQCS_ERR_ARG;
  if (!targets || !m) return fail(JUQCS_ERR_ARG, "null targets or matrix");
  if (k < 1 || k > 6 || k > st->n) return fail(JUQCS_ERR_ARG, "k must be in [1, min(6, n)]");
  if (st->dt == JUQCS_ENC2) return fail(JUQCS_ERR_DTYPE, "fused blocks need C128 or C64");
  if (mode < JUQCS_MMA_FP64 || mode > JUQCS_MMA_AUTO) return fail(JUQCS_ERR_ARG, "bad mma mode");
  int phys[6];
  for (int j = 0; j < k; ++j) {
    if (juqcs_status rc = check_qubit(st, targets[j])) return rc;
    for (int i = 0; i < j; ++i)
      if (targets[i] == targets[j]) return fail(JUQCS_ERR_QUBIT, "repeated target");
    phys[j] = st->phys[targets[j]];
  }
  const int K = 1 << k;
  if (!finite8(m, 2 * K * K)) return fail(JUQCS_ERR_NUMERIC, "non-finite matrix entry");
  std::vector<C> mm(K * K);
  for (int i = 0; i < K * K; ++i) mm[i] = C{m[2 * i], m[2 * i + 1]};
  return apply_fused_phys(st, k, phys, mm.data(), mode);
}

juqcs_status juqcs_run_circuit(juqcs_state* st, const juqcs_gate* gates, size_t count,
                               juqcs_plan_opts* opts) {
  if (check_state(st)) return JUQCS_ERR_ARG;
  if (count > 0 && !gates) return fail(JUQCS_ERR_ARG, "null gate array");
  juqcs_plan_opts dflt{};
  dflt.mode = JUQCS_PLAN_AUTO;
  juqcs_plan_opts* o = opts ? opts : &dflt;
  if (o->mode < JUQCS_PLAN_PLAIN || o->mode > JUQCS_PLAN_AUTO)
    return fail(JUQCS_ERR_ARG, "bad plan mode");
  std::vector<Gate> g;
  if (juqcs_status rc = decode_all(st, gates, count, &g)) return rc;
  juqcs_plan_opts tuned = *o;
  if (o->mode == JUQCS_PLAN_AUTO && tuned_options(structure_key(st, gates, count), &tuned)) {
    tuned.profile = o->profile;
    juqcs_status rc = juqcs_run_circuit(st, gates, count, &tuned);
    o->passes = tuned.passes;
    o->gates = tuned.gates;
    o->kernel_ms = tuned.kernel_ms;
    o->bytes = tuned.bytes;
    o->flops = tuned.flops;
    o->mma_flops = tuned.mma_flops;
    return rc;
  }
  int mode = o->mode == JUQCS_PLAN_AUTO ? JUQCS_PLAN_TILE : o->mode;
  if (st->dt == JUQCS_ENC2) mode = JUQCS_PLAN_TILE;
  o->gates = (int64_t)count;
  o->passes = 0;
  o->kernel_ms = 0.0;
  o->flops = 0.0;
  for (const Gate& x : g) o->flops += gate_flops(x) * std::ldexp(1.0, st->n);
  st->bytes = 0.0;
  st->mma_flops = 0.0;
  st->profiling = o->profile != 0;
  juqcs_status rc = run_planned(st, g, mode, o);
  if (st->profiling) o->kernel_ms = prof_collect(st);
  st->profiling = false;
  o->bytes = st->bytes;
  o->mma_flops = st->mma_flops;
  return rc;
}

juqcs_status juqcs_autotune(juqcs_state* st, const juqcs_gate* gates, size_t count,
                            juqcs_tune_result* out) {
  if (check_state(st)) return JUQCS_ERR_ARG;
  if (!out) return fail(JUQCS_ERR_ARG, "null output");
  if (count > 0 && !gates) return fail(JUQCS_ERR_ARG, "null gate array");
  *out = juqcs_tune_result{};
  hipEvent_t a = nullptr, b = nullptr;
  hipError_t e = hipEventCreate(&a);
  if (e == hipSuccess) e = hipEventCreate(&b);
  if (e != hipSuccess) return hip_fail(e, "hipEventCreate");
  juqcs_status err = JUQCS_OK;
  int trials = 0;
  const char* verbose = std::getenv("JUQCS_TUNE_VERBOSE");
  const bool say = verbose && verbose[0] == '1';
  // one timed run from |0...0>; infinite if the options are rejected
  auto time_run = [&](juqcs_plan_opts o) {
    o.profile = 0;
    if (err != JUQCS_OK) return 1e300;  // no more device work after a device error
    if (juqcs_state_init(st, 0) != JUQCS_OK) return 1e300;
    if (hipEventRecord(a, st->stream) != hipSuccess) return 1e300;
    const juqcs_status rc = juqcs_run_circuit(st, gates, count, &o);
    (void)hipEventRecord(b, st->stream);
    (void)hipEventSynchronize(b);
    if (rc == JUQCS_ERR_HIP) err = rc;
    float ms = 0.0f;
    if (rc != JUQCS_OK || hipEventElapsedTime(&ms, a, b) != hipSuccess) return 1e300;
    ++trials;
    if (say)
      std::fprintf(stderr, "juqcs_autotune: mode %d fuse_k %d tile_bits %d low_bits %d pass_gates %d "
                   "relabel %d: %.3f ms\n", o.mode, o.fuse_k, o.tile_bits, o.low_bits, o.pass_gates,
                   o.relabel, ms);
    return (double)ms;
  };
  // the better of two runs (the first run of a kernel also pays for loading it)
  auto measure = [&](const juqcs_plan_opts& o, double best) {
    double t = time_run(o);
    if (t < 2.0 * best) t = std::min(t, time_run(o));
    return t;
  };
  juqcs_plan_opts cur{};
  cur.mode = JUQCS_PLAN_TILE;
  const double t_default = measure(cur, 1e300);
  double best = t_default;
  juqcs_plan_opts bo = cur;
  // a candidate must win by more than the run-to-run spread (about 1%)
  constexpr double kMargin = 0.98;
  auto consider = [&](juqcs_plan_opts o) {
    const double t = measure(o, best);
    if (t < kMargin * best) {
      best = t;
      bo = o;
    }
  };
  const bool c128 = st->dt == JUQCS_C128, enc2 = st->dt == JUQCS_ENC2;
  const std::vector<int> low_v = c128 ? std::vector<int>{4, 5, 6} : std::vector<int>{5, 6, 7, 8};
  const std::vector<int> tb_v = c128 ? std::vector<int>{12, 13} : std::vector<int>{12, 13, 14};
  const std::vector<int> cap_v = c128 ? std::vector<int>{-1, 60, 40, 25} : std::vector<int>{-1, 90, 60, 40};
  // coordinate descent over the tile options, each from the best so far
  if (!enc2)
    for (int v : low_v) {
      juqcs_plan_opts o = bo;
      o.low_bits = v;
      consider(o);
    }
  for (int v : tb_v) {
    juqcs_plan_opts o = bo;
    o.tile_bits = v;
    if (o.low_bits == 0 && !enc2) o.low_bits = c128 ? 5 : 7;
    consider(o);
  }
  for (int v : {2, 4}) {
    juqcs_plan_opts o = bo;
    o.fuse_k = v;
    consider(o);
  }
  for (int v : cap_v) {
    juqcs_plan_opts o = bo;
    o.pass_gates = v;
    consider(o);
  }
  {
    juqcs_plan_opts o = bo;
    o.relabel = -1;
    consider(o);
  }
  // dense fused blocks on the matrix cores (full precision of the state)
  if (!enc2)
    for (int k = 3; k <= 6 && k <= st->n; ++k) {
      juqcs_plan_opts o{};
      o.mode = JUQCS_PLAN_FUSED;
      o.fuse_k = k;
      o.mma = JUQCS_MMA_AUTO;
      consider(o);
    }
  // one pass per gate: only where that cannot take long
  if (!enc2 && (st->n <= 24 || count <= 32)) {
    juqcs_plan_opts o{};
    o.mode = JUQCS_PLAN_PLAIN;
    consider(o);
  }
  // confirm a change against the defaults: three runs of each, interleaved,
  // medians compared
  double t_def = t_default;
  const bool changed = bo.mode != cur.mode || bo.fuse_k != cur.fuse_k || bo.mma != cur.mma ||
                       bo.tile_bits != cur.tile_bits || bo.low_bits != cur.low_bits ||
                       bo.pass_gates != cur.pass_gates || bo.relabel != cur.relabel;
  if (best < 1e299 && changed) {
    double tb[3], td[3];
    for (int i = 0; i < 3; ++i) {
      td[i] = time_run(cur);
      tb[i] = time_run(bo);
    }
    std::sort(tb, tb + 3);
    std::sort(td, td + 3);
    t_def = td[1];
    best = tb[1];
    if (!(best < 0.99 * t_def)) {
      bo = cur;
      best = t_def;
    }
  }
  (void)hipEventDestroy(a);
  (void)hipEventDestroy(b);
  if (err != JUQCS_OK) return err;
  if (!(best < 1e299)) return fail(JUQCS_ERR_UNSUPPORTED, "no planner option ran this circuit");
  out->opts = bo;
  out->opts.profile = 0;
  out->ms = best;
  out->default_ms = t_def;
  out->trials = trials;
  out->key = structure_key(st, gates, count);
  std::lock_guard<std::mutex> lock(g_tune_mu);
  TuneEntry& te = g_tune[out->key];
  te.r = *out;
  te.n = st->n;
  te.dtype = st->dt;
  return JUQCS_OK;
}

juqcs_status juqcs_tune_lookup(const juqcs_state* st, const juqcs_gate* gates, size_t count,
                               juqcs_tune_result* out) {
  if (check_state(st)) return JUQCS_ERR_ARG;
  if (!out || (count > 0 && !gates)) return fail(JUQCS_ERR_ARG, "null argument");
  const uint64_t key = structure_key(st, gates, count);
  std::lock_guard<std::mutex> lock(g_tune_mu);
  auto it = g_tune.find(key);
  if (it == g_tune.end()) return fail(JUQCS_ERR_ARG, "no tuning entry for this circuit");
  *out = it->second.r;
  return JUQCS_OK;
}

juqcs_status juqcs_tune_clear(void) {
  std::lock_guard<std::mutex> lock(g_tune_mu);
  g_tune.clear();
  return JUQCS_OK;
}

juqcs_status juqcs_tune_save(const char* path) {
  if (!path) return fail(JUQCS_ERR_ARG, "null path");
  std::lock_guard<std::mutex> lock(g_tune_mu);
  FILE* f = std::fopen(path, "w");
  if (!f) return fail(JUQCS_ERR_ARG, std::string("cannot write ") + path);
  std::fprintf(f, "{\"juqcs_tune\": 1, \"entries\": [\n");
  size_t i = 0;
  for (const auto& kv : g_tune) {
    const juqcs_tune_result& r = kv.second.r;
    std::fprintf(f,
                 " {\"key\": \"%016llx\", \"n\": %d, \"dtype\": %d, \"mode\": %d, \"fuse_k\": %d, "
                 "\"mma\": %d, \"tile_bits\": %d, \"low_bits\": %d, \"pass_gates\": %d, "
                 "\"relabel\": %d, \"ms\": %.6f, \"default_ms\": %.6f, \"trials\": %d}%s\n",
                 (unsigned long long)kv.first, kv.second.n, kv.second.dtype, r.opts.mode, r.opts.fuse_k,
                 r.opts.mma, r.opts.tile_bits, r.opts.low_bits, r.opts.pass_gates, r.opts.relabel, r.ms,
                 r.default_ms, r.trials, ++i < g_tune.size() ? "," : "");
  }
  std::fprintf(f, "]}\n");
  const bool ok = std::fclose(f) == 0;
  if (!ok) return fail(JUQCS_ERR_ARG, std::string("cannot write ") + path);
  return JUQCS_OK;
}

juqcs_status juqcs_tune_load(const char* path) {
  if (!path) return fail(JUQCS_ERR_ARG, "null path");
  FILE* f = std::fopen(path, "r");
  if (!f) return fail(JUQCS_ERR_ARG, std::string("cannot read ") + path);
  std::string text;
  char buf[4096];
  size_t got;
  while ((got = std::fread(buf, 1, sizeof buf, f)) > 0) text.append(buf, got);
  std::fclose(f);
  if (text.find("\"juqcs_tune\"") == std::string::npos) return fail(JUQCS_ERR_ARG, "not a tuning table");
  // every object after "entries": numbers by name, the key as hex text
  auto number = [](const std::string& obj, const char* name, double* v) {
    const std::string pat = std::string("\"") + name + "\":";
    const size_t at = obj.find(pat);
    if (at == std::string::npos) return false;
    char* end = nullptr;
    *v = std::strtod(obj.c_str() + at + pat.size(), &end);
    return end != obj.c_str() + at + pat.size();
  };
  std::map<uint64_t, TuneEntry> add;
  size_t p = text.find("\"entries\"");
  if (p == std::string::npos) return fail(JUQCS_ERR_ARG, "tuning table without entries");
  while ((p = text.find('{', p)) != std::string::npos) {
    const size_t q = text.find('}', p);
    if (q == std::string::npos) return fail(JUQCS_ERR_ARG, "malformed tuning table");
    const std::string obj = text.substr(p, q - p + 1);
    p = q + 1;
    const size_t kat = obj.find("\"key\": \"");
    if (kat == std::string::npos) return fail(JUQCS_ERR_ARG, "tuning entry without key");
    const uint64_t key = std::strtoull(obj.c_str() + kat + 8, nullptr, 16);
    double v[12];
    const char* names[12] = {"n", "dtype", "mode", "fuse_k", "mma", "tile_bits", "low_bits",
                             "pass_gates", "relabel", "ms", "default_ms", "trials"};
    for (int i = 0; i < 12; ++i)
      if (!number(obj, names[i], &v[i])) return fail(JUQCS_ERR_ARG, std::string("tuning entry without ") + names[i]);
    if (v[2] < JUQCS_PLAN_PLAIN || v[2] > JUQCS_PLAN_FUSED) return fail(JUQCS_ERR_ARG, "tuning entry with a bad mode");
    TuneEntry te;
    te.n = (int)v[0];
    te.dtype = (int)v[1];
    te.r.opts.mode = (int32_t)v[2];
    te.r.opts.fuse_k = (int32_t)v[3];
    te.r.opts.mma = (int32_t)v[4];
    te.r.opts.tile_bits = (int32_t)v[5];
    te.r.opts.low_bits = (int32_t)v[6];
    te.r.opts.pass_gates = (int32_t)v[7];
    te.r.opts.relabel = (int32_t)v[8];
    te.r.ms = v[9];
    te.r.default_ms = v[10];
    te.r.trials = (int32_t)v[11];
    te.r.key = key;
    add[key] = te;
  }
  std::lock_guard<std::mutex> lock(g_tune_mu);
  for (auto& kv : add) g_tune[kv.first] = kv.second;
  return JUQCS_OK;
}

}  // extern "C"

namespace {

juqcs_status run_planned(juqcs_state* st, const std::vector<Gate>& g, int mode,
                         juqcs_plan_opts* o) {
  if (mode == JUQCS_PLAN_PLAIN) {
    for (const Gate& x : g) {
      if (juqcs_status rc = apply_gate_plain(st, x)) return rc;
      ++o->passes;
    }
    return JUQCS_OK;
  }
  if (mode == JUQCS_PLAN_TILE) {
    int64_t passes = 0;
    juqcs_status rc =
        tile_gates(st, g, o->low_bits, o->tile_bits, &passes, o->fuse_k, o->pass_gates, o->relabel);
    o->passes = passes;
    return rc;
  }
  // FUSED
  int k = o->fuse_k == 0 ? 5 : o->fuse_k;
  if (k < 1 || k > 6) return fail(JUQCS_ERR_ARG, "fuse_k must be in [1, 6]");
  k = std::min(k, st->n);
  juqcs_mma mode_mma = (juqcs_mma)o->mma;
  if (mode_mma == JUQCS_MMA_FP64 && st->dt == JUQCS_C64) mode_mma = JUQCS_MMA_FP32;
  std::vector<FusedBlock> blocks;
  plan_fused(st->n, k, g, &blocks);
  for (const FusedBlock& b : blocks) {
    if (juqcs_status rc = apply_fused_phys(st, (int)b.targets.size(), b.targets.data(),
                                           b.m.data(), mode_mma))
      return rc;
    ++o->passes;
  }
  return JUQCS_OK;
}

}  // namespace

extern "C" {

juqcs_status juqcs_amplitudes_device(juqcs_state* st, const uint64_t* d_idx, size_t count,
                                     double* d_out) {
  if (check_state(st)) return JUQCS_ERR_ARG;
  if (count > 0 && (!d_idx || !d_out)) return fail(JUQCS_ERR_ARG, "null index or output");
  int8_t phys[64];
  for (int q = 0; q < 64; ++q) phys[q] = (int8_t)st->phys[q];
  hipError_t e = launch_gather(st->dt, st->amps, st->scales, st->n, st->B, d_idx, count, phys,
                               st->gf, d_out, st->stream);
  if (e != hipSuccess) return hip_fail(e, "gather launch");
  return JUQCS_OK;
}

juqcs_status juqcs_amplitudes(juqcs_state* st, const uint64_t* idx, size_t count, double* out) {
  if (check_state(st)) return JUQCS_ERR_ARG;
  if (count > 0 && (!idx || !out)) return fail(JUQCS_ERR_ARG, "null index or output");
  for (size_t i = 0; i < count; ++i)
    if (st->n < 64 && (idx[i] >> st->n) != 0) return fail(JUQCS_ERR_ARG, "index >= 2^n");
  const size_t chunk = 1 << 18;
  for (size_t off = 0; off < count; off += chunk) {
    const size_t m = std::min(chunk, count - off);
    char* d_idx = nullptr;
    if (juqcs_status rc = upload(st, idx + off, m * sizeof(uint64_t), &d_idx)) return rc;
    double* d_out = (double*)ring_alloc(st, m * 2 * sizeof(double));
    if (!d_out) return fail(JUQCS_ERR_SIZE, "workspace too small");
    if (juqcs_status rc = juqcs_amplitudes_device(st, (const uint64_t*)d_idx, m, d_out)) return rc;
    hipError_t e = hipMemcpyAsync(out + 2 * off, d_out, m * 2 * sizeof(double),
                                  hipMemcpyDeviceToHost, st->stream);
    if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync D2H");
    if (juqcs_status rc = sync(st)) return rc;
  }
  return JUQCS_OK;
}

juqcs_status juqcs_norm(juqcs_state* st, double* out) {
  if (check_state(st)) return JUQCS_ERR_ARG;
  if (!out) return fail(JUQCS_ERR_ARG, "null output");
  double* partials = (double*)(st->work + kPartialOff);
  double* res = (double*)(st->work + kResultOff);
  hipError_t e = launch_norm(st->dt, st->amps, st->scales, st->n, st->B, partials, res, st->stream);
  if (e != hipSuccess) return hip_fail(e, "norm launch");
  e = hipMemcpyAsync(out, res, sizeof(double), hipMemcpyDeviceToHost, st->stream);
  if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync D2H");
  if (juqcs_status rc = sync(st)) return rc;
  *out *= st->gf.re * st->gf.re + st->gf.im * st->gf.im;
  if (!std::isfinite(*out)) return fail(JUQCS_ERR_NUMERIC, "norm is not finite");
  return JUQCS_OK;
}

juqcs_status juqcs_set_global_factor(juqcs_state* st, const double g[2]) {
  if (check_state(st)) return JUQCS_ERR_ARG;
  if (!g) return fail(JUQCS_ERR_ARG, "null factor");
  if (!finite8(g, 2)) return fail(JUQCS_ERR_NUMERIC, "non-finite factor");
  st->gf = C{g[0], g[1]};
  return JUQCS_OK;
}

juqcs_status juqcs_mul_global_factor(juqcs_state* st, const double f[2]) {
  if (check_state(st)) return JUQCS_ERR_ARG;
  if (!f) return fail(JUQCS_ERR_ARG, "null factor");
  if (!finite8(f, 2)) return fail(JUQCS_ERR_NUMERIC, "non-finite factor");
  st->gf = cmul(st->gf, C{f[0], f[1]});
  return JUQCS_OK;
}

juqcs_status juqcs_get_global_factor(const juqcs_state* st, double g[2]) {
  if (check_state(st)) return JUQCS_ERR_ARG;
  if (!g) return fail(JUQCS_ERR_ARG, "null output");
  g[0] = st->gf.re;
  g[1] = st->gf.im;
  return JUQCS_OK;
}

juqcs_status juqcs_renormalize(juqcs_state* st, double* norm_before) {
  if (check_state(st)) return JUQCS_ERR_ARG;
  double nrm = 0.0;
  if (juqcs_status rc = juqcs_norm(st, &nrm)) return rc;
  if (!(nrm > 0.0)) return fail(JUQCS_ERR_NUMERIC, "cannot renormalise a zero state");
  const double f = 1.0 / std::sqrt(nrm);
  st->gf = C{st->gf.re * f, st->gf.im * f};
  if (norm_before) *norm_before = nrm;
  return JUQCS_OK;
}

juqcs_status juqcs_scale(juqcs_state* st, double factor) {
  if (check_state(st)) return JUQCS_ERR_ARG;
  if (!std::isfinite(factor)) return fail(JUQCS_ERR_NUMERIC, "non-finite factor");
  if (st->dt == JUQCS_ENC2 && !(factor > 0)) return fail(JUQCS_ERR_ARG, "ENC2 scale factor must be > 0");
  hipError_t e = launch_scale(st->dt, st->amps, st->scales, st->n, st->B, factor, st->stream);
  if (e != hipSuccess) return hip_fail(e, "scale launch");
  st->size *= std::fabs(factor);
  return JUQCS_OK;
}

juqcs_status juqcs_expectations(juqcs_state* st, double* out) {
  if (check_state(st)) return JUQCS_ERR_ARG;
  if (!out) return fail(JUQCS_ERR_ARG, "null output");
  const int n = st->n;
  double* partials = (double*)ring_alloc(st, expect_partials_bytes());
  if (!partials) return fail(JUQCS_ERR_SIZE, "workspace too small for expectation partials");
  double* res = (double*)(st->work + kResultOff);  // 3 sums per physical bit
  // first pass: the low b bits; then L contiguous bits plus up to b - L
  // gathered bits not covered yet per pass
  const int b = std::min(n, expect_max_bits(st->dt, n, st->B)), L = expect_low_bits(st->dt, n, st->B);
  TileGeom g{};
  g.n = n;
  g.block_bits = st->B;
  g.L = b;
  g.H = 0;
  g.b = b;
  hipError_t e = launch_expect(st->dt, st->amps, st->scales, g, 0, partials, res, st->stream);
  if (e != hipSuccess) return hip_fail(e, "expectation launch");
  for (int covered = b; covered < n;) {
    const int H = std::min(b - L, n - covered);
    // a last pass with fewer new bits keeps the full tile size: bits already
    // covered (just below the new ones) fill the tile and are not reduced
    // again (small tiles would make the pass launch-bound)
    const int fill = std::min(b - L - H, covered - L);
    g.L = L;
    g.H = fill + H;
    g.b = L + fill + H;
    for (int i = 0; i < fill; ++i) g.hbits[i] = covered - fill + i;
    for (int i = 0; i < H; ++i) g.hbits[fill + i] = covered + i;
    e = launch_expect(st->dt, st->amps, st->scales, g, L + fill, partials, res + 3 * covered, st->stream);
    if (e != hipSuccess) return hip_fail(e, "expectation launch");
    covered += H;
  }
  std::vector<double> sums(3 * n);
  e = hipMemcpyAsync(sums.data(), res, 3 * n * sizeof(double), hipMemcpyDeviceToHost, st->stream);
  if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync D2H");
  if (juqcs_status rc = sync(st)) return rc;
  const double g2 = st->gf.re * st->gf.re + st->gf.im * st->gf.im;
  for (int q = 0; q < n; ++q)
    for (int c = 0; c < 3; ++c) out[3 * q + c] = 0.5 * (1.0 - g2 * sums[3 * st->phys[q] + c]);
  return JUQCS_OK;
}

juqcs_status juqcs_permute(juqcs_state* st, const int* new_phys) {
  if (check_state(st)) return JUQCS_ERR_ARG;
  if (!new_phys) return fail(JUQCS_ERR_ARG, "null permutation");
  std::vector<char> seen(st->n, 0);
  for (int q = 0; q < st->n; ++q) {
    if (new_phys[q] < 0 || new_phys[q] >= st->n) return fail(JUQCS_ERR_QUBIT, "position out of range");
    if (seen[new_phys[q]]) return fail(JUQCS_ERR_QUBIT, "not a permutation");
    seen[new_phys[q]] = 1;
  }
  return move_layout(st, new_phys);
}

juqcs_status juqcs_state_canonicalize(juqcs_state* st) {
  if (check_state(st)) return JUQCS_ERR_ARG;
  std::vector<int> id(st->n);
  for (int q = 0; q < st->n; ++q) id[q] = q;
  return move_layout(st, id.data());
}

juqcs_status juqcs_get_layout(const juqcs_state* st, int* phys) {
  if (check_state(st)) return JUQCS_ERR_ARG;
  if (!phys) return fail(JUQCS_ERR_ARG, "null output");
  for (int q = 0; q < st->n; ++q) phys[q] = st->phys[q];
  return JUQCS_OK;
}

juqcs_status juqcs_encode2(const void* d_src, juqcs_dtype src, uint64_t count, int block_bits,
                           void* d_codes, void* d_scales, void* hip_stream) {
  if (src != JUQCS_C128 && src != JUQCS_C64) return fail(JUQCS_ERR_DTYPE, "source must be C128 or C64");
  if (block_bits < 3 || block_bits > 12) return fail(JUQCS_ERR_ARG, "block_bits must be in [3, 12]");
  if (count > 0 && (!d_src || !d_codes || !d_scales)) return fail(JUQCS_ERR_ARG, "null buffer");
  hipError_t e = launch_encode2(d_src, src, count, block_bits, d_codes, d_scales,
                                (hipStream_t)hip_stream);
  if (e != hipSuccess) return hip_fail(e, "encode2 launch");
  return JUQCS_OK;
}

juqcs_status juqcs_decode2(const void* d_codes, const void* d_scales, uint64_t count,
                           int block_bits, void* d_dst, juqcs_dtype dst, void* hip_stream) {
  if (dst != JUQCS_C128 && dst != JUQCS_C64) return fail(JUQCS_ERR_DTYPE, "target must be C128 or C64");
  if (block_bits < 3 || block_bits > 12) return fail(JUQCS_ERR_ARG, "block_bits must be in [3, 12]");
  if (count > 0 && (!d_codes || !d_scales || !d_dst)) return fail(JUQCS_ERR_ARG, "null buffer");
  hipError_t e = launch_decode2(d_codes, d_scales, count, block_bits, d_dst, dst,
                                (hipStream_t)hip_stream);
  if (e != hipSuccess) return hip_fail(e, "decode2 launch");
  return JUQCS_OK;
}

juqcs_status juqcs_copy(void* d_dst, const void* d_src, size_t bytes, void* hip_stream) {
  if (bytes == 0) return JUQCS_OK;
  if (!d_dst || !d_src) return fail(JUQCS_ERR_ARG, "null buffer");
  if ((bytes & 15) || ((uintptr_t)d_dst & 15) || ((uintptr_t)d_src & 15))
    return fail(JUQCS_ERR_ARG, "copy needs 16-byte multiples and alignment");
  hipError_t e = launch_copy(d_dst, d_src, bytes, (hipStream_t)hip_stream);
  if (e != hipSuccess) return hip_fail(e, "copy launch");
  return JUQCS_OK;
}

}  // extern "C"
