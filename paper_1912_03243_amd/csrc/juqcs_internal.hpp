// Internal declarations shared by the kernel translation units and the
// host-side engine of libjuqcs_gpu.  Not installed; the public interface is
// include/juqcs_gpu.h.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cstddef>
#include <cmath>
#include <cstdint>
#include <string>
#include <vector>

#include "juqcs_gpu.h"

namespace juqcs {

// ---------------------------------------------------------------------------
// Complex arithmetic on interleaved (re, im) storage.  The alignment makes a
// C128 amplitude one 16-byte load and a C64 amplitude one 8-byte load.
// ---------------------------------------------------------------------------
template <typename T>
struct alignas(2 * sizeof(T)) cplx {
  T re, im;
};

template <typename T>
__host__ __device__ inline cplx<T> cmul(cplx<T> a, cplx<T> b) {
  return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
// acc + a*b as four fused multiply-adds (one rounding each)
template <typename T>
__host__ __device__ inline cplx<T> cmad(cplx<T> a, cplx<T> b, cplx<T> acc) {
  acc.re = fma(a.re, b.re, acc.re);
  acc.re = fma(-a.im, b.im, acc.re);
  acc.im = fma(a.re, b.im, acc.im);
  acc.im = fma(a.im, b.re, acc.im);
  return acc;
}

template <typename T>
struct Mat2 {
  cplx<T> m[4];  // row-major
};
template <typename T>
struct Mat4 {
  cplx<T> m[16];  // row-major, index b_q0 + 2 b_q1
};

// Streaming accesses to state vectors: non-temporal, so data a pass touches
// once does not evict from L2 the coefficients and tables it keeps
// re-reading.  V is a scalar or a clang vector type.
template <typename V>
__device__ __forceinline__ V ld_stream(const V* p) {
  return __builtin_nontemporal_load(p);
}
template <typename V>
__device__ __forceinline__ void st_stream(V* p, V v) {
  __builtin_nontemporal_store(v, p);
}

template <typename T>
__device__ __forceinline__ cplx<T> ld_amp(const cplx<T>* p) {
  typedef T v2 __attribute__((ext_vector_type(2)));
  const v2 v = __builtin_nontemporal_load(reinterpret_cast<const v2*>(p));
  return cplx<T>{v.x, v.y};
}
template <typename T>
__device__ __forceinline__ void st_amp(cplx<T>* p, cplx<T> a) {
  typedef T v2 __attribute__((ext_vector_type(2)));
  __builtin_nontemporal_store(v2{a.re, a.im}, reinterpret_cast<v2*>(p));
}

// Insert a zero bit at position pos of x (bits >= pos move up by one).
__host__ __device__ inline uint64_t insert_zero(uint64_t x, int pos) {
  const uint64_t low = x & ((uint64_t(1) << pos) - 1);
  return ((x >> pos) << (pos + 1)) | low;
}

// ---------------------------------------------------------------------------
// Tile passes: 2^b amplitudes per workgroup, made of 2^H chunks of 2^L
// contiguous amplitudes; local index bit j < L is physical bit j, local bit
// L + i is physical bit hbits[i].  Ops act on local bits.
// ---------------------------------------------------------------------------
constexpr int kMaxGather = 10;  // gathered chunk bits of a tile pass
constexpr int kPassOps = 48;    // most ops the planner puts in one pass
constexpr int kHbitsCap = 12;   // fused blocks reuse the struct: 2k <= 12
constexpr int kSwapCap = 8;     // relabel swaps at the end of one pass

struct TileGeom {
  int32_t n, L, H, b;
  int32_t hbits[kHbitsCap];      // ascending physical positions (>= L)
  int32_t block_bits;            // ENC2 only
  int32_t maxk;                  // widest op of the pass (1..4)
  int32_t mat_count;             // coefficients of the pass's ops, from ops[0].moff on
  int32_t mma_count;             // 8x8 (TOP_DENSE3) ops of the pass
  // Relabeling: after its ops the pass writes the tile
  // back with local bits swap_a[i] and swap_b[i] exchanged (disjoint pairs),
  // i.e. the qubits at those two physical positions trade places.
  int32_t nswap;
  int8_t swap_a[kSwapCap], swap_b[kSwapCap];
};

// Local index after the pass's relabel swaps (an involution: the swaps are
// disjoint transpositions of bit positions).
// The loop has a fixed trip count so that a kernel reads the pairs from its
// argument block with constant offsets (no vector memory loads).
__host__ __device__ inline int swap_local(int e, const TileGeom& g) {
  for (int i = 0; i < kSwapCap; ++i) {
    if (i < g.nswap) {
      const int a = g.swap_a[i], c = g.swap_b[i];
      const int x = ((e >> a) ^ (e >> c)) & 1;
      e ^= (x << a) | (x << c);
    }
  }
  return e;
}

enum TileOpKind : int32_t {
  TOP_DENSE1 = 0,  // 2x2 on local bit a
  TOP_DENSE2 = 1,  // 4x4 on local bits (a, b), index b_a + 2 b_b
  TOP_DIAG2 = 2,   // phases d[b_a + 2 b_b] (b may equal -1: d[b_a])
  TOP_DENSE3 = 3,  // 8x8 on local bits bits[0..3) (matrix order)
  TOP_DENSE4 = 4,  // 16x16 on local bits bits[0..4)
  TOP_PERM = 5,    // monomial on local bits bits[0..k), k <= 3: out[r] =
                   // c[r] in[sigma(r)], sigma(r) in bits 3r..3r+2 of a
  TOP_DENSE3G = 6, // 8x8 on bits[0..3) in three-product form (FP64 pipelined
                   // kernels only): per row r, 24 reals Re m_r., (Re + Im) m_r.,
                   // (Im - Re) m_r.
};

struct TileOp {
  int32_t kind;
  int32_t a, b;
  int32_t k;
  int32_t bits[4];
  int64_t moff;  // offset of the matrix in the complex coefficient array
};

// A tile pass: geometry plus a range of ops.
struct TilePass {
  TileGeom g;
  int32_t op_begin, op_count;
};

// ---------------------------------------------------------------------------
// Register-resident tile programs (block_ops.hpp, block.cpp)
// ---------------------------------------------------------------------------
constexpr int kBlkRegs = 4;      // register bits: 2^4 amplitudes per thread
constexpr int kBlkThrBits = 9;   // most thread bits of a tile (2^13 amplitudes)
// A layer: sign changes of register-bit pairs and bits, then at most one
// rotation per register bit.
template <typename T>
struct alignas(16) BlkLayer {
  int32_t flags;
  int32_t pairs;                // pair_bit of every pair that changes sign where both are set
  int32_t pad[2];
  uint32_t tmask[kBlkRegs];     // thread bits whose parity signs C + i S of register bit j
  T c[3 * kBlkRegs];            // C, S, t at 3 j
};
struct BlkMore {  // what few layers need
  uint64_t gmask[kBlkRegs];     // bits of the tile number that join tmask's
  int32_t col_begin[kBlkRegs], col_end[kBlkRegs];  // phases that join C + i S per thread
};
enum BlkFlags : int32_t {  // J: register bit
  BLK_ROT = 1 << 0,      // << J: phase C + i S on the set half, then [[1, -t], [t, 1]]
  BLK_OUTER = 1 << 4,    // << J: C, S take signs or phases of outer bits
  BLK_NEG = 1 << 8,      // << J: no rotation, the set half changes sign by the masks
  BLK_COL = 1 << 12,     // << J: C + i S takes the collected phases
  BLK_GMASK = 1 << 16,   // << J: gmask counts
  BLK_NEGS = 15 << 8,
};
// Bit of a pair of register bits: neighbours first (0-2), then the others.
constexpr int pair_bit(int i, int j) { return j == i + 1 ? i : j == i + 2 ? 3 + i : 5; }
// Kinds of misc ops: one bit each, so that the kernels test them one by one (a
// chain of comparisons is made a tree of branches whose joins copy all
// amplitudes).
constexpr uint32_t blk_dense(int j) { return 1u << j; }  // dense 2x2 on register bit j, 8 reals
// the halves of register bit j trade places where bit i is set (i = j: where
// all mask bits are)
constexpr uint32_t blk_swap(int j, int i) { return 1u << (4 + 4 * j + i); }
// C + i S where all mask bits and both register bits (i < j) are set; on none
constexpr uint32_t blk_phase() { return 1u << 21; }
constexpr uint32_t blk_phase(int i, int j) { return 1u << (22 + pair_bit(i, j)); }
// sign by the parity of the masked bits and of the register bits cm
constexpr uint32_t blk_signs(uint32_t cm) { return 1u << 20 | cm << 28; }
struct BlkOp {     // coefficients: 8 reals per op
  uint32_t kind;   // (entries of a col list, C + i S where all mask bits are set: 0)
  uint32_t tmask;  // thread bits (of the thread index)
  uint64_t gmask;  // bits of the tile number
  int32_t col_begin, col_end;  // phases: phases that join per thread
};
enum BlkExchange : int32_t { BLK_STAY, BLK_WAVE, BLK_CROSS };  // nothing, within waves, across waves
struct BlkStage {
  int32_t misc_begin, misc_end;
  int32_t layer_begin, layer_end;  // an even number
  int32_t exchange;           // what comes before this stage
  int32_t row[kBlkRegs];      // LDS byte offset of each register bit
  int32_t thr[kBlkThrBits];   // of each thread bit
};
struct BlkGeom {
  int32_t n, b, L, H;            // as TileGeom
  int32_t hbits[kMaxGather];
  int32_t nst;                   // stages
  int32_t tile_sync;             // waves hold other LDS slots in the last stage than in the first
  int32_t block_bits;            // ENC2 only
  // physical bit of each thread and register bit as the tile is read and as
  // it is written (through the pass's relabel swaps)
  int32_t ld_thr[kBlkThrBits], ld_reg[kBlkRegs], st_thr[kBlkThrBits], st_reg[kBlkRegs];
  uint64_t st_flip;              // physical bits that are written complemented
};
struct BlkPass {
  BlkGeom g;
  int32_t stage_begin;
  int32_t pad;
};
struct BlkDev {  // a plan in device memory
  const BlkStage* stages;
  const void* layers;  // BlkLayer<T>
  const BlkMore* more; // one per layer
  const BlkOp* ops;
  const void* ocoef;   // 8 per op
};

struct BatchGroup {  // every tile of one pass of one circuit
  uint64_t state_off;    // byte offset of the circuit's C64 state
  uint64_t src_off;      // of the state that the pass reads (register-resident passes)
  int64_t first_chunk;   // first ticket of this group
  int32_t circuit;
  int32_t pass;          // index into the BatchPass array
  int32_t chunk_tiles;   // tiles claimed per ticket
  int32_t init;          // 1: start from |0...0> instead of loading
};

// ---------------------------------------------------------------------------
// Kernel launchers (defined in the .hip files).  All asynchronous on stream.
// Return hipSuccess or the launch error.
// ---------------------------------------------------------------------------
hipError_t launch_init(juqcs_dtype dt, void* amps, void* scales, int n,
                       int block_bits, uint64_t idx, hipStream_t s);
hipError_t launch_1q(juqcs_dtype dt, void* amps, int n, int t, int c,
                     const cplx<double> u[4], hipStream_t s);
hipError_t launch_diag(juqcs_dtype dt, void* amps, int n, uint64_t mask,
                       cplx<double> phase, hipStream_t s);
hipError_t launch_2q(juqcs_dtype dt, void* amps, int n, int q0, int q1,
                     const cplx<double> m[16], hipStream_t s);
hipError_t launch_norm(juqcs_dtype dt, const void* amps, const void* scales,
                       int n, int block_bits, double* partials, double* out,
                       hipStream_t s);
hipError_t launch_gather(juqcs_dtype dt, const void* amps, const void* scales,
                         int n, int block_bits, const uint64_t* idx,
                         uint64_t count, const int8_t* phys, cplx<double> g, double* out,
                         hipStream_t s);
hipError_t launch_scale(juqcs_dtype dt, void* amps, void* scales, int n,
                        int block_bits, double f, hipStream_t s);
hipError_t launch_copy(void* dst, const void* src, size_t bytes, hipStream_t s);
// Zeroes bytes (a multiple of 4, 4-byte aligned) with a kernel.
hipError_t launch_zero(void* p, size_t bytes, hipStream_t s);

hipError_t launch_tile(juqcs_dtype dt, void* amps, void* scales,
                       const TileGeom& g, const TileOp* d_ops, int nops,
                       const void* d_mats, hipStream_t s);
// Whether launch_tile runs a pass on a pipelined (fixed tile size) kernel.
bool tile_pipelined(juqcs_dtype dt, const TileGeom& g, int nops);
int tile_max_bits(juqcs_dtype dt);
// Expectation values of sigma^x,y,z for the tile bits jlo..b-1 of geometry
// g (b <= expect_max_bits, at most 16 bits per launch):
// out3[3 (j - jlo) + c].  partials: expect_partials_bytes() of device memory.
int expect_max_bits(juqcs_dtype dt, int n, int block_bits);
// least contiguous bits of its passes after the first
int expect_low_bits(juqcs_dtype dt, int n, int block_bits);
size_t expect_partials_bytes();
hipError_t launch_expect(juqcs_dtype dt, const void* amps, const void* scales, const TileGeom& g,
                         int jlo, double* partials, double* out3, hipStream_t s);

// Register-resident tile passes (k_block.hip): tile sizes that have a kernel.
bool block_sized(juqcs_dtype dt, int b);
// p: the pass, d_pass the same in device memory.
bool block_codes_sized(int block_bits, int b);
hipError_t launch_block(juqcs_dtype dt, void* amps, void* scales, const BlkPass& p, const BlkPass* d_pass, const BlkDev& d,
                        hipStream_t s);
// Rounds of many states' passes (C64): groups [g0, g1) of tiles of 2^b
// amplitudes, chunks [c0, c1), claimed through *ticket.
hipError_t launch_block_round(int b, char* states, const BatchGroup* groups, int g0, int g1,
                              const BlkPass* passes, const BlkDev& d, uint64_t* ticket, long long c0,
                              long long c1, hipStream_t s);
// Workgroups of a kernel that fit on the device at once (cached per kernel).
uint64_t resident_blocks(const void* kern, int threads);

// What a pass of 2^b-amplitude tiles may carry so that it runs on the
// pipelined kernel: coefficients (staged in LDS by the two-byte kernels) and
// 8x8 ops (whose tables the FP32 kernels build in LDS); 0 = no limit.
int tile_mat_cap(juqcs_dtype dt, int b);
int tile_mma_cap(juqcs_dtype dt, int b);

hipError_t launch_fused(juqcs_dtype dt, void* amps, int n, int k,
                        const int* targets, const void* d_mat, juqcs_mma mode,
                        hipStream_t s);

hipError_t launch_encode2(const void* src, juqcs_dtype sdt, uint64_t count,
                          int block_bits, void* codes, void* scales,
                          hipStream_t s);
hipError_t launch_decode2(const void* codes, const void* scales,
                          uint64_t count, int block_bits, void* dst,
                          juqcs_dtype ddt, hipStream_t s);
// ---------------------------------------------------------------------------
// Batches (k_batch.hip, batch.cpp)
// ---------------------------------------------------------------------------
struct BatchPass {  // one tile pass of one circuit
  TileGeom g;
  int32_t op_begin, op_count;
};


struct BatchDevice {
  const BatchGroup* groups;
  int ngroups;
  const BatchPass* passes;
  const TileOp* ops;
  const cplx<float>* mats;
  uint64_t* tickets;               // one counter per round (device)
  int nrounds;                     // round r: pass r of every circuit that has one
  std::vector<int32_t> round_group;    // host: first group of each round (+ end)
  std::vector<int64_t> round_chunk;    // host: first chunk of each round (+ end)
  int count;
  long long nchunks;
  // Register-resident passes: sub-round k of round r (tiles of 2^(11 + k)
  // amplitudes) is entry kBlkTileSizes r + k of the tables (+ end)
  const BatchGroup* bgroups = nullptr;
  const BlkPass* bpasses = nullptr;
  BlkDev bdev{};
  uint64_t* btickets = nullptr;   // one per sub-round
  std::vector<int32_t> bround_group;
  std::vector<int64_t> bround_chunk;
};
constexpr int kBlkTileSizes = 3, kBlkMinTile = 11;

int batch_max_bits();
int batch_mma_cap();  // 8x8 ops per pass whose tables the batch kernel holds in LDS
int batch_max_gather();  // most gathered chunk bits of a batch pass
hipError_t launch_batch(char* states, const BatchDevice& d, hipStream_t s);
hipError_t launch_batch_gather(const char* states, const uint64_t* state_off, const int32_t* nq,
                               const int8_t* pos, int count, int m, const uint64_t* idx, double* out,
                               hipStream_t s);
hipError_t launch_batch_norms(const char* states, const uint64_t* state_off, const int32_t* nq,
                              int count, double* out, hipStream_t s);

// Entangling-gate decomposition (Eq. (3)) on the device.
constexpr int kBranchMaxParts = 8;    // parts of a decomposition
constexpr int kBranchMaxQubits = 240; // kBranchMaxParts parts of at most 30 qubits
constexpr int kBranchMaxWords = 4;    // 64-bit words per bitstring
// Bitstring split table (int32 entries): [0, P] part starts into the runs,
// then the runs: qubits q, q + 1, .. q + len - 1 of one bitstring word on bits
// d, d + 1, .. of the part's index (q | d << 8 | (len - 1) << 16).
constexpr int kBranchTabInts = kBranchMaxParts + 1 + kBranchMaxQubits;
// Sets *bad (device int) when a bitstring has a bit at or above n.
hipError_t launch_branch_split(const uint64_t* z, int words, long long count, int P, int n,
                               const int32_t* tab, uint32_t* zp, int* bad, hipStream_t s);
// The leaves of each part: first[p] .. first[p + 1], and where a sum reads
// interleaved states, log2 of how many of them (0: the state as it lies) and
// the byte offset of their interleaved amplitudes.
struct BranchLeaves {
  int32_t first[kBranchMaxParts + 1];
  int32_t shift[kBranchMaxParts];
  uint64_t base[kBranchMaxParts];
};
// Amplitude z of the 2^r states (r >= 1) at state_off[0 .. 2^r) goes to dst[z 2^r + i].
hipError_t launch_branch_interleave(const char* states, const uint64_t* state_off, int r, int nloc, void* dst,
                                    hipStream_t s);
// acc[k] += sum over the group's g branches (in order) of prod_p
// psi_{tab[j P + p]}[zp[p count + k]] (FP64); the first group starts from
// zero and the last one multiplies by scale.
hipError_t launch_branch_gather_accum(const char* states, const uint64_t* state_off, int P,
                                      const BranchLeaves& leaves, bool interleaved, long long g,
                                      const int32_t* tab, const uint32_t* zp, long long count, double* acc,
                                      bool first, bool last, double scale, hipStream_t s);
// The same sum when the group has at most kBranchSumValues states, stored
// part by part (part p: circuits first[p] .. first[p + 1]): every thread
// gathers its coefficient's amplitude of each state into LDS once, then sums
// the branches from there; byte p of tab8[j] is branch j's circuit of part p.
constexpr int kBranchSumValues = 48;
constexpr int kBranchSumThreads = 128;
hipError_t launch_branch_sum_lds(const char* states, const uint64_t* state_off, int P,
                                 const BranchLeaves& leaves, bool interleaved, long long g, const uint64_t* tab8,
                                 const uint32_t* zp, long long count, double* acc, bool first, bool last,
                                 double scale, hipStream_t s);

// ---------------------------------------------------------------------------
// Host-side planning (planner.cpp)
// ---------------------------------------------------------------------------
struct Gate {  // decoded gate: matrix on 1 or 2 qubits (physical positions)
  int nq;
  int q[2];
  cplx<double> m[16];  // 2x2 (first 4) or 4x4, index b_q0 + 2 b_q1
  bool diag;
  // Bit j: the tile selection may count on the gate being diagonal on q[j]
  // (it commutes with other gates that are, and q[j] may lie outside the tile).
  int diag_on = 0;
};

bool decode_gate(const juqcs_gate& g, int n, Gate* out, std::string* err);
// Algorithmic flops per state amplitude of a gate (planner.cpp).
double gate_flops(const Gate& g);

struct TilePlan {
  std::vector<TilePass> passes;
  std::vector<TileOp> ops;
  std::vector<cplx<double>> mats;
  // for every op: the gates folded into it, in merge order, so the matrices
  // can be rebuilt for gates with other values but the same structure
  std::vector<std::vector<int>> op_gates;
  std::vector<Gate> src;  // those gates, on the physical bits of their passes (two-byte plans only)
  int64_t gates = 0;
};

// Recomputes every op matrix of plan from gates (same qubits and zero
// pattern as the gates the plan was made for).
void rebuild_mats(const std::vector<Gate>& gates, TilePlan* plan);

// Tile selection alone: the passes (geometry) and the gates each absorbs.
struct TileSchedule {
  std::vector<TilePass> passes;
  std::vector<std::vector<int>> taken;
  int64_t gates = 0;
  // Relabeling schedules only: the absorbed gates on the physical bits of
  // their pass (taken indexes these), the index of each in the input gate
  // list, and final_pos[p] = where the qubit at physical bit p before the
  // schedule sits after it.
  std::vector<Gate> tgates;
  std::vector<int> tsrc;
  std::vector<int> final_pos;
};
// max_take > 0 caps the gates one pass absorbs (later gates wait for the
// next pass), which moves on-chip work from crowded passes to light ones.
void select_tiles(int n, int L, int b, int block_bits, const std::vector<Gate>& gates,
                  TileSchedule* sched, int max_take = 0);
// Same with relabeling: between passes, qubits of the finished tile may take
// over the low L physical bits (swapped in by the finished pass's store), so
// that the next tile is any b qubits of which at least L were in the
// finished one.  Fills sched->tgates and sched->final_pos.
void select_tiles_relabel(int n, int L, int b, int block_bits, const std::vector<Gate>& gates,
                          TileSchedule* sched, int max_take = 0);
// Fuses every pass's gates into ops of at most kin qubits.  A pass whose
// coefficients would exceed max_mats (> 0), or whose 8x8 ops would exceed
// max_mma (> 0), is split into consecutive passes of the same geometry (the
// relabel swaps go with the last of them).  taken indexes sched.tgates when
// that is non-empty, else gates; plan->op_gates index the same vector.
void emit_schedule(const TileSchedule& sched, const std::vector<Gate>& gates, int kin,
                   TilePlan* plan, int max_mats = 0, int max_mma = 0);

// Plans tile passes for gates (physical qubits).  L, b: low contiguous bits
// and total tile bits; the low L bits are always tile bits.
// relabel: plan with select_tiles_relabel; *final_pos (if given) receives
// the schedule's final_pos (identity without relabeling).
void plan_tiles(int n, int L, int b, int block_bits, const std::vector<Gate>& gates,
                TilePlan* plan, int kin = 2, int max_mats = 0, int max_take = 0,
                int max_mma = 0, bool relabel = false, std::vector<int>* final_pos = nullptr);

// Host values of register-resident programs: eleven bits more than FP64, so that
// what is rounded to a state's precision is rounded once.
using BlkReal = long double;

// A gate of a register-resident tile program (block.cpp).
struct BlkGate {
  enum Kind { ROT, DENSE, PHASE1, CPHASE, CNOT } kind = DENSE;
  int q[2] = {0, -1};       // CNOT: control, target
  bool formb = false;       // ROT: lam R diag(1, ph), R = [[1, -t], [t, 1]] or (formb) [[t, -1], [1, t]]
                            // = [[1, t], [-t, 1]] [[0, -1], [1, 0]]
  BlkReal t = 0;
  cplx<BlkReal> ph{1, 0};   // phase of the set half (ROT, PHASE1) or quarter (CPHASE)
  cplx<BlkReal> lam{1, 0};  // scalar factor (ROT, PHASE1)
  double share = 0.5;       // ROT: how much of the state's norm its set half holds, as far as is known
  cplx<BlkReal> m[4];       // DENSE
};
struct BlkPlan {
  std::vector<BlkPass> passes;
  std::vector<BlkStage> stages;
  std::vector<BlkLayer<double>> layers;
  std::vector<BlkMore> more;
  std::vector<BlkOp> ops;
  std::vector<double> ocoef;
};
// Rewrites a circuit as rotations, phases, controlled phases and CNOTs: the
// single-qubit gates between two others merge, and left diagonals move on
// to the qubit's next gate.  tol: the largest relative miss of a matrix
// entry by the rotation form (else the gate stays dense).  False when a
// two-qubit gate is neither a controlled phase nor a CNOT.
// keep: phases that happen to be 1 stay in the list, so that its shape (kinds
// and qubits) is the same for circuits that differ in their diagonals' values.
// order: which of the gates, in which order (null: all as they come).
// basis: the basis state that the circuit starts from (null: any state).
bool block_gates(int n, const std::vector<Gate>& gates, double tol, std::vector<BlkGate>* out, bool keep = false,
                 const std::vector<int>* order = nullptr, const uint64_t* basis = nullptr);
// A number that tells apart lists whose plans differ in more than coefficients:
// kinds, qubits, forms, and which phases and scalars are 1 or -1.
uint64_t block_shape(const std::vector<BlkGate>& gates);
// Appends one pass: geometry tg, its gates and the physical bits of their qubits.
// low: low bits that the first and the last stage keep on lanes (contiguous
// accesses of 2^low amplitudes).
void plan_block_pass(const TileGeom& tg, const std::vector<const BlkGate*>& gates,
                     const std::vector<std::array<int, 2>>& at, bool fp64, int low, BlkPlan* plan, int codes = 0);
// Plans a circuit as register-resident passes (arguments as plan_tiles);
// false when it holds gates they do not take.
bool plan_block(int n, int L, int b, const std::vector<Gate>& gates, bool fp64, int max_take, bool relabel,
                BlkPlan* plan, std::vector<int>* final_pos, const uint64_t* basis = nullptr);

// The relative miss of a matrix entry by the rotation form up to which a
// gate is not kept dense: an FP64 rounding step, or far below an FP32 one.
// (Haar circuits in FP64: one rotation in 250 stays dense, against one in 20
// at 2^-53; errors of 20 layers 1.28e-15 against 1.21e-15.)
inline double block_tol(bool fp64) { return fp64 ? 0x1p-52 : 1e-9; }
// Tile selection of a rewritten circuit; plans of circuits of the same shape
// (kinds and qubits) can be built on it with other values.
struct BlkSchedule {
  TileSchedule sched;
  std::vector<Gate> shape;
  std::vector<BlkGate::Kind> kinds;
  int low = 0;
};
void block_schedule(int n, int L, int b, const std::vector<BlkGate>& bg, int max_take, bool relabel, bool strict,
                    BlkSchedule* out);
// Appends the schedule's passes with bg's values; false when bg has another shape
// or coefficients that the precision cannot hold.
bool block_build(const BlkSchedule& bs, const std::vector<BlkGate>& bg, bool fp64, BlkPlan* plan);

// The passes of a tile plan of two-byte amplitudes (scale blocks of 2^block_bits)
// as register-resident programs: the same gates between the same encodings.
// False if a pass has gates that they do not do, or coefficients out of range.
bool block_tile_plan(const TilePlan& tp, int block_bits, BlkPlan* plan);

// Byte image of a plan for the device (reals in the state's precision) and
// where its parts lie.
struct BlkSizes {
  size_t passes = 0, stages = 0, layers = 0, ops = 0;
  BlkSizes() = default;
  explicit BlkSizes(const BlkPlan& p)
      : passes(p.passes.size()), stages(p.stages.size()), layers(p.layers.size()), ops(p.ops.size()) {}
  void grow(const BlkSizes& z) {  // each the larger of the two
    passes = std::max(passes, z.passes);
    stages = std::max(stages, z.stages);
    layers = std::max(layers, z.layers);
    ops = std::max(ops, z.ops);
  }
};
// Appends p to all (indices moved).
void append_plan(const BlkPlan& p, BlkPlan* all);
struct BlkLayout {
  size_t o_geoms, o_layers, o_more, o_ops, o_ocoef, total;  // o_geoms: BlkPass
};
BlkLayout block_layout(const BlkSizes& z, bool fp64);
BlkLayout block_image(const BlkPlan& plan, bool fp64, char* image);  // image: zeroed, layout's total bytes
inline BlkDev block_device(const BlkLayout& l, const char* dev) {
  return BlkDev{(const BlkStage*)dev, dev + l.o_layers, (const BlkMore*)(dev + l.o_more),
                (const BlkOp*)(dev + l.o_ops), dev + l.o_ocoef};
}

struct FusedBlock {
  std::vector<int> targets;           // physical
  std::vector<cplx<double>> m;        // 2^k x 2^k
};
void plan_fused(int n, int kmax, const std::vector<Gate>& gates,
                std::vector<FusedBlock>* blocks);

void set_error(const std::string& msg);

}  // namespace juqcs
