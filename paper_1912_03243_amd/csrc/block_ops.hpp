// Register-resident tile programs.  A workgroup holds a tile of 2^TB
// amplitudes in registers, 2^K per thread: K tile bits are register bits, the
// others are thread bits.  A pass is a list of stages; each stage applies
// gates whose targets are register bits to the registers, and between stages
// the tile is redistributed through LDS so that other tile bits become
// register bits.  Gates are applied one by one instead of as fused dense
// matrices:
//  * a 2x2 unitary is diag(l, m) R diag(1, p) with R = [[1, -t], [t, 1]], |t| <=
//    1, after a flip of the bit where needed: the left diagonal commutes with
//    the controlled phases that follow and joins the qubit's next gate, a flip
//    only changes the place that the tile is written to (the host does both),
//    p costs 2 and R 2 operations per amplitude, against the 26 of a dense 8x8
//    block for 3 to 4 such gates;
//  * controlled phases and controls need no register bit for the other
//    qubit: a thread bit (or a bit outside the tile) gives a sign or a phase
//    per thread, which joins the next gate's p.
// Bound: FP64/FP32 vector arithmetic (4 operations per gate and amplitude) on
// passes of many gates, HBM on light ones; the exchange is one LDS write and
// read of the tile per stage.
#pragma once

#include "tile_ops.hpp"

namespace juqcs {
namespace blk {

// Plans are read through constant-address-space pointers: uniform reads go
// through the scalar cache whatever else the kernel writes.
template <typename X>
using Const = const X __attribute__((address_space(4)))*;
template <typename X>
__device__ __forceinline__ Const<X> as_const(const void* p) {
  return (Const<X>)(const X*)p;
}

// x with its sign flipped where the top bit of s is set.
__device__ __forceinline__ float flip(float x, uint32_t s) {
  return __uint_as_float(__float_as_uint(x) ^ s);
}
__device__ __forceinline__ double flip(double x, uint32_t s) {
  return __hiloint2double(__double2hiint(x) ^ (int)s, __double2loint(x));
}

template <typename T, int K>
struct Regs {
  static constexpr int R = 1 << K;
  typedef T v2 __attribute__((ext_vector_type(2)));
  v2 a[R];  // native vectors stay in registers

  // y *= C + i S on the amplitudes with register bit J set, then the rotation
  // [[1, -t], [t, 1]].  nS = -S, nt = -t: a multiply-add without a sign
  // modifier that adds to its own register takes 4 bytes of code instead of
  // 8, and code is what the four SIMDs of a CU run short of here.
  template <int J>
  __device__ __forceinline__ void rot(T C, T S, T nS, T t, T nt) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if ((r >> J) & 1) continue;
      const int s = r | (1 << J);
      const T yr = fma(nS, a[s].y, C * a[s].x);
      const T yi = fma(S, a[s].x, C * a[s].y);
      a[s].x = fma(t, a[r].x, yr);
      a[s].y = fma(t, a[r].y, yi);
      a[r].x = fma(nt, yr, a[r].x);
      a[r].y = fma(nt, yi, a[r].y);
    }
  }

  // dense complex 2x2 on register bit J (m: 8 reals, row-major)
  template <int J>
  __device__ __forceinline__ void dense(const T* m) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if ((r >> J) & 1) continue;
      const int s = r | (1 << J);
      const T xr = a[r].x, xi = a[r].y, yr = a[s].x, yi = a[s].y;
      a[r].x = fma(-m[3], yi, fma(m[2], yr, fma(-m[1], xi, m[0] * xr)));
      a[r].y = fma(m[3], yr, fma(m[2], yi, fma(m[1], xr, m[0] * xi)));
      a[s].x = fma(-m[7], yi, fma(m[6], yr, fma(-m[5], xi, m[4] * xr)));
      a[s].y = fma(m[7], yr, fma(m[6], yi, fma(m[5], xr, m[4] * xi)));
    }
  }

  // pairs of register bit J trade places: those whose register index holds
  // the bits of M, or (M = 0) all of the thread's where on is set
  template <int J, int M>
  __device__ __forceinline__ void swap_if(bool on) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (((r >> J) & 1) || (r & M) != M) continue;
      const int s = r | (1 << J);
      const v2 x = a[r], y = a[s];
      const bool t = M != 0 || on;
      a[r].x = t ? y.x : x.x;
      a[r].y = t ? y.y : x.y;
      a[s].x = t ? x.x : y.x;
      a[s].y = t ? x.y : y.y;
    }
  }

  // amplitudes whose register index holds every bit of M change sign (by s)
  template <int M>
  __device__ __forceinline__ void neg(uint32_t s) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if ((r & M) != M) continue;
      a[r].x = flip(a[r].x, s);
      a[r].y = flip(a[r].y, s);
    }
  }

  // sign by s and the parity of the register bits cm (uniform)
  __device__ __forceinline__ void signs(int cm, uint32_t s) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const uint32_t t = s ^ ((uint32_t)__popc(r & cm) << 31);
      a[r].x = flip(a[r].x, t);
      a[r].y = flip(a[r].y, t);
    }
  }

  // amplitudes whose register index holds every bit of M times C + i S
  template <int M>
  __device__ __forceinline__ void phase(T C, T S) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if ((r & M) != M) continue;
      const T x = a[r].x;
      a[r].x = fma(-S, a[r].y, C * x);
      a[r].y = fma(S, x, C * a[r].y);
    }
  }
};

// Sign (top bit) of the masked thread and tile-number bits.
__device__ __forceinline__ uint32_t parity_sign(uint32_t x, uint64_t y) {
  return (uint32_t)(__popc(x) + __popcll(y)) << 31;
}

// C + i S times the phases [c0, c1) of a thread.
template <typename T>
__device__ __forceinline__ void collect(Const<BlkOp> ops, Const<T> oc, int c0, int c1, uint32_t tid,
                                        uint64_t tau, T* C, T* S) {
  T x = *C, y = *S;
  for (int o = c0; o < c1; ++o) {
    const T p = oc[8 * o], q = oc[8 * o + 1];
    const uint32_t tm = ops[o].tmask;
    const uint64_t gm = ops[o].gmask;
    const bool on = (tid & tm) == tm && (tau & gm) == gm;
    const T u = fma(-q, y, p * x), v = fma(q, x, p * y);
    x = on ? u : x;
    y = on ? v : y;
  }
  *C = x;
  *S = y;
}

// Ops off the fast path, one after the other.
template <typename T, int K>
__device__ __forceinline__ void run_misc(Regs<T, K>& v, Const<BlkOp> ops, Const<T> oc, int o0, int o1,
                                         uint32_t tid, uint64_t tau) {
  static_assert(K == 4, "the kinds name four register bits");
  for (int o = o0; o < o1; ++o) {
    const uint32_t tm = ops[o].tmask;
    const uint64_t gm = ops[o].gmask;
    uint32_t kind = ops[o].kind;
    asm volatile("" : "+s"(kind));  // independent bits, as far as the compiler knows
    T c[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) c[i] = oc[8 * o + i];
    const bool on = (tid & tm) == tm && (tau & gm) == gm;
    if (kind & blk_dense(0)) v.template dense<0>(c);
    if (kind & blk_dense(1)) v.template dense<1>(c);
    if (kind & blk_dense(2)) v.template dense<2>(c);
    if (kind & blk_dense(3)) v.template dense<3>(c);
#define JUQCS_SWAP(J, I) \
  if (kind & blk_swap(J, I)) v.template swap_if<J, (I == J ? 0 : 1 << I)>(on);
#define JUQCS_SWAPS(J)                        \
  if (kind & (blk_swap(J, 0) * 15)) {         \
    JUQCS_SWAP(J, 0)                          \
    JUQCS_SWAP(J, 1)                          \
    JUQCS_SWAP(J, 2)                          \
    JUQCS_SWAP(J, 3)                          \
  }
    JUQCS_SWAPS(0)
    JUQCS_SWAPS(1)
    JUQCS_SWAPS(2)
    JUQCS_SWAPS(3)
#undef JUQCS_SWAPS
#undef JUQCS_SWAP
    if (kind & blk_signs(0)) v.signs((int)(kind >> 28), parity_sign(tid & tm, tau & gm));
    if (kind & (blk_phase() * 127)) {
      T C = c[0], S = c[1];
      collect(ops, oc, ops[o].col_begin, ops[o].col_end, tid, tau, &C, &S);
      if (kind & blk_phase()) v.template phase<0>(C, S);
      if (kind & blk_phase(0, 1)) v.template phase<3>(C, S);
      if (kind & blk_phase(0, 2)) v.template phase<5>(C, S);
      if (kind & blk_phase(0, 3)) v.template phase<9>(C, S);
      if (kind & blk_phase(1, 2)) v.template phase<6>(C, S);
      if (kind & blk_phase(1, 3)) v.template phase<10>(C, S);
      if (kind & blk_phase(2, 3)) v.template phase<12>(C, S);
    }
  }
}

// A layer's record in scalar registers.
template <typename T>
struct LayerRec {
  int flags, pairs;
  uint32_t tm[kBlkRegs];
  T c[3 * kBlkRegs];
  __device__ __forceinline__ void read(Const<BlkLayer<T>> y) {
    flags = y->flags;
    pairs = y->pairs;
#pragma unroll
    for (int i = 0; i < kBlkRegs; ++i) tm[i] = y->tmask[i];
#pragma unroll
    for (int i = 0; i < 3 * kBlkRegs; ++i) c[i] = y->c[i];
  }
  // all of it has arrived from here on: one wait instead of one per use
  __device__ __forceinline__ void arrive() {
#pragma unroll
    for (int i = 0; i < kBlkRegs; ++i)
      asm volatile("" : "+s"(c[3 * i]), "+s"(c[3 * i + 1]), "+s"(c[3 * i + 2]), "+s"(tm[i]));
    asm volatile("" : "+s"(flags), "+s"(pairs));
  }
};

// A scalar as a vector operand: FP32 multiply-adds with a scalar operand
// issue at half the rate.
template <typename T>
__device__ __forceinline__ T in_vgpr(T x) {
  asm volatile("" : "+v"(x));
  return x;
}

// Sign changes and rotations of one layer.  Straight-line code with a scalar
// branch around each part, so that the registers are updated in place; a
// switch over single ops made the compiler copy all of them at every join and
// waited for each op's parameters (brick30 pass of 84 rotations: 36 ms).
template <typename T, int K>
__device__ __forceinline__ void run_layer(Regs<T, K>& v, const LayerRec<T>& y, Const<BlkMore> more,
                                          Const<BlkOp> ops, Const<T> oc, uint32_t tid, uint64_t tau) {
  static_assert(K == 4, "the flags name four register bits");
  auto sign = [&](int j) {
    const uint64_t gm = y.flags & (BLK_GMASK << j) ? tau & more->gmask[j] : 0;
    return parity_sign(tid & y.tm[j], gm);
  };
#define JUQCS_PAIR(I, J) \
  if (y.pairs & (1 << pair_bit(I, J))) v.template neg<((1 << I) | (1 << J))>(0x80000000u);
  if (y.pairs) {
    JUQCS_PAIR(0, 1)
    JUQCS_PAIR(1, 2)
    JUQCS_PAIR(2, 3)
    if (y.pairs >> 3) {
      JUQCS_PAIR(0, 2)
      JUQCS_PAIR(1, 3)
      JUQCS_PAIR(0, 3)
    }
  }
#undef JUQCS_PAIR
  if (y.flags & BLK_NEGS) {
    if (y.flags & (BLK_NEG << 0)) v.template neg<1>(sign(0));
    if (y.flags & (BLK_NEG << 1)) v.template neg<2>(sign(1));
    if (y.flags & (BLK_NEG << 2)) v.template neg<4>(sign(2));
    if (y.flags & (BLK_NEG << 3)) v.template neg<8>(sign(3));
  }
#define JUQCS_ROT(J)                                                                     \
  if (y.flags & (BLK_ROT << J)) {                                                        \
    T C = in_vgpr(y.c[3 * J]), S = in_vgpr(y.c[3 * J + 1]);                              \
    const T t = in_vgpr(y.c[3 * J + 2]);                                                 \
    if (y.flags & (BLK_OUTER << J)) {                                                    \
      if (y.flags & (BLK_COL << J))                                                      \
        collect(ops, oc, more->col_begin[J], more->col_end[J], tid, tau, &C, &S);        \
      const uint32_t sg = sign(J);                                                       \
      C = flip(C, sg);                                                                   \
      S = flip(S, sg);                                                                   \
    }                                                                                    \
    v.template rot<J>(C, S, in_vgpr(-S), t, in_vgpr(-t));                                \
  }
  JUQCS_ROT(0)
  JUQCS_ROT(1)
  JUQCS_ROT(2)
  JUQCS_ROT(3)
#undef JUQCS_ROT
}

// Applies layers [l0, l1) (an even number) of a stage to the registers.  tid:
// thread index; tau: tile number (its bits are the qubits outside the tile).
// Two records take turns: one is read while the other one's layer runs (the
// plan ends with spare records).
template <typename T, int K>
__device__ __forceinline__ void run_layers(Regs<T, K>& v, const BlkDev& d, int l0, int l1,
                                           uint32_t tid, uint64_t tau) {
  Const<BlkLayer<T>> y = as_const<BlkLayer<T>>(d.layers) + l0;
  const Const<BlkLayer<T>> end = as_const<BlkLayer<T>>(d.layers) + l1;
  Const<BlkMore> more = as_const<BlkMore>(d.more) + l0;
  const Const<BlkOp> ops = as_const<BlkOp>(d.ops);
  const Const<T> oc = as_const<T>(d.ocoef);
  LayerRec<T> a, b;
  a.read(y);
  while (y < end) {
    a.arrive();
    b.read(y + 1);
    run_layer<T, K>(v, a, more, ops, oc, tid, tau);
    b.arrive();
    y += 2;
    a.read(y);
    run_layer<T, K>(v, b, more + 1, ops, oc, tid, tau);
    more += 2;
  }
}

// Byte offset in LDS of a thread's share of the tile in a stage's layout.
template <int TBITS>
__device__ __forceinline__ int stage_base(Const<BlkStage> s, int tid) {
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int u = 0;  // wave-uniform part
#pragma unroll
  for (int i = 6; i < TBITS; ++i) u ^= -((wave >> (i - 6)) & 1) & s->thr[i];
  int b = u;
#pragma unroll
  for (int i = 0; i < (TBITS < 6 ? TBITS : 6); ++i) b ^= -((tid >> i) & 1) & s->thr[i];
  return b;
}

// LDS byte offsets of a thread's amplitudes: b, then one more register bit at
// a time (the four row offsets stay scalar).
template <int K>
__device__ __forceinline__ void stage_rows(Const<BlkStage> s, int b, int* o) {
  o[0] = b;
#pragma unroll
  for (int j = 0; j < K; ++j)
#pragma unroll
    for (int r = 0; r < (1 << j); ++r) o[r | (1 << j)] = o[r] ^ s->row[j];
}

__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Redistributes the tile from the layout of stage a to that of stage b (and
// does the CNOTs planned between them: they only change which slot b's
// threads read).
// Every thread writes the amplitudes that it holds to their own slots and
// reads the next stage's from theirs: a slot is only ever written by the
// thread that read it last, so one barrier per exchange is enough, and none
// where the wave bits stay the same (the exchange then stays within each
// wave).  FP64 tiles go through LDS one component at a time: at 8 bytes per
// amplitude two workgroups share a CU.
template <typename T, int TB, int K>
__device__ __forceinline__ void exchange(Regs<T, K>& v, char* sh, Const<BlkStage> a, Const<BlkStage> b,
                                         int tid) {
  constexpr int R = 1 << K;
  typedef T v2 __attribute__((ext_vector_type(2)));
  int o[R];
  const bool cross = b->exchange == BLK_CROSS;
  const auto sync = [&]() {
    if (cross) __syncthreads();
    else wave_fence();
  };
  // the addresses of one direction at a time: both would not fit the registers
  int wb = stage_base<TB - K>(a, tid), rb = stage_base<TB - K>(b, tid);
  stage_rows<K>(a, wb, o);
  if constexpr (sizeof(T) == 8) {
#pragma unroll
    for (int r = 0; r < R; ++r) *reinterpret_cast<T*>(sh + o[r]) = v.a[r].x;
    sync();
    asm volatile("" : "+v"(rb));
    stage_rows<K>(b, rb, o);
#pragma unroll
    for (int r = 0; r < R; ++r) v.a[r].x = *reinterpret_cast<const T*>(sh + o[r]);
    sync();
    asm volatile("" : "+v"(wb));
    stage_rows<K>(a, wb, o);
#pragma unroll
    for (int r = 0; r < R; ++r) *reinterpret_cast<T*>(sh + o[r]) = v.a[r].y;
    sync();
    asm volatile("" : "+v"(rb));
    stage_rows<K>(b, rb, o);
#pragma unroll
    for (int r = 0; r < R; ++r) v.a[r].y = *reinterpret_cast<const T*>(sh + o[r]);
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r) *reinterpret_cast<v2*>(sh + o[r]) = v.a[r];
    stage_rows<K>(b, rb, o);
    sync();
#pragma unroll
    for (int r = 0; r < R; ++r) v.a[r] = *reinterpret_cast<const v2*>(sh + o[r]);
  }
}

// Runs a pass's stages on the tile in v.  sh: 8 bytes of LDS per amplitude.
template <typename T, int TB, int K>
__device__ __forceinline__ void run_stages(Regs<T, K>& v, char* sh, const BlkDev& d, int nst,
                                           uint64_t tau) {
  const Const<BlkStage> st = as_const<BlkStage>(d.stages);
  const int tid = (int)threadIdx.x;
  for (int s = 0; s < nst; ++s) {
    if (s > 0 && st[s].exchange != BLK_STAY) {
      // an opaque copy: masks of its bits kept from stage to stage would hold
      // scalar registers that the layers' coefficients need
      int t = tid;
      asm volatile("" : "+v"(t));
      exchange<T, TB, K>(v, sh, st + s - 1, st + s, t);
    }
    // misc ops come before a stage's layers: within the loop over the layers
    // the compiler would copy the registers at their joins every time
    if (st[s].misc_begin < st[s].misc_end)
      run_misc<T, K>(v, as_const<BlkOp>(d.ops), as_const<T>(d.ocoef), st[s].misc_begin, st[s].misc_end,
                     (uint32_t)tid, tau);
    run_layers<T, K>(v, d, st[s].layer_begin, st[s].layer_end, (uint32_t)tid, tau);
  }
}

}  // namespace blk
}  // namespace juqcs
