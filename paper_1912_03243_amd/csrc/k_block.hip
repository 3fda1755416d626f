// Tile passes on register-resident tiles (block_ops.hpp): one HBM read and
// write of the state per pass, a program of stages in between.
#include "block_ops.hpp"

namespace juqcs {

namespace {

using blk::as_const;
using blk::Const;
using blk::Regs;
using blk::run_stages;

// Base index of tile tau: tau's bits fill the non-tile positions in order.
__device__ __forceinline__ uint64_t block_base(uint64_t tau, Const<BlkGeom> g) {
  uint64_t base = tau << g->L;
#pragma unroll
  for (int j = 0; j < kMaxGather; ++j)
    if (j < g->H) base = insert_zero(base, g->hbits[j]);
  return base;
}

// Sum of the amplitude offsets of the set bits of x.
template <int N>
__device__ __forceinline__ uint64_t place(uint32_t x, Const<int32_t> pos) {
  uint64_t o = 0;
#pragma unroll
  for (int i = 0; i < N; ++i) o |= (uint64_t)((x >> i) & 1) << pos[i];
  return o;
}

// Addresses of a thread's 2^K amplitudes: base, then one more register bit at
// a time (adding the K strides one by one keeps 2^K scalar offsets out of the
// scalar registers).
template <int K, typename V>
__device__ __forceinline__ void amp_ptrs(V* base, Const<int32_t> reg, V** p) {
  p[0] = base;
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const uint64_t d = uint64_t(1) << reg[j];
#pragma unroll
    for (int r = 0; r < (1 << j); ++r) p[r | (1 << j)] = p[r] + d;
  }
}

// The same with offset bits that may already be set in off (complemented
// bits): the register strides toggle them.
template <int K, typename V>
__device__ __forceinline__ void amp_ptrs_flip(V* base, uint64_t off, Const<int32_t> reg, V** p) {
  p[0] = base + off;
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const uint64_t b = uint64_t(1) << reg[j];
    const int64_t d = (off & b) ? -(int64_t)b : (int64_t)b;
#pragma unroll
    for (int r = 0; r < (1 << j); ++r) p[r | (1 << j)] = p[r] + d;
  }
}

// At most 128 registers per thread, so that 16 waves share a CU: while a
// workgroup's tile is on its way from or to HBM, the others compute.  (With
// the next tile prefetched into registers instead, FP64 had room for 8 waves:
// brick30 175 ms per step against 165.)
template <typename T, int TB, int K>
__global__ __launch_bounds__(1 << (TB - K), 4) void k_block(cplx<T>* __restrict__ psi,
                                                                const BlkGeom* __restrict__ geom,
                                                                BlkDev d, int n, int nst, int tile_sync) {
  constexpr int R = 1 << K, TBITS = TB - K;
  __shared__ alignas(16) char sh[8 << TB];
  typedef T v2 __attribute__((ext_vector_type(2)));
  v2* gp = reinterpret_cast<v2*>(psi);
  const uint64_t ntiles = uint64_t(1) << (n - TB);
  const uint64_t per = ntiles / gridDim.x, extra = ntiles % gridDim.x, bi = blockIdx.x;
  uint64_t tau = bi * per + (bi < extra ? bi : extra);
  const uint64_t tau_end = tau + per + (bi < extra ? 1 : 0);
  if (tau >= tau_end) return;
  // The geometry is read again for every tile, through an opaque pointer:
  // kept over the layers it would hold the scalar registers that their
  // coefficients need.
  const auto geometry = [&]() {
    const BlkGeom* p = geom;
    asm volatile("" : "+s"(p));
    return as_const<BlkGeom>(p);
  };
  const uint64_t lt = place<TBITS>(threadIdx.x, geometry()->ld_thr);
  const uint64_t wt = place<TBITS>(threadIdx.x, geometry()->st_thr) ^ geometry()->st_flip;
  auto load = [&](uint64_t t, v2* a) {
    const Const<BlkGeom> g = geometry();
    v2* p[R];
    amp_ptrs<K>(gp + block_base(t, g) + lt, g->ld_reg, p);
#pragma unroll
    for (int r = 0; r < R; ++r) a[r] = ld_stream(p[r]);
  };
  Regs<T, K> v;
  load(tau, v.a);
  for (;;) {
    run_stages<T, TB, K>(v, sh, d, nst, tau);
    {
      const Const<BlkGeom> g = geometry();
      v2* p[R];
      amp_ptrs_flip<K>(gp + block_base(tau, g), wt, g->st_reg, p);
#pragma unroll
      for (int r = 0; r < R; ++r) st_stream(p[r], v.a[r]);
    }
    if (++tau >= tau_end) break;
    load(tau, v.a);
    if (tile_sync) __syncthreads();
  }
}

}  // namespace

bool block_sized(juqcs_dtype dt, int b) {
  if (dt == JUQCS_C128) return b >= 11 && b <= 13;
  if (dt == JUQCS_C64) return b >= 11 && b <= 13;
  return false;
}

hipError_t launch_block(juqcs_dtype dt, void* amps, const BlkGeom& g,
                        const BlkGeom* d_geom, const BlkDev& d, hipStream_t s) {
  const uint64_t ntiles = uint64_t(1) << (g.n - g.b);
#define JUQCS_BLOCK(T, TB)                                                                     \
  do {                                                                                         \
    const uint64_t slots = resident_blocks((const void*)k_block<T, TB, kBlkRegs>, 1 << (TB - kBlkRegs)); \
    hipLaunchKernelGGL((k_block<T, TB, kBlkRegs>), dim3((unsigned)(ntiles < slots ? ntiles : slots)),    \
                       dim3(1 << (TB - kBlkRegs)), 0, s, (cplx<T>*)amps, d_geom, d, g.n, g.nst, g.tile_sync); \
  } while (0)
  if (dt == JUQCS_C128 && g.b == 13) JUQCS_BLOCK(double, 13);
  else if (dt == JUQCS_C128 && g.b == 12) JUQCS_BLOCK(double, 12);
  else if (dt == JUQCS_C128 && g.b == 11) JUQCS_BLOCK(double, 11);
  else if (dt == JUQCS_C64 && g.b == 13) JUQCS_BLOCK(float, 13);
  else if (dt == JUQCS_C64 && g.b == 12) JUQCS_BLOCK(float, 12);
  else if (dt == JUQCS_C64 && g.b == 11) JUQCS_BLOCK(float, 11);
  else return hipErrorInvalidValue;
#undef JUQCS_BLOCK
  return hipGetLastError();
}

}  // namespace juqcs
