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
// brick30 175 ms per step where this form took 165; it takes 157 now.)
// The geometry is read again for every tile, through an opaque pointer: kept
// over the layers it would hold the scalar registers that their coefficients
// need.
__device__ __forceinline__ Const<BlkGeom> geometry(const BlkPass* p) {
  asm volatile("" : "+s"(p));
  return as_const<BlkGeom>(&p->g);
}

template <typename T, int TB, int K>
__global__ __launch_bounds__(1 << (TB - K), 4) void k_block(cplx<T>* __restrict__ psi,
                                                            const BlkPass* __restrict__ pass, BlkDev d, int n,
                                                            int nst, int tile_sync) {
  constexpr int R = 1 << K, TBITS = TB - K;
  __shared__ alignas(16) char sh[8 << TB];
  typedef T v2 __attribute__((ext_vector_type(2)));
  v2* gp = reinterpret_cast<v2*>(psi);
  const uint64_t ntiles = uint64_t(1) << (n - TB);
  const uint64_t per = ntiles / gridDim.x, extra = ntiles % gridDim.x, bi = blockIdx.x;
  uint64_t tau = bi * per + (bi < extra ? bi : extra);
  const uint64_t tau_end = tau + per + (bi < extra ? 1 : 0);
  if (tau >= tau_end) return;
  const uint64_t lt = place<TBITS>(threadIdx.x, geometry(pass)->ld_thr);
  const uint64_t wt = place<TBITS>(threadIdx.x, geometry(pass)->st_thr) ^ geometry(pass)->st_flip;
  const auto load = [&](uint64_t t, v2* a) {
    const Const<BlkGeom> g = geometry(pass);
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
      const Const<BlkGeom> g = geometry(pass);
      v2* p[R];
      amp_ptrs_flip<K>(gp + block_base(tau, g), wt, g->st_reg, p);
#pragma unroll
      for (int r = 0; r < R; ++r) st_stream(p[r], v.a[r]);
    }
    if (++tau >= tau_end) break;
    load(tau, v.a);  // on its way while the waves wait for each other (20 brick layers on 30 qubits: 175 -> 170 ms)
    if (tile_sync) __syncthreads();
  }
}

// Two-byte amplitudes: register bits 0..2 of the first and the last stage
// are the 8 amplitudes of a 16-byte group of codes, the last register bit
// tells a thread's two groups apart, and the lowest lane bits of the last
// stage are the rest of a scale block.  A pass decodes and encodes in
// registers: against tiles decoded into LDS and encoded from there, it needs
// no LDS access but the exchanges.  A pass over 2^33 amplitudes without
// rotations takes 9.9 ms (tiles in LDS: 21.5; its 32 GiB of traffic 6.6), and
// 12 ms without the next tile's codes in flight; 29 qubits with a rotation and
// a phase each 1.27 ms a pass of five to six rotations, vector instructions.
typedef int32_t codes4 __attribute__((ext_vector_type(4)));
constexpr float kTiny = 7.888609052210118e-31f;  // 2^-100: smaller block maxima code as zero

// Eight amplitudes from their codes: code c is byte c + 128 of w ^ 0x80.., and
// fma(c + 128, d, -128 d) rounds c d once (128 d is exact below 2^121; larger
// states take the fused passes.  Testing for it here took 1.4% of the passes of
// 29 qubits).
template <typename V>
__device__ __forceinline__ void decode_group(const codes4& w, float d, V* a) {
  const float off = -128.0f * d;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t u = (uint32_t)w[j] ^ 0x80808080u;
    a[2 * j] = V{__builtin_fmaf((float)(u & 0xffu), d, off), __builtin_fmaf((float)((u >> 8) & 0xffu), d, off)};
    a[2 * j + 1] =
        V{__builtin_fmaf((float)((u >> 16) & 0xffu), d, off), __builtin_fmaf((float)(u >> 24), d, off)};
  }
}

template <typename V>
__device__ __forceinline__ uint32_t group_max(const V* a) {
  float m = 0.0f;  // (fmaxf would canonicalise every argument first)
#pragma unroll
  for (int j = 0; j < 8; ++j) asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(a[j].x), "v"(a[j].y));
  return __float_as_uint(m);
}

// Codes of eight amplitudes: x = a r clamped to +-127, then rounded to an
// integer by adding 1.5 2^23, which leaves it in the sum's low byte.
template <typename V>
__device__ __forceinline__ codes4 encode_group(const V* a, float r) {
  const auto code = [&](float x) {
    return __float_as_uint(__builtin_amdgcn_fmed3f(x * r, -127.0f, 127.0f) + 12582912.0f);
  };
  codes4 w;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t lo = __builtin_amdgcn_perm(code(a[2 * j].y), code(a[2 * j].x), 0x0c0c0400u);
    const uint32_t hi = __builtin_amdgcn_perm(code(a[2 * j + 1].y), code(a[2 * j + 1].x), 0x0c0c0400u);
    w[j] = (int32_t)(lo | hi << 16);
  }
  return w;
}

template <int TB, int K>
__global__ __launch_bounds__(1 << (TB - K), 4) void k_block_codes(int8_t* __restrict__ codes,
                                                                  float* __restrict__ scales,
                                                                  const BlkPass* __restrict__ pass, BlkDev d,
                                                                  int n, int nst, int tile_sync, int B) {
  constexpr int TBITS = TB - K;
  static_assert(K == 4, "two groups of codes per thread");
  __shared__ alignas(16) char sh[8 << TB];
  const uint64_t ntiles = uint64_t(1) << (n - TB);
  const uint64_t per = ntiles / gridDim.x, extra = ntiles % gridDim.x, bi = blockIdx.x;
  uint64_t tau = bi * per + (bi < extra ? bi : extra);
  const uint64_t tau_end = tau + per + (bi < extra ? 1 : 0);
  if (tau >= tau_end) return;
  const uint64_t lt = place<TBITS>(threadIdx.x, geometry(pass)->ld_thr);
  const uint64_t wt = place<TBITS>(threadIdx.x, geometry(pass)->st_thr) ^ (geometry(pass)->st_flip & ~uint64_t(7));
  // the next tile's codes (8 registers) come in while a tile is worked on
  codes4 w0, w1;
  float s0, s1;
  const auto fetch = [&](uint64_t t) {
    const Const<BlkGeom> g = geometry(pass);
    const uint64_t a0 = block_base(t, g) + lt, a1 = a0 + (uint64_t(1) << g->ld_reg[3]);
    w0 = ld_stream(reinterpret_cast<const codes4*>(codes + 2 * a0));
    w1 = ld_stream(reinterpret_cast<const codes4*>(codes + 2 * a1));
    s0 = ld_stream(&scales[a0 >> B]);
    s1 = ld_stream(&scales[a1 >> B]);
  };
  Regs<float, K> v;
  fetch(tau);
  for (;;) {
    decode_group(w0, s0 / 127.0f, v.a);
    decode_group(w1, s1 / 127.0f, v.a + 8);
    fetch(tau + 1 < tau_end ? tau + 1 : tau);
    run_stages<float, TB, K>(v, sh, d, nst, tau);
    {
      const Const<BlkGeom> g = geometry(pass);
      const uint64_t hi = uint64_t(1) << g->st_reg[3], a0 = block_base(tau, g) | wt, a1 = a0 ^ hi;
      const int flip = (int)(g->st_flip & 7);
      // a block's groups are the lanes that differ in the lowest B - 3 bits
      uint32_t m0 = group_max(v.a), m1 = group_max(v.a + 8);
      for (int x = 1; x < 1 << (B - 3); x <<= 1) {
        const uint32_t o0 = (uint32_t)__shfl_xor((int)m0, x, 64), o1 = (uint32_t)__shfl_xor((int)m1, x, 64);
        m0 = o0 > m0 ? o0 : m0;
        m1 = o1 > m1 ? o1 : m1;
      }
      const auto put = [&](const auto* a, uint32_t m, uint64_t at) {
        const float s = __uint_as_float(m);
        const bool zero = !(s >= kTiny);
        codes4 w = encode_group(a, 127.0f / s);
        if (flip & 1)
#pragma unroll
          for (int j = 0; j < 4; ++j) w[j] = (int32_t)__builtin_amdgcn_alignbit((uint32_t)w[j], (uint32_t)w[j], 16);
        if (flip & 2) w = codes4{w[1], w[0], w[3], w[2]};
        if (flip & 4) w = codes4{w[2], w[3], w[0], w[1]};
        if (zero) w = codes4{0, 0, 0, 0};
        st_stream(reinterpret_cast<codes4*>(codes + 2 * at), w);
        if ((threadIdx.x & ((1 << (B - 3)) - 1)) == 0) st_stream(&scales[at >> B], zero ? 0.0f : s);
      };
      put(v.a, m0, a0);
      put(v.a + 8, m1, a1);
    }
    if (++tau >= tau_end) break;
    if (tile_sync) __syncthreads();
  }
}

// One round of many C64 states: workgroups claim chunks of tiles through the
// ticket counter until none are left (none ever waits for another).  States
// are read and written through the caches.  A round goes over all of its
// states, so they stay there from pass to pass only where they take less than
// the 256 MiB last-level cache together: the levels of small decompositions,
// not those of 42 qubits in halves with 8 crossings (98 GB at 3.1 TB/s).
template <int TB, int K>
__global__ __launch_bounds__(1 << (TB - K), 4) void k_block_round(
    char* __restrict__ states, const BatchGroup* __restrict__ groups, int g0, int g1,
    const BlkPass* __restrict__ passes, BlkDev d, unsigned long long* __restrict__ ticket, long long c0,
    long long c1) {
  constexpr int R = 1 << K, TBITS = TB - K;
  __shared__ alignas(16) char sh[8 << TB];
  __shared__ long long s_t;
  __shared__ int s_g;
  typedef float v2 __attribute__((ext_vector_type(2)));
  const BlkStage* const stages = d.stages;
  for (;;) {
    __syncthreads();  // the last chunk's exchanges are done with sh
    if (threadIdx.x == 0) {
      const long long t = c0 + (long long)atomicAdd(ticket, 1ull);
      int g = -1;
      if (t < c1) {  // last group of the round whose first chunk is <= t
        int lo = g0, hi = g1 - 1;
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (groups[mid].first_chunk <= t) lo = mid;
          else hi = mid - 1;
        }
        g = lo;
      }
      s_t = t;
      s_g = g;
    }
    __syncthreads();
    const int gi = __builtin_amdgcn_readfirstlane(s_g);
    if (gi < 0) break;  // every workgroup leaves once the round's tickets run out
    const int t_lo = __builtin_amdgcn_readfirstlane((int)s_t), t_hi = __builtin_amdgcn_readfirstlane((int)(s_t >> 32));
    const long long t = ((long long)t_hi << 32) | (uint32_t)t_lo;
    const Const<BatchGroup> grp = as_const<BatchGroup>(groups + gi);
    const BlkPass* pass = passes + grp->pass;
    v2* dst = reinterpret_cast<v2*>(states + grp->state_off);
    const v2* src = reinterpret_cast<const v2*>(states + grp->src_off);
    const bool init = grp->init != 0;
    uint64_t tau = (uint64_t)(t - grp->first_chunk) * grp->chunk_tiles;
    const uint64_t tau_end = tau + grp->chunk_tiles;
    const int nst = geometry(pass)->nst, tile_sync = geometry(pass)->tile_sync;
    d.stages = stages + as_const<BlkPass>(pass)->stage_begin;
    const uint64_t lt = place<TBITS>(threadIdx.x, geometry(pass)->ld_thr);
    const uint64_t wt = place<TBITS>(threadIdx.x, geometry(pass)->st_thr) ^ geometry(pass)->st_flip;
    const auto load = [&](uint64_t t, v2* a) {
      const Const<BlkGeom> g = geometry(pass);
      if (init) {  // first pass: the state is |0...0>
#pragma unroll
        for (int r = 0; r < R; ++r) a[r] = v2{r == 0 && t == 0 && lt == 0 ? 1.0f : 0.0f, 0.0f};
      } else {
        const v2* p[R];
        amp_ptrs<K>(src + block_base(t, g) + lt, g->ld_reg, p);
#pragma unroll
        for (int r = 0; r < R; ++r) a[r] = *p[r];
      }
    };
    Regs<float, K> v;
    load(tau, v.a);
    for (;;) {
      run_stages<float, TB, K>(v, sh, d, nst, tau);
      {
        const Const<BlkGeom> g = geometry(pass);
        v2* p[R];
        amp_ptrs_flip<K>(dst + block_base(tau, g), wt, g->st_reg, p);
#pragma unroll
        for (int r = 0; r < R; ++r) *p[r] = v.a[r];
      }
      if (++tau >= tau_end) break;
      load(tau, v.a);
      if (tile_sync) __syncthreads();
    }
  }
}

}  // namespace

bool block_sized(juqcs_dtype dt, int b) {
  return (dt == JUQCS_C128 || dt == JUQCS_C64) && b >= kBlkMinTile && b < kBlkMinTile + kBlkTileSizes;
}

// Blocks of 8 to 512 amplitudes: a block's groups of 8 are lanes of a wave.
bool block_codes_sized(int block_bits, int b) { return block_bits >= 3 && block_bits <= 9 && b == 13; }

hipError_t launch_block(juqcs_dtype dt, void* amps, void* scales, const BlkPass& p, const BlkPass* d_pass, const BlkDev& d,
                        hipStream_t s) {
  const BlkGeom& g = p.g;
  const uint64_t ntiles = uint64_t(1) << (g.n - g.b);
  BlkDev dev = d;
  dev.stages += p.stage_begin;
#define JUQCS_BLOCK(T, TB)                                                                     \
  do {                                                                                         \
    const uint64_t slots = resident_blocks((const void*)k_block<T, TB, kBlkRegs>, 1 << (TB - kBlkRegs)); \
    hipLaunchKernelGGL((k_block<T, TB, kBlkRegs>), dim3((unsigned)(ntiles < slots ? ntiles : slots)),    \
                       dim3(1 << (TB - kBlkRegs)), 0, s, (cplx<T>*)amps, d_pass, dev, g.n, g.nst, g.tile_sync); \
  } while (0)
  if (dt == JUQCS_C128 && g.b == 13) JUQCS_BLOCK(double, 13);
  else if (dt == JUQCS_C128 && g.b == 12) JUQCS_BLOCK(double, 12);
  else if (dt == JUQCS_C128 && g.b == 11) JUQCS_BLOCK(double, 11);
  else if (dt == JUQCS_C64 && g.b == 13) JUQCS_BLOCK(float, 13);
  else if (dt == JUQCS_C64 && g.b == 12) JUQCS_BLOCK(float, 12);
  else if (dt == JUQCS_C64 && g.b == 11) JUQCS_BLOCK(float, 11);
  else if (dt == JUQCS_ENC2 && block_codes_sized(g.block_bits, g.b)) {
    const uint64_t slots = resident_blocks((const void*)k_block_codes<13, kBlkRegs>, 1 << (13 - kBlkRegs));
    hipLaunchKernelGGL((k_block_codes<13, kBlkRegs>), dim3((unsigned)(ntiles < slots ? ntiles : slots)),
                       dim3(1 << (13 - kBlkRegs)), 0, s, (int8_t*)amps, (float*)scales, d_pass, dev, g.n, g.nst,
                       g.tile_sync, g.block_bits);
  }
  else return hipErrorInvalidValue;
#undef JUQCS_BLOCK
  return hipGetLastError();
}

hipError_t launch_block_round(int b, char* states, const BatchGroup* groups, int g0, int g1,
                              const BlkPass* passes, const BlkDev& d, uint64_t* ticket, long long c0,
                              long long c1, hipStream_t s) {
  if (c1 <= c0) return hipSuccess;
#define JUQCS_ROUND(TB)                                                                            \
  do {                                                                                             \
    const uint64_t slots = resident_blocks((const void*)k_block_round<TB, kBlkRegs>, 1 << (TB - kBlkRegs)); \
    const uint64_t grid = (uint64_t)(c1 - c0) < slots ? (uint64_t)(c1 - c0) : slots;               \
    hipLaunchKernelGGL((k_block_round<TB, kBlkRegs>), dim3((unsigned)grid), dim3(1 << (TB - kBlkRegs)), 0, s, \
                       states, groups, g0, g1, passes, d, (unsigned long long*)ticket, c0, c1);    \
  } while (0)
  if (b == 13) JUQCS_ROUND(13);
  else if (b == 12) JUQCS_ROUND(12);
  else if (b == 11) JUQCS_ROUND(11);
  else return hipErrorInvalidValue;
#undef JUQCS_ROUND
  return hipGetLastError();
}

}  // namespace juqcs
