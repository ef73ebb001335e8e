// Device code of the lattice (populations, streaming, collision) shared by
// the kernel translation units (included only by the .hip files).
#pragma once

#include <hip/hip_fp16.h>

#include "common.h"

namespace lbmib {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Fourth word of a raw buffer resource on this architecture (32-bit data
// format; stride 0, so the range check is against the byte count)
constexpr int kBufferWord3 = 0x00020000;

constexpr float kW0 = 1.0f / 3.0f;
constexpr float kW1 = 1.0f / 18.0f;
constexpr float kW2 = 1.0f / 36.0f;

template <int ST>
struct PopIO;

__device__ constexpr float weight(int q) { return q == 0 ? kW0 : (q < 7 ? kW1 : kW2); }

// Load / store of population q as the deviation g = f - w_q.
template <>
struct PopIO<kFp32> {
  using T = float;
  using Raw = unsigned;
  static constexpr int kNtAux = 2;  // non-temporal buffer loads (the nt bit)
  __device__ static inline float decode(Raw r, int, float) { return __uint_as_float(r); }
  __device__ static inline float ld(const float* p, int, float) { return __builtin_nontemporal_load(p); }
  __device__ static inline float ld_cached(const float* p, int, float) { return *p; }
  __device__ static inline void st(float* p, int, float v, float) { __builtin_nontemporal_store(v, p); }
  __device__ static inline void st_wt(float* p, int, float v, float) { stream_store(p, v); }
};

template <>
struct PopIO<kFp16> {
  using T = __half;
  using Raw = unsigned short;
  static constexpr int kNtAux = 0;  // half loads stay plain (measured faster)
  __device__ static inline float decode(Raw r, int, float inv) { return __half2float(__ushort_as_half(r)) * inv; }
  __device__ static inline float ld(const __half* p, int, float inv) { return __half2float(*p) * inv; }
  __device__ static inline float ld_cached(const __half* p, int q, float inv) { return ld(p, q, inv); }
  __device__ static inline void st(__half* p, int, float v, float scale) { *p = __float2half_rn(v * scale); }
  __device__ static inline void st_wt(__half* p, int, float v, float scale) {
    stream_store(reinterpret_cast<unsigned short*>(p), __half_as_ushort(__float2half_rn(v * scale)));
  }
};

// Unshifted storage of f itself (rounded at the scale of w_q ~ 1/3): the
// reference that shows what the shifted forms gain.
template <>
struct PopIO<kFp32Plain> {
  using T = float;
  using Raw = unsigned;
  static constexpr int kNtAux = 2;
  __device__ static inline float decode(Raw r, int q, float) { return __uint_as_float(r) - weight(q); }
  __device__ static inline float ld(const float* p, int q, float) {
    return __builtin_nontemporal_load(p) - weight(q);
  }
  __device__ static inline float ld_cached(const float* p, int q, float) { return *p - weight(q); }
  __device__ static inline void st(float* p, int q, float v, float) { __builtin_nontemporal_store(v + weight(q), p); }
  __device__ static inline void st_wt(float* p, int q, float v, float) { stream_store(p, v + weight(q)); }
};

// In-place FP32 deviations: the element type and decoding of kFp32; its loads
// and stores are the buffer forms of sc_node_inplace.
template <>
struct PopIO<kFp32InPlace> : PopIO<kFp32> {};

// Offsets (in nodes, periodic wrap folded in) of the six face neighbours.
struct Nbr {
  int xm, xp, ym, yp, zm, zp;
};

__device__ inline Nbr neighbours(int x, int y, int z, int nx, int ny, int nz) {
  const int sz = nx * ny;
  Nbr o;
  o.xm = (x == 0) ? nx - 1 : -1;
  o.xp = (x == nx - 1) ? -(nx - 1) : 1;
  o.ym = (y == 0) ? (ny - 1) * nx : -nx;
  o.yp = (y == ny - 1) ? -(ny - 1) * nx : nx;
  o.zm = (z == 0) ? (nz - 1) * sz : -sz;
  o.zp = (z == nz - 1) ? -(nz - 1) * sz : sz;
  return o;
}

// Pull the 19 deviations of node `base` from the source populations.
// NTLD: non-temporal loads (populations of the last-level-cache size) or
// plain ones (larger sets: 2 % faster on 10 GB of populations, 8 % slower at
// 128^3).
template <int ST, bool NTLD = true, bool OFF32 = false>
__device__ inline void pull(const typename PopIO<ST>::T* __restrict__ src, int64_t base, const Nbr& o, float inv,
                            float* g, uint32_t set_bytes = 0) {
  using IO = PopIO<ST>;
  const int off[kQ] = {0,
                       o.xm, o.xp, o.ym, o.yp, o.zm, o.zp,
                       o.xm + o.ym, o.xp + o.yp, o.xm + o.yp, o.xp + o.ym,
                       o.xm + o.zm, o.xp + o.zp, o.xm + o.zp, o.xp + o.zm,
                       o.ym + o.zm, o.yp + o.zp, o.ym + o.zp, o.yp + o.zm};
  const int lane = (int)(base % kPopBlock);
  if constexpr (OFF32) {
    // A population set below 4 GiB (set_bytes): buffer loads with a 32-bit
    // byte offset per node and the population's constant offset split into a
    // scalar part (multiples of 4 KiB) and the instruction's immediate field,
    // so each load takes one offset register and no 64-bit address
    // arithmetic.  Node m sits at element (m / 256) * 19 * 256 + m % 256 =
    // m + 4608 (m >> 8) of population 0; in bytes, with M = m * sizeof(T):
    // M + 4608 sizeof(T) (M >> (8 + log2 sizeof(T))).  Per population: one
    // add (the neighbour's M), one shift, one 24-bit multiply-add
    // (m >> 8 < 2^23).
    using T = typename PopIO<ST>::T;
    using Raw = typename IO::Raw;
    constexpr uint32_t kSz = (uint32_t)sizeof(T);
    constexpr int kSh = 8 + (kSz == 4 ? 2 : kSz == 2 ? 1 : 0);
    constexpr uint32_t kBlockStep = (kQ - 1) * kPopBlock * kSz;
    constexpr int kAux = NTLD ? IO::kNtAux : 0;
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(src), (short)0, (int)set_bytes, kBufferWord3);
    const uint32_t M = (uint32_t)base * kSz;
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      const uint32_t Mn = M + (uint32_t)off[q] * kSz;  // the neighbour's node, in bytes (wraps to in-box)
      const uint32_t b = __umul24(Mn >> kSh, kBlockStep) + Mn;
      const uint32_t c = (uint32_t)q * kPopBlock * kSz;  // population q's block offset
      Raw r;
      if constexpr (kSz == 2)
        r = __builtin_amdgcn_raw_buffer_load_b16(rs, b + (c & 4095u), c & ~4095u, kAux);
      else
        r = __builtin_amdgcn_raw_buffer_load_b32(rs, b + (c & 4095u), c & ~4095u, kAux);
      g[q] = IO::decode(r, q, inv);
    }
    return;
  } else {
  // larger sets: addresses relative to the node's own population block,
  // 32-bit lane and population offsets, one 64-bit multiply-add per
  // population for the block
  const typename PopIO<ST>::T* bp = src + (base / kPopBlock) * (int64_t)(kQ * kPopBlock);
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    const int rel = lane + off[q];
    const int db = rel >> 8;  // floor(rel / kPopBlock): arithmetic shift, kPopBlock = 256
    const typename PopIO<ST>::T* a = bp + (int64_t)db * (kQ * kPopBlock) + (q * kPopBlock + (rel & (kPopBlock - 1)));
    if constexpr (NTLD)
      g[q] = IO::ld(a, q, inv);
    else
      g[q] = IO::ld_cached(a, q, inv);
  }
  }
}

struct Moments {
  float drho, rho, jx, jy, jz;
};

__device__ inline Moments moments(const float* g) {
  Moments m;
  float s = g[0];
#pragma unroll
  for (int q = 1; q < kQ; ++q) s += g[q];
  m.drho = s;
  m.rho = 1.0f + s;
  m.jx = (g[1] - g[2]) + (g[7] - g[8]) + (g[9] - g[10]) + (g[11] - g[12]) + (g[13] - g[14]);
  m.jy = (g[3] - g[4]) + (g[7] - g[8]) - (g[9] - g[10]) + (g[15] - g[16]) + (g[17] - g[18]);
  m.jz = (g[5] - g[6]) + (g[11] - g[12]) - (g[13] - g[14]) + (g[15] - g[16]) - (g[17] - g[18]);
  return m;
}

// BGK collision of one direction pair (+c, -c) with weight w.
//   e    = c . u_eq, the equilibrium velocity projection
//   cu,cf = c . u and c . F (Guo source), uf = u . F
// Every sum of two products is written as an explicit fmaf: left to the
// compiler, which product is fused can differ between template instances of
// the caller and change the last bit, and the launch variants of the step
// must agree bit for bit.
// 1/rho from the hardware reciprocal (within one ulp; rho stays near 1 in
// these flows), in place of the correctly rounded division sequence
__device__ inline float inv_density(float rho) { return __builtin_amdgcn_rcpf(rho); }

// SRC = false: the source term is zero (no force at the node, or Shan-Chen
// forcing) and is left out of the arithmetic; the populations are the same
// as with the zero term added (up to the sign of an exact zero).
template <bool SRC>
__device__ inline void collide_pair(float& gp, float& gm, float w, float om, float drho, float rho,
                                    float usq15, float e, float src_a, float cu, float cf,
                                    float uf) {
  const float sym = w * (drho + rho * fmaf(4.5f * e, e, -usq15));
  const float wr3 = w * rho * 3.0f;
  const float eqp = fmaf(wr3, e, sym), eqm = fmaf(-wr3, e, sym);
  if constexpr (SRC) {
    // Guo source: src_a (1 - om/2) w [3 (c - u).F + 9 (c.u)(c.F)]
    const float sw = src_a * w;
    const float s_sym = sw * fmaf(9.0f * cu, cf, -3.0f * uf);
    const float sw3 = sw * 3.0f;
    const float sp = fmaf(sw3, cf, s_sym), sm = fmaf(-sw3, cf, s_sym);
    gp = gp + om * (eqp - gp) + sp;
    gm = gm + om * (eqm - gm) + sm;
  } else {
    gp = gp + om * (eqp - gp);
    gm = gm + om * (eqm - gm);
  }
}

// BGK collision of all 19 populations (with the Guo source when SRC).
template <bool SRC>
__device__ inline void collide_all(float* g, const Moments& m, float om, float ex, float ey, float ez, float src_a,
                                   float ux, float uy, float uz, float Fx, float Fy, float Fz) {
  const float usq15 = 1.5f * fmaf(ez, ez, fmaf(ey, ey, ex * ex));
  const float uf = SRC ? fmaf(uz, Fz, fmaf(uy, Fy, ux * Fx)) : 0.0f;
  // rest population
  {
    const float eq0 = kW0 * (m.drho - m.rho * usq15);
    if constexpr (SRC)
      g[0] = g[0] + om * (eq0 - g[0]) + src_a * kW0 * (-3.0f * uf);
    else
      g[0] = g[0] + om * (eq0 - g[0]);
  }
  // faces
  collide_pair<SRC>(g[1], g[2], kW1, om, m.drho, m.rho, usq15, ex, src_a, ux, Fx, uf);
  collide_pair<SRC>(g[3], g[4], kW1, om, m.drho, m.rho, usq15, ey, src_a, uy, Fy, uf);
  collide_pair<SRC>(g[5], g[6], kW1, om, m.drho, m.rho, usq15, ez, src_a, uz, Fz, uf);
  // edges
  collide_pair<SRC>(g[7], g[8], kW2, om, m.drho, m.rho, usq15, ex + ey, src_a, ux + uy, Fx + Fy, uf);
  collide_pair<SRC>(g[9], g[10], kW2, om, m.drho, m.rho, usq15, ex - ey, src_a, ux - uy, Fx - Fy, uf);
  collide_pair<SRC>(g[11], g[12], kW2, om, m.drho, m.rho, usq15, ex + ez, src_a, ux + uz, Fx + Fz, uf);
  collide_pair<SRC>(g[13], g[14], kW2, om, m.drho, m.rho, usq15, ex - ez, src_a, ux - uz, Fx - Fz, uf);
  collide_pair<SRC>(g[15], g[16], kW2, om, m.drho, m.rho, usq15, ey + ez, src_a, uy + uz, Fy + Fz, uf);
  collide_pair<SRC>(g[17], g[18], kW2, om, m.drho, m.rho, usq15, ey - ez, src_a, uy - uz, Fy - Fz, uf);
}

// Workgroup -> logical block.  Workgroups are handed to the 8 XCDs round
// robin; with `remap` each XCD instead receives one contiguous range of
// logical blocks, so the cache lines shared by neighbouring blocks (the
// x-shifted pulls straddle block edges) stay in one XCD's L2.
__device__ inline int logical_block(int remap, int nblocks) {
  if (!remap) return blockIdx.x;
  const int per = (int)gridDim.x / 8;  // grid is a multiple of 8 when remapping
  return (blockIdx.x % 8) * per + blockIdx.x / 8;
}

// ---- in-place storage (one population set) ------------------------------------
// The AA access pattern (Bailey, Myre, Walsh, Lilja and Lerner, "Accelerating
// lattice Boltzmann fluid flow simulations using graphics processors", ICPP
// 2009): one set of deviations, updated in place.  With the state after an
// odd number of steps (and the initial state) holding f*_q(x) in slot q of
// node x + c_q, an even step n reads the incoming f_q(x) from its own slot q
// and writes f*_q(x) back to slot opposite(q) of the same node; after it,
// slot opposite(q) of node x holds f*_q(x), so an odd step reads f_q(x) =
// f*_q(x - c_q) from slot opposite(q) of node x - c_q and writes f*_q(x) to
// slot q of node x + c_q, which restores the first arrangement.  Every node
// reads and writes the same 19 slots and no other node touches them in that
// step, so the launches of one step (bulk and near blocks) may run
// concurrently, as with two sets.  The moments, forcing and collision are
// the same as for two sets, so the results equal the two-set storage bit for bit.
// Loads and stores go through a buffer resource bounded by the set's size.

// Node offsets of the upstream neighbours x - c_q, periodic wrap folded in.
__device__ inline void upstream_offsets(const Nbr& o, int* off) {
  const int t[kQ] = {0,
                     o.xm, o.xp, o.ym, o.yp, o.zm, o.zp,
                     o.xm + o.ym, o.xp + o.yp, o.xm + o.yp, o.xp + o.ym,
                     o.xm + o.zm, o.xp + o.zp, o.xm + o.zp, o.xp + o.zm,
                     o.ym + o.zm, o.yp + o.zp, o.ym + o.zp, o.yp + o.zm};
#pragma unroll
  for (int q = 0; q < kQ; ++q) off[q] = t[q];
}

// Byte offset of population 0 of node byte offset M = m * 4 in the block layout
// (m + 4608 (m >> 8) elements, see pull).
__device__ inline uint32_t inplace_node_bytes(uint32_t M) {
  return __umul24(M >> 10, (uint32_t)((kQ - 1) * kPopBlock * 4)) + M;
}

__device__ inline __amdgpu_buffer_rsrc_t inplace_rsrc(const Dev& d) {
  return __builtin_amdgcn_make_buffer_rsrc(d.pop[0], (short)0, (int)(uint32_t)(kQ * d.pstride * 4), kBufferWord3);
}

// Slot q of the node at byte offset b (from inplace_node_bytes), as float.
__device__ inline float inplace_load(__amdgpu_buffer_rsrc_t rs, uint32_t b, int q) {
  const uint32_t c = (uint32_t)q * kPopBlock * 4u;
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, b + (c & 4095u), c & ~4095u, 0));
}

// Stores written through (system-coherent, the sc0 sc1 bits) while the set
// is of the order of the last-level cache, non-temporal above.
template <int AUX>
__device__ inline void inplace_store(__amdgpu_buffer_rsrc_t rs, uint32_t b, int q, float v) {
  const uint32_t c = (uint32_t)q * kPopBlock * 4u;
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rs, b + (c & 4095u), c & ~4095u, AUX);
}
constexpr int kAuxWriteThrough = 17;  // sc0 | sc1
constexpr int kAuxNonTemporal = 2;    // nt

// The state after `steps` steps, f*_q(x) of node x (byte offset M), into g.
__device__ inline void inplace_post(__amdgpu_buffer_rsrc_t rs, uint32_t M, const int* off, int64_t steps, float* g) {
  if (steps & 1) {
    const uint32_t b = inplace_node_bytes(M);
#pragma unroll
    for (int q = 0; q < kQ; ++q) g[q] = inplace_load(rs, b, opposite(q));
  } else {
#pragma unroll
    for (int q = 0; q < kQ; ++q) g[q] = inplace_load(rs, inplace_node_bytes(M + (uint32_t)off[opposite(q)] * 4u), q);
  }
}

template <int AUX>
__device__ inline void inplace_push(__amdgpu_buffer_rsrc_t rs, uint32_t M, const int* off, bool odd, const float* g) {
  if (!odd) {
    const uint32_t b = inplace_node_bytes(M);
#pragma unroll
    for (int q = 0; q < kQ; ++q) inplace_store<AUX>(rs, b, opposite(q), g[q]);
  } else {
#pragma unroll
    for (int q = 0; q < kQ; ++q) inplace_store<AUX>(rs, inplace_node_bytes(M + (uint32_t)off[opposite(q)] * 4u), q, g[q]);
  }
}

// ---- one node of the fused step ------------------------------------------------
// In two parts, so that a caller can do other work between the loads and the
// collision: sc_load gathers the 19 incoming deviations, sc_finish does the
// moments, forcing, BGK collision and stores.

// The FP64 time-average sums of a node in a sampled step: loaded with the
// populations, so that their latency overlaps (a load issued after the stores
// left a full memory latency exposed per block).
struct AvgSums {
  double x, y, z;
};

__device__ inline AvgSums avg_load(const Dev& d, int64_t base, bool avg) {
  AvgSums a{0.0, 0.0, 0.0};
  if (avg) {
    a.x = d.uavg[base];
    a.y = d.uavg[d.pstride + base];
    a.z = d.uavg[2 * d.pstride + base];
  }
  return a;
}

template <int ST, bool NTLD, bool OFF32>
__device__ inline void sc_load(const Dev& d, const Nbr& o, int64_t base, int64_t n, float* g) {
  if constexpr (ST == kFp32InPlace) {
    const __amdgpu_buffer_rsrc_t rs = inplace_rsrc(d);
    const uint32_t M = (uint32_t)base * 4u;
    if (!(n & 1)) {
      const uint32_t b = inplace_node_bytes(M);
#pragma unroll
      for (int q = 0; q < kQ; ++q) g[q] = inplace_load(rs, b, q);
    } else {
      int off[kQ];
      upstream_offsets(o, off);
#pragma unroll
      for (int q = 0; q < kQ; ++q)
        g[q] = inplace_load(rs, inplace_node_bytes(M + (uint32_t)off[q] * 4u), opposite(q));
    }
  } else {
    using T = typename PopIO<ST>::T;
    pull<ST, NTLD, OFF32>(static_cast<const T*>(d.pop[n & 1]), base, o, d.fp16_inv, g,
                          (uint32_t)(kQ * d.pstride * (int64_t)sizeof(T)));
  }
}

// The stores of a node's 19 post-collision deviations.  SERIAL (in-place
// storage): a full-grid launch with no concurrent kernels, whose odd-step
// stores go plain (the L2 merges the partial lines of the neighbours'
// scattered runs: 128^3 FP32 launch 48.1 against 50.2 us written through);
// beside the immersed-boundary kernels they stay written through (plain:
// step 58.9 against 56.8 us, the L2 taken from the concurrent kernels).
// WT: whether the stores are written through, 0 / 1, or 2: as d.small_pops says.
// EARLY: the population set to write is `set`, else it is looked up here.
template <int ST, bool OFF32, bool SERIAL, int WT = 2, bool EARLY = false>
__device__ inline void sc_store(const Dev& d, const Nbr& o, int64_t base, int64_t n, const float* g, void* set) {
  if constexpr (ST == kFp32InPlace) {
    const __amdgpu_buffer_rsrc_t rs = inplace_rsrc(d);
    const uint32_t M = (uint32_t)base * 4u;
    const bool odd = (n & 1) != 0;
    int off[kQ];
    upstream_offsets(o, off);
    const bool through = WT == 2 ? d.small_pops != 0 : WT == 1;
    if (!through)
      inplace_push<kAuxNonTemporal>(rs, M, off, odd, g);
    else if (SERIAL && odd)
      inplace_push<0>(rs, M, off, true, g);
    else
      inplace_push<kAuxWriteThrough>(rs, M, off, odd, g);
  } else {
    using IO = PopIO<ST>;
    using T = typename IO::T;
    T* __restrict__ dst = static_cast<T*>(EARLY ? set : d.pop[(n + 1) & 1]);
    T* bq;
    if constexpr (OFF32) {
      // 32-bit byte offsets from the set's start (see pull): one offset
      // register for all 19 stores, the population's q * 256 elements are a
      // constant the store instruction carries
      constexpr uint32_t kSz = (uint32_t)sizeof(T);
      constexpr int kSh = 8 + (kSz == 4 ? 2 : kSz == 2 ? 1 : 0);
      const uint32_t M = (uint32_t)base * kSz;
      bq = reinterpret_cast<T*>(reinterpret_cast<char*>(dst) + (__umul24(M >> kSh, (kQ - 1) * kPopBlock * kSz) + M));
    } else {
      bq = dst + (base / kPopBlock) * (int64_t)(kQ * kPopBlock) + (int)(base % kPopBlock);
    }
    if (WT == 2 ? d.small_pops != 0 : WT == 1) {
#pragma unroll
      for (int q = 0; q < kQ; ++q) IO::st_wt(bq + q * kPopBlock, q, g[q], d.fp16_scale);
    } else {
#pragma unroll
      for (int q = 0; q < kQ; ++q) IO::st(bq + q * kPopBlock, q, g[q], d.fp16_scale);
    }
  }
}

// Moments, forcing, BGK collision and stores of a node with the total force
// density (Fx, Fy, Fz).
// `forced`: write u at this node (markers may interpolate there).
// `avg`: add u to the node's time-average sums (a sampled step).
// MOM: also record (rho, u) of the node in d.mom.
template <int ST, bool MOM, bool OFF32, bool SERIAL, int WT = 2, bool EARLY = false>
__device__ inline void sc_finish(const Dev& d, const Box& B, const Nbr& o, int64_t base, int64_t n, float* g, float Fx,
                                 float Fy, float Fz, bool forced, bool avg, const AvgSums& a, void* set = nullptr) {
  const int64_t ps = d.pstride;
  const Moments m = moments(g);
  const float ir = inv_density(m.rho);
  const float ux = (m.jx + 0.5f * Fx) * ir;
  const float uy = (m.jy + 0.5f * Fy) * ir;
  const float uz = (m.jz + 0.5f * Fz) * ir;
  if (forced) {
    d.u[base] = ux;
    d.u[ps + base] = uy;
    d.u[2 * ps + base] = uz;
  }
  if constexpr (MOM) {
    const f32x4 rec = {m.rho, ux, uy, uz};
    __builtin_nontemporal_store(rec, reinterpret_cast<f32x4*>(d.mom) + base);
  }
  float ex = ux, ey = uy, ez = uz, src_a = 1.0f - 0.5f * B.omega;
  if (B.forcing == kShanChen) {
    ex = (m.jx + B.tau * Fx) * ir;
    ey = (m.jy + B.tau * Fy) * ir;
    ez = (m.jz + B.tau * Fz) * ir;
    src_a = 0.0f;
  }
  // no force at the node (most nodes) or Shan-Chen forcing: no source term
  if (src_a != 0.0f && (Fx != 0.0f || Fy != 0.0f || Fz != 0.0f))
    collide_all<true>(g, m, B.omega, ex, ey, ez, src_a, ux, uy, uz, Fx, Fy, Fz);
  else
    collide_all<false>(g, m, B.omega, ex, ey, ez, src_a, ux, uy, uz, Fx, Fy, Fz);
  sc_store<ST, OFF32, SERIAL, WT, EARLY>(d, o, base, n, g, set);
  if (avg) {
    double* __restrict__ acc = d.uavg;
    acc[base] = a.x + (double)ux;
    acc[ps + base] = a.y + (double)uy;
    acc[2 * ps + base] = a.z + (double)uz;
  }
}

// One node: `forced` nodes read the spread force density F and write u.
// EARLY: the address of the set to write is looked up before the populations are
// loaded, not before the stores, which a persistent workgroup's next block waits for
// (64 boxes, 17.6 M nodes, one per compute unit: 705 us per step, else 730; one
// workgroup per block gains nothing).
template <int ST, bool MOM = false, bool NTLD = true, bool OFF32 = false, bool SERIAL = false, bool EARLY = false>
__device__ inline void sc_node(const Dev& d, const Box& B, int x, int y, int z, int64_t base, int64_t n, bool forced,
                               bool avg) {
  static_assert(!MOM || ST != kFp32InPlace, "the in-place storage does not record moments");
  const Nbr o = neighbours(x, y, z, B.nx, B.ny, B.nz);
  const AvgSums a = avg_load(d, base, avg);
  void* const set = EARLY ? d.pop[(n + 1) & 1] : nullptr;
  float g[kQ];
  sc_load<ST, NTLD, OFF32>(d, o, base, n, g);
  float Fx = B.gx, Fy = B.gy, Fz = B.gz;
  if (forced) {
    Fx += d.F[base];
    Fy += d.F[d.pstride + base];
    Fz += d.F[2 * d.pstride + base];
  }
  sc_finish<ST, MOM, OFF32, SERIAL, 2, EARLY>(d, B, o, base, n, g, Fx, Fy, Fz, forced, avg, a, set);
}

// Whether step n adds to the time-average sums (uniform over a launch).
__device__ inline bool avg_sampled(const Dev& d, int64_t n) {
  return d.uavg != nullptr && n >= d.avg_t0 && (n - d.avg_t0) % d.avg_every == 0;
}

// One block of BS nodes.  `bulk`: none of its nodes is forced (every node a
// stencil reaches lies in a near block, and an active tile's other nodes carry
// F = 0).
template <int ST, int BS, bool NTLD, bool SERIAL, bool MOM = false, bool EARLY = false>
__device__ inline void sc_block(const Dev& d, int blk, int64_t n, bool bulk, bool avg) {
  const int b = d.nboxes == 1 ? 0 : d.sc_block_box[blk];
  const Box B = d.boxes[b];
  const int first = d.nboxes == 1 ? 0 : d.sc_box_block0[b];
  const int id = (blk - first) * BS + (int)threadIdx.x;
  if (id >= B.n) return;
  const int yz = (int)divide((uint32_t)id, B.div_nx);
  const int x = id - yz * B.nx;
  const int z = (int)divide((uint32_t)yz, B.div_ny);
  const int y = yz - z * B.ny;
  bool forced = false;
  if (!bulk) {
    const int tile = B.tile0 + (x / kTile) + B.tx * ((y / kTile) + B.ty * (z / kTile));
    forced = d.stamp[tile] == (int)n;
  }
  // the two addressing forms as separate code (a population set below 4 GiB
  // takes 32-bit offsets; the in-place set always does)
  if (ST == kFp32InPlace || d.pops32)
    sc_node<ST, MOM, NTLD, true, SERIAL, EARLY>(d, B, x, y, z, B.node0 + id, n, forced, avg);
  else
    sc_node<ST, MOM, NTLD, false, SERIAL, EARLY>(d, B, x, y, z, B.node0 + id, n, forced, avg);
}

}  // namespace
}  // namespace lbmib
