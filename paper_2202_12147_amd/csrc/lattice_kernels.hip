// Lattice kernels: fused pull stream-collide, macroscopic output, and the
// FP64 conservation reductions.
//
// Fluid model (paper Sec. 2.1): D3Q19 BGK, Eq. (lbe) with the second-order
// equilibrium of Eq. (lbm:equilibrium); moments rho = sum f, rho u_eq =
// sum f c + tau F for the Shan-Chen force scheme (Eq. sc), physical velocity
// rho u = sum f c + F/2.  The Guo scheme uses u in the equilibrium and adds
// (1 - 1/(2 tau)) w_i [3 (c_i - u) + 9 (c_i.u) c_i].F.
//
// Storage holds g_i = f_i - w_i (deviation from the rest state), so the
// O(1e-5) flow signal is not swamped by the O(1/3) weights in FP32; FP16
// storage holds g_i * S rounded to nearest even; the unshifted reference
// storage holds f_i.  Arithmetic is FP32 on g in all three.
//
// Streaming is "pull": node x gathers g*_i(x - c_i) from the source parity and
// writes its 19 post-collision values to the same node of the other parity,
// so every read and write of a wavefront covers consecutive x (coalesced);
// only the c_x = +-1 loads are shifted by one element.
#include "common.h"
#include "lattice_device.h"
#include "bead_terms.h"
#include "near_marks.h"
#include "step_launch.h"

#include <hip/hip_ext.h>

#include <algorithm>
#include <mutex>

namespace lbmib {

namespace {

// Launch modes: every node of the grid, F and u where the node's tile is stamped
// active for this step (kLaunchAll); and the two of the two-stream schedule:
// every block except those marked near at the previous step,
// never forced (kLaunchBulk), and one workgroup per listed near block
// (kLaunchActive).  AVG: the variant launched while a time average of u runs
// (the sampling test and the sums); without it the averaging code is compiled
// out.
template <int ST, int BS, int MODE, bool AVG, bool NTLD>
__global__ __launch_bounds__(BS) void k_stream_collide(Dev d, int remap, int nblocks, int resident) {
  const int64_t n = *d.step + d.sub;
  const int64_t pn = n - 1;  // the step whose bead statistics marked the near blocks
  const int pp = (int)(pn & 1), pf = near_slot(pn);
  const bool avg = AVG && avg_sampled(d, n);
  if constexpr (MODE == kLaunchActive) {
    if ((int)blockIdx.x >= d.max_near + d.nbeads) {
      // the total force of each marker at step n (the observable; the
      // spreading formed the same sums from the split parts)
      const int m = ((int)blockIdx.x - d.max_near - d.nbeads) * BS + (int)threadIdx.x;
      if (m < d.nm) {
        const BeadTerms t = d.bterms[d.marker_info[m].x];
        float f[3];
        marker_total(d, m, t, f);
        d.fm[m] = f[0];
        d.fm[d.nm + m] = f[1];
        d.fm[2 * d.nm + m] = f[2];
      }
      return;
    }
    if ((int)blockIdx.x >= d.max_near) {
      // the near blocks of step n + 1 around bead blockIdx.x - max_near, from
      // the bead region its statistics kernel found at step n
      const int b = (int)blockIdx.x - d.max_near;
      const BeadState& st = d.bstate[b];
      const int box = d.beads[b].box;
      __shared__ int reg[6];
      if (threadIdx.x < 3) {
        reg[threadIdx.x] = st.lo[threadIdx.x];
        reg[3 + threadIdx.x] = st.hi[threadIdx.x];
      }
      __syncthreads();
      mark_near_blocks(d, d.boxes[box], box, reg, reg + 3, n);
      return;
    }
    const int cnt = min(d.near_count[pp], d.max_near);
    if ((int)blockIdx.x < cnt)
      sc_block<ST, BS, NTLD, false>(d, d.near_list[pp * d.max_near + blockIdx.x], n, false, avg);
  } else if constexpr (MODE == kLaunchBulk) {
    // Persistent launches (resident > 0) walk the blocks statically here
    // (FP16 storage; FP32 launches k_stream_collide_claimed instead): FP16
    // blocks take half the time of FP32 ones and the FP16 step is bound by
    // the immersed-boundary chain, so claiming blocks costs more than it
    // balances (58.8 against 57.7 us per 128^3 step).  With `remap` each XCD
    // walks one contiguous range of blocks, else the blocks go grid-stride
    // (round robin over the XCDs).
    if (resident && remap) {
      const int per = (nblocks + 7) / 8;  // logical blocks per XCD
      const int xcd = blockIdx.x % 8, g8 = (int)gridDim.x / 8;
      for (int j = blockIdx.x / 8; j < per; j += g8) {
        const int blk = xcd * per + j;
        if (blk < nblocks && d.near[pf * d.nsc + blk] != (int)pn) sc_block<ST, BS, NTLD, false>(d, blk, n, true, avg);
      }
    } else if (resident) {
      for (int blk = blockIdx.x; blk < nblocks; blk += (int)gridDim.x)
        if (d.near[pf * d.nsc + blk] != (int)pn) sc_block<ST, BS, NTLD, false>(d, blk, n, true, avg);
    } else {
      const int blk = logical_block(remap, nblocks);
      if (blk < nblocks && d.near[pf * d.nsc + blk] != (int)pn) sc_block<ST, BS, NTLD, false>(d, blk, n, true, avg);
    }
  } else {
    const int blk = logical_block(remap, nblocks);
    if (blk < nblocks) sc_block<ST, BS, NTLD, true>(d, blk, n, false, avg);
  }
}

// Persistent bulk launch with claimed blocks (FP32 storage; the same launch
// mode and arguments as k_stream_collide<..., kLaunchBulk, ...> with resident > 0;
// a kernel of its own so that the claim slots in LDS are not allocated by the
// other launches).
//
// The workgroups of group g = blockIdx.x mod G (G = 8 when the grid allows:
// the workgroups of one XCD) claim the group's blocks one at a time from
// the group's counter, so workgroups slowed by the concurrent
// immersed-boundary kernels take fewer blocks.  64 boxes of 32 to 96 nodes an
// edge, 17.6 M nodes, us per step claimed and with a static split: 512/1 706 and
// 1080, 512/2 872 and 1021, 256/2 700 and 1100, 256/4 884 and 1005 (block /
// resident; one workgroup per block 685).  The group's blocks are g, g + G,
// g + 2G, ... (round robin), or, with `remap`, one contiguous range per
// group.  The claim of the next block is issued before the current block's
// work, which hides its latency; two claim slots need one barrier per block.
// Odd steps walk each group's blocks in reverse, so a step starts on the
// blocks the previous one wrote last, the likeliest to be still in the
// last-level cache.
template <int ST, int BS, bool AVG, bool NTLD>
__global__ __launch_bounds__(BS) void k_stream_collide_claimed(Dev d, int remap, int nblocks, int resident) {
  (void)resident;
  const int64_t n = *d.step + d.sub;
  const int64_t pn = n - 1;  // the step whose bead statistics marked the near blocks
  const int pf = near_slot(pn);
  const bool avg = AVG && avg_sampled(d, n);
  __shared__ int next[2];
  const int G = min(kXcds, (int)gridDim.x), g = (int)blockIdx.x % G;
  const int per = (nblocks + G - 1) / G;
  int* const ctr = d.work + ((int)(n & 1) * kXcds + g) * kWorkStride;
  if ((int)blockIdx.x < G && threadIdx.x == 0)
    d.work[((int)((n + 1) & 1) * kXcds + (int)blockIdx.x) * kWorkStride] = 0;
  if (threadIdx.x == 0) next[0] = atomicAdd(ctr, 1);
  __syncthreads();
  for (int i = 0;; ++i) {
    const int j = next[i & 1];  // uniform over the workgroup
    if (j >= per) break;
    // slot (i + 1) & 1 was last read in iteration i - 1, before its barrier
    if (threadIdx.x == 0) next[(i + 1) & 1] = atomicAdd(ctr, 1);
    const int jj = (n & 1) ? per - 1 - j : j;
    const int blk = remap ? g * per + jj : g + G * jj;
    if (blk < nblocks && d.near[pf * d.nsc + blk] != (int)pn)
      sc_block<ST, BS, NTLD, false, false, true>(d, blk, n, true, avg);
    __syncthreads();
  }
}

// FP32, recording (rho, u) per node (segment recompute of the adjoint), in the
// two modes of the two-stream schedule, workgroups of kScBlock nodes.
template <int MODE>
__global__ __launch_bounds__(kScBlock) void k_stream_collide_mom(Dev d, int nblocks) {
  const int64_t n = *d.step + d.sub;
  const int64_t pn = n - 1;
  const int pp = (int)(pn & 1), pf = near_slot(pn);
  if constexpr (MODE == kLaunchActive) {
    const int cnt = min(d.near_count[pp], d.max_near);
    if ((int)blockIdx.x < cnt)
      sc_block<kFp32, kScBlock, true, false, true>(d, d.near_list[pp * d.max_near + blockIdx.x], n, false, false);
  } else {
    const int blk = blockIdx.x;
    if (blk < nblocks && d.near[pf * d.nsc + blk] != (int)pn)
      sc_block<kFp32, kScBlock, true, false, true>(d, blk, n, true, false);
  }
}

// Advance the step counter past an enqueued chunk of `count` steps.
__global__ void k_tick(int64_t* step, int count) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *step += count;
}

// u_n and rho_n of the last completed step n = step - 1 (zero before any step).
template <int ST>
__global__ __launch_bounds__(kScBlock) void k_velocity(Dev d, float* __restrict__ uo,
                                                        float* __restrict__ ro) {
  using T = typename PopIO<ST>::T;
  const int blk = blockIdx.x;
  const int b = d.nboxes == 1 ? 0 : d.block_box[blk];
  const Box B = d.boxes[b];
  const int id = (blk - B.block0) * kScBlock + (int)threadIdx.x;
  if (id >= B.n) return;
  const int64_t c = *d.step;
  // outputs box after box: velocity [box][3][n_box], density [box][n_box]
  const int64_t ob = 3 * B.node0 + id, nb = B.n, orho = B.node0 + id;
  if (c == 0) {
    if (uo) {
      uo[ob] = 0.0f;
      uo[nb + ob] = 0.0f;
      uo[2 * nb + ob] = 0.0f;
    }
    if (ro) ro[orho] = 1.0f;
    return;
  }
  const int64_t n = c - 1;
  const int nx = B.nx, ny = B.ny, nz = B.nz;
  const int x = id % nx;
  const int yz = id / nx;
  const int y = yz % ny;
  const int z = yz / ny;
  const Nbr o = neighbours(x, y, z, nx, ny, nz);
  const int64_t ps = d.pstride;
  const int64_t base = B.node0 + id;
  float g[kQ];
  // the incoming populations of step n (two sets: still in the set step n
  // read), or, in place, the post-collision ones, whose momentum is j + F
  // (the collision adds the force density once, Guo or Shan-Chen)
  float hf = 0.5f;
  if constexpr (ST == kFp32InPlace) {
    int off[kQ];
    upstream_offsets(o, off);
    inplace_post(inplace_rsrc(d), (uint32_t)base * 4u, off, c, g);
    hf = -0.5f;
  } else {
    const T* src = static_cast<const T*>(d.pop[n & 1]);
    pull<ST>(src, base, o, d.fp16_inv, g);
  }
  const Moments m = moments(g);
  float Fx = B.gx, Fy = B.gy, Fz = B.gz;
  const int tile = B.tile0 + (x / kTile) + B.tx * ((y / kTile) + B.ty * (z / kTile));
  if (d.stamp[tile] == (int)n) {
    Fx += d.F[base];
    Fy += d.F[ps + base];
    Fz += d.F[2 * ps + base];
  }
  const float ir = inv_density(m.rho);
  if (uo) {
    uo[ob] = (m.jx + hf * Fx) * ir;
    uo[nb + ob] = (m.jy + hf * Fy) * ir;
    uo[2 * nb + ob] = (m.jz + hf * Fz) * ir;
  }
  if (ro) ro[orho] = m.rho;
}

// Exchange of population deviations with the host order, box after box, each
// [q][node] in FP64: host value px_from + i is px_buf[i].  The conversions are
// those of the storage types (g exactly; half precision rounded to nearest
// even on the way in).  Bound by the copy over the host link that follows or
// precedes it (97x65x131: 12 ms for 125 MB into untouched host memory, 38 ms
// with the conversion in a host loop over the whole device image).
template <int ST>
__global__ __launch_bounds__(256) void k_populations(Dev d) {
  using T = typename PopIO<ST>::T;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= d.px_count) return;
  const int64_t hi = d.px_from + i;
  int b = 0;  // last box whose values start at or before hi
  for (int lo = 0, up = d.nboxes; up - lo > 1;) {
    const int mid = (lo + up) / 2;
    if (kQ * d.boxes[mid].node0 <= hi) lo = b = mid;
    else up = mid;
  }
  const Box& B = d.boxes[b];
  const int64_t r = hi - kQ * B.node0;
  const int q = (int)(r / B.n);
  const int id = (int)(r - q * B.n);
  const int64_t c = *d.step;
  int64_t at = pop_index(q, B.node0 + id);
  if constexpr (ST == kFp32InPlace) {
    // after an odd number of steps f*_q(x) sits in slot opposite(q) of node x,
    // else in slot q of node x + c_q, the upstream node of the opposite direction
    if (c & 1) {
      at = pop_index(opposite(q), B.node0 + id);
    } else {
      const int x = id % B.nx, yz = id / B.nx, y = yz % B.ny, z = yz / B.ny;
      int off[kQ];
      upstream_offsets(neighbours(x, y, z, B.nx, B.ny, B.nz), off);
      int o = 0;
#pragma unroll
      for (int k = 0; k < kQ; ++k) o = k == opposite(q) ? off[k] : o;
      at = pop_index(q, B.node0 + id + o);
    }
  }
  T* const p = static_cast<T*>(d.pop[c & 1]) + at;
  const float w = q == 0 ? kW0 : (q < 7 ? kW1 : kW2);
  if (d.px_set) {
    const double v = d.px_buf[i];
    if constexpr (ST == kFp16) *p = __float2half_rn((float)v * d.fp16_scale);
    else if constexpr (ST == kFp32Plain) *p = (float)((double)w + v);
    else *p = (float)v;
  } else {
    if constexpr (ST == kFp16) d.px_buf[i] = (double)(__half2float(*p) / d.fp16_scale);
    else if constexpr (ST == kFp32Plain) d.px_buf[i] = (double)*p - (double)w;
    else d.px_buf[i] = (double)*p;
  }
}

// Time-average of u: the FP64 sums over `count` sampled steps divided by the
// count (zero without samples), box after box as [box][3][n_box].
__global__ __launch_bounds__(kScBlock) void k_average_out(Dev d, int64_t count, float* __restrict__ uo) {
  const int blk = blockIdx.x;
  const int b = d.nboxes == 1 ? 0 : d.block_box[blk];
  const Box B = d.boxes[b];
  const int id = (blk - B.block0) * kScBlock + (int)threadIdx.x;
  if (id >= B.n) return;
  const int64_t ob = 3 * B.node0 + id, nb = B.n, base = B.node0 + id, ps = d.pstride;
  const double inv = count > 0 ? 1.0 / (double)count : 0.0;
  uo[ob] = (float)(d.uavg[base] * inv);
  uo[nb + ob] = (float)(d.uavg[ps + base] * inv);
  uo[2 * nb + ob] = (float)(d.uavg[2 * ps + base] * inv);
}

// Block sum of 4 doubles through wavefront shuffles, result in thread 0.
__device__ inline void block_sum4(double* v) {
  __shared__ double part[kScBlock / 64][4];
#pragma unroll
  for (int k = 0; k < 4; ++k)
    for (int s = 32; s > 0; s >>= 1) v[k] += __shfl_xor(v[k], s, 64);
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  if (lane == 0)
    for (int k = 0; k < 4; ++k) part[wave][k] = v[k];
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 0; k < 4; ++k) {
      double s = 0;
      for (int w = 0; w < kScBlock / 64; ++w) s += part[w][k];
      v[k] = s;
    }
  }
}

// Stage 1: per-block FP64 sums of g and g c over the current state.
template <int ST>
__global__ __launch_bounds__(kScBlock) void k_conserved_partial(Dev d, int box, double* __restrict__ part) {
  using IO = PopIO<ST>;
  using T = typename IO::T;
  const int64_t c = *d.step;
  const T* src = static_cast<const T*>(d.pop[c & 1]);
  double v[4] = {0, 0, 0, 0};
  for (int b = 0; b < d.nboxes; ++b) {
    if (box >= 0 && b != box) continue;
    const Box B = d.boxes[b];
    for (int64_t id = (int64_t)blockIdx.x * kScBlock + threadIdx.x; id < B.n;
         id += (int64_t)gridDim.x * kScBlock) {
      float g[kQ];
      if constexpr (ST == kFp32InPlace) {
        // each node's own 19 post-collision values, wherever they are stored
        const int x = (int)(id % B.nx), yz = (int)(id / B.nx), y = yz % B.ny, z = yz / B.ny;
        int off[kQ];
        upstream_offsets(neighbours(x, y, z, B.nx, B.ny, B.nz), off);
        inplace_post(inplace_rsrc(d), (uint32_t)(B.node0 + id) * 4u, off, c, g);
      } else {
#pragma unroll
        for (int q = 0; q < kQ; ++q) g[q] = IO::ld(src + pop_index(q, B.node0 + id), q, d.fp16_inv);
      }
      const Moments m = moments(g);
      v[0] += (double)m.drho;
      v[1] += (double)m.jx;
      v[2] += (double)m.jy;
      v[3] += (double)m.jz;
    }
  }
  block_sum4(v);
  if (threadIdx.x == 0)
    for (int k = 0; k < 4; ++k) part[4 * blockIdx.x + k] = v[k];
}

// Stage 2: one block folds the partials in a fixed order; `mass0` (the sum
// of the weights, one per node, or 0 when the caller adds it) is added to the
// mass sum last.
__global__ __launch_bounds__(kScBlock) void k_conserved_final(const double* __restrict__ part,
                                                               int nparts, double* __restrict__ out,
                                                               double mass0) {
  double v[4] = {0, 0, 0, 0};
  for (int i = threadIdx.x; i < nparts; i += kScBlock)
    for (int k = 0; k < 4; ++k) v[k] += part[4 * i + k];
  block_sum4(v);
  if (threadIdx.x == 0) {
    out[0] = v[0] + mass0;
    for (int k = 1; k < 4; ++k) out[k] = v[k];
  }
}

// Plain device copy, one 16-byte vector per thread over a grid that covers
// the buffer, non-temporal loads and stores: the achievable-bandwidth
// reference for the HBM roofline.
__global__ __launch_bounds__(256) void k_copy(const f32x4* __restrict__ src, f32x4* __restrict__ dst,
                                              int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
    __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

}  // namespace

void launch_copy(const void* src, void* dst, int64_t bytes, hipStream_t s) {
  const int64_t n = bytes / 16;
  const int blocks = (int)std::min<int64_t>((n + 255) / 256, (int64_t)1 << 30);
  hipLaunchKernelGGL(k_copy, dim3(blocks), dim3(256), 0, s, static_cast<const f32x4*>(src),
                     static_cast<f32x4*>(dst), n);
}

// Launch through hipExtLaunchKernelGGL when timing: the start / stop events are
// stamped by the kernel's own dispatch packet, so the elapsed time is the
// kernel's duration without the cost of separate event packets.
template <class K>
static void launch_k(K kernel, int grid, int block, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1, const Dev& d,
                     int remap, int nblocks, int resident) {
  if (ev0)
    hipExtLaunchKernelGGL(kernel, dim3(grid), dim3(block), 0, s, ev0, ev1, 0, d, remap, nblocks, resident);
  else
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(block), 0, s, d, remap, nblocks, resident);
}

struct ScArgs {
  int mode, block, nblocks, remap, resident, ncu;
  hipStream_t s;
  hipEvent_t ev0, ev1;
};

template <int ST, int MODE, bool AVG, bool NTLD>
static void launch_sc_mode(const Dev& d, const ScArgs& p) {
  int grid = p.remap ? (p.nblocks + 7) / 8 * 8 : p.nblocks;
  int resident = 0;
  if (MODE == kLaunchActive) grid = d.max_near + (d.near_mark ? d.nbeads + (d.nm + p.block - 1) / p.block : 0);
  if (MODE == kLaunchBulk && p.resident > 0) {
    resident = p.resident;
    grid = p.remap ? std::min(grid, p.ncu * resident) / 8 * 8 : std::min(grid, p.ncu * resident);
  }
  if (MODE == kLaunchBulk && resident > 0 && ST != kFp16) {
    if (p.block == 128)
      launch_k(k_stream_collide_claimed<ST, 128, AVG, NTLD>, grid, 128, p.s, p.ev0, p.ev1, d, p.remap, p.nblocks, resident);
    else if (p.block == 512)
      launch_k(k_stream_collide_claimed<ST, 512, AVG, NTLD>, grid, 512, p.s, p.ev0, p.ev1, d, p.remap, p.nblocks, resident);
    else
      launch_k(k_stream_collide_claimed<ST, 256, AVG, NTLD>, grid, 256, p.s, p.ev0, p.ev1, d, p.remap, p.nblocks, resident);
    return;
  }
  if (p.block == 128)
    launch_k(k_stream_collide<ST, 128, MODE, AVG, NTLD>, grid, 128, p.s, p.ev0, p.ev1, d, p.remap, p.nblocks, resident);
  else if (p.block == 512)
    launch_k(k_stream_collide<ST, 512, MODE, AVG, NTLD>, grid, 512, p.s, p.ev0, p.ev1, d, p.remap, p.nblocks, resident);
  else
    launch_k(k_stream_collide<ST, 256, MODE, AVG, NTLD>, grid, 256, p.s, p.ev0, p.ev1, d, p.remap, p.nblocks, resident);
}

template <int ST, bool AVG, bool NTLD>
static void launch_sc_ld(const Dev& d, const ScArgs& p) {
  if (p.mode == kLaunchBulk)
    launch_sc_mode<ST, kLaunchBulk, AVG, NTLD>(d, p);
  else if (p.mode == kLaunchActive)
    launch_sc_mode<ST, kLaunchActive, AVG, NTLD>(d, p);
  else
    launch_sc_mode<ST, kLaunchAll, AVG, NTLD>(d, p);
}

// FP16 pulls are plain loads in either regime, and the in-place set has one
// load form (one instance each)
template <int ST, bool AVG>
static void launch_sc_avg(const Dev& d, const ScArgs& p) {
  constexpr bool kOne = ST == kFp16 || ST == kFp32InPlace;
  if (kOne || d.small_pops)
    launch_sc_ld<ST, AVG, true>(d, p);
  else
    launch_sc_ld<ST, AVG, kOne>(d, p);
}

template <int ST>
static void launch_sc_st(const Dev& d, const ScArgs& p) {
  if (d.uavg)
    launch_sc_avg<ST, true>(d, p);
  else
    launch_sc_avg<ST, false>(d, p);
}

void launch_stream_collide(const Dev& d, int storage, int mode, int block, int nblocks, int remap,
                           int resident, int ncu, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  if (mode >= kLaunchStepFirst) {
    launch_step(d, storage, mode, nblocks, s, ev0, ev1);
    return;
  }
  const ScArgs p{mode, block, nblocks, remap, resident, ncu, s, ev0, ev1};
  if (storage == kFp16)
    launch_sc_st<kFp16>(d, p);
  else if (storage == kFp32Plain)
    launch_sc_st<kFp32Plain>(d, p);
  else if (storage == kFp32InPlace)
    launch_sc_st<kFp32InPlace>(d, p);
  else
    launch_sc_st<kFp32>(d, p);
}

void launch_stream_collide_mom(const Dev& d, int mode, int nblocks, hipStream_t s) {
  if (mode == kLaunchActive)
    hipLaunchKernelGGL(k_stream_collide_mom<kLaunchActive>, dim3(d.max_near), dim3(kScBlock), 0, s, d, nblocks);
  else if (mode == kLaunchBulk)
    hipLaunchKernelGGL(k_stream_collide_mom<kLaunchBulk>, dim3(nblocks), dim3(kScBlock), 0, s, d, nblocks);
  else
    launch_step_mom(d, mode, nblocks, s);
}

void launch_tick(const Dev& d, int count, hipStream_t s) {
  hipLaunchKernelGGL(k_tick, dim3(1), dim3(64), 0, s, d.step, count);
}

void launch_velocity(const Dev& d, int storage, int nblocks, float* u_out, float* rho_out,
                     hipStream_t s) {
  if (d.px_buf) {
    const int grid = (int)((d.px_count + 255) / 256);
    if (storage == kFp16)
      hipLaunchKernelGGL(k_populations<kFp16>, dim3(grid), dim3(256), 0, s, d);
    else if (storage == kFp32Plain)
      hipLaunchKernelGGL(k_populations<kFp32Plain>, dim3(grid), dim3(256), 0, s, d);
    else if (storage == kFp32InPlace)
      hipLaunchKernelGGL(k_populations<kFp32InPlace>, dim3(grid), dim3(256), 0, s, d);
    else
      hipLaunchKernelGGL(k_populations<kFp32>, dim3(grid), dim3(256), 0, s, d);
    return;
  }
  if (storage == kFp16)
    hipLaunchKernelGGL(k_velocity<kFp16>, dim3(nblocks), dim3(kScBlock), 0, s, d, u_out, rho_out);
  else if (storage == kFp32Plain)
    hipLaunchKernelGGL(k_velocity<kFp32Plain>, dim3(nblocks), dim3(kScBlock), 0, s, d, u_out, rho_out);
  else if (storage == kFp32InPlace)
    hipLaunchKernelGGL(k_velocity<kFp32InPlace>, dim3(nblocks), dim3(kScBlock), 0, s, d, u_out, rho_out);
  else
    hipLaunchKernelGGL(k_velocity<kFp32>, dim3(nblocks), dim3(kScBlock), 0, s, d, u_out, rho_out);
}

void launch_average_out(const Dev& d, int nblocks, int64_t count, float* u_out, hipStream_t s) {
  hipLaunchKernelGGL(k_average_out, dim3(nblocks), dim3(kScBlock), 0, s, d, count, u_out);
}

void launch_conserved(const Dev& d, int storage, int box, double* partial, int nparts, double* out,
                      hipStream_t s, double mass0) {
  if (storage == kFp16)
    hipLaunchKernelGGL(k_conserved_partial<kFp16>, dim3(nparts), dim3(kScBlock), 0, s, d, box, partial);
  else if (storage == kFp32Plain)
    hipLaunchKernelGGL(k_conserved_partial<kFp32Plain>, dim3(nparts), dim3(kScBlock), 0, s, d, box, partial);
  else if (storage == kFp32InPlace)
    hipLaunchKernelGGL(k_conserved_partial<kFp32InPlace>, dim3(nparts), dim3(kScBlock), 0, s, d, box, partial);
  else
    hipLaunchKernelGGL(k_conserved_partial<kFp32>, dim3(nparts), dim3(kScBlock), 0, s, d, box, partial);
  hipLaunchKernelGGL(k_conserved_final, dim3(1), dim3(kScBlock), 0, s, partial, nparts, out, mass0);
}

// ---- static scratch of the allocation-free conserved sums ---------------------
// The partial sums of lbm_batch_get_conserved_noalloc live in this array, one
// copy per GPU for the life of the process.  In host code `scratch` names a
// host-side stand-in, not device memory: its address on a GPU comes from
// hipGetSymbolAddress, called once per device while that device is current.
static __device__ __align__(256) double scratch[4 * kNoAllocParts];

namespace {
constexpr int kMaxDevices = 64;
std::mutex scratch_mutex;
double* scratch_addr[kMaxDevices] = {};
}  // namespace

hipError_t resolve_conserved_scratch(int device, double** out) {
  *out = nullptr;
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(scratch_mutex);
  if (!scratch_addr[device]) {
    double* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(reinterpret_cast<void**>(&p), HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    scratch_addr[device] = p;
  }
  *out = scratch_addr[device];
  return hipSuccess;
}

}  // namespace lbmib
