// The fused step: two launches per step, on one stream.
//
//   k_step_a  patch workgroups: interpolation and advection of step n - 1,
//             then the membrane forces and partial bead statistics of step n,
//             one workgroup per surface patch of a bead (at most kPatchOwn
//             nodes it owns, plus the neighbours its elements touch, advected
//             redundantly);
//             block workgroups: stream-collide of step n for a share of the
//             blocks away from the swimmers.
//   k_step_b  spreading workgroups: one z slab of one near tile each; F is
//             summed in LDS and the slab's nodes are collided with it at once;
//             bead workgroups: bead state, total marker forces, near tiles of
//             step n + 1;
//             block workgroups: stream-collide of the remaining blocks.
//
// The markers' chain of a step (interpolation, forces, spreading, collision
// near the beads) is serial and bound by memory latency, while the rest of the
// grid is bound by bandwidth.  Both run inside the same two launches: the
// chain's workgroups come first in the grid, the blocks fill the other compute
// units, and there is no second stream, whose cross-stream graph edges cost
// about 5 us of queue time each.
//
// Per step, against the chain in five kernels on a second stream beside one
// launch of the other blocks (us): 32^3 36.0 to 19.5, 64^3 36.3 to 26.5, 96^3
// 45.9 to 33.6, 128^3 in place 56.9 to 52.9 and with two sets 58.4 to 55.4,
// 256x128x128 127.5 to 109.3, 1024x256x256 2152 to 1751.  At 128^3 in place
// k_step_a takes 22.6 us and k_step_b 29.4 (13.0 and 13.1 without blocks).
//
// What a launch reads was written by an earlier launch, except for data of the
// same workgroup: k_step_a reads the positions in d.pos and writes d.pos_new;
// k_step_b reads d.pos_new and its bead workgroups copy it to d.pos.  The near
// tiles of step n come from the bead regions of step n - 1 grown by
// kNearMargin nodes (a marker moves by far less than one node per step), so
// both launches of step n know which nodes the spreading workgroups collide.
#include "common.h"
#include "bead_terms.h"
#include "ibm_device.h"
#include "lattice_device.h"
#include "near_marks.h"
#include "step_launch.h"

#include <hip/hip_ext.h>

namespace lbmib {

namespace {

constexpr int kWaves = kStepBlock / 64;

constexpr int kSlabNodes = kTile * kTile * kSlabLayers;
constexpr int kSubsets = kWaves / kSlabLayers;  // wavefronts that share a layer

// Population sizes (Dev::small_pops, Dev::pops32), as a template parameter of
// the step kernels: small (both sets within kWriteThroughBytes: stores written
// through, non-temporal pulls), one set below 4 GiB (32-bit addresses), larger.
enum { kSmall = 0, kLarge = 1, kHuge = 2 };
// What a launch records besides: nothing, the time average of u (Dev::uavg), or
// (rho, u) of every node (Dev::mom).
enum { kPlain = 0, kAverage = 1, kMoments = 2 };
template <int SZ>
constexpr bool kNtLd = SZ == kSmall;
template <int SZ>
constexpr bool kOff32 = SZ != kHuge;
template <int SZ>
constexpr int kThrough = SZ == kSmall ? 1 : 0;

// A product rounded by itself: left to the compiler, the first addition of the
// reduction after it may be fused with it in one kernel and not in another,
// and every split of a run into calls has to give the same bits.
__device__ inline float mul_rn(float a, float b) {
#pragma clang fp contract(off)
  return a * b;
}

// A value known to be the same in every lane, in scalar registers.
__device__ inline int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ inline int4 uniform(int4 v) { return make_int4(uniform(v.x), uniform(v.y), uniform(v.z), uniform(v.w)); }

__device__ inline float uniform(float v) { return __int_as_float(uniform(__float_as_int(v))); }
__device__ inline int64_t uniform(int64_t v) {
  return (int64_t)((uint64_t)(uint32_t)uniform((int)v) | (uint64_t)(uint32_t)uniform((int)(v >> 32)) << 32);
}
__device__ inline double uniform(double v) {
  return __hiloint2double(uniform(__double2hiint(v)), uniform(__double2loint(v)));
}
__device__ inline StepBox uniform(const StepBox& b) {
  return StepBox{uniform(b.bead0), uniform(b.nbeads), uniform(b.patch0), uniform(b.npatch),
                 uniform(b.m0),    uniform(b.m_end),  uniform(b.list0),  uniform(b.workers)};
}
__device__ inline Box uniform(const Box& b) {
  Box r = b;
  r.nx = uniform(b.nx);
  r.ny = uniform(b.ny);
  r.nz = uniform(b.nz);
  r.tx = uniform(b.tx);
  r.ty = uniform(b.ty);
  r.tz = uniform(b.tz);
  r.node0 = uniform(b.node0);
  r.tile0 = uniform(b.tile0);
  r.forcing = uniform(b.forcing);
  r.tau = uniform(b.tau);
  r.omega = uniform(b.omega);
  r.gx = uniform(b.gx);
  r.gy = uniform(b.gy);
  r.gz = uniform(b.gz);
  for (int a = 0; a < 3; ++a) r.inv[a] = uniform(b.inv[a]);
  return r;
}

// ---- blocks -----------------------------------------------------------------------
// Stream-collide of block j in walking order, leaving out the nodes of near
// tiles.  The populations are loaded before the block's mark is looked at, so
// that no memory trip precedes them.  With populations of the last-level
// cache's size odd steps walk in reverse: a step starts on the blocks the
// previous one wrote last, the likeliest to be still in it.
template <int ST, int EX, int SZ>
__device__ inline void step_bulk(const Dev& d, int j, int64_t n) {
  const int blk = SZ == kSmall && (n & 1) ? d.nstep - 1 - j : j;
  const int slot = (int)(n & 1);
  const int mark = d.step_near[slot * d.nstep + blk];
  const bool avg = EX == kAverage && avg_sampled(d, n);
  const int b = d.nboxes == 1 ? 0 : d.step_block_box[blk];
  const Box B = d.boxes[b];
  const int first = d.nboxes == 1 ? 0 : d.step_box_block0[b];
  const int id = (blk - first) * kStepBlock + (int)threadIdx.x;
  if (id >= B.n) return;
  const int yz = (int)divide((uint32_t)id, B.div_nx);
  const int x = id - yz * B.nx;
  const int z = (int)divide((uint32_t)yz, B.div_ny);
  const int y = yz - z * B.ny;
  const int64_t base = B.node0 + id;
  const Nbr o = neighbours(x, y, z, B.nx, B.ny, B.nz);
  const AvgSums sums = avg_load(d, base, avg);
  float g[kQ];
  sc_load<ST, kNtLd<SZ>, kOff32<SZ>>(d, o, base, n, g);
  if (mark == (int)n) {
    const int tile = B.tile0 + (x / kTile) + B.tx * ((y / kTile) + B.ty * (z / kTile));
    if (d.near_tile[slot * d.ntiles + tile] == (int)n) return;
  }
  sc_finish<ST, EX == kMoments, kOff32<SZ>, false, kThrough<SZ>>(d, B, o, base, n, g, B.gx, B.gy, B.gz, false, avg,
                                                                 sums);
}

// ---- interpolation ------------------------------------------------------------------
// U = sum over the stencil of Delta u: 16 lanes per marker, lane l the row of
// nodes (y, z) = (l mod NW, l / NW) of the stencil, NW loads along x each; the
// rows are added by DPP moves within the 16 lanes.  `c` holds the box-local
// node offset of each stencil coordinate along x and the row's base.
constexpr int kRowLanes = 16;

template <int NW>
struct RowStencil {
  float wx[NW], wyz;
  int c[NW];  // node of (x_k, y, z) in the box
};

template <int NW>
struct RowValues {
  float v[3][NW];
};

template <int NW>
__device__ inline RowValues<NW> row_load(const float* u, int64_t ps, const RowStencil<NW>& r) {
  RowValues<NW> q;
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int k = 0; k < NW; ++k) q.v[a][k] = u[a * ps + r.c[k]];
  return q;
}

// The marker's U, in every lane of its group (`in`: the lane holds a row).
template <int NW>
__device__ inline float3 row_sum(const RowValues<NW>& q, const RowStencil<NW>& r, bool in) {
  float s[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    float t = q.v[a][0] * r.wx[0];
#pragma unroll
    for (int k = 1; k < NW; ++k) t = fmaf(q.v[a][k], r.wx[k], t);
    s[a] = group_reduce<kRowLanes>(in ? mul_rn(t, r.wyz) : 0.0f);
  }
  return make_float3(s[0], s[1], s[2]);
}

// ---- patches ------------------------------------------------------------------------
// One workgroup per patch.  The work is bound by instruction issue and by the
// three dependent memory trips (tables, positions, velocities), so nothing is
// computed twice: one thread per (local node, axis) makes the kernel weights and
// node offsets of that axis, one thread per element makes all its corner
// forces, and the node sums gather them from LDS in the lane order of
// vertex_forces_block.
template <int NW>
__device__ inline void patch_block(const Dev& d, int p, int advance, int64_t n) {
  constexpr int G = kStepBlock / kRowLanes;             // markers interpolated per pass
  constexpr int U = NW == 4 ? 2 : 3;                    // passes in flight
  constexpr int kLanes = 32, kTriLanes = 8;             // force lanes per node
  constexpr int R = kPatchOwn * kLanes / kStepBlock;    // force rounds
  constexpr int kTriWaves = 2, kHingeWaves = 3;
  __shared__ double lp[3][kPatchLocal];
  __shared__ float wgt[3][NW][kPatchLocal];
  __shared__ int idx[3][NW][kPatchLocal];
  __shared__ int lid[kPatchLocal];
  __shared__ float ftri[3][3 * kPatchTri], farea[3][kPatchTri], fhinge[3][4 * kPatchHinge];
  static_assert(3 * kPatchLocal <= kStepBlock && kPatchOwn <= 64 && kPatchVol == 128 && kWaves == 8, "patch threads");
  const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64;
  const int4 pi = uniform(d.patch[p]);
  const int b = pi.x, own = pi.z & 0xffff, local = pi.z >> 16, ntri = pi.w & 0xffff, nhinge = pi.w >> 16;
  const int nm = d.nm;
  int slots[R];
#pragma unroll
  for (int r = 0; r < R; ++r) slots[r] = d.patch_lane[(size_t)p * (kPatchOwn * kLanes) + r * kStepBlock + tid];
  const Bead Bd = d.beads[b];
  const Box B = uniform(d.boxes[pi.y]);
  const int li = tid / 3, la = tid - 3 * li;
  if (li < local) {
    const int m = d.patch_marker[(size_t)p * kPatchLocal + li];
    const double x = d.pos[la * nm + m];
    lp[la][li] = x;
    if (la == 0) lid[li] = m;
    if (advance) {
      const int N = la == 0 ? B.nx : (la == 1 ? B.ny : B.nz);
      const int stride = la == 0 ? 1 : (la == 1 ? B.nx : B.nx * B.ny);
      const double inv = la == 0 ? B.inv[0] : (la == 1 ? B.inv[1] : B.inv[2]);
      const int base = stencil_base<NW>(x);
      int c = wrap(base, N, inv);
#pragma unroll
      for (int k = 0; k < NW; ++k) {
        wgt[la][k][li] = phi_fused<NW>((float)((double)(base + k) - x));
        idx[la][k][li] = c * stride;
        c = c + 1 == N ? 0 : c + 1;
      }
    }
  }
  __syncthreads();
  if (advance) {
    // group g of 16 lanes takes the local markers g, g + G, ...
    const int g = tid / kRowLanes, ln = tid % kRowLanes;
    const int yk = ln % NW, zk = ln / NW;
    const bool in = ln < NW * NW;
    const float* const u = d.u + B.node0;
    for (int i0 = 0; i0 < local; i0 += G * U) {
      RowStencil<NW> r[U];
      RowValues<NW> q[U];
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int i = i0 + k * G + g;
        const bool on = i < local && in;
        r[k].wyz = 0.0f;
#pragma unroll
        for (int x = 0; x < NW; ++x) {
          r[k].wx[x] = 0.0f;
          q[k].v[0][x] = q[k].v[1][x] = q[k].v[2][x] = 0.0f;
        }
        if (on) {
          r[k].wyz = wgt[1][yk][i] * wgt[2][zk][i];
          const int row = idx[1][yk][i] + idx[2][zk][i];
#pragma unroll
          for (int x = 0; x < NW; ++x) {
            r[k].wx[x] = wgt[0][x][i];
            r[k].c[x] = row + idx[0][x][i];
          }
          q[k] = row_load<NW>(u, d.pstride, r[k]);
        }
      }
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int i = i0 + k * G + g;
        const float3 v = row_sum<NW>(q[k], r[k], i < local && in);
        if (i < local && ln == 0) {
          // the entry is touched by this group only
          lp[0][i] += (double)v.x;
          lp[1][i] += (double)v.y;
          lp[2][i] += (double)v.z;
          if (i < own) {
            const int m = lid[i];
            d.U[m] = v.x;
            d.U[nm + m] = v.y;
            d.U[2 * nm + m] = v.z;
          }
        }
      }
    }
    __syncthreads();
  }
  // elements, by wave: triangles, hinges, position statistics, volume
  auto at = [&](int v) { return make_double3(lp[0][v], lp[1][v], lp[2][v]); };
  if (wave < kTriWaves) {
    for (int t = tid; t < ntri; t += 64 * kTriWaves) {
      const int2 e = d.patch_tri[(size_t)p * kPatchTri + t];
      const TriangleTerms T = triangle_terms(d, Bd, e.x, at(e.y & 1023), at((e.y >> 10) & 1023), at((e.y >> 20) & 1023));
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const float3 f = corner_force(T, k);
        ftri[0][3 * t + k] = f.x;
        ftri[1][3 * t + k] = f.y;
        ftri[2][3 * t + k] = f.z;
      }
      farea[0][t] = T.area.x;
      farea[1][t] = T.area.y;
      farea[2][t] = T.area.z;
    }
  } else if (wave < kTriWaves + kHingeWaves) {
    for (int t = tid - 64 * kTriWaves; t < nhinge; t += 64 * kHingeWaves) {
      const int4 e = d.patch_hinge[(size_t)p * kPatchHinge + t];
      const HingeTerms T = hinge_terms(d, Bd, e.x, at(e.y & 0xffff), at((e.y >> 16) & 0xffff), at(e.z & 0xffff),
                                       at((e.z >> 16) & 0xffff));
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float3 f = role_force(T, T.fa[k], T.fb[k]);
        fhinge[0][4 * t + k] = f.x;
        fhinge[1][4 * t + k] = f.y;
        fhinge[2][4 * t + k] = f.z;
      }
    }
  } else if (wave == 5) {
    const bool in = lane < own;
    double* const out = d.part + (size_t)p * kPartVals;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const double v = in ? lp[k][lane] : 0.0;
      if (in) d.pos_new[k * nm + lid[lane]] = v;
      const double s = wave_reduce<kRedSum>(v), lo = wave_reduce<kRedMin>(in ? v : 1e300),
                   hi = wave_reduce<kRedMax>(in ? v : -1e300);
      if (lane == 0) {
        out[k] = s;
        out[3 + k] = lo;
        out[6 + k] = hi;
      }
    }
  } else {
    // volume about the bead's previous centre (any point serves: the surface
    // is closed), and one lane of the swimmer's first patch its driving forces
    const int tv = d.patch_vol[(size_t)p * kPatchVol + tid - 384];
    const double cx = d.bstate[b].c[0], cy = d.bstate[b].c[1], cz = d.bstate[b].c[2];
    double v = 0.0;
    if (tv >= 0) {
      const int i0 = tv & 1023, i1 = (tv >> 10) & 1023, i2 = (tv >> 20) & 1023;
      const double ax = lp[0][i0] - cx, ay = lp[1][i0] - cy, az = lp[2][i0] - cz;
      const double bx = lp[0][i1] - cx, by = lp[1][i1] - cy, bz = lp[2][i1] - cz;
      const double qx = lp[0][i2] - cx, qy = lp[1][i2] - cy, qz = lp[2][i2] - cz;
      v = ax * (by * qz - bz * qy) + ay * (bz * qx - bx * qz) + az * (bx * qy - by * qx);
    }
    v = wave_reduce<kRedSum>(v);
    if (lane == 0) d.part[(size_t)p * kPartVals + 9 + (wave - 6)] = v;
    if (tid == 384 && Bd.slot == 0 && p == Bd.patch0) {
      const Swimmer& S = d.swimmers[Bd.swimmer];
      const double t = (double)n;
      d.drive[Bd.swimmer] = make_double2(S.A * sin(S.omega * t + S.phi0), S.B * sin(S.omega * t + S.phi0 + S.alpha));
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int j = (r * kStepBlock + tid) / kLanes, fl = tid % kLanes;
    float fx = 0, fy = 0, fz = 0, gx = 0, gy = 0, gz = 0;
    if (slots[r] >= 0) {
      if (fl < kTriLanes) {
        const int t = slots[r] / 3;
        fx = ftri[0][slots[r]];
        fy = ftri[1][slots[r]];
        fz = ftri[2][slots[r]];
        gx = farea[0][t];
        gy = farea[1][t];
        gz = farea[2][t];
      } else {
        fx = fhinge[0][slots[r]];
        fy = fhinge[1][slots[r]];
        fz = fhinge[2][slots[r]];
      }
    }
    fx = group_reduce<kLanes>(fx);
    fy = group_reduce<kLanes>(fy);
    fz = group_reduce<kLanes>(fz);
    gx = group_reduce<kTriLanes>(gx);
    gy = group_reduce<kTriLanes>(gy);
    gz = group_reduce<kTriLanes>(gz);
    if (j < own && fl == 0) {
      const int m = lid[j];
      d.fmem[m] = fx;
      d.fmem[nm + m] = fy;
      d.fmem[2 * nm + m] = fz;
      d.gvol[m] = gx;
      d.gvol[nm + m] = gy;
      d.gvol[2 * nm + m] = gz;
    }
  }
}

// Whether a bead's near range holds tile (tx, ty, tz): all are in [0, T).
__device__ inline bool in_run(int t, int t0, int cnt, int T) {
  const int r = t - t0;
  return (r < 0 ? r + T : r) < cnt;
}
__device__ inline bool near_covers(const NearRange& s, int tx, int ty, int tz, const Box& B) {
  return in_run(tx, s.t0[0], s.cnt[0], B.tx) && in_run(ty, s.t0[1], s.cnt[1], B.ty) && in_run(tz, s.t0[2], s.cnt[2], B.tz);
}

// ---- slab list ------------------------------------------------------------------------
// The slabs of step n in box `box`, from the near ranges: one entry per z slab
// of every near tile, {tile of the box * slabs per tile + slab, first marker of the
// first bead whose range holds the tile, the holding beads of the box (two
// words)}.  One workgroup; the order does not matter, since slabs are independent.
// k_step_b waits for it, so the tiles of all beads are dealt to the threads at
// once, and what is left serial is one test per bead.  us per step, bead after
// bead and at once: 8 swimmers of 162-node beads in 96^3 151.6 and 47.0, in 128^3
// 168.5 and 71.5; 4 in 64^3 58.0 and 26.7; 2 in 96^3 36.9 and 33.6.
__device__ inline void list_block(const Dev& d, int box, int64_t n) {
  __shared__ NearRange range[kFoldBeads];
  __shared__ int end[kFoldBeads];  // tiles of the beads up to this one
  __shared__ int count;
  const int tid = threadIdx.x;
  const StepBox X = d.step_box[box];
  const Box B = d.boxes[box];
  static_assert(kFoldBeads == 64, "a bead per lane of the first wavefront, a bit of the cover mask each");
  if (tid < kFoldBeads) {
    int tiles = 0;
    if (tid < X.nbeads) {
      const NearRange r = d.near_range[(n & 1) * d.nbeads + X.bead0 + tid];
      range[tid] = r;
      tiles = r.cnt[0] * r.cnt[1] * r.cnt[2];
    }
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) {
      const int below = __shfl_up(tiles, s, 64);
      if (tid >= s) tiles += below;
    }
    end[tid] = tiles;
    if (tid == 0) count = 0;
  }
  __syncthreads();
  const int total = end[kFoldBeads - 1];
  int b = 0;
  for (int i = tid; i < total; i += kStepBlock) {
    while (i >= end[b]) ++b;
    const NearRange S = range[b];
    const int t = i - (b > 0 ? end[b - 1] : 0);
    int tx = S.t0[0] + t % S.cnt[0], ty = S.t0[1] + (t / S.cnt[0]) % S.cnt[1], tz = S.t0[2] + t / (S.cnt[0] * S.cnt[1]);
    if (tx >= B.tx) tx -= B.tx;
    if (ty >= B.ty) ty -= B.ty;
    if (tz >= B.tz) tz -= B.tz;
    unsigned long long cover = 0;
    for (int j = 0; j < X.nbeads; ++j)
      if (near_covers(range[j], tx, ty, tz, B)) cover |= 1ull << j;
    if (cover & ((1ull << b) - 1)) continue;  // an earlier bead's range holds the tile
    const int slabs = (min(kTile, B.nz - tz * kTile) + kSlabLayers - 1) / kSlabLayers;
    const int at = atomicAdd(&count, slabs);
    const int first = d.beads[X.bead0 + b].first;
    for (int p = 0; p < slabs; ++p)
      d.slab_list[X.list0 + at + p] = make_int4((tx + B.tx * (ty + B.ty * tz)) * kSlabParts + p, first,
                                                (int)(uint32_t)cover, (int)(uint32_t)(cover >> 32));
  }
  __syncthreads();
  if (tid == 0) d.slab_count[box] = count;
}

template <int ST, int NW, int EX, int SZ>
__global__ __launch_bounds__(kStepBlock, 4) void k_step_a(Dev d, int advance, int nchain) {
  const int64_t n = uniform(*d.step) + d.sub;
  const int i = blockIdx.x;
  if (i < d.npatch)
    patch_block<NW>(d, i, advance, n);
  else if (i < nchain)
    list_block(d, i - d.npatch, n);
  else
    step_bulk<ST, EX, SZ>(d, i - nchain, n);
}

// ---- spreading and near tiles -----------------------------------------------------------
// A marker's stencil on a slab: the kernel weights at the slab's eight x and
// eight y coordinates and, per layer, the force times the z weight; zero
// outside the stencil, so every node adds every entry without a test.
struct alignas(16) StepEntry {
  float wx[kTile], wy[kTile];
  float f[kSlabLayers][4];
};

// Value k = x, y, z (sums) or 3 (6 V) of patch p.
__device__ inline double patch_value(const Dev& d, int p, int k) {
  const double* const v = d.part + (size_t)p * kPartVals;
  return k < 3 ? v[k] : v[9] + v[10];
}

// Per bead: what the terms need besides the folded sums.
struct TermInputs {
  int slot, nv;
  float kv;
  double V0;
  double k[2], L0[2];
  double2 drive;
};

// Swimmer s owns beads 3s, 3s + 1, 3s + 2, which lets every load issue at once.
__device__ inline TermInputs term_inputs(const Dev& d, int b) {
  const int sw = b / 3;
  const Bead& q = d.beads[b];
  const Swimmer& S = d.swimmers[sw];
  return TermInputs{b - 3 * sw, q.nv, q.kv, q.V0, {S.k[0], S.k[1]}, {S.L0[0], S.L0[1]}, d.drive[sw]};
}

// Terms of a bead from the centres of its swimmer's beads, c[bead][4] (the
// fourth value of each: 6 V), as bead_terms.
__device__ inline BeadTerms step_terms(const TermInputs& q, const double* c) {
  double f[3] = {q.slot == 0 ? q.drive.x : (q.slot == 2 ? q.drive.y : -q.drive.x - q.drive.y), 0.0, 0.0};
#pragma unroll
  for (int sp = 0; sp < 2; ++sp) {
    const int outer = 2 * sp;
    if (q.slot != outer && q.slot != 1) continue;
    const double dx = c[4 * outer] - c[4], dy = c[4 * outer + 1] - c[5], dz = c[4 * outer + 2] - c[6];
    const double len = sqrt(dx * dx + dy * dy + dz * dz);
    const double s = (q.slot == outer ? -1.0 : 1.0) * q.k[sp] * (len - q.L0[sp]) / len;
    f[0] += s * dx;
    f[1] += s * dy;
    f[2] += s * dz;
  }
  const float inv = 1.0f / (float)q.nv;
  BeadTerms t;
  t.pv = (float)(q.kv * (c[4 * q.slot + 3] / 6.0 - q.V0) / (6.0 * q.V0));
  t.share[0] = (float)f[0] * inv;
  t.share[1] = (float)f[1] * inv;
  t.share[2] = (float)f[2] * inv;
  return t;
}

// A marker's bead, position and split force (bead_terms.h), as loaded.
struct StepMarker {
  int bead;  // -1: none
  double x[3];
  float fm[3], gv[3];
  __device__ inline void load(const Dev& d, int m, int end) {
    bead = -1;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      x[a] = 0.0;
      fm[a] = gv[a] = 0.0f;
    }
    if (m >= end) return;
    bead = d.marker_bead[m];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      x[a] = d.pos_new[a * d.nm + m];
      fm[a] = d.fmem[a * d.nm + m];
      gv[a] = d.gvol[a * d.nm + m];
    }
  }
};

// Spreading into one slab (kSlabLayers z layers) of a near tile and the
// collision of its nodes.  The workgroup is short and bound by its chain of
// memory trips, so these are kept to three: its table entry; the near ranges,
// the patch values and the markers; (the populations come meanwhile).
template <int ST, int NW, int EX, int SZ>
__device__ inline void spread_block(const Dev& d, int sblk, int collide, int64_t n) {
  __shared__ StepEntry ent[kStepBlock];
  __shared__ float acc[kWaves][3][64];
  __shared__ int wave_cnt[kWaves];
  __shared__ int nonfinite;  // the chunk has a force or a position that is not finite
  __shared__ BeadTerms terms[kFoldBeads];
  __shared__ double fv[kFoldBeads * 4];
  static_assert(sizeof(ent) >= sizeof(double) * 4 * kFoldPatches, "patch values fit the entries' LDS");
  const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
  int box = 0, c = sblk;
  if (d.nboxes > 1) {
    const int2 e = d.step_spread[sblk];
    box = uniform(e.x);
    c = uniform(e.y);
  }
  const StepBox X = uniform(d.step_box[box]);
  const int count = uniform(d.slab_count[box]);
  const int bead0 = X.bead0, nb = X.nbeads, m_end = X.m_end;
  const Box B = uniform(d.boxes[box]);
  // a box's markers that all fit one chunk are loaded at once, else those of
  // the slab's first bead on when the entry is known
  const bool one_chunk = X.m_end - X.m0 <= kStepBlock;
  StepMarker q;
  if (one_chunk) q.load(d, X.m0 + tid, m_end);
  int4 entry = uniform(d.slab_list[X.list0 + min(c, max(count - 1, 0))]);
  const bool avg = EX == kAverage && avg_sampled(d, n);
  // markers of the box's beads, by lane
  const int lane_first = lane < nb ? d.beads[bead0 + lane].first : 0x7fffffff;
  const int lane_end = lane < nb ? lane_first + d.beads[bead0 + lane].nv : 0;
  // what the bead terms are made of, loaded with the ranges and the markers
  double pv[2] = {0.0, 0.0};
  int p0 = 0, np = 0;
  double inv_nv = 0.0;
  TermInputs in{};
  static_assert(4 * kFoldPatches <= 2 * kStepBlock && kFoldBeads <= 64, "patch values per thread");
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int t = r * kStepBlock + tid;
    if (t < 4 * X.npatch) pv[r] = patch_value(d, X.patch0 + (t >> 2), t & 3);
  }
  if (tid < 4 * nb) {
    const Bead& bd = d.beads[bead0 + (tid >> 2)];
    p0 = bd.patch0 - X.patch0;
    np = bd.npatch;
    inv_nv = bd.inv_nv;
  }
  if (tid < nb) in = term_inputs(d, bead0 + tid);
  if (c >= count) return;
  double* const pbuf = reinterpret_cast<double*>(ent);
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int t = r * kStepBlock + tid;
    if (t < 4 * X.npatch) pbuf[t] = pv[r];
  }
  __syncthreads();
  if (tid < 4 * nb) {
    const int k = tid & 3;
    double v = 0.0;
#pragma unroll 4
    for (int j = 0; j < np; ++j) v += pbuf[4 * (p0 + j) + k];
    fv[tid] = k < 3 ? v * inv_nv : v;
  }
  __syncthreads();
  if (tid < nb) terms[tid] = step_terms(in, fv + 4 * (tid - in.slot));
  for (;;) {
    const int tile = entry.x / kSlabParts, part = entry.x % kSlabParts;
    const int tx = tile % B.tx, ty = (tile / B.tx) % B.ty, tz = tile / (B.tx * B.ty);
    const unsigned long long cover = (uint64_t)(uint32_t)entry.z | (uint64_t)(uint32_t)entry.w << 32;
    const int m0 = one_chunk ? X.m0 : entry.y;
    if (!one_chunk) q.load(d, m0 + tid, m_end);
    const int ox = tx * kTile, oy = ty * kTile, oz = tz * kTile + kSlabLayers * part;
    const int ex = min(kTile, B.nx - ox), ey = min(kTile, B.ny - oy), ez = min(kSlabLayers, B.nz - oz);
    if (part == 0 && tid == 0) d.stamp[B.tile0 + tile] = (int)n;
    // the slab's nodes, one per thread of the first waves: their populations
    // are loaded before the spreading, which hides the latency
    const int lx = tid % kTile, ly = (tid / kTile) % kTile, lz = tid / (kTile * kTile);
    const bool node_in = tid < kSlabNodes && lx < ex && ly < ey && lz < ez;
    const int x = ox + lx, y = oy + ly, z = oz + lz;
    const int64_t base = B.node0 + ((int64_t)z * B.ny + y) * B.nx + x;
    float g[kQ];
    AvgSums sums{0.0, 0.0, 0.0};
    if (collide && node_in) {
      const Nbr o = neighbours(x, y, z, B.nx, B.ny, B.nz);
      sums = avg_load(d, base, avg);
      sc_load<ST, kNtLd<SZ>, kOff32<SZ>>(d, o, base, n, g);
    }
    // this lane's node in layer wave / kSubsets, summed over the entries e =
    // wave mod kSubsets
    float sx = 0.0f, sy = 0.0f, sz = 0.0f;
    const int layer = wave / kSubsets, subset = wave % kSubsets;
    // One chunk of markers (one per thread) into the slab's sums: those of
    // covering beads whose stencils meet the slab are compacted in marker
    // order; each lane adds them at its node.  Fixed order, no atomics, and no
    // addition waits on LDS (sums held in LDS cost one dependent LDS round
    // trip per entry).
    auto spread_chunk = [&]() {
      bool take = q.bead >= 0;
      const int i = q.bead - bead0;
      int off[3], first_node[3];
      take = take && ((cover >> (i & 63)) & 1ull);
      if (take) {
        const int org[3] = {ox, oy, oz}, ext[3] = {ex, ey, ez}, N[3] = {B.nx, B.ny, B.nz};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          first_node[a] = stencil_base<NW>(q.x[a]);
          const int r = wrap(first_node[a] - org[a], N[a], B.inv[a]);
          take = take && (r < ext[a] || r >= N[a] - NW + 1);
          off[a] = r < ext[a] ? r : r - N[a];
        }
      }
      const unsigned long long mask = __ballot(take);
      const int before = __popcll(mask & ((1ull << lane) - 1ull));
      __syncthreads();  // previous chunk's entries fully consumed, bead terms made
      if (lane == 0) wave_cnt[wave] = __popcll(mask);
      if (tid == 0) nonfinite = 0;
      __syncthreads();
      int at = before, total = 0;
      for (int w = 0; w < kWaves; ++w) {
        if (w < wave) at += wave_cnt[w];
        total += wave_cnt[w];
      }
      if (take) {
        StepEntry& E = ent[at];
        const BeadTerms t = terms[i];
        float w[3][NW];
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
          for (int k = 0; k < NW; ++k) w[a][k] = phi_fused<NW>((float)((double)(first_node[a] + k) - q.x[a]));
        float4* const zero = reinterpret_cast<float4*>(E.wx);
#pragma unroll
        for (int k = 0; k < 4; ++k) zero[k] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
        for (int k = 0; k < NW; ++k) {
          if ((unsigned)(off[0] + k) < (unsigned)kTile) E.wx[off[0] + k] = w[0][k];
          if ((unsigned)(off[1] + k) < (unsigned)kTile) E.wy[off[1] + k] = w[1][k];
        }
        const float fx = total_force(q.fm[0], q.gv[0], t.pv, t.share[0]),
                    fy = total_force(q.fm[1], q.gv[1], t.pv, t.share[1]),
                    fz = total_force(q.fm[2], q.gv[2], t.pv, t.share[2]);
        // a sum that is not finite has a term that is not
        if (!(fabsf(fx + fy + fz + (float)(q.x[0] + q.x[1] + q.x[2])) < INFINITY)) nonfinite = 1;
#pragma unroll
        for (int l = 0; l < kSlabLayers; ++l) {
          float wz = 0.0f;
#pragma unroll
          for (int k = 0; k < NW; ++k) wz = l - off[2] == k ? w[2][k] : wz;
          *reinterpret_cast<float4*>(E.f[l]) =
              wz != 0.0f ? make_float4(wz * fx, wz * fy, wz * fz, 0.0f) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
      }
      __syncthreads();
      auto add = [&](const StepEntry& E) {
        const float w = E.wx[lane % kTile] * E.wy[lane / kTile];
        const float4 f = *reinterpret_cast<const float4*>(E.f[layer]);
        sx = fmaf(w, f.x, sx);
        sy = fmaf(w, f.y, sy);
        sz = fmaf(w, f.z, sz);
      };
      if (!nonfinite) {
#pragma unroll 4
        for (int e = subset; e < total; e += kSubsets) add(ent[e]);
      } else {  // not beyond the stencils, where the weights are zero
        for (int e = subset; e < total; e += kSubsets)
          if (ent[e].wx[lane % kTile] != 0.0f && ent[e].wy[lane / kTile] != 0.0f) add(ent[e]);
      }
    };
    // the box's markers from the first covering bead's on, kStepBlock at a
    // time, leaving out the chunks that hold no marker of a covering bead; the
    // next chunk is loaded before the current one is worked on
    for (int at = m0;;) {
      int next = at + kStepBlock;
      for (; next < m_end; next += kStepBlock) {
        const bool meets = lane < nb && ((cover >> lane) & 1ull) && lane_first < next + kStepBlock && lane_end > next;
        if (__ballot(meets)) break;
      }
      StepMarker ahead;
      if (next < m_end) ahead.load(d, next + tid, m_end);
      spread_chunk();
      if (next >= m_end) break;
      q = ahead;
      at = next;
    }
    acc[wave][0][lane] = sx;
    acc[wave][1][lane] = sy;
    acc[wave][2][lane] = sz;
    __syncthreads();
    if (node_in) {
      float ax = 0, ay = 0, az = 0;
#pragma unroll
      for (int k = 0; k < kSubsets; ++k) {
        ax += acc[lz * kSubsets + k][0][lane];
        ay += acc[lz * kSubsets + k][1][lane];
        az += acc[lz * kSubsets + k][2][lane];
      }
      d.F[base] = ax;
      d.F[d.pstride + base] = ay;
      d.F[2 * d.pstride + base] = az;
      if (collide) {
        const Nbr o = neighbours(x, y, z, B.nx, B.ny, B.nz);
        sc_finish<ST, EX == kMoments, kOff32<SZ>, false, kThrough<SZ>>(d, B, o, base, n, g, B.gx + ax, B.gy + ay, B.gz + az, true,
                                                             avg, sums);
      }
    }
    c += X.workers;
    if (c >= count) return;
    entry = uniform(d.slab_list[X.list0 + c]);
    __syncthreads();  // the sums are read before the next slab's are written
  }
}

// ---- bead bookkeeping -----------------------------------------------------------------------
// The near tiles of step v around a bead with the region [lo, hi]: the bead's
// tile range, the tiles' stamps, and the flags of the blocks they meet.  One
// workgroup.
__device__ inline void mark_near_tiles(const Dev& d, const Bead& Bd, int b, const int* lo, const int* hi, int64_t v) {
  const Box B = d.boxes[Bd.box];
  const int T[3] = {B.tx, B.ty, B.tz}, N[3] = {B.nx, B.ny, B.nz};
  const int reserved[3] = {Bd.tiles_x, Bd.tiles_y, Bd.tiles_z};
  const int slot = (int)(v & 1);
  NearRange r;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    tile_run(lo[a] - kNearMargin, hi[a] + kNearMargin, N[a], T[a], r.t0[a], r.cnt[a]);
    if (r.cnt[a] > reserved[a]) {
      if (threadIdx.x == 0) atomicOr(d.overflow, 1);
      r.cnt[a] = reserved[a];
    }
    r.cnt[a] = max(r.cnt[a], 0);
  }
  if (threadIdx.x == 0) d.near_range[slot * d.nbeads + b] = r;
  const int first = d.nboxes == 1 ? 0 : d.step_box_block0[Bd.box];
  const int rows = r.cnt[0] * r.cnt[1] * r.cnt[2] * kTile * kTile;
  for (int i = threadIdx.x; i < rows; i += blockDim.x) {
    const int row = i % (kTile * kTile), tt = i / (kTile * kTile);
    const int tx = pmod(r.t0[0] + tt % r.cnt[0], B.tx), ty = pmod(r.t0[1] + (tt / r.cnt[0]) % r.cnt[1], B.ty),
              tz = pmod(r.t0[2] + tt / (r.cnt[0] * r.cnt[1]), B.tz);
    if (row == 0) d.near_tile[slot * d.ntiles + B.tile0 + tx + B.tx * (ty + B.ty * tz)] = (int)v;
    const int y = ty * kTile + row % kTile, z = tz * kTile + row / kTile;
    if (y >= B.ny || z >= B.nz) continue;
    const int id = (z * B.ny + y) * B.nx + tx * kTile;  // first node of the row
    const int end = id + min(kTile, B.nx - tx * kTile) - 1;
    int* const flags = d.step_near + (size_t)slot * d.nstep + first;
    flags[id / kStepBlock] = (int)v;
    flags[end / kStepBlock] = (int)v;
  }
}

// One workgroup per bead: bead state from the patch values, the total
// force of each marker, the markers' new positions into d.pos, and the near
// tiles of step n + 1.
template <int NW>
__device__ inline void bead_block(const Dev& d, int b, int64_t n) {
  __shared__ double val[3 * kPartVals], cen[12];
  __shared__ BeadTerms sterm;
  __shared__ int reg[6];
  const int tid = threadIdx.x;
  const Bead Bd = d.beads[b];
  const Box B = d.boxes[Bd.box];
  const TermInputs in = term_inputs(d, b);
  const int s0 = b - in.slot;  // first bead of the swimmer
  if (tid < 3 * kPartVals) {
    const int i = tid / kPartVals, k = tid % kPartVals;
    const Bead& q = d.beads[s0 + i];
    const double* const src = d.part + (size_t)q.patch0 * kPartVals;
    const bool sum = k < 3 || k >= 9;
    double s = sum ? 0.0 : src[k];
#pragma unroll 8
    for (int j = 0; j < q.npatch; ++j) {
      const double x = k == 9 ? src[j * kPartVals + 9] + src[j * kPartVals + 10] : src[j * kPartVals + k];
      s = sum ? s + x : (k < 6 ? fmin(s, x) : fmax(s, x));
    }
    val[tid] = s;
    if (k < 3) cen[4 * i + k] = s * q.inv_nv;
    if (k == 9) cen[4 * i + 3] = s;
  }
  __syncthreads();
  if (tid == 0) {
    sterm = step_terms(in, cen);
    d.bstate[b].V = cen[4 * in.slot + 3] / 6.0;
  } else if (tid >= 64 && tid < 67) {
    const int a = tid - 64;
    const double* const v = val + kPartVals * in.slot;
    BeadState& st = d.bstate[b];
    st.c[a] = cen[4 * in.slot + a];
    const int lo = stencil_base<NW>(v[3 + a]), hi = stencil_base<NW>(v[6 + a]) + NW - 1;
    st.lo[a] = reg[a] = lo;
    st.hi[a] = reg[3 + a] = hi;
    int t0, cnt;
    tile_run(lo, hi, a == 0 ? B.nx : (a == 1 ? B.ny : B.nz), a == 0 ? B.tx : (a == 1 ? B.ty : B.tz), t0, cnt);
    st.tlo[a] = t0;
    st.tcnt[a] = max(cnt, 0);
  }
  __syncthreads();
  mark_near_tiles(d, Bd, b, reg, reg + 3, n + 1);
  if (d.near) mark_near_blocks(d, B, Bd.box, reg, reg + 3, n);  // for the reverse sweep
  const BeadTerms t = sterm;
  const int nm = d.nm;
  for (int i = tid; i < Bd.nv; i += kStepBlock) {
    const int m = Bd.first + i;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      d.pos[a * nm + m] = d.pos_new[a * nm + m];
      d.fm[a * nm + m] = total_force(d.fmem[a * nm + m], d.gvol[a * nm + m], t.pv, t.share[a]);
    }
  }
}

// Grid: the spreading workgroups, one workgroup per bead, then the blocks from
// `share` on.
template <int ST, int NW, int EX, int SZ>
__global__ __launch_bounds__(kStepBlock, 4) void k_step_b(Dev d, int collide, int share) {
  const int64_t n = uniform(*d.step) + d.sub;
  int i = blockIdx.x;
  if (i < d.step_spread_blocks) {
    spread_block<ST, NW, EX, SZ>(d, i, collide, n);
  } else if ((i -= d.step_spread_blocks) < d.nbeads) {
    bead_block<NW>(d, i, n);
  } else {
    step_bulk<ST, EX, SZ>(d, share + i - d.nbeads, n);
  }
}

// Advection of the last step of a sequence, in place, and the step counter.
template <int NW>
__global__ __launch_bounds__(256) void k_step_end(Dev d) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *d.step += d.tick;
  const int gid = blockIdx.x * 256 + threadIdx.x;
  const int m = gid / kRowLanes, ln = gid % kRowLanes;
  const int yk = ln % NW, zk = ln / NW;
  const bool in = m < d.nm && ln < NW * NW;
  double3 p = make_double3(0, 0, 0);
  RowStencil<NW> r{};
  RowValues<NW> q{};
  if (in) {
    p = load_pos(d.pos, d.nm, m);
    const Box B = d.boxes[d.nboxes == 1 ? 0 : d.marker_info[m].y];
    const int bx = stencil_base<NW>(p.x), by = stencil_base<NW>(p.y) + yk, bz = stencil_base<NW>(p.z) + zk;
    r.wyz = phi_fused<NW>((float)((double)by - p.y)) * phi_fused<NW>((float)((double)bz - p.z));
    const int row = (wrap(bz, B.nz, B.inv[2]) * B.ny + wrap(by, B.ny, B.inv[1])) * B.nx;
    int x = wrap(bx, B.nx, B.inv[0]);
#pragma unroll
    for (int k = 0; k < NW; ++k) {
      r.wx[k] = phi_fused<NW>((float)((double)(bx + k) - p.x));
      r.c[k] = row + x;
      x = x + 1 == B.nx ? 0 : x + 1;
    }
    q = row_load<NW>(d.u + B.node0, d.pstride, r);
  }
  const float3 v = row_sum<NW>(q, r, in);
  if (in && ln == 0) {
    d.U[m] = v.x;
    d.U[d.nm + m] = v.y;
    d.U[2 * d.nm + m] = v.z;
    d.pos[m] = p.x + (double)v.x;
    d.pos[d.nm + m] = p.y + (double)v.y;
    d.pos[2 * d.nm + m] = p.z + (double)v.z;
  }
}

__global__ __launch_bounds__(256) void k_step_mark(Dev d) {
  const int b = blockIdx.x;
  const BeadState& st = d.bstate[b];
  mark_near_tiles(d, d.beads[b], b, st.lo, st.hi, *d.step + d.sub);
}

// ---- launches ---------------------------------------------------------------------------------
template <class K, class... Args>
void launch_ev(K kernel, int grid, int lds, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1, const Args&... args) {
  if (ev0)
    hipExtLaunchKernelGGL(kernel, dim3(grid), dim3(kStepBlock), lds, s, ev0, ev1, 0, args...);
  else
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kStepBlock), lds, s, args...);
}

// k_step_a is launched with unused LDS up to a total of kStepALds, so that two of its
// workgroups fit a compute unit as of k_step_b (128 registers) and a third does not,
// whatever its kernel width needs: 16 wavefronts stream faster than 24 (1024x256x256
// 1803 us per step with three, 1747 with two; 128^3 in place 53.8 and 53.4; width 2
// 1742 and 1699, 56.2 and 53.3; one of k_step_b's per unit: 60.3).
constexpr int kStepALds = 57344;
template <int NW>
constexpr int kPatchLds = kPatchLocal * (3 * (int)sizeof(double) + 3 * NW * (int)(sizeof(float) + sizeof(int)) + (int)sizeof(int)) +
                          3 * (int)sizeof(float) * (3 * kPatchTri + kPatchTri + 4 * kPatchHinge);
static_assert(3 * kStepALds > 160 * 1024 && kPatchLds<4> < kStepALds, "two workgroups per compute unit, not three");

struct StepArgs {
  int b, x, y;  // launch (0: a, 1: b) and its two integer arguments
  hipStream_t s;
  hipEvent_t ev0, ev1;
};

template <int ST, int NW, int EX, int SZ>
void launch_step_i(const Dev& d, const StepArgs& p) {
  if (p.b == 0)
    launch_ev(k_step_a<ST, NW, EX, SZ>, d.npatch + d.nboxes + p.y, kStepALds - kPatchLds<NW>, p.s, p.ev0, p.ev1, d, p.x, d.npatch + d.nboxes);
  else
    launch_ev(k_step_b<ST, NW, EX, SZ>, d.step_spread_blocks + d.nbeads + (p.x ? d.nstep - p.y : 0), 0, p.s, p.ev0,
              p.ev1, d, p.x, p.y);
}

template <int ST, int NW, int EX>
void launch_step_n(const Dev& d, const StepArgs& p) {
  if (d.small_pops)
    launch_step_i<ST, NW, EX, kSmall>(d, p);
  else if (ST == kFp32InPlace || d.pops32)
    launch_step_i<ST, NW, EX, kLarge>(d, p);
  else
    launch_step_i<ST, NW, EX, ST == kFp32InPlace ? kLarge : kHuge>(d, p);
}

template <int ST, int NW>
void launch_step_w(const Dev& d, const StepArgs& p) {
  if (d.uavg)
    launch_step_n<ST, NW, kAverage>(d, p);
  else
    launch_step_n<ST, NW, kPlain>(d, p);
}

template <int ST>
void launch_step_st(const Dev& d, const StepArgs& p) {
  if (d.width == 2)
    launch_step_w<ST, 2>(d, p);
  else if (d.width == 3)
    launch_step_w<ST, 3>(d, p);
  else
    launch_step_w<ST, 4>(d, p);
}

StepArgs step_args(int mode, int share, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  const bool second = mode == kLaunchStepB || mode == kLaunchStepSpread;
  return {second, mode == kLaunchStepA || mode == kLaunchStepB, share, s, ev0, ev1};
}

void launch_step_sto(const Dev& d, int storage, const StepArgs& p) {
  if (storage == kFp32Plain)
    launch_step_st<kFp32Plain>(d, p);
  else if (storage == kFp32InPlace)
    launch_step_st<kFp32InPlace>(d, p);
  else
    launch_step_st<kFp32>(d, p);
}

}  // namespace

void launch_step(const Dev& d, int storage, int mode, int share, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  launch_step_sto(d, storage, step_args(mode, share, s, ev0, ev1));
}

void launch_step_mom(const Dev& d, int mode, int share, hipStream_t s) {
  const StepArgs p = step_args(mode, share, s, nullptr, nullptr);
  if (d.width == 2)
    launch_step_n<kFp32, 2, kMoments>(d, p);
  else if (d.width == 3)
    launch_step_n<kFp32, 3, kMoments>(d, p);
  else
    launch_step_n<kFp32, 4, kMoments>(d, p);
}

void launch_step_end(const Dev& d, hipStream_t s) {
  const int blocks = (int)(((int64_t)d.nm * kRowLanes + 255) / 256);
  if (d.width == 2) hipLaunchKernelGGL(k_step_end<2>, dim3(blocks), dim3(256), 0, s, d);
  else if (d.width == 3) hipLaunchKernelGGL(k_step_end<3>, dim3(blocks), dim3(256), 0, s, d);
  else hipLaunchKernelGGL(k_step_end<4>, dim3(blocks), dim3(256), 0, s, d);
}

void launch_step_mark(const Dev& d, hipStream_t s) {
  hipLaunchKernelGGL(k_step_mark, dim3(d.nbeads), dim3(256), 0, s, d);
}

}  // namespace lbmib
