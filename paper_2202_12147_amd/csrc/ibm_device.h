// Device code of the immersed boundary and the membranes (delta kernels,
// reductions, element forces) shared by the kernel translation units
// (included only by the .hip files).
#pragma once

#include "common.h"

namespace lbmib {

namespace {

__device__ inline int pmod(int a, int b) {
  int r = a % b;
  return r < 0 ? r + b : r;
}

// phi of the delta kernel.
template <int NW>
__device__ inline float phi(float r) {
  r = fabsf(r);
  if constexpr (NW == 2) {
    return r < 1.0f ? 1.0f - r : 0.0f;
  } else if constexpr (NW == 3) {
    if (r <= 0.5f) return (1.0f + sqrtf(1.0f - 3.0f * r * r)) * (1.0f / 3.0f);
    if (r <= 1.5f) return (5.0f - 3.0f * r - sqrtf(fmaxf(0.0f, 1.0f - 3.0f * (1.0f - r) * (1.0f - r)))) * (1.0f / 6.0f);
    return 0.0f;
  } else {
    if (r <= 1.0f) return (3.0f - 2.0f * r + sqrtf(1.0f + 4.0f * r - 4.0f * r * r)) * 0.125f;
    if (r <= 2.0f) return (5.0f - 2.0f * r - sqrtf(fmaxf(0.0f, -7.0f + 12.0f * r - 4.0f * r * r))) * 0.125f;
    return 0.0f;
  }
}

// a mod N in [0, N) with invN = 1/N in FP64: the quotient is off by at most one
// for every 32-bit a, and no integer division is made (about 40 instructions).
__device__ inline int wrap(int a, int N, double invN) {
  const int q = (int)floor((double)a * invN);
  int r = a - q * N;
  if (r < 0) r += N;
  if (r >= N) r -= N;
  return r;
}

// phi for the fused step.  The sums of products are explicit fmaf (which
// product is fused could otherwise differ between kernels), and both branches
// share one square root, sqrt(1 - 3 s^2) (three-point) or sqrt(2 - (1 - 2 s)^2)
// (four-point), with s the distance folded into the inner interval.
template <int NW>
__device__ inline float phi_fused(float r) {
  r = fabsf(r);
  if constexpr (NW == 2) {
    return r < 1.0f ? 1.0f - r : 0.0f;
  } else if constexpr (NW == 3) {
    const bool inner = r <= 0.5f;
    const float s = inner ? r : 1.0f - r;
    const float q = sqrtf(fmaxf(0.0f, fmaf(-3.0f * s, s, 1.0f)));
    const float in = (1.0f + q) * (1.0f / 3.0f), out = (fmaf(-3.0f, r, 5.0f) - q) * (1.0f / 6.0f);
    return inner ? in : (r <= 1.5f ? out : 0.0f);
  } else {
    // 1 + 4 r - 4 r^2 = 2 - (1 - 2 r)^2 and -7 + 12 r - 4 r^2 = 2 - (3 - 2 r)^2
    const bool inner = r <= 1.0f;
    const float e = inner ? 3.0f : 5.0f;
    const float t = fmaf(-2.0f, r, e - 2.0f);
    const float q = sqrtf(fmaxf(0.0f, fmaf(-t, t, 2.0f)));
    const float v = fmaf(-2.0f, r, e) + (inner ? q : -q);
    return r <= 2.0f ? v * 0.125f : 0.0f;
  }
}

// First stencil node of a marker coordinate.  The clamp keeps the integer
// conversion defined when a diverged run produces non-finite positions (fmax
// returns the finite operand for NaN); the bead-region check then reports it.
template <int NW>
__device__ inline int stencil_base(double r) {
  r = fmin(fmax(r, -1.0e9), 1.0e9);
  if constexpr (NW == 3) return (int)floor(r + 0.5) - 1;
  if constexpr (NW == 4) return (int)floor(r) - 1;
  return (int)floor(r);
}

__device__ inline double3 load_pos(const double* pos, int nm, int m) {
  return make_double3(pos[m], pos[nm + m], pos[2 * nm + m]);
}

// ---- wavefront reductions ---------------------------------------------------
// Within rows of 16 lanes by DPP moves: pairs and quads by quad permutations,
// then the mirrored half row and the mirrored row, after which every lane of
// a row holds the row's total.  Each step is a register move of the ALU; a
// shuffle routes every step through the LDS unit.
constexpr int kDppXor1 = 0xB1;         // quad_perm [1, 0, 3, 2]
constexpr int kDppXor2 = 0x4E;         // quad_perm [2, 3, 0, 1]
constexpr int kDppHalfMirror = 0x141;  // lane i <- lane 7 - i of its half row
constexpr int kDppMirror = 0x140;      // lane i <- lane 15 - i of its row

template <int CTRL>
__device__ inline float dpp_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
template <int CTRL>
__device__ inline double dpp_move(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}

enum { kRedSum, kRedMin, kRedMax };
template <int OP, typename T>
__device__ inline T red_op(T a, T b) {
  if constexpr (OP == kRedSum) return a + b;
  else if constexpr (OP == kRedMin) return fmin(a, b);  // a NaN operand is dropped
  else return fmax(a, b);
}

// The reduction over each aligned group of L lanes (L a power of two up to
// 64), the result in every lane of the group; the steps beyond a row of 16
// are shuffles.
template <int L, int OP = kRedSum, typename T>
__device__ inline T group_reduce(T v) {
  if constexpr (L >= 2) v = red_op<OP>(v, dpp_move<kDppXor1>(v));
  if constexpr (L >= 4) v = red_op<OP>(v, dpp_move<kDppXor2>(v));
  if constexpr (L >= 8) v = red_op<OP>(v, dpp_move<kDppHalfMirror>(v));
  if constexpr (L >= 16) v = red_op<OP>(v, dpp_move<kDppMirror>(v));
#pragma unroll
  for (int s = 16; s < L; s <<= 1) v = red_op<OP>(v, __shfl_xor(v, s, 64));
  return v;
}

// The reduction over the whole wavefront, the result in every lane: row
// totals by DPP, then the four rows read out and combined in a fixed order.
template <int OP>
__device__ inline double wave_reduce(double v) {
  v = group_reduce<16, OP>(v);
  double r[4];
#pragma unroll
  for (int k = 0; k < 4; ++k)
    r[k] = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 16 * k),
                            __builtin_amdgcn_readlane(__double2loint(v), 16 * k));
  return red_op<OP>(red_op<OP>(r[0], r[1]), red_op<OP>(r[2], r[3]));
}

// ---- membrane forces ------------------------------------------------------------
// Skalak force on corner `corner` of triangle t.  With
// Delta = g - G0 (metric change, formed in FP64), I1 = G0^-1 : Delta,
// I2 = (det g - det G0)/det G0 and the stress P = dW/dg written so that its
// O(1) parts cancel analytically:
//   P = ks A0/4 [(2 I1 + 2 C I2) G0^-1 + (2 C I2 - 2) adj(Delta)/det G0],
// dW/de1 = 2 (P11 e1 + P12 e2), dW/de2 = 2 (P12 e1 + P22 e2), e_a = r_a - r_0.
// The triangle's area vector (r1 - r0) x (r2 - r0), formed in FP64, goes to
// `area`: the volume force of the corner is -pv times it (bead_terms.h).
struct TriangleTerms {
  float P11, P12, P22;  // dW/dg
  float e1[3], e2[3];
  float3 area;
};

__device__ inline TriangleTerms triangle_terms(const Dev& d, const Bead& Bd, int t, const double3& p0,
                                               const double3& p1, const double3& p2) {
  const double e1x = p1.x - p0.x, e1y = p1.y - p0.y, e1z = p1.z - p0.z;
  const double e2x = p2.x - p0.x, e2y = p2.y - p0.y, e2z = p2.z - p0.z;
  const double G11d = d.G0[t], G12d = d.G0[d.ntri + t], G22d = d.G0[2 * d.ntri + t];
  const float D11 = (float)(e1x * e1x + e1y * e1y + e1z * e1z - G11d);
  const float D12 = (float)(e1x * e2x + e1y * e2y + e1z * e2z - G12d);
  const float D22 = (float)(e2x * e2x + e2y * e2y + e2z * e2z - G22d);
  const float G11 = (float)G11d, G12 = (float)G12d, G22 = (float)G22d;
  const float Gi11 = d.G0inv[t], Gi12 = d.G0inv[d.ntri + t], Gi22 = d.G0inv[2 * d.ntri + t];
  const float idet = d.idetG0[t];
  const float I1 = Gi11 * D11 + 2.0f * Gi12 * D12 + Gi22 * D22;
  const float I2 = (G11 * D22 + G22 * D11 - 2.0f * G12 * D12 + (D11 * D22 - D12 * D12)) * idet;
  const float k4 = 0.25f * Bd.ks * d.A0[t];
  const float a = k4 * (2.0f * I1 + 2.0f * Bd.C * I2);
  const float bq = k4 * (2.0f * Bd.C * I2 - 2.0f) * idet;
  TriangleTerms T;
  T.P11 = fmaf(bq, D22, a * Gi11);
  T.P12 = fmaf(-bq, D12, a * Gi12);
  T.P22 = fmaf(bq, D11, a * Gi22);
  T.e1[0] = (float)e1x;
  T.e1[1] = (float)e1y;
  T.e1[2] = (float)e1z;
  T.e2[0] = (float)e2x;
  T.e2[1] = (float)e2y;
  T.e2[2] = (float)e2z;
  T.area = make_float3((float)(e1y * e2z - e1z * e2y), (float)(e1z * e2x - e1x * e2z), (float)(e1x * e2y - e1y * e2x));
  return T;
}

// Force -(ca e1 + cb e2) on one corner.
__device__ inline float3 corner_force(const TriangleTerms& T, int corner) {
  float ca, cb;
  if (corner == 1) {
    ca = 2.0f * T.P11;
    cb = 2.0f * T.P12;
  } else if (corner == 2) {
    ca = 2.0f * T.P12;
    cb = 2.0f * T.P22;
  } else {
    ca = -2.0f * (T.P11 + T.P12);
    cb = -2.0f * (T.P12 + T.P22);
  }
  return make_float3(-fmaf(ca, T.e1[0], cb * T.e2[0]), -fmaf(ca, T.e1[1], cb * T.e2[1]),
                     -fmaf(ca, T.e1[2], cb * T.e2[2]));
}

__device__ inline float3 triangle_corner(const Dev& d, const Bead& Bd, int t, int corner, int i0, int i1,
                                         int i2, float3& area) {
  const double3 p0 = load_pos(d.pos, d.nm, i0);
  const double3 p1 = load_pos(d.pos, d.nm, i1);
  const double3 p2 = load_pos(d.pos, d.nm, i2);
  const double e1x = p1.x - p0.x, e1y = p1.y - p0.y, e1z = p1.z - p0.z;
  const double e2x = p2.x - p0.x, e2y = p2.y - p0.y, e2z = p2.z - p0.z;
  const double G11d = d.G0[t], G12d = d.G0[d.ntri + t], G22d = d.G0[2 * d.ntri + t];
  const float D11 = (float)(e1x * e1x + e1y * e1y + e1z * e1z - G11d);
  const float D12 = (float)(e1x * e2x + e1y * e2y + e1z * e2z - G12d);
  const float D22 = (float)(e2x * e2x + e2y * e2y + e2z * e2z - G22d);
  const float G11 = (float)G11d, G12 = (float)G12d, G22 = (float)G22d;
  const float Gi11 = d.G0inv[t], Gi12 = d.G0inv[d.ntri + t], Gi22 = d.G0inv[2 * d.ntri + t];
  const float idet = d.idetG0[t];
  const float I1 = Gi11 * D11 + 2.0f * Gi12 * D12 + Gi22 * D22;
  const float I2 = (G11 * D22 + G22 * D11 - 2.0f * G12 * D12 + (D11 * D22 - D12 * D12)) * idet;
  const float k4 = 0.25f * Bd.ks * d.A0[t];
  const float a = k4 * (2.0f * I1 + 2.0f * Bd.C * I2);
  const float bq = k4 * (2.0f * Bd.C * I2 - 2.0f) * idet;
  const float P11 = a * Gi11 + bq * D22;
  const float P12 = a * Gi12 - bq * D12;
  const float P22 = a * Gi22 + bq * D11;
  const float e1[3] = {(float)e1x, (float)e1y, (float)e1z};
  const float e2[3] = {(float)e2x, (float)e2y, (float)e2z};
  float ca, cb;  // force = -(ca e1 + cb e2) from the Skalak energy
  if (corner == 1) {
    ca = 2.0f * P11;
    cb = 2.0f * P12;
  } else if (corner == 2) {
    ca = 2.0f * P12;
    cb = 2.0f * P22;
  } else {
    ca = -2.0f * (P11 + P12);
    cb = -2.0f * (P12 + P22);
  }
  area = make_float3((float)(e1y * e2z - e1z * e2y), (float)(e1z * e2x - e1x * e2z), (float)(e1x * e2y - e1y * e2x));
  return make_float3(-(ca * e1[0] + cb * e2[0]), -(ca * e1[1] + cb * e2[1]), -(ca * e1[2] + cb * e2[2]));
}

// Kantor-Nelson bending force -kt sin(theta - theta0) d theta / d x_role on one
// vertex of hinge h (x1, x2 shared edge; x3, x4 opposite).  With
// nA = (x2-x1) x (x3-x1), nB = (x1-x2) x (x4-x2), e = x2 - x1:
//   d theta/d x3 = -|e| nA/|nA|^2,  d theta/d x4 = -|e| nB/|nB|^2,
//   d theta/d x1 = -((x3-x2).e^) nA/|nA|^2 + ((x2-x4).e^) nB/|nB|^2,
//   d theta/d x2 = -((x1-x3).e^) nA/|nA|^2 + ((x4-x1).e^) nB/|nB|^2.
// sin(theta - theta0) = sin theta cos theta0 - cos theta sin theta0 with
// cos theta = nA.nB/(|nA||nB|), sin theta = (nA x nB).e^/(|nA||nB|), in FP64.
struct HingeTerms {
  float dW;                  // -dW/d theta applies to every role
  float nA[3], nB[3];
  float fa[4], fb[4];        // d theta/d x_role = fa nA + fb nB
};

__device__ inline HingeTerms hinge_terms(const Dev& d, const Bead& Bd, int h, const double3& x1, const double3& x2,
                                         const double3& x3, const double3& x4) {
  const double ex = x2.x - x1.x, ey = x2.y - x1.y, ez = x2.z - x1.z;
  const double ax = x3.x - x1.x, ay = x3.y - x1.y, az = x3.z - x1.z;
  const double bx = x4.x - x2.x, by = x4.y - x2.y, bz = x4.z - x2.z;
  const double nAx = ey * az - ez * ay, nAy = ez * ax - ex * az, nAz = ex * ay - ey * ax;
  const double nBx = -(ey * bz - ez * by), nBy = -(ez * bx - ex * bz), nBz = -(ex * by - ey * bx);
  const double iA = 1.0 / (nAx * nAx + nAy * nAy + nAz * nAz);
  const double iB = 1.0 / (nBx * nBx + nBy * nBy + nBz * nBz);
  const double E2 = ex * ex + ey * ey + ez * ez;
  const double E = sqrt(E2);
  const double iE = 1.0 / E;
  const double ehx = ex * iE, ehy = ey * iE, ehz = ez * iE;
  const double cx = nAy * nBz - nAz * nBy, cy = nAz * nBx - nAx * nBz, cz = nAx * nBy - nAy * nBx;
  const double inorm = sqrt(iA * iB);
  const double sn = (cx * ehx + cy * ehy + cz * ehz) * inorm;
  const double cs = (nAx * nBx + nAy * nBy + nAz * nBz) * inorm;
  HingeTerms T;
  T.dW = Bd.kt * (float)(sn * d.th0cs[h] - cs * d.th0cs[d.nh + h]);
  T.nA[0] = (float)nAx;
  T.nA[1] = (float)nAy;
  T.nA[2] = (float)nAz;
  T.nB[0] = (float)nBx;
  T.nB[1] = (float)nBy;
  T.nB[2] = (float)nBz;
  // projections on the edge: (x3 - x1), (x4 - x2); the others differ by E
  const double pa = ax * ehx + ay * ehy + az * ehz, pb = bx * ehx + by * ehy + bz * ehz;
  T.fa[0] = (float)((E - pa) * iA);  // -((x3 - x2).e^) / |nA|^2
  T.fb[0] = (float)(-pb * iB);       // ((x2 - x4).e^) / |nB|^2
  T.fa[1] = (float)(pa * iA);        // -((x1 - x3).e^) / |nA|^2
  T.fb[1] = (float)((E + pb) * iB);  // ((x4 - x1).e^) / |nB|^2
  T.fa[2] = (float)(-E * iA);
  T.fb[2] = 0.0f;
  T.fa[3] = 0.0f;
  T.fb[3] = (float)(-E * iB);
  return T;
}

__device__ inline float3 role_force(const HingeTerms& T, float fa, float fb) {
  return make_float3(-T.dW * fmaf(fa, T.nA[0], fb * T.nB[0]), -T.dW * fmaf(fa, T.nA[1], fb * T.nB[1]),
                     -T.dW * fmaf(fa, T.nA[2], fb * T.nB[2]));
}

__device__ inline float3 bending_role(const Dev& d, const Bead& Bd, int h, int role, int4 v) {
  const int nh = d.nh;
  const double3 x1 = load_pos(d.pos, d.nm, v.x);
  const double3 x2 = load_pos(d.pos, d.nm, v.y);
  const double3 x3 = load_pos(d.pos, d.nm, v.z);
  const double3 x4 = load_pos(d.pos, d.nm, v.w);
  const double ex = x2.x - x1.x, ey = x2.y - x1.y, ez = x2.z - x1.z;
  const double ax = x3.x - x1.x, ay = x3.y - x1.y, az = x3.z - x1.z;
  const double bx = x4.x - x2.x, by = x4.y - x2.y, bz = x4.z - x2.z;
  const double nAx = ey * az - ez * ay, nAy = ez * ax - ex * az, nAz = ex * ay - ey * ax;
  const double nBx = -(ey * bz - ez * by), nBy = -(ez * bx - ex * bz), nBz = -(ex * by - ey * bx);
  const double nA2 = nAx * nAx + nAy * nAy + nAz * nAz;
  const double nB2 = nBx * nBx + nBy * nBy + nBz * nBz;
  const double E = sqrt(ex * ex + ey * ey + ez * ez);
  const double iE = 1.0 / E;
  const double ehx = ex * iE, ehy = ey * iE, ehz = ez * iE;
  const double cx = nAy * nBz - nAz * nBy, cy = nAz * nBx - nAx * nBz, cz = nAx * nBy - nAy * nBx;
  const double inorm = 1.0 / sqrt(nA2 * nB2);
  const double sn = (cx * ehx + cy * ehy + cz * ehz) * inorm;
  const double cs = (nAx * nBx + nAy * nBy + nAz * nBz) * inorm;
  const float dW = Bd.kt * (float)(sn * d.th0cs[h] - cs * d.th0cs[nh + h]);
  double ca, cb;  // d theta / d x_role = ca nA/|nA|^2 + cb nB/|nB|^2
  if (role == 2) {
    ca = -E;
    cb = 0;
  } else if (role == 3) {
    ca = 0;
    cb = -E;
  } else if (role == 0) {
    ca = -((x3.x - x2.x) * ehx + (x3.y - x2.y) * ehy + (x3.z - x2.z) * ehz);
    cb = (x2.x - x4.x) * ehx + (x2.y - x4.y) * ehy + (x2.z - x4.z) * ehz;
  } else {
    ca = -((x1.x - x3.x) * ehx + (x1.y - x3.y) * ehy + (x1.z - x3.z) * ehz);
    cb = (x4.x - x1.x) * ehx + (x4.y - x1.y) * ehy + (x4.z - x1.z) * ehz;
  }
  const float fa = (float)(ca / nA2), fb = (float)(cb / nB2);
  return make_float3(-dW * (fa * (float)nAx + fb * (float)nBx), -dW * (fa * (float)nAy + fb * (float)nBy),
                     -dW * (fa * (float)nAz + fb * (float)nBz));
}

// Tiles of the node run [lo, hi] (unwrapped) on a periodic axis of N nodes in
// T tiles: from the wrapped first node, counted on in periodic tile order
// (tile T follows tile T - 1).  Node lo + j lies in tile (u / N) T +
// (u mod N) / kTile (mod T), u = (lo mod N) + j, which rises by at most one
// per node, so the run's nodes fill the tile run [t0, t0 + cnt) also on an
// edge that is not a whole number of tiles.  A run shorter than the edge
// wraps at most once.  cnt = 0: no run (non-finite positions).
__device__ inline void tile_run(int lo, int hi, int N, int T, int& t0, int& cnt) {
  const int lw = pmod(lo, N);
  const int hw = lw + (hi - lo);
  t0 = lw / kTile;
  cnt = T;
  if (hw < lw)
    cnt = 0;
  else if (hw - lw + 1 < N)
    cnt = (hw < N ? hw / kTile : T + (hw - N) / kTile) - t0 + 1;
  if (cnt >= T) {
    t0 = 0;
    cnt = T;
  }
}

// ---- stencils and tiles ------------------------------------------------------------

// Offset of a marker's stencil from the tile origin, taking the periodic image
// that meets the tile; returns false when no image meets it.
template <int NW>
__device__ inline bool stencil_offset(int base, int origin, int extent, int N, int& off) {
  const int r = pmod(base - origin, N);
  if (r < extent) {
    off = r;
    return true;
  }
  if (r >= N - NW + 1) {
    off = r - N;
    return true;
  }
  return false;
}

}  // namespace
}  // namespace lbmib
