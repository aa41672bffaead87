// Device helpers and constants shared by the trace kernels (k_trace) and the single-round
// kernels: ray keys, slab test, unit-sphere leaf terms, real spherical harmonics, and the
// per-lane stack sizes. Included inside namespace grtx's anonymous namespace of each
// source, so every file gets its own copies.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "grtx_internal.h"

namespace grtx {
namespace {

#ifndef GRTX_LDS_STACK
#define GRTX_LDS_STACK 16
#endif
constexpr int kTraceBlock = 256;
constexpr int kWaves = kTraceBlock / 64;
constexpr int kLdsStack = GRTX_LDS_STACK;  // per-lane stack entries held in LDS
// The build keeps no tree deeper than GRTX_MAX_TREE_DEPTH internal nodes on a path (it
// measures the restructured tree and falls back to the plain radix tree, at most 96 deep
// over distinct 95-bit keys); a record's children lie one to three levels below it, so a
// path visits at most that many records, each leaving at most three entries pending.
constexpr int kMaxStack = 3 * GRTX_MAX_TREE_DEPTH + 16;
constexpr int kSpillRows = kMaxStack - kLdsStack;
constexpr uint64_t kEmptyKey = (0x7F800000ull << 32) | 0xFFFFFFFFull;  // (+inf, max)

__device__ __forceinline__ float key_t(uint64_t k) { return __uint_as_float((uint32_t)(k >> 32)); }
__device__ __forceinline__ uint64_t make_key(float t, uint32_t id) {
  return ((uint64_t)__float_as_uint(t) << 32) | id;
}

// Robust reciprocal for the slab test: zero components become a huge finite value of
// the same sign, so that 0 * inv never produces NaN.
__device__ __forceinline__ float safe_inv(float d) {
  const float tiny = 1e-20f;
  float ad = fabsf(d);
  return 1.0f / copysignf(ad > tiny ? ad : tiny, d);
}

struct Slab {
  float tn, tf;
};

__device__ __forceinline__ Slab slab(float lox, float loy, float loz, float hix, float hiy, float hiz, float ox,
                                     float oy, float oz, float ix, float iy, float iz) {
  float t0x = (lox - ox) * ix, t1x = (hix - ox) * ix;
  float t0y = (loy - oy) * iy, t1y = (hiy - oy) * iy;
  float t0z = (loz - oz) * iz, t1z = (hiz - oz) * iz;
  Slab s;
  s.tn = fmaxf(fmaxf(fminf(t0x, t1x), fminf(t0y, t1y)), fminf(t0z, t1z));
  s.tf = fminf(fminf(fmaxf(t0x, t1x), fmaxf(t0y, t1y)), fmaxf(t0z, t1z));
  return s;
}

// Real spherical harmonics up to band 3 (orthonormal, Condon-Shortley phase) as
// polynomials in the unit direction. Y_l^m = sqrt(2) K_l^|m| (-1)^m (cos|sin)(|m| phi)
// sin^|m|(theta) P_l^(|m|)(cos theta), with K_l^m = sqrt((2l+1)/(4 pi) (l-|m|)!/(l+|m|)!)
// and P_l^(m) the m-th derivative of the Legendre polynomial.
constexpr double cx_sqrt(double x) {
  double r = x > 1.0 ? x : 1.0;
  for (int i = 0; i < 100; ++i) r = 0.5 * (r + x / r);
  return r;
}
constexpr double kPi = 3.14159265358979323846;
constexpr double K(int l, int am, double fac_ratio) { return cx_sqrt((2.0 * l + 1.0) / (4.0 * kPi) * fac_ratio); }
constexpr float SH00 = (float)K(0, 0, 1.0);
constexpr float SH1 = (float)K(1, 0, 1.0);                                   // sqrt(3/4pi)
constexpr float SH20 = (float)(K(2, 0, 1.0) * 0.5);                          // K20 / 2 * (3z^2 - 1)
constexpr float SH21 = (float)(cx_sqrt(2.0) * K(2, 1, 1.0 / 6.0) * 3.0);     // -xz, -yz
constexpr float SH22 = (float)(cx_sqrt(2.0) * K(2, 2, 1.0 / 24.0) * 3.0);    // (x^2-y^2), 2xy
constexpr float SH30 = (float)(K(3, 0, 1.0) * 0.5);                          // (5z^3 - 3z)
constexpr float SH31 = (float)(cx_sqrt(2.0) * K(3, 1, 1.0 / 12.0) * 0.5);    // -(15z^2-3) x|y
constexpr float SH32 = (float)(cx_sqrt(2.0) * K(3, 2, 1.0 / 120.0) * 15.0);  // z (x^2-y^2), 2xyz
constexpr float SH33 = (float)(cx_sqrt(2.0) * K(3, 3, 1.0 / 720.0) * 15.0);  // -(x^3-3xy^2), -(3x^2y-y^3)

// Contraction is written out (fmaf, and none elsewhere) here and in the functions below: the
// trace's kernels share them, and an image must not depend on which kernel rendered it.
__device__ __forceinline__ void sh_basis(float x, float y, float z, int L, float* Y) {
#pragma clang fp contract(off)
  Y[0] = SH00;
  if (L < 1) return;
  Y[1] = -SH1 * y;
  Y[2] = SH1 * z;
  Y[3] = -SH1 * x;
  if (L < 2) return;
  const float xx = x * x, yy = y * y, zz = z * z;
  const float xxyy = fmaf(x, x, -yy);
  Y[4] = SH22 * 2.f * x * y;
  Y[5] = -SH21 * y * z;
  Y[6] = SH20 * fmaf(zz, 3.f, -1.f);
  Y[7] = -SH21 * x * z;
  Y[8] = SH22 * xxyy;
  if (L < 3) return;
  const float zz15 = fmaf(zz, 15.f, -3.f);
  Y[9] = -SH33 * fmaf(y, 3.f * xx, -(y * yy));
  Y[10] = SH32 * 2.f * x * y * z;
  Y[11] = -SH31 * y * zz15;
  Y[12] = SH30 * fmaf(z, 5.f * zz, -3.f * z);
  Y[13] = -SH31 * x * zz15;
  Y[14] = SH32 * z * xxyy;
  Y[15] = -SH33 * fmaf(x, xx, -3.f * x * yy);
}
// The basis at direction d, made unit here.
__device__ __forceinline__ void sh_basis_of(float dx, float dy, float dz, int L, float* Y) {
#pragma clang fp contract(off)
  const float dn = rsqrtf(fmaf(dz, dz, fmaf(dy, dy, dx * dx)));
  sh_basis(dx * dn, dy * dn, dz * dn, L, Y);
}

// Sphere leaf: ray in the unit-sphere frame of instance record (r0, r1, r2).
struct SphereHit {
  float a, b, c2;  // v.v, u.v, |u x v|^2
};

__device__ __forceinline__ SphereHit sphere_terms(float4 r0, float4 r1, float4 r2, float ox, float oy, float oz,
                                                  float dx, float dy, float dz) {
#pragma clang fp contract(off)
  const float fx = ox - r0.w, fy = oy - r1.w, fz = oz - r2.w;
  auto dot = [](float ax, float ay, float az, float bx, float by, float bz) __attribute__((always_inline)) {
#pragma clang fp contract(off)
    return fmaf(az, bz, fmaf(ax, bx, ay * by));
  };
  const float ux = dot(r0.x, r0.y, r0.z, fx, fy, fz);
  const float uy = dot(r1.x, r1.y, r1.z, fx, fy, fz);
  const float uz = dot(r2.x, r2.y, r2.z, fx, fy, fz);
  const float vx = dot(r0.x, r0.y, r0.z, dx, dy, dz);
  const float vy = dot(r1.x, r1.y, r1.z, dx, dy, dz);
  const float vz = dot(r2.x, r2.y, r2.z, dx, dy, dz);
  const float cx = fmaf(uy, vz, -(uz * vy)), cy = fmaf(uz, vx, -(ux * vz)), cz = fmaf(ux, vy, -(uy * vx));
  SphereHit h;
  h.a = dot(vx, vy, vz, vx, vy, vz);
  h.b = dot(ux, uy, uz, vx, vy, vz);
  h.c2 = dot(cx, cy, cz, cx, cy, cz);
  return h;
}

// Distance at which the ray of `h` (one that meets the sphere) enters it.
__device__ __forceinline__ float sphere_entry(const SphereHit& h) {
#pragma clang fp contract(off)
  return (-h.b - __builtin_amdgcn_sqrtf(fmaxf(h.a - h.c2, 0.f))) * __builtin_amdgcn_rcpf(h.a);
}

// Eq. 2 at the point of maximum response: alpha, 1 - alpha, and minus its distance. Hardware
// reciprocal and exp2 (about 1 ulp each); the exponent lies in [-log2(o / alpha_min), 0], far
// from the denormal range a library exp2f guards.
struct HitAlpha {
  float alpha, rest, neg_t;
};
__device__ __forceinline__ HitAlpha hit_alpha(const SphereHit& h, float4 r3) {
#pragma clang fp contract(off)
  const float inva = __builtin_amdgcn_rcpf(h.a);
  const float e = __builtin_amdgcn_exp2f(-r3.y * (h.c2 * inva));
  HitAlpha q;
  q.alpha = r3.x * e;
  q.rest = fmaf(-r3.x, e, 1.f);
  q.neg_t = h.b * inva;
  return q;
}

// Colour of Gaussian `gid` for a ray with SH basis Y: 0.5 + sum Y sh per channel.
__device__ __forceinline__ void sh_colour(const float* __restrict__ sh, uint32_t gid, int degree, const float* Y,
                                          float c[3]) {
#pragma clang fp contract(off)
  c[0] = c[1] = c[2] = 0.5f;
  const int ncoef = (degree + 1) * (degree + 1);
  if (degree == 3) {
    // all twelve loads in flight at once, then the sums
    const float4* sp4 = reinterpret_cast<const float4*>(sh + (int64_t)gid * 48);
    float4 shv[12];
#pragma unroll
    for (int q = 0; q < 12; ++q) shv[q] = sp4[q];
#pragma unroll
    for (int q = 0; q < 12; ++q) {
      const float* vv = reinterpret_cast<const float*>(&shv[q]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int f = 4 * q + e;
        c[f % 3] = fmaf(Y[f / 3], vv[e], c[f % 3]);
      }
    }
  } else {
    const float* sc = sh + (int64_t)gid * 3 * ncoef;
#pragma unroll
    for (int f = 0; f < 16; ++f) {
      if (f < ncoef) {
        c[0] = fmaf(Y[f], sc[3 * f + 0], c[0]);
        c[1] = fmaf(Y[f], sc[3 * f + 1], c[1]);
        c[2] = fmaf(Y[f], sc[3 * f + 2], c[2]);
      }
    }
  }
}

}  // namespace
}  // namespace grtx
