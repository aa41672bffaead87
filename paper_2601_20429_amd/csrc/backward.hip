// Backward pass of the Gaussian ray tracer for gfx950.
//
// The forward image of a ray is front-to-back compositing (Eq. 1) of its blended hits,
// in blend order, with alpha at the point of maximum response (Eq. 2) and colour from
// SH at the ray direction:
//   C = sum_i T_i a_i c_i + T_N bg,   D = sum_i T_i a_i t_i,   O = 1 - T_N,
//   T_i = prod_{j<i} (1 - a_j).
// With S_i = sum_{j>i} T_j a_j c_j + T_N bg (everything behind hit i):
//   dC/dc_i = T_i a_i,  dC/da_i = T_i c_i - S_i / (1 - a_i),
//   dD/dt_i = T_i a_i,  dD/da_i = T_i t_i - (sum_{j>i} T_j a_j t_j) / (1 - a_i),
//   dO/da_i = T_N / (1 - a_i).
// The suffix sums come from the forward outputs (C, D, T_N) minus running prefix sums,
// so one pass in blend order suffices. Per hit, with M = S^-1 R^T, f = o - mu,
// u = M f, v = M d, t = -(u.v)/(v.v), p = u + t v (closest approach in the whitened
// frame), m2 = |p|^2 and a = opacity * exp(-m2/2):
//   dm2/du = 2p, dm2/dv = 2 t p, dt/du = -v/(v.v), dt/dv = -(u + 2 t v)/(v.v),
//   dL/dM = g_u f^T + g_v d^T, dL/dmu = -M^T g_u, dL/ds_i = -(1/s_i) sum_j g_M[i][j] M[i][j],
//   dL/dR[j][i] = g_M[i][j] / s_i, then through R(q/|q|) to q; dL/do = dL/da * a / o;
//   dL/dsh[l,m,ch] = dL/dc_ch * [c_ch > 0] * Y_lm(d).
// The sum over rays is done without atomics and in a fixed order, in three kernels. k_bwd_hits
// replays each ray and writes one 32-byte record per (ray, blended hit): dL/da, dL/dt and the
// colour factors dL/dc * T a [c > 0]; the records' positions are sorted by Gaussian (stable, so
// their order, fixed by rays and lists, is kept inside a Gaussian); k_bwd_sums walks the sorted records in equal shares,
// forms each record's gradients of mean, scale, rotation, opacity and SH (colour factor x
// Y(ray direction)), adds them up per Gaussian and, for a Gaussian whose records lie within the
// share, adds the totals to the caller's arrays; k_bwd_join adds up the Gaussians that reach
// over the end of a share. Results are deterministic.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "grtx_internal.h"

namespace grtx {
namespace {

constexpr int kBlock = 256;

constexpr double cx_sqrt(double x) {
  double r = x > 1.0 ? x : 1.0;
  for (int i = 0; i < 100; ++i) r = 0.5 * (r + x / r);
  return r;
}
constexpr double kPi = 3.14159265358979323846;
// K_l^m = sqrt((2l+1)/(4 pi) (l-m)!/(l+m)!)
constexpr double Klm(int l, double fac_ratio) { return cx_sqrt((2.0 * l + 1.0) / (4.0 * kPi) * fac_ratio); }
constexpr float B00 = (float)Klm(0, 1.0);
constexpr float B1 = (float)Klm(1, 1.0);
constexpr float B20 = (float)(Klm(2, 1.0) * 0.5);
constexpr float B21 = (float)(cx_sqrt(2.0) * Klm(2, 1.0 / 6.0) * 3.0);
constexpr float B22 = (float)(cx_sqrt(2.0) * Klm(2, 1.0 / 24.0) * 3.0);
constexpr float B30 = (float)(Klm(3, 1.0) * 0.5);
constexpr float B31 = (float)(cx_sqrt(2.0) * Klm(3, 1.0 / 12.0) * 0.5);
constexpr float B32 = (float)(cx_sqrt(2.0) * Klm(3, 1.0 / 120.0) * 15.0);
constexpr float B33 = (float)(cx_sqrt(2.0) * Klm(3, 1.0 / 720.0) * 15.0);

// Real SH basis (orthonormal, Condon-Shortley phase) as polynomials of the unit direction.
__device__ __forceinline__ void basis(float x, float y, float z, int L, float* Y) {
  Y[0] = B00;
  if (L < 1) return;
  Y[1] = -B1 * y;
  Y[2] = B1 * z;
  Y[3] = -B1 * x;
  if (L < 2) return;
  const float xx = x * x, yy = y * y, zz = z * z;
  Y[4] = B22 * 2.f * x * y;
  Y[5] = -B21 * y * z;
  Y[6] = B20 * (3.f * zz - 1.f);
  Y[7] = -B21 * x * z;
  Y[8] = B22 * (xx - yy);
  if (L < 3) return;
  Y[9] = -B33 * (3.f * xx * y - yy * y);
  Y[10] = B32 * 2.f * x * y * z;
  Y[11] = -B31 * y * (15.f * zz - 3.f);
  Y[12] = B30 * (5.f * zz * z - 3.f * z);
  Y[13] = -B31 * x * (15.f * zz - 3.f);
  Y[14] = B32 * z * (xx - yy);
  Y[15] = -B33 * (xx * x - 3.f * x * yy);
}

struct BwdArgs {
  const float* means;
  const float* scales;
  const float* quats;
  const float* opac;
  const float* sh;
  int sh_degree;
  const float* ray_o;
  const float* ray_d;
  int64_t n_rays;
  const float* rgb;
  const float* depth;
  const float* opacity;
  const int32_t* hit_ids;
  const int32_t* hit_counts;
  int hit_cap;
  const float* g_rgb;
  const float* g_depth;
  const float* g_opacity;
  int64_t n_gauss;
  float4* gauss;             // per Gaussian: 4 x float4
  const uint32_t* pair_off;  // per ray: records of the rays before it
  float4* rec;               // per (ray, hit): 2 x float4
  uint32_t* key;             // per record: Gaussian index (n_gauss: of no Gaussian)
};

// Record layout: (dL/da, dL/dt, gc.r, gc.g), (gc.b, ray index bits, G, t). The records of four
// neighbouring rays are interleaved by hit number: rays side by side meet a Gaussian at about
// the same one, and the sums below, which take the records by Gaussian, find some of them in
// one 128-byte line.

// Records per ray (the blended hits the forward pass listed, at most hit_cap).
__global__ void __launch_bounds__(kBlock) k_bwd_count(const int32_t* __restrict__ hit_counts, int64_t n, int cap,
                                                      uint32_t* __restrict__ cnt, unsigned int* truncated) {
  const int64_t r = blockIdx.x * (int64_t)kBlock + threadIdx.x;
  if (r >= n) return;
  int c = hit_counts[r];
  if (c > cap) {
    atomicAdd(truncated, 1u);
    c = cap;
  }
  cnt[r] = (uint32_t)(c < 0 ? 0 : c);
}

// What of a Gaussian does not depend on the ray, once for all its hits (13 divisions and a square
// root): M = S^-1 R^T by rows, mean, opacity.
struct Shape {
  float M[3][3], mu[3], opac;
};

__device__ __forceinline__ Shape load_shape(const float4* gauss, int64_t i) {
  const float4 a = gauss[4 * i], b = gauss[4 * i + 1], c = gauss[4 * i + 2], e = gauss[4 * i + 3];
  return Shape{{{a.x, a.y, a.z}, {a.w, b.x, b.y}, {b.z, b.w, c.x}}, {c.y, c.z, c.w}, e.x};
}

__global__ void __launch_bounds__(kBlock) k_bwd_shapes(BwdArgs A) {
  const int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x;
  if (i >= A.n_gauss) return;
  const float4 q4 = reinterpret_cast<const float4*>(A.quats)[i];
  const float qn = sqrtf(q4.x * q4.x + q4.y * q4.y + q4.z * q4.z + q4.w * q4.w);
  const float w = q4.x / qn, x = q4.y / qn, y = q4.z / qn, z = q4.w / qn;
  float R[3][3];
  R[0][0] = 1.f - 2.f * (y * y + z * z); R[0][1] = 2.f * (x * y - w * z);       R[0][2] = 2.f * (x * z + w * y);
  R[1][0] = 2.f * (x * y + w * z);       R[1][1] = 1.f - 2.f * (x * x + z * z); R[1][2] = 2.f * (y * z - w * x);
  R[2][0] = 2.f * (x * z - w * y);       R[2][1] = 2.f * (y * z + w * x);       R[2][2] = 1.f - 2.f * (x * x + y * y);
  float M[9];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float s = A.scales[3 * i + a];
#pragma unroll
    for (int b = 0; b < 3; ++b) M[3 * a + b] = R[b][a] / s;
  }
  A.gauss[4 * i] = make_float4(M[0], M[1], M[2], M[3]);
  A.gauss[4 * i + 1] = make_float4(M[4], M[5], M[6], M[7]);
  A.gauss[4 * i + 2] = make_float4(M[8], A.means[3 * i], A.means[3 * i + 1], A.means[3 * i + 2]);
  A.gauss[4 * i + 3] = make_float4(A.opac[i], 0.f, 0.f, 0.f);
}

// A hit's geometry: f = o - mu, u = M f, v = M d and v.v.
struct Geom {
  float f[3], u[3], v[3], vv;
};

__device__ __forceinline__ Geom geometry(const Shape& g, const float* o, const float* d) {
  Geom h;
#pragma unroll
  for (int a = 0; a < 3; ++a) h.f[a] = o[a] - g.mu[a];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    h.u[a] = g.M[a][0] * h.f[0] + g.M[a][1] * h.f[1] + g.M[a][2] * h.f[2];
    h.v[a] = g.M[a][0] * d[0] + g.M[a][1] * d[1] + g.M[a][2] * d[2];
  }
  h.vv = h.v[0] * h.v[0] + h.v[1] * h.v[1] + h.v[2] * h.v[2];
  return h;
}

// Lane J of the row of 16, for all its lanes.
template <int J>
__device__ __forceinline__ float row_lane(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + J, 0xF, 0xF, true));
}

// The compositing of up to 16 hits, one per lane of the row, in their order: a lane runs the
// ray's sums up to its own hit (T before it, C and D with it).
struct Sums {
  float T, C[3], D;
};
template <int J>
__device__ __forceinline__ void replay(int sub, int most, float alpha, float rest, const float* c, float t, Sums& s) {
  if constexpr (J < 16) {
    if (J % 4 == 0 && J >= most) return;  // (no row of the wave has a hit there)
    const float a = row_lane<J>(alpha), rest_j = row_lane<J>(rest), t_j = row_lane<J>(t);
    const float c0 = row_lane<J>(c[0]), c1 = row_lane<J>(c[1]), c2 = row_lane<J>(c[2]);
    if (sub >= J) {
      const float w = s.T * a;
      s.C[0] += w * c0;
      s.C[1] += w * c1;
      s.C[2] += w * c2;
      s.D += w * t_j;
      if (sub > J) s.T *= rest_j;
    }
    replay<J + 1>(sub, most, alpha, rest, c, t, s);
  }
}

// Replays the rays: sixteen lanes per ray, a hit per lane. Bound by cache accesses (16 a hit, for
// its shape and SH) and issue; a lane per ray, hit after hit, has the longest ray set the end.
// 10.7M hits of 262144 rays, degree 3: 1266 us by lane, 369 us so. (Quads that read each hit's SH
// by whole lines: 316 us, but then the colour's terms add up in another order, and a
// gradient of scale, where terms a thousand times larger cancel, moves by up to 0.3% of its rms.)
// For the same reason the sums along the ray stay in hit order, the suffix C - sum cancelling
// against the forward's, and 1 - alpha and dL/dM are written out as fused operations.
constexpr int kLanes = 16;
__global__ void __launch_bounds__(kBlock) k_bwd_hits(BwdArgs A) {
  const int64_t r0 = (blockIdx.x * (int64_t)kBlock + threadIdx.x) / kLanes;
  const int sub = threadIdx.x & (kLanes - 1);
  const int64_t r = min(r0, A.n_rays - 1);
  int n = A.hit_counts[r];
  n = r0 >= A.n_rays ? 0 : n > A.hit_cap ? A.hit_cap : n;
  if (!__any(n > 0)) return;
  const float o[3] = {A.ray_o[3 * r], A.ray_o[3 * r + 1], A.ray_o[3 * r + 2]};
  const float d[3] = {A.ray_d[3 * r], A.ray_d[3 * r + 1], A.ray_d[3 * r + 2]};
  n = max(n, 0);
  int nr[4];  // the hits of the wave's rays
#pragma unroll
  for (int k = 0; k < 4; ++k) nr[k] = __builtin_amdgcn_readlane(n, 16 * k);
  const int row = (threadIdx.x & 63) / kLanes;
  const uint32_t base = __builtin_amdgcn_readfirstlane(A.pair_off[r]);  // of the wave's first ray
  const float TN = 1.f - A.opacity[r];
  float Cf[3], gC[3];
#pragma unroll
  for (int ch = 0; ch < 3; ++ch) {
    Cf[ch] = A.rgb[3 * r + ch];  // includes T_N * bg
    gC[ch] = A.g_rgb ? A.g_rgb[3 * r + ch] : 0.f;
  }
  const float Df = A.depth[r];
  const float gD = A.g_depth ? A.g_depth[r] : 0.f;
  const float gO = A.g_opacity ? A.g_opacity[r] : 0.f;
  const float dn = rsqrtf(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
  float Y[16];
  basis(d[0] * dn, d[1] * dn, d[2] * dn, A.sh_degree, Y);
  const int ncoef = (A.sh_degree + 1) * (A.sh_degree + 1);
  const int32_t* ids = A.hit_ids + r * A.hit_cap;

  Sums run = {1.f, {0.f, 0.f, 0.f}, 0.f};
  int32_t ahead = sub < n ? ids[sub] : -1;
  for (int h0 = 0; __any(h0 < n); h0 += kLanes) {
    const int h = h0 + sub;
    const int32_t id = ahead;
    ahead = h + kLanes < n ? ids[h + kLanes] : -1;
    const bool hit = h < n && id >= 0 && id < A.n_gauss;
    float alpha = 0.f, rest = 1.f, G = 0.f, ta = 0.f, c[3] = {0.f, 0.f, 0.f};
    bool pos[3] = {false, false, false};
    if (hit) {
      const int64_t i = id;
      const Shape shape = load_shape(A.gauss, i);
      float acc[3] = {0.5f, 0.5f, 0.5f};
      if (A.sh_degree == 3) {
        // the 48 coefficients as twelve 16-B loads
        const float4* sp4 = reinterpret_cast<const float4*>(A.sh + i * 48);
        float4 shv[12];
#pragma unroll
        for (int q = 0; q < 12; ++q) shv[q] = sp4[q];
#pragma unroll
        for (int q = 0; q < 12; ++q) {
          const float e[4] = {shv[q].x, shv[q].y, shv[q].z, shv[q].w};
#pragma unroll
          for (int k = 0; k < 4; ++k) acc[(4 * q + k) % 3] += Y[(4 * q + k) / 3] * e[k];
        }
      } else {
        const float* shp = A.sh + i * 3 * ncoef;
#pragma unroll
        for (int k = 0; k < 9; ++k)
          if (k < ncoef)
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) acc[ch] += Y[k] * shp[3 * k + ch];
      }
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) {
        pos[ch] = acc[ch] > 0.f;
        c[ch] = pos[ch] ? acc[ch] : 0.f;
      }
      const Geom g = geometry(shape, o, d);
      ta = -(g.u[0] * g.v[0] + g.u[1] * g.v[1] + g.u[2] * g.v[2]) / g.vv;
      const float p[3] = {g.u[0] + ta * g.v[0], g.u[1] + ta * g.v[1], g.u[2] + ta * g.v[2]};
      G = expf(-0.5f * (p[0] * p[0] + p[1] * p[1] + p[2] * p[2]));
      alpha = shape.opac * G;
      rest = fmaf(-shape.opac, G, 1.f);  // 1 - alpha, from the product before it is rounded
    }
    const int most = max(max(nr[0], nr[1]), max(nr[2], nr[3])) - h0;  // hits of the fullest row here
    Sums own = run;
    replay<0>(sub, most, alpha, rest, c, ta, own);
    // the ray's sums so far, for its next 16 hits: those of its last lane
    run.T = row_lane<15>(own.T * rest);
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) run.C[ch] = row_lane<15>(own.C[ch]);
    run.D = row_lane<15>(own.D);
    if (h < n) {
      // ---- compositing derivatives
      const float wgt = own.T * alpha;
      const float inv1ma = 1.f / rest;
      float gA = 0.f;
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) {
        const float behind = Cf[ch] - own.C[ch];  // S_i (includes T_N bg)
        gA += gC[ch] * (own.T * c[ch] - behind * inv1ma);
      }
      gA += gD * (own.T * ta - (Df - own.D) * inv1ma);
      gA += gO * (TN * inv1ma);
      uint32_t pi = base;
#pragma unroll
      for (int k = 0; k < 4; ++k) pi += (uint32_t)(min(nr[k], h) + (k < row && nr[k] > h ? 1 : 0));
      float4* rp = A.rec + 2 * (int64_t)pi;
      rp[0] = make_float4(gA, gD * wgt, pos[0] ? gC[0] * wgt : 0.f, pos[1] ? gC[1] * wgt : 0.f);
      rp[1] = make_float4(pos[2] ? gC[2] * wgt : 0.f, __uint_as_float((uint32_t)r), G, ta);
      A.key[pi] = hit ? (uint32_t)id : (uint32_t)A.n_gauss;  // not a Gaussian of this scene: sorted last
    }
  }
}

// Total number of records: the last ray's offset plus its count.
__global__ void k_bwd_total(const uint32_t* __restrict__ off, const uint32_t* __restrict__ cnt, int64_t R,
                            uint32_t* __restrict__ total) {
  if (threadIdx.x == 0) *total = off[R - 1] + cnt[R - 1];
}

// The sorted records in kShares equal shares of whole tiles of 64, a wave for each: an even
// split however the records lie among the Gaussians (from none to a hundred thousand each).
constexpr int kShares = 4096;
__device__ __forceinline__ int64_t share_size(int64_t P) {
  return max((int64_t)64, (P + (int64_t)kShares * 64 - 1) / ((int64_t)kShares * 64) * 64);
}

struct SumArgs {
  BwdArgs in;
  const uint32_t* key;    // sorted
  const uint32_t* order;  // sorted position -> record
  const uint32_t* total;
  float* part;  // [kShares][2][64]: sums of the Gaussian that a share begins inside of, and of
                // the one that it ends inside of
  float* d_means;
  float* d_scales;
  float* d_quats;
  float* d_opac;
  float* d_sh;
};

// A record's row in LDS (an odd stride: no bank conflicts): g_u, dL/dM, the sums of dL/dM M per
// axis and dL/do, which add up to the gradients of mean, rotation, scale and opacity (the rest is
// linear and the same for all records of a Gaussian), three colour factors, the basis at its ray
// and a one.
constexpr int kTotals = 16;
constexpr int kRow = kTotals + 3 + 16 + 2;
__device__ __forceinline__ void record_row(const BwdArgs& A, uint32_t id, uint32_t rec, float* row) {
  const float4 a = A.rec[2 * (int64_t)rec], b = A.rec[2 * (int64_t)rec + 1];
  const Shape shape = load_shape(A.gauss, id);
  const float gA = a.x, gT = a.y, G = b.z, ta = b.w;
  const int64_t r = __float_as_uint(b.y);
  const float o[3] = {A.ray_o[3 * r], A.ray_o[3 * r + 1], A.ray_o[3 * r + 2]};
  const float d[3] = {A.ray_d[3 * r], A.ray_d[3 * r + 1], A.ray_d[3 * r + 2]};
  const Geom g = geometry(shape, o, d);
  // ---- alpha -> opacity, m2, t
  const float gm2 = gA * (-0.5f * (shape.opac * G));
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float p = g.u[k] + ta * g.v[k];
    const float gu = gm2 * 2.f * p - gT * g.v[k] / g.vv;
    const float gv = gm2 * 2.f * ta * p - gT * (g.u[k] + 2.f * ta * g.v[k]) / g.vv;
    // ---- u = M f, v = M d
    row[k] = gu;
    float gs = 0.f;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const float gM = fmaf(gu, g.f[j], gv * d[j]);
      row[3 + 3 * k + j] = gM;
      gs += gM * shape.M[k][j];
    }
    row[12 + k] = gs;
  }
  row[15] = gA * G;
  // ---- SH: dL/dsh = colour factor x Y
  row[kTotals] = a.z;
  row[kTotals + 1] = a.w;
  row[kTotals + 2] = b.x;
  const float dn = rsqrtf(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
  float Y[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) Y[k] = 0.f;
  basis(d[0] * dn, d[1] * dn, d[2] * dn, A.sh_degree, Y);
#pragma unroll
  for (int k = 0; k < 16; ++k) row[kTotals + 3 + k] = Y[k];
  row[kRow - 2] = 1.f;
}

// From a Gaussian's totals to its gradients.
__device__ __forceinline__ void add_shape(const SumArgs& A, int64_t i, const float* total) {
  const Shape shape = load_shape(A.in.gauss, i);
  const float4 q4 = reinterpret_cast<const float4*>(A.in.quats)[i];
  const float qn = sqrtf(q4.x * q4.x + q4.y * q4.y + q4.z * q4.z + q4.w * q4.w);
  const float w = q4.x / qn, x = q4.y / qn, y = q4.z / qn, z = q4.w / qn;
  float gR[3][3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    A.d_means[3 * i + k] += -(shape.M[0][k] * total[0] + shape.M[1][k] * total[1] + shape.M[2][k] * total[2]);
    const float s = A.in.scales[3 * i + k];
#pragma unroll
    for (int j = 0; j < 3; ++j) gR[j][k] = total[3 + 3 * k + j] / s;
    A.d_scales[3 * i + k] += -total[12 + k] / s;
  }
  // ---- R(qhat) -> qhat -> q
  const float gw = 2.f * (-z * gR[0][1] + y * gR[0][2] + z * gR[1][0] - x * gR[1][2] - y * gR[2][0] + x * gR[2][1]);
  const float gx = 2.f * (y * gR[0][1] + z * gR[0][2] + y * gR[1][0] - 2.f * x * gR[1][1] - w * gR[1][2] +
                          z * gR[2][0] + w * gR[2][1] - 2.f * x * gR[2][2]);
  const float gy = 2.f * (-2.f * y * gR[0][0] + x * gR[0][1] + w * gR[0][2] + x * gR[1][0] + z * gR[1][2] -
                          w * gR[2][0] + z * gR[2][1] - 2.f * y * gR[2][2]);
  const float gz = 2.f * (-2.f * z * gR[0][0] - w * gR[0][1] + x * gR[0][2] + w * gR[1][0] - 2.f * z * gR[1][1] +
                          y * gR[1][2] + x * gR[2][0] + y * gR[2][1]);
  const float dot = w * gw + x * gx + y * gy + z * gz;
  A.d_quats[4 * i] += (gw - w * dot) / qn;
  A.d_quats[4 * i + 1] += (gx - x * dot) / qn;
  A.d_quats[4 * i + 2] += (gy - y * dot) / qn;
  A.d_quats[4 * i + 3] += (gz - z * dot) / qn;
  A.d_opac[i] += total[15];
}

// One share of the sorted records, 64 at a time: a lane turns one into its row, then every lane
// adds up one of the 64 totals over the rows, four partial sums at a time, and passes it on when
// the Gaussian changes: SH at once, 48 neighbouring floats, the others by a lane per Gaussian,
// kWaiting of them at a time. Two LDS reads and one fma per record for all 64 (a wave per
// Gaussian that ended in 59 sums over its lanes spent its time on those: 354 shuffles for some
// 30 records): 611 us for 10.7M hits, 243 us so, bound by the records' lines (128 bytes
// fetched for 32).
constexpr int kWaiting = 8;
__global__ void __launch_bounds__(64) k_bwd_sums(SumArgs A) {
  __shared__ float s_row[64 * kRow];
  __shared__ float s_total[kWaiting][kTotals];
  __shared__ uint32_t s_id[kWaiting];
  const int lane = threadIdx.x;
  const int64_t P = *A.total;
  const int64_t size = share_size(P);
  const int64_t begin = blockIdx.x * size;
  const int64_t end = min(P, begin + size);
  if (begin >= end) return;
  const uint32_t none = (uint32_t)A.in.n_gauss;
  const int nsh = 3 * (A.in.sh_degree + 1) * (A.in.sh_degree + 1);
  const int ia = lane < 48 ? kTotals + lane % 3 : lane < 48 + kTotals ? lane - 48 : 0;
  const int ib = lane < 48 ? kTotals + 3 + lane / 3 : kRow - 2;
  uint32_t cur = A.key[begin];
  bool inside = begin > 0 && A.key[begin - 1] == cur;  // its first records are another share's
  float sum[4] = {0.f, 0.f, 0.f, 0.f};
  int waiting = 0;
  float sh = lane < nsh && cur < none ? A.d_sh[(int64_t)cur * nsh + lane] : 0.f;  // read ahead
  auto finish = [&]() {
    __syncthreads();
    if (lane < waiting) add_shape(A, s_id[lane], s_total[lane]);
    __syncthreads();
    waiting = 0;
  };
  auto pass_on = [&](bool goes_on) {
    const float all = (sum[0] + sum[1]) + (sum[2] + sum[3]);
    if (inside || goes_on) {
      A.part[(int64_t)blockIdx.x * 128 + (inside ? 0 : 64) + lane] = all;
    } else if (cur < none) {
      if (lane < nsh)
        A.d_sh[(int64_t)cur * nsh + lane] = sh + all;
      if (lane >= 48 && lane < 48 + kTotals) s_total[waiting][lane - 48] = all;
      if (lane == 0) s_id[waiting] = cur;
      if (++waiting == kWaiting) finish();
    }
  };
  uint32_t k_ahead = A.key[min(begin + lane, end - 1)], p_ahead = A.order[min(begin + lane, end - 1)];
  for (int64_t t = begin; t < end; t += 64) {
    const uint32_t k = k_ahead, rec = p_ahead;
    const int64_t next = min(t + 64 + lane, end - 1);
    k_ahead = A.key[next];
    p_ahead = A.order[next];
    const int n = (int)min((int64_t)64, end - t);
    if (lane < n && k < none) record_row(A.in, k, rec, s_row + lane * kRow);
    const uint32_t before = __shfl_up(k, 1);
    const uint64_t starts = __ballot(lane < n && k != (lane == 0 ? cur : before));
    __syncthreads();
    for (int j = 0; j < n;) {
      if ((starts >> j) & 1) {
        pass_on(false);
        inside = false;
        sum[0] = sum[1] = sum[2] = sum[3] = 0.f;
        cur = __builtin_amdgcn_readlane(k, j);
        sh = lane < nsh && cur < none ? A.d_sh[(int64_t)cur * nsh + lane] : 0.f;
      }
      const uint64_t rest = j == 63 ? 0 : starts >> (j + 1);
      const int stop = rest ? min(n, j + 1 + __builtin_ctzll(rest)) : n;
      if (cur >= none) {
        j = stop;
        continue;
      }
      for (; j + 4 <= stop; j += 4) {
#pragma unroll
        for (int q = 0; q < 4; ++q) sum[q] += s_row[(j + q) * kRow + ia] * s_row[(j + q) * kRow + ib];
      }
      if (j < stop) sum[0] += s_row[j * kRow + ia] * s_row[j * kRow + ib];
      if (j + 1 < stop) sum[1] += s_row[(j + 1) * kRow + ia] * s_row[(j + 1) * kRow + ib];
      if (j + 2 < stop) sum[2] += s_row[(j + 2) * kRow + ia] * s_row[(j + 2) * kRow + ib];
      j = stop;
    }
    __syncthreads();
  }
  pass_on(end < P && A.key[end] == cur);
  finish();
}

// The Gaussians whose records reach over the end of a share: the share in which one begins adds
// up its own part and those of the shares that follow.
__global__ void __launch_bounds__(64) k_bwd_join(SumArgs A) {
  __shared__ float s_total[kTotals];
  const int lane = threadIdx.x;
  const int64_t P = *A.total;
  const int64_t size = share_size(P);
  const int64_t begin = blockIdx.x * size;
  const int64_t end = begin + size;
  if (end >= P) return;
  const uint32_t cur = A.key[end];
  if (cur >= (uint32_t)A.in.n_gauss || A.key[end - 1] != cur) return;
  if (begin > 0 && A.key[begin - 1] == cur) return;  // it began in an earlier share
  float all = A.part[(int64_t)blockIdx.x * 128 + 64 + lane];
  for (int64_t c = blockIdx.x + 1; c * size < P; c += 64) {
    // how many of the next 64 shares begin inside of it
    const int64_t at = (c + lane) * size;
    const uint64_t in = __ballot(at < P && A.key[min(at, P - 1)] == cur);
    const int n = in == ~0ull ? 64 : __builtin_ctzll(~in);
#pragma unroll 8
    for (int j = 0; j < n; ++j) all += A.part[(c + j) * 128 + lane];
    if (n < 64) break;
  }
  const int nsh = 3 * (A.in.sh_degree + 1) * (A.in.sh_degree + 1);
  if (lane < nsh) A.d_sh[(int64_t)cur * nsh + lane] += all;
  if (lane >= 48 && lane < 48 + kTotals) s_total[lane - 48] = all;
  __syncthreads();
  if (lane == 0) add_shape(A, cur, s_total);
}

__global__ void k_zero_u32(unsigned int* p) { *p = 0u; }

inline unsigned grid(int64_t n, int per = kBlock) { return (unsigned)std::max<int64_t>(1, (n + per - 1) / per); }


}  // namespace

// Hit-list capacity of the re-trace when the forward outputs carry no list.
constexpr int kRetraceCap = 256;

grtx_status trace_backward(const Bvh* bvh, const grtx_gaussians* g, const grtx_rays* r, const grtx_trace_params* p,
                           const grtx_trace_outputs* fwd, const float* grad_rgb, const float* grad_depth,
                           const float* grad_opacity, const grtx_gaussian_grads* grads, unsigned int* truncated,
                           hipStream_t s) {
  const int64_t R = r->count;
  const int64_t N = g->count;
  hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(1), 0, s, truncated);
  GRTX_LAUNCH_CHECK();
  if (R == 0 || N == 0) return GRTX_OK;
  const bool retrace = fwd->hit_ids == nullptr;
  const int cap = !retrace ? fwd->hit_capacity : (fwd->hit_capacity > 0 ? fwd->hit_capacity : kRetraceCap);
  // every record of the pass lives in scratch sized for the bound rays x cap, so that the
  // host never waits for the actual number (which stays on the device)
  const int64_t Pmax = R * (int64_t)cap;
  if (Pmax >= ((int64_t)1 << 32) - 1) {
    set_error("trace_backward: %lld rays x %d listed hits exceed 2^32 records", (long long)R, cap);
    return GRTX_ERR_INVALID_ARG;
  }
  Scratch sc(s);
  grtx_trace_outputs fo = *fwd;
  if (retrace) {
    // the blended ids are not given: trace again with a list (the trace is deterministic,
    // so its outputs equal the forward's)
    float* outs = nullptr;
    GRTX_TRY(sc.get(&outs, 5 * R));
    GRTX_TRY(sc.get(&fo.hit_ids, Pmax));
    GRTX_TRY(sc.get(&fo.hit_counts, R));
    fo.rgb = outs;
    fo.depth = outs + 3 * R;
    fo.opacity = outs + 4 * R;
    fo.stats = nullptr;
    fo.hit_capacity = cap;
    GRTX_TRY(trace(bvh, r, p, &fo, s));
  }
  // 1. records per ray, their offsets and the total (on the device)
  uint32_t *cnt = nullptr, *off = nullptr, *total = nullptr;
  GRTX_TRY(sc.get(&cnt, R));
  GRTX_TRY(sc.get(&off, R));
  GRTX_TRY(sc.get(&total, 1));
  hipLaunchKernelGGL(k_bwd_count, dim3(grid(R)), dim3(kBlock), 0, s, fo.hit_counts, R, cap, cnt, truncated);
  GRTX_LAUNCH_CHECK();
  GRTX_TRY(exclusive_scan_u32(cnt, off, R, s));
  hipLaunchKernelGGL(k_bwd_total, dim3(1), dim3(64), 0, s, off, cnt, R, total);
  // 2. one record per (ray, blended hit)
  BwdArgs a{};
  a.means = g->means;
  a.scales = g->scales;
  a.quats = g->quats;
  a.opac = g->opacities;
  a.sh = g->sh;
  a.sh_degree = g->sh_degree;
  a.ray_o = r->origins;
  a.ray_d = r->dirs;
  a.n_rays = R;
  a.rgb = fo.rgb;
  a.depth = fo.depth;
  a.opacity = fo.opacity;
  a.hit_ids = fo.hit_ids;
  a.hit_counts = fo.hit_counts;
  a.hit_cap = cap;
  a.g_rgb = grad_rgb;
  a.g_depth = grad_depth;
  a.g_opacity = grad_opacity;
  a.n_gauss = N;
  a.pair_off = off;
  GRTX_TRY(sc.get(&a.gauss, 4 * N));
  hipLaunchKernelGGL(k_bwd_shapes, dim3(grid(N)), dim3(kBlock), 0, s, a);
  GRTX_TRY(sc.get(&a.rec, 2 * Pmax));
  GRTX_TRY(sc.get(&a.key, Pmax));
  hipLaunchKernelGGL(k_bwd_hits, dim3(grid(R * kLanes)), dim3(kBlock), 0, s, a);
  GRTX_LAUNCH_CHECK();
  // 3. group by Gaussian, keeping the records' order inside a Gaussian
  int bits = 1;  // keys are 0..N (N marks a record of no Gaussian)
  while (bits < 32 && ((int64_t)1 << bits) <= N) ++bits;
  uint32_t *vals = nullptr, *tkeys = nullptr, *tvals = nullptr, *skey = nullptr, *sval = nullptr;
  GRTX_TRY(sc.get(&vals, Pmax));
  GRTX_TRY(sc.get(&tkeys, Pmax));
  GRTX_TRY(sc.get(&tvals, Pmax));
  GRTX_TRY(sort_positions(a.key, vals, tkeys, tvals, Pmax, bits, s, total, &skey, &sval));
  // 4. per-Gaussian sums
  SumArgs sa{};
  sa.in = a;
  sa.key = skey;
  sa.order = sval;
  sa.total = total;
  GRTX_TRY(sc.get(&sa.part, (size_t)kShares * 2 * 64));
  sa.d_means = grads->means;
  sa.d_scales = grads->scales;
  sa.d_quats = grads->quats;
  sa.d_opac = grads->opacities;
  sa.d_sh = grads->sh;
  hipLaunchKernelGGL(k_bwd_sums, dim3(kShares), dim3(64), 0, s, sa);
  hipLaunchKernelGGL(k_bwd_join, dim3(kShares), dim3(64), 0, s, sa);
  GRTX_LAUNCH_CHECK();
  return GRTX_OK;
}

}  // namespace grtx
