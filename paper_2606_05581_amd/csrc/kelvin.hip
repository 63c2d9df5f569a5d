// The exterior estimate in the Kelvin-inverted domain (Sec. 3.3, The Kelvin
// Transform; eqs. exterior-jump-kernel-final, killing-measure-poisson-kernel,
// main-exterior-estimator; Sec. 4, spherical triangular elements).
//
// Coordinates are relative to an inversion centre inside the shape. The map
// x -> x / |x|^2 sends the unbounded exterior to a bounded domain whose
// boundary is the image of the mesh: each planar triangle becomes a piece of
// a sphere through the origin (or of the plane itself when it passes through
// the centre), bounded by three circular arcs, the images of its edges. Walks
// in that domain always end, so Walk-on-Spheres applies with the exact
// distance to these curved elements. Everything here is FP64: element
// spheres of triangles whose planes pass near the centre have huge radii,
// and the distance is written stably in that limit.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>

#include "msk_internal.h"
#include "kelvin.h"
#include "philox.h"
#include "search.h"

// wavefronts per SIMD the persistent walk kernel is compiled for
#ifndef MSK_KELVIN_WAVES_PER_EU
#define MSK_KELVIN_WAVES_PER_EU 4
#endif
namespace msk {

namespace {

// The element distance is evaluated exactly as written, with no fused
// multiply-adds, in these helpers as in the functions that use them: the
// result then does not depend on how the compiler inlines them.
__host__ __device__ __forceinline__ double dot(const double a[3], const double b[3]) {
#pragma clang fp contract(off)
  return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}

__host__ __device__ __forceinline__ void invert(const double x[3], double y[3]) {
#pragma clang fp contract(off)
  const double s = 1.0 / dot(x, x);
  y[0] = x[0] * s; y[1] = x[1] * s; y[2] = x[2] * s;
}

__host__ __device__ __forceinline__ void cross(const double u[3], const double v[3], double o[3]) {
#pragma clang fp contract(off)
  o[0] = u[1] * v[2] - u[2] * v[1];
  o[1] = u[2] * v[0] - u[0] * v[2];
  o[2] = u[0] * v[1] - u[1] * v[0];
}

// Offer a candidate point q at squared distance d2 with barycentrics l.
struct Best {
  double d2;
  double q[3];
  double l[3];
};
__host__ __device__ __forceinline__ void offer(Best& b, double d2, const double q[3], double l0, double l1, double l2) {
  if (d2 < b.d2) {
    b.d2 = d2;
    b.q[0] = q[0]; b.q[1] = q[1]; b.q[2] = q[2];
    b.l[0] = l0; b.l[1] = l1; b.l[2] = l2;
  }
}

// The image of the edge [P, Q] (primal, relative to the centre): end points,
// and the nearest point of the arc. The line through P and Q, at foot point f
// from the centre, maps to the circle through the origin in the plane of
// (0, P, Q) with centre f / (2 |f|^2) and radius 1 / (2 |f|); the circle
// point nearest to x is the radial projection of x's in-plane position, and
// it lies on the edge's arc when its image is between P and Q. A line
// through the centre maps to itself: the arc is then the straight segment
// between the end points' images. Everything that does not depend on x is
// computed once per inverted mesh (edge_prepare, kelvin_prepare_kernel);
// edge_eval does the rest, with the same operations in the same order as
// one function evaluating both would. (ia, ib) are the edge's vertex slots.
__host__ __device__ void edge_prepare(const double P[3], const double Q[3], KelvinEdge& E) {
#pragma clang fp contract(off)
  double kp[3], kq[3];
  invert(P, kp);
  invert(Q, kq);
  for (int k = 0; k < 3; ++k) E.e[k] = Q[k] - P[k];
  E.ee = dot(E.e, E.e);
  E.kind = 0;
  E.pad = 0;
  for (int k = 0; k < 3; ++k) E.m[k] = E.c[k] = 0.0;
  E.rho = 0.0;
  E.pqmax = fmax(dot(P, P), dot(Q, Q));
  if (!(E.ee > 0.0)) return;
  const double tf = -dot(P, E.e) / E.ee;
  const double f[3] = {P[0] + tf * E.e[0], P[1] + tf * E.e[1], P[2] + tf * E.e[2]};
  const double ff = dot(f, f);
  double m[3];
  cross(P, Q, m);
  const double mm = dot(m, m);
  if (ff > 1e-24 * E.pqmax && mm > 0.0) {
    E.kind = 1;
    const double ml = 1.0 / sqrt(mm);
    for (int k = 0; k < 3; ++k) E.m[k] = m[k] * ml;
    for (int k = 0; k < 3; ++k) E.c[k] = f[k] / (2.0 * ff);
    E.rho = 1.0 / (2.0 * sqrt(ff));
  } else {
    E.kind = 2;
    for (int k = 0; k < 3; ++k) E.m[k] = kq[k] - kp[k];  // the segment's direction g
    E.rho = dot(E.m, E.m);                               // |g|^2
  }
}

// FP64 operations are counted (kCount) as additions, multiplications,
// divisions and square roots, one each, up to each exit: dot 5, inversion 9.
template <bool kCount>
__host__ __device__ void edge_eval(const double x[3], const double P[3], const double kp[3], const double kq[3],
                                   const KelvinEdge& E, int ia, int ib, Best& b, uint64_t& ops) {
#pragma clang fp contract(off)
  double d[3];
  double l[3] = {0.0, 0.0, 0.0};
  for (int k = 0; k < 3; ++k) d[k] = x[k] - kp[k];
  l[ia] = 1.0;
  offer(b, dot(d, d), kp, l[0], l[1], l[2]);
  for (int k = 0; k < 3; ++k) d[k] = x[k] - kq[k];
  l[ia] = 0.0; l[ib] = 1.0;
  offer(b, dot(d, d), kq, l[0], l[1], l[2]);
  if constexpr (kCount) ops += 16;
  if (E.kind == 0) return;
  if (E.kind == 1) {
    const double* m = E.m;
    const double* c = E.c;
    const double mx = dot(m, x);
    const double u[3] = {x[0] - mx * m[0] - c[0], x[1] - mx * m[1] - c[1], x[2] - mx * m[2] - c[2]};
    const double ul = sqrt(dot(u, u));
    if constexpr (kCount) ops += 20;
    if (!(ul > 0.0)) return;
    const double pt[3] = {c[0] + E.rho * u[0] / ul, c[1] + E.rho * u[1] / ul, c[2] + E.rho * u[2] / ul};
    // the origin is the image of the line's point at infinity: every point of
    // the segment's image lies at least 1 / max(|P|, |Q|) from it
    if constexpr (kCount) ops += 15;
    if (!(dot(pt, pt) * E.pqmax >= 1.0 - 1e-9)) return;
    double y[3];
    invert(pt, y);
    const double yd[3] = {y[0] - P[0], y[1] - P[1], y[2] - P[2]};
    const double t = dot(yd, E.e) / E.ee;
    if constexpr (kCount) ops += 18;
    if (t >= 0.0 && t <= 1.0) {
      if constexpr (kCount) ops += 9;
      for (int k = 0; k < 3; ++k) d[k] = x[k] - pt[k];
      l[ia] = 1.0 - t; l[ib] = t;
      offer(b, dot(d, d), pt, l[0], l[1], l[2]);
    }
  } else {
    const double* g = E.m;
    const double gg = E.rho;
    double s = gg > 0.0 ? ((x[0] - kp[0]) * g[0] + (x[1] - kp[1]) * g[1] + (x[2] - kp[2]) * g[2]) / gg : 0.0;
    s = fmin(1.0, fmax(0.0, s));
    const double pt[3] = {kp[0] + s * g[0], kp[1] + s * g[1], kp[2] + s * g[2]};
    double y[3];
    invert(pt, y);
    const double yd[3] = {y[0] - P[0], y[1] - P[1], y[2] - P[2]};
    const double t = dot(yd, E.e) / E.ee;
    for (int k = 0; k < 3; ++k) d[k] = x[k] - pt[k];
    l[ia] = 1.0 - t; l[ib] = t;
    offer(b, dot(d, d), pt, l[0], l[1], l[2]);
    if constexpr (kCount) ops += 42;
  }
}

}  // namespace

// The plane of triangle (a, b, c) as used by the distance below: unit normal
// n and offset cpl = n . a, or false for a (numerically) degenerate triangle.
__host__ __device__ bool kelvin_plane(const double a[3], const double b[3], const double c[3], double n[3],
                                      double& cpl) {
#pragma clang fp contract(off)
  double ab[3], ac[3];
  for (int k = 0; k < 3; ++k) {
    ab[k] = b[k] - a[k];
    ac[k] = c[k] - a[k];
  }
  cross(ab, ac, n);
  const double nl = sqrt(dot(n, n));
  if (!(nl > 1e-12 * fmax(dot(ab, ab), dot(ac, ac)))) return false;
  for (int k = 0; k < 3; ++k) n[k] /= nl;
  cpl = dot(n, a);
  return true;
}

// Squared distance from x to the image of triangle T, its nearest point and
// the barycentrics of that point's image in T. The triangle's plane
// n . y = c maps to the sphere through the origin with centre n / (2c) and
// radius 1 / (2|c|); with v = c x - n/2 the signed distance of x to it is
// (|c| |x|^2 - sign(c) n . x) / (|v| + 1/2) and the radial projection moves x
// by that distance along sign(c) v / |v|, which tends to the plane's own
// projection as c -> 0. The projection belongs to the patch when its image
// lies in T; otherwise the nearest point is on the patch's boundary (distance
// to a sphere's points grows with their angle from the radial projection).
// Every point of the patch lies on that sphere (or plane), so its distance
// bounds the patch's from below: when its square exceeds `bound` (with a
// relative margin for rounding) the element cannot come nearer than bound and
// INFINITY is returned without the boundary arcs.
template <bool kCount>
__host__ __device__ double kelvin_tri_d2_t(const double x[3], const KelvinTri& T, const KelvinPre& R, double q[3],
                                           double l[3], double bound, uint64_t& ops) {
#pragma clang fp contract(off)
  Best b;
  b.d2 = INFINITY;
  if (T.has_plane) {
    const double* n = T.n;
    const double c = T.cpl;
    double p[3];
    if (c != 0.0) {
      const double sg = c > 0.0 ? 1.0 : -1.0;
      const double v[3] = {c * x[0] - 0.5 * n[0], c * x[1] - 0.5 * n[1], c * x[2] - 0.5 * n[2]};
      const double vl = sqrt(dot(v, v));
      const double sd = (fabs(c) * dot(x, x) - sg * dot(n, x)) / (vl + 0.5);
      if constexpr (kCount) ops += 32;
      if (sd * sd > bound * (1.0 + 1e-9)) return INFINITY;
      for (int k = 0; k < 3; ++k) p[k] = x[k] - sd * sg * v[k] / vl;
      if constexpr (kCount) ops += 10;
    } else {
      const double nx = dot(n, x);
      if constexpr (kCount) ops += 7;
      if (nx * nx > bound * (1.0 + 1e-9)) return INFINITY;
      for (int k = 0; k < 3; ++k) p[k] = x[k] - nx * n[k];
      if constexpr (kCount) ops += 6;
    }
    if constexpr (kCount) ops += 6;
    if (dot(p, p) * T.M2 >= 1.0 - 1e-9) {  // image points lie at least 1 / max|vertex| from the origin
      double y[3], ay[3], w[3], ab[3], ac[3], nn[3];
      invert(p, y);
      for (int k = 0; k < 3; ++k) {
        ay[k] = y[k] - T.a[k];
        ab[k] = T.b[k] - T.a[k];
        ac[k] = T.c[k] - T.a[k];
      }
      // barycentrics of y's projection on the plane
      cross(ab, ac, nn);
      const double nl = dot(nn, n);
      cross(ay, ac, w);
      const double l1 = dot(w, n) / nl;
      cross(ab, ay, w);
      const double l2 = dot(w, n) / nl;
      const double l0 = 1.0 - l1 - l2;
      if constexpr (kCount) ops += 64;
      if (l0 >= 0.0 && l1 >= 0.0 && l2 >= 0.0) {
        const double d[3] = {x[0] - p[0], x[1] - p[1], x[2] - p[2]};
        offer(b, dot(d, d), p, l0, l1, l2);
        if constexpr (kCount) ops += 8;
      }
    }
  }
  edge_eval<kCount>(x, T.a, R.k[0], R.k[1], R.edge[0], 0, 1, b, ops);
  edge_eval<kCount>(x, T.b, R.k[1], R.k[2], R.edge[1], 1, 2, b, ops);
  edge_eval<kCount>(x, T.c, R.k[2], R.k[0], R.edge[2], 2, 0, b, ops);
  q[0] = b.q[0]; q[1] = b.q[1]; q[2] = b.q[2];
  l[0] = b.l[0]; l[1] = b.l[1]; l[2] = b.l[2];
  return b.d2;
}

// The point-independent part of every element (leaf order): the images of
// its vertices and its edges' constants.
__global__ void kelvin_prepare_kernel(const KelvinTri* __restrict__ tris, int64_t n, KelvinPre* __restrict__ pre) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n || tris[s].orig == kPadTri) return;
  const KelvinTri& T = tris[s];
  KelvinPre R;
  invert(T.a, R.k[0]);
  invert(T.b, R.k[1]);
  invert(T.c, R.k[2]);
  edge_prepare(T.a, T.b, R.edge[0]);
  edge_prepare(T.b, T.c, R.edge[1]);
  edge_prepare(T.c, T.a, R.edge[2]);
  pre[s] = R;
}

// Smallest distance of the origin from triangle (a, b, c).
__device__ double origin_distance(const double a[3], const double b[3], const double c[3], const double n[3],
                                  double cpl, bool plane) {
  double best = INFINITY;
  bool inside = plane;
  const double* P[3] = {a, b, c};
  for (int s = 0; s < 3; ++s) {
    const double *u = P[s], *v = P[(s + 1) % 3];
    const double e[3] = {v[0] - u[0], v[1] - u[1], v[2] - u[2]};
    const double ee = dot(e, e);
    const double t = ee > 0.0 ? fmin(1.0, fmax(0.0, -dot(u, e) / ee)) : 0.0;
    const double p[3] = {u[0] + t * e[0], u[1] + t * e[1], u[2] + t * e[2]};
    best = fmin(best, dot(p, p));
    double m[3];
    const double w[3] = {cpl * n[0] - u[0], cpl * n[1] - u[1], cpl * n[2] - u[2]};
    cross(e, w, m);
    inside = inside && dot(m, n) >= 0.0;
  }
  return inside ? fmin(fabs(cpl), sqrt(best)) : sqrt(best);
}

// Prefilter records of the elements (slots, pads among them): the flat
// triangle of the vertices' images, and a bound h (field F) on how far any
// point of the curved element lies from it, and any of its points from the
// element. The element is kappa(T), kappa(y) = y / |y|^2, and the flat triangle
// the linear interpolation of kappa at T's vertices: with |D^2 kappa(y)[e, e]|
// = 2 |e|^2 / |y|^3 and rmin the smallest |y| on T they differ by at most
// (1/2) (2 / rmin^3) sum_i lambda_i |v_i - y|^2 <= L^2 / (3 rmin^3), L the
// longest edge; L^2 / (2 rmin^3) is taken. Records are in units of 1 / scale.
__global__ void kelvin_quick_kernel(const KelvinTri* __restrict__ tris, int64_t n, double scale,
                                    float4* __restrict__ quick) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n + kQuickPad) return;
  float4* q = quick + quick_index(i);
  if (i >= n || tris[i].orig == kPadTri) {
    quick_pad(q);
    return;
  }
  const KelvinTri& T = tris[i];
  double ka[3], kb[3], kc[3], l2 = 0.0;
  invert(T.a, ka);
  invert(T.b, kb);
  invert(T.c, kc);
  for (int s = 0; s < 3; ++s) {
    const double *u = s == 0 ? T.a : (s == 1 ? T.b : T.c), *v = s == 0 ? T.b : (s == 1 ? T.c : T.a);
    const double e[3] = {v[0] - u[0], v[1] - u[1], v[2] - u[2]};
    l2 = fmax(l2, dot(e, e));
  }
  const double r = origin_distance(T.a, T.b, T.c, T.n, T.cpl, T.has_plane != 0);
  const double h = l2 / (2.0 * r * r * r) * (1.0 + 1e-6) * scale;
  for (int c = 0; c < 3; ++c) {
    ka[c] *= scale;
    kb[c] *= scale;
    kc[c] *= scale;
  }
  if (!(h < 1e20) || !quick_frame(ka, kb, kc, q, h, 0.0)) quick_always(ka, q, 1e30f, 0.0f);
}

namespace {

// Curved elements of the inverted domain in the wavefront-shared search.
// Values are distances: the prefilter's flat one (quick_flat) less and plus h,
// m2 the bound on the distance in FP32. All FP32 quantities (boxes, records,
// pt, m2) are in units of 1 / scale, a power of two near the domain's size, so
// that their squares stay in range whatever the mesh's units. The FP32 roundings (of the point, of
// the frame and in quick_flat, at most 16 u (R + |x|) together, u = 2^-24, R
// the domain's radius) and the boxes' stand in pt.w, twice that bound. The
// exact test is the FP64 one; the owner keeps the lexicographic minimum of
// (squared distance, original index).
struct ArcEl {
  static constexpr uint32_t kQuickFlops = 0;  // not counted: exact tests, their operations and the boxes' are
  const Node4* node0;
  const KelvinTri* tris;
  const KelvinPre* pre;
  const float4* quick0;
  double scale;
  struct Owners {
    double x[64][3];
    unsigned long long key[64];  // squared distance (bits)
    uint32_t orig[64];
    int32_t slot[64];
  };
  static __device__ __forceinline__ float keep(float m2, const float4& q) {
    return (m2 + fabsf(q.w)) * (1.0f + 0x1p-20f);
  }
  static __device__ __forceinline__ float keep_wide(float m2, const float4& q) { return keep(m2, q); }
  static __device__ __forceinline__ float boxes(float m2, const float4& q) {
    const float s = (m2 + fabsf(q.w)) * (1.0f + 0x1p-20f);
    return fminf(s * s * (1.0f + 0x1p-20f), 0x1.fffffep127f);
  }
  template <typename Scratch>
  __device__ __forceinline__ const Node4* nodes(Scratch*, uint32_t) const {
    return node0;
  }
  template <typename Scratch>
  __device__ __forceinline__ void quick(Scratch*, uint32_t, const float4& p, int64_t i, float& lo, float& up,
                                        bool& always) const {
    values(p.x, p.y, p.z, i, lo, up, always);
  }
  __device__ __forceinline__ void values(float x, float y, float z, int64_t i, float& lo, float& up,
                                         bool& always) const {
    float w2, F, G;
    const float d2 = quick_flat(x, y, z, quick0, i, w2, F, G);
    const float d = __builtin_amdgcn_sqrtf(d2);
    lo = d * (1.0f - 0x1p-20f) - F;
    up = d * (1.0f + 0x1p-20f) + F;
    always = F > 1e28f;
  }
  template <bool kStats, typename Scratch>
  __device__ __forceinline__ void exact(Scratch* W, uint32_t o, int32_t s, bool now, const float4&,
                                        TravCount& cnt) const {
    if (!now) return;
    const double x[3] = {W->own.x[o][0], W->own.x[o][1], W->own.x[o][2]};
    const unsigned long long before = W->own.key[o];
    double q[3], l[3];
    uint64_t ops = 0;
    if (kStats) ++cnt.tris;
    const double d = kelvin_tri_d2_t<kStats>(x, tris[s], pre[s], q, l, __longlong_as_double((long long)before), ops);
    if (kStats) cnt.flops += ops;
    const unsigned long long bits = (unsigned long long)__double_as_longlong(d);
    if (d < INFINITY && bits <= before) {
      const uint32_t orig = (uint32_t)tris[s].orig;
      atomicMin(&W->own.key[o], bits);
      atomicMin(&W->m2[o], __float_as_uint((float)(sqrt(d) * scale * (1.0 + 1e-6))));
      lds_order();
      const unsigned long long now_best = W->own.key[o];
      if (bits == now_best) {
        // the lanes that hold a new minimum forget the index of the old one,
        // then the smallest of theirs (and of an equal old one's) stays
        if (now_best < before) W->own.orig[o] = (uint32_t)INT_MAX;
        lds_order();
        atomicMin(&W->own.orig[o], orig);
        lds_order();
        if (W->own.orig[o] == orig) W->own.slot[o] = s;
      }
    }
  }
};

__device__ __forceinline__ ArcEl arc_elements(const KelvinDev& K) {
  return ArcEl{K.nodes, K.tris, K.pre, K.quick, K.scale};
}

// Sets up owner `lane`'s search at x with the first bound of slot `warm` (or
// of the leaf a descent reaches, if negative).
template <typename Scratch>
__device__ __forceinline__ void arc_start(const KelvinDev& K, const ArcEl& el, Scratch* W, uint32_t lane,
                                          const double x[3], int32_t warm) {
  const float px = (float)(x[0] * K.scale), py = (float)(x[1] * K.scale), pz = (float)(x[2] * K.scale);
  if (warm < 0) warm = nearest_leaf(K.nodes, px, py, pz);
  float m2 = INFINITY;
  if (warm >= 0) {
    float lo;
    bool always;
    el.values(px, py, pz, quick_index(warm), lo, m2, always);
  }
  // 16 u (R + sqrt(3) |x|_inf), twice, rounded up
  const float pm = fmaxf(fabsf(px), fmaxf(fabsf(py), fabsf(pz)));
  W->pt[lane] = make_float4(px, py, pz, 0x1p-19f * ((float)(K.radius * K.scale) * 1.0001f + 1.75f * pm));
  W->m2[lane] = __float_as_uint(m2);
  for (int c = 0; c < 3; ++c) W->own.x[lane][c] = x[c];
  W->own.key[lane] = (unsigned long long)__double_as_longlong(INFINITY);
  W->own.orig[lane] = (uint32_t)INT_MAX;
  W->own.slot[lane] = -1;
}

// Answer of an owner whose search has ended and whose pending tests are done
// (as search_answer of the triangles): false if the search has to run again on
// exact values.
template <typename Scratch>
__device__ __forceinline__ bool arc_answer(const KelvinDev& K, Scratch* W, uint32_t lane, double& d2, int32_t& slot) {
  d2 = __longlong_as_double((long long)W->own.key[lane]);
  slot = W->own.slot[lane];
  const float4 q = W->pt[lane];
  const float d = (float)(sqrt(d2) * K.scale * (1.0 - 1e-6));
  if (q.w >= 0.0f && d > ArcEl::keep(__uint_as_float(W->m2[lane]), q)) {
    W->m2[lane] = __float_as_uint((float)(sqrt(d2) * K.scale * (1.0 + 1e-6)));
    W->pt[lane].w = -q.w;
    return false;
  }
  return true;
}

}  // namespace

namespace {

__device__ __forceinline__ void frame(const double n[3], double e1[3], double e2[3]) {
  const double sg = n[2] >= 0.0 ? 1.0 : -1.0;
  const double a = -1.0 / (sg + n[2]);
  const double b = n[0] * n[1] * a;
  e1[0] = 1.0 + sg * n[0] * n[0] * a; e1[1] = sg * b; e1[2] = -sg * n[0];
  e2[0] = b; e2[1] = sg + n[1] * n[1] * a; e2[2] = -n[1];
}

// The move of step k from x at squared distance d2 to the surface: a uniform
// point of the sphere of radius d (1 - kappa) - delta, drawn from the Philox
// block (row, walk, k, step purpose).
__device__ __forceinline__ void kelvin_move(const KelvinDev& K, uint32_t row, uint32_t walk, int64_t k, double d2,
                                            double x[3]) {
#pragma clang fp contract(off)
  const uint4 u = philox10(make_uint4(row, walk, (uint32_t)k, (kPurposeStep << 24) | (K.mesh_id & 0xFFFFFFu)),
                           K.seed_lo, K.seed_hi);
  const double u0 = unit_f(u.x), u1 = unit_f(u.y);
  const double r = sqrt(d2) * (1.0 - K.kappa) - K.delta;
  const double z = 1.0 - 2.0 * u0;
  const double rxy = 2.0 * sqrt(u0 * (1.0 - u0));
  double sp, cp;
  sincospi(2.0 * u1, &sp, &cp);
  x[0] += r * rxy * cp;
  x[1] += r * rxy * sp;
  x[2] += r * z;
}

}  // namespace

// Largest ball in the inverted domain touching its boundary at s~_i (unit
// normal n~_i pointing out of the domain): bisection over [0, r_max], a
// radius accepted when the centre c = s~ - r n~ is at least r - min(tol,
// r/1024) from the inverted surface and the ball lies within the domain's
// bound. Three levels per round: the eight lanes of a row take the (up to)
// seven midpoints of the next three levels at once (lane k heap node k of that
// subtree: node 1 the current midpoint, nodes 2k and 2k + 1 the midpoints of
// its halves), then all follow the path the sequential bisection takes through
// them. Every midpoint is formed by the operations of the sequential loop, so
// the radius is that loop's. Whether some element lies nearer to c than t is
// asked of the wavefront-shared search, bounded by t; it ends once an upper
// value says so and the exact one confirms it. (One depth-first search per
// lane: 21.6 ms for 1,024 rows on 79,380 elements; now 0.4 ms.) rows_per_wave (1, 2, 4 or
// 8) is as low as still gives every resident wavefront rows. queries[i] counts
// the iters decisions.
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MSK_KELVIN_WAVES_PER_EU)))
kelvin_tangent_kernel(KelvinDev K, const double* __restrict__ st, const double* __restrict__ nt, int64_t n_rows,
                      int32_t rows_per_wave, double r_max, int32_t iters, double tol, double* __restrict__ radius,
                      unsigned long long* __restrict__ queries) {
#pragma clang fp contract(off)
  __shared__ SearchScratch<ArcEl, true> coop[4];
  const int wi = (int)uniform(threadIdx.x >> 6);
  SearchScratch<ArcEl, true>* W = &coop[wi];
  const uint32_t lane = __lane_id();
  const int sub = (int)(lane & 7u), gbase = (int)(lane & ~7u);
  const ArcEl el = arc_elements(K);
  TravCount cnt;
  uint32_t size = 0, npend = 0;
  for (int64_t base = ((int64_t)blockIdx.x * 4 + wi) * rows_per_wave; base < n_rows;
       base += (int64_t)gridDim.x * 4 * rows_per_wave) {
    const int64_t i = base + (lane >> 3);
    const bool valid = (int32_t)(lane >> 3) < rows_per_wave && i < n_rows;
    double s[3] = {0.0, 0.0, 0.0}, n[3] = {0.0, 0.0, 0.0};
    if (valid)
      for (int c = 0; c < 3; ++c) {
        s[c] = st[3 * i + c];
        n[c] = nt[3 * i + c];
      }
    double lo = 0.0, hi = r_max;
    for (int32_t done = 0; done < iters;) {
      const int levels = min(3, iters - done);
      bool inside = false, fresh = false;
      double t = 0.0;
      if (valid && sub >= 1 && sub < (1 << levels)) {
        double a = lo, b = hi;
        const int depth = 31 - __clz(sub);  // bits of the node index below its leading one
        for (int j = depth - 1; j >= 0; --j) {
          const double m = 0.5 * (a + b);
          if ((sub >> j) & 1)
            a = m;
          else
            b = m;
        }
        const double mid = 0.5 * (a + b);
        const double c[3] = {s[0] - mid * n[0], s[1] - mid * n[1], s[2] - mid * n[2]};
        t = mid - fmin(tol, mid * (1.0 / 1024.0));
        inside = sqrt(dot(c, c)) + mid <= K.radius;
        fresh = inside && t > 0.0;
        if (fresh) {
          arc_start(K, el, W, lane, c, -1);
          // elements at t or farther do not matter; an upper value below
          // `stop` means an exact distance below t
          W->m2[lane] = min(W->m2[lane], __float_as_uint((float)(t * K.scale * (1.0 + 1e-6))));
          W->own.key[lane] = (unsigned long long)__double_as_longlong(t * t * (1.0 + 1e-9));
          W->stop[lane] = fmaxf(0.0f, (float)(t * K.scale * (1.0 - 1e-6)) - W->pt[lane].w);
        }
      }
      bool closer = false, open = fresh;
      search_push(W, lane, fresh, K.entry, size);
      while (true) {
        const bool step = size == 0;
        search_pass<false, true>(el, W, lane, !step, ~0ull, size, npend, cnt);
        if (!step) continue;
        bool again = false;
        if (open) {
          closer = W->own.slot[lane] >= 0 && sqrt(__longlong_as_double((long long)W->own.key[lane])) < t;
          // bounded by an upper value that no exact one has confirmed: search
          // on exact values only
          again = !closer && W->pt[lane].w >= 0.0f && __uint_as_float(W->m2[lane]) < (float)(t * K.scale * (1.0 - 1e-6));
          open = again;
          if (again) {
            W->pt[lane].w = -W->pt[lane].w;
            W->m2[lane] = __float_as_uint((float)(t * K.scale * (1.0 + 1e-6)));
          }
        }
        search_push(W, lane, again, K.entry, size);
        if (size == 0) break;
      }
      const unsigned long long mask = __ballot(inside && !closer);  // every lane of the wavefront takes part
      int node = 1;
      for (int l = 0; l < levels; ++l) {
        const double mid = 0.5 * (lo + hi);
        const int bit = (int)((mask >> (gbase + node)) & 1ull);
        if (bit)
          lo = mid;
        else
          hi = mid;
        node = 2 * node + bit;
      }
      done += levels;
    }
    if (valid && sub == 0) {
      radius[i] = lo;
      queries[i] = (unsigned long long)iters;
    }
  }
}

// Walks [0, n_rows 2 pairs) are the jump term's: walk 2j + a of row i starts
// at point a of antithetic pair j on the row's tangent ball, drawn with
// density proportional to the ball jump kernel outside the cap
// (u = sin(theta/2) with density ~ 1/u^2 on [u0, 1], inverted in closed form;
// azimuth uniform, + pi for the partner). The next n_kill walks are the
// killing term's, from the origin (the image of infinity), with Philox row
// 0xFFFFFFFF and walk index k; their first step, from near the middle of a
// round shape, shares one answer. The launch is persistent: a wavefront claims
// walks for its idle lanes from a counter, its walks' searches share its
// stack, and walks whose search has ended wait until a quarter of the
// wavefront's do, then finish their step together; each walk's result depends
// on its index only. At most `owners` lanes carry a walk. Each walk logs its
// status, terminal original triangle, the barycentrics of that triangle's
// vertices 1 and 2 at the terminal point's image, its query count, and the
// factor g = 1/|t~| of its rank-one update.
//   With a depth-first search per lane and every listed element tested in
// FP64, 38.5 element tests of up to 354 operations per search, 98,304 walks on
// 79,380 elements took 79.6 ms; now 6.5 ms, bound by the longest walks' chains of
// searches.
// The counting instantiation (kCount) runs the same walks and adds the
// searches' node visits, exact element tests and operations (68 FP32 ones per
// node for its boxes, the FP64 ones of the exact tests) to stats[0..2]. The
// prefilter's are not counted.
template <bool kCount>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MSK_KELVIN_WAVES_PER_EU)))
kelvin_stream_kernel(
    KelvinDev K, const double* __restrict__ st, const double* __restrict__ nt, const double* __restrict__ radius,
    int64_t n_rows, int64_t pairs, double u0, int64_t n_kill, int32_t owners, int32_t* __restrict__ log_status,
    int32_t* __restrict__ log_tri, float* __restrict__ log_bary, int32_t* __restrict__ log_q, double* __restrict__ g,
    unsigned long long* __restrict__ row_queries, unsigned long long* kill_queries, unsigned long long* next_walk,
    unsigned long long* __restrict__ stats) {
  __shared__ SearchScratch<ArcEl> coop[4];
  const int wi = (int)uniform(threadIdx.x >> 6);
  SearchScratch<ArcEl>* W = &coop[wi];
  const int64_t n_jump = n_rows * 2 * pairs, total = n_jump + n_kill;
  const uint32_t lane = __lane_id();
  const ArcEl el = arc_elements(K);
  TravCount cnt;
  int64_t id = -1, i = -1, k = 0;
  uint32_t row = 0, walk = 0;
  double x[3] = {0.0, 0.0, 0.0};
  int32_t mode = 0;  // 0 no walk, 1 searching, 2 search ended
  uint32_t size = 0, npend = 0;
  bool drained = false;
  auto log_walk = [&](int32_t status, int32_t nq, int32_t orig, const double q[3], const double l[3]) {
    log_status[id] = status;
    log_tri[id] = orig;
    log_bary[2 * id] = (float)l[1];
    log_bary[2 * id + 1] = (float)l[2];
    log_q[id] = nq;
    g[id] = 1.0 / sqrt(dot(q, q));
    if (i >= 0)
      atomicAdd(row_queries + i, (unsigned long long)nq);
    else
      atomicAdd(kill_queries, (unsigned long long)nq);
    mode = 0;
  };
  while (true) {
    if (mode == 1 && W->open[lane] == 0) mode = 2;
    size = uniform(size);
    drained = uniform(drained ? 1u : 0u) != 0;
    const uint64_t pend = __ballot(mode == 2), busy = __ballot(mode == 1) | pend;
    const uint64_t idle0 = drained ? 0ull : __ballot(mode == 0 && lane < (uint32_t)owners);
    const bool step = size == 0 || (size <= (uint32_t)kRootLimit &&
                                    (int)__popcll(pend | idle0) >= min(16, (int)(__popcll(busy | idle0) + 3) >> 2));
    search_pass<kCount>(el, W, lane, !step, pend, size, npend, cnt);
    if (!step) continue;
    bool fresh = false, go = false;  // go: a new search at x, warm-started from `warm`
    int32_t warm = -1;
    if (mode == 2) {
      double d2;
      int32_t slot;
      if (!arc_answer(K, W, lane, d2, slot)) {
        fresh = true;
        mode = 1;
      } else if (slot < 0) {  // no element at a finite distance (never for a finite x): no triangle for the products to read
        const double none[3] = {0.0, 0.0, 0.0};
        log_walk(kCapped, (int32_t)(k + 1), -1, none, none);
      } else if (k >= K.max_steps || d2 < K.eps2) {
        // the walk ends at its position's nearest point: that element's test
        // once more (the step cap's search is the one at k = max_steps)
        double q[3], l[3];
        uint64_t none = 0;
        const KelvinTri& T = K.tris[slot];
        (void)kelvin_tri_d2_t<false>(x, T, K.pre[slot], q, l, INFINITY, none);
        log_walk(k >= K.max_steps ? kCapped : kHit, (int32_t)(k + 1), T.orig, q, l);
      } else {
        kelvin_move(K, row, walk, k, d2, x);
        ++k;
        warm = slot;
        go = true;
      }
    }
    // idle lanes claim the next walks
    const uint64_t idle = drained ? 0ull : __ballot(mode == 0 && lane < (uint32_t)owners);
    if (idle != 0) {
      unsigned long long first = 0;
      const int lead = __ffsll((unsigned long long)idle) - 1;
      if ((int)lane == lead) first = atomicAdd(next_walk, (unsigned long long)__popcll(idle));
      first = (unsigned long long)__shfl(first, lead);
      const int64_t claim = (int64_t)first + (int64_t)mbcnt64(idle);
      drained = (int64_t)first + (int64_t)__popcll(idle) >= total;
      if (((idle >> lane) & 1ull) && claim < total) {
        id = claim;
        k = 0;
        if (id < n_jump) {
          i = id / (2 * pairs);
          const int64_t w = id - i * 2 * pairs;
          const double r = radius[i];
          if (!(r > 0.0)) {
            log_status[id] = -1;
            log_tri[id] = -1;
            log_bary[2 * id] = log_bary[2 * id + 1] = 0.0f;
            log_q[id] = 0;
            g[id] = 0.0;
          } else {
            row = (uint32_t)i;
            walk = (uint32_t)w;
            const uint4 u = philox10(
                make_uint4(row, (uint32_t)(w >> 1), 0u, (kPurposeBall << 24) | (K.mesh_id & 0xFFFFFFu)), K.seed_lo,
                K.seed_hi);
            const double xi = unit_f(u.x), eta = unit_f(u.y);
            const double su = 1.0 / (1.0 / u0 - xi * (1.0 / u0 - 1.0));
            const double ct = 1.0 - 2.0 * su * su, sn = 2.0 * su * sqrt(fmax(0.0, 1.0 - su * su));
            double sp, cp;
            sincospi(2.0 * eta + ((w & 1) ? 1.0 : 0.0), &sp, &cp);
            const double n[3] = {nt[3 * i], nt[3 * i + 1], nt[3 * i + 2]};
            double e1[3], e2[3];
            frame(n, e1, e2);
            for (int c3 = 0; c3 < 3; ++c3) {
              const double c = st[3 * i + c3] - r * n[c3];
              x[c3] = c + r * (ct * n[c3] + sn * (cp * e1[c3] + sp * e2[c3]));
            }
            go = true;
          }
        } else {
          i = -1;
          row = 0xFFFFFFFFu;
          walk = (uint32_t)(id - n_jump);
          x[0] = x[1] = x[2] = 0.0;
          go = true;
          if (K.origin_known && K.max_steps > 0) {  // the first step's shared answer
            if (K.origin_d2 < K.eps2) {
              log_walk(kHit, 1, K.origin_orig, K.origin_q, K.origin_l);
              go = false;
            } else {
              kelvin_move(K, row, walk, 0, K.origin_d2, x);
              k = 1;
            }
          }
        }
      }
    }
    if (go) {
      arc_start(K, el, W, lane, x, warm);
      mode = 1;
      fresh = true;
    }
    search_push(W, lane, fresh, K.entry, size);
    if (drained && __ballot(mode != 0) == 0) break;
  }
  if constexpr (kCount) {
    atomicAdd(stats, (unsigned long long)cnt.nodes);
    atomicAdd(stats + 1, (unsigned long long)cnt.tris);
    atomicAdd(stats + 2, (unsigned long long)cnt.flops);
  }
}

// Nearest inverted element of each query point (inverted space, relative to
// the centre), on the shared search: query j of wavefront g is j G + g, G the
// number of wavefronts, at most `owners` of them at a time.
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MSK_KELVIN_WAVES_PER_EU)))
kelvin_closest_kernel(KelvinDev K, const double* __restrict__ Q, int64_t nq, int32_t owners, int32_t* __restrict__ tri,
                      double* __restrict__ d2, double* __restrict__ qpt, double* __restrict__ bary) {
  __shared__ SearchScratch<ArcEl> coop[4];
  const int wi = (int)uniform(threadIdx.x >> 6);
  SearchScratch<ArcEl>* W = &coop[wi];
  const uint32_t lane = __lane_id();
  const int64_t G = (int64_t)gridDim.x * 4, g = (int64_t)blockIdx.x * 4 + wi;
  const ArcEl el = arc_elements(K);
  TravCount cnt;
  int32_t mode = 0;
  int64_t next = 0, qi = 0;
  double x[3] = {0.0, 0.0, 0.0};
  uint32_t size = 0, npend = 0;
  bool drained = false;
  while (true) {
    if (mode == 1 && W->open[lane] == 0) mode = 2;
    size = uniform(size);
    const uint64_t pend = __ballot(mode == 2), busy = __ballot(mode == 1) | pend;
    const bool step = size == 0 || (size <= (uint32_t)kRootLimit &&
                                    (int)__popcll(pend) >= min(16, (int)(__popcll(busy) + 3) >> 2));
    search_pass<false>(el, W, lane, !step, pend, size, npend, cnt);
    if (!step) continue;
    bool fresh = false;
    if (mode == 2) {
      double best;
      int32_t slot;
      if (arc_answer(K, W, lane, best, slot)) {
        double q[3] = {0.0, 0.0, 0.0}, l[3] = {0.0, 0.0, 0.0};
        uint64_t none = 0;
        int32_t orig = 0;  // no finite distance: the lowest element at infinity
        if (slot >= 0) {
          (void)kelvin_tri_d2_t<false>(x, K.tris[slot], K.pre[slot], q, l, INFINITY, none);
          orig = K.tris[slot].orig;
        }
        d2[qi] = best;
        tri[qi] = orig;
        for (int c = 0; c < 3; ++c) {
          qpt[3 * qi + c] = q[c];
          bary[3 * qi + c] = l[c];
        }
        mode = 0;
      } else {
        fresh = true;
        mode = 1;
      }
    }
    const uint64_t idle = drained ? 0ull : __ballot(mode == 0 && lane < (uint32_t)owners);
    if (idle != 0) {
      const int64_t q = (next + (int64_t)mbcnt64(idle)) * G + g;
      const bool take = ((idle >> lane) & 1ull) && q < nq;
      if (take) {
        qi = q;
        for (int c = 0; c < 3; ++c) x[c] = Q[3 * qi + c];
        arc_start(K, el, W, lane, x, -1);
        const float4 p = W->pt[lane];
        if (!(fabsf(p.x) <= 0x1p60f && fabsf(p.y) <= 0x1p60f && fabsf(p.z) <= 0x1p60f)) {
          // its squares leave FP32's range, or it is no number: every element
          // lies within the allowance, and exact values alone decide
          W->pt[lane] = make_float4(0.0f, 0.0f, 0.0f, -0x1p41f);
          W->m2[lane] = __float_as_uint(INFINITY);
        }
        mode = 1;
        fresh = true;
      }
      const uint32_t got = (uint32_t)__popcll(__ballot(take));
      drained = got < (uint32_t)__popcll(idle);
      next += got;
    }
    search_push(W, lane, fresh, K.entry, size);
    if (drained && __ballot(mode != 0) == 0) break;
  }
}

hipError_t launch_kelvin_tangent(const KelvinDev& K, const double* st, const double* nt, int64_t n_rows, double r_max,
                                 int32_t iters, double tol, int32_t n_cu, double* radius, unsigned long long* queries,
                                 hipStream_t s) {
  if (n_rows <= 0) return hipSuccess;
  const int64_t waves = 16ll * n_cu;
  int32_t rows = 1;
  while (rows < 8 && rows * waves < n_rows) rows *= 2;
  const int64_t blocks = std::min<int64_t>(4ll * n_cu, (n_rows + rows * 4 - 1) / (rows * 4));
  hipLaunchKernelGGL(kelvin_tangent_kernel, dim3((unsigned)blocks), dim3(256), 0, s, K, st, nt, n_rows, rows, r_max,
                     iters, tol, radius, queries);
  return hipGetLastError();
}

// Owners of a wavefront and workgroups for n searches: all resident
// wavefronts (4 per SIMD), each with as few at a time as still covers n.
static void spread(int64_t n, int32_t n_cu, int32_t* owners, int64_t* blocks) {
  const int64_t waves = 16ll * n_cu;
  *owners = (int32_t)std::min<int64_t>(64, (n + waves - 1) / waves);
  *blocks = std::min<int64_t>(4ll * n_cu, (n + 4 * *owners - 1) / (4 * *owners));
}

hipError_t launch_kelvin_walks(const KelvinDev& K, const double* st, const double* nt, const double* radius,
                               int64_t n_rows, int64_t pairs, double u0, int64_t n_kill, int32_t* log_status,
                               int32_t* log_tri, float* log_bary, int32_t* log_q, double* g,
                               unsigned long long* row_queries, unsigned long long* kill_queries,
                               unsigned long long* next_walk, unsigned long long* stats, int32_t n_cu, hipStream_t s) {
  const int64_t n = n_rows * 2 * pairs + n_kill;
  if (n <= 0) return hipSuccess;
  if (n_cu < 1) return hipErrorInvalidValue;
  int32_t owners;
  int64_t blocks;
  spread(n, n_cu, &owners, &blocks);
  if (stats)
    hipLaunchKernelGGL(kelvin_stream_kernel<true>, dim3((unsigned)blocks), dim3(256), 0, s, K, st, nt, radius, n_rows,
                       pairs, u0, n_kill, owners, log_status, log_tri, log_bary, log_q, g, row_queries, kill_queries,
                       next_walk, stats);
  else
    hipLaunchKernelGGL(kelvin_stream_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, s, K, st, nt, radius,
                       n_rows, pairs, u0, n_kill, owners, log_status, log_tri, log_bary, log_q, g, row_queries,
                       kill_queries, next_walk, stats);
  return hipGetLastError();
}

hipError_t launch_kelvin_prepare(const KelvinTri* tris, int64_t n, double scale, KelvinPre* pre, float4* quick,
                                 hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(kelvin_prepare_kernel, dim3((unsigned)((n + 127) / 128)), dim3(128), 0, s, tris, n, pre);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kelvin_quick_kernel, dim3((unsigned)((n + kQuickPad + 127) / 128)), dim3(128), 0, s, tris, n,
                     scale, quick);
  return hipGetLastError();
}

hipError_t launch_kelvin_closest(const KelvinDev& K, const double* Q, int64_t nq, int32_t n_cu, int32_t* tri, double* d2,
                                 double* qpt, double* bary, hipStream_t s) {
  if (nq <= 0) return hipSuccess;
  int32_t owners;
  int64_t blocks;
  spread(nq, n_cu, &owners, &blocks);
  hipLaunchKernelGGL(kelvin_closest_kernel, dim3((unsigned)blocks), dim3(256), 0, s, K, Q, nq, owners, tri, d2, qpt,
                     bary);
  return hipGetLastError();
}

}  // namespace msk
