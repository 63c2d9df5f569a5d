// HIP kernels of the Walk-on-Spheres DtN estimator for gfx950.
//
// One wavefront lane carries one walk. Each step asks the BVH for the exact
// nearest triangle (the empty-ball radius, Sec. 2 "Walk-on-Spheres"), stops
// in the eps-shell, and otherwise jumps to a uniform point of the ball. The
// walk's hit is scattered into its row as c = b(s) - b(t) (Sec. 3.1, Alg. 1,
// eq. naive-stiffness-matrix). The persistent form keeps every lane busy by
// refilling finished lanes from a work queue (walks of a wavefront have very
// different lengths), with one queue per XCD over a contiguous, Z-ordered
// range of rows so that each XCD's L2 sees one region of the surface.
#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>
#include <cstring>

#include "msk_internal.h"
#include "philox.h"
#include "search.h"

namespace msk {

// A mesh's descriptor, which no kernel writes: read through the scalar cache
// where the mesh is the same for all lanes (wave_meshes).
typedef const __attribute__((address_space(4))) MeshDev ConstMesh;

__device__ __forceinline__ TriRec gload_tri(const TriRec* tris, int64_t i) {
  return TriRec{gload4(tris, 3 * i), gload4(tris, 3 * i + 1), gload4(tris, 3 * i + 2)};
}
__device__ __forceinline__ uint4 draw(const WalkLaunch& L, uint32_t row, uint32_t walk, uint32_t step,
                                      uint32_t purpose, uint32_t mesh) {
  return philox10(make_uint4(row, walk, step, (purpose << 24) | (mesh & 0xFFFFFFu)), L.seed_lo, L.seed_hi);
}

// --------------------------------------------------- FP32 closest point
// Squared distance from p to triangle T, evaluated in a fixed order with
// every product and sum rounded on its own (no contraction into FMA), so
// that it is reproducible bit for bit: Voronoi regions tested in the order
// vertex a, vertex b, edge ab, vertex c, edge ac, edge bc, face; face-region
// numerators n.(u x v) with n = ab x ac; face distance (n.ap)^2 / (n.n).
// (l1, l2) are the barycentric weights of vertices b and c.
//
// In the face region the barycentrics are returned as numerators (l1, l2 =
// vb, vc) over `den` (left unchanged in the other regions); they are divided
// only where a walk's final nearest point is used. A face whose squared
// plane distance exceeds `reject` by a safe margin returns +inf without
// dividing: it cannot beat or tie a current best of `reject`. Distances that
// are returned are exactly the values above.
__host__ __device__ __forceinline__ float tri_dist2(float px, float py, float pz, const TriRec& T, float reject,
                                                   float& l1, float& l2, float& den_out, int& region) {
#pragma clang fp contract(off)
  const float ax = T.a.x, ay = T.a.y, az = T.a.z;
  const float bx = T.b.x, by = T.b.y, bz = T.b.z;
  const float cx = T.c.x, cy = T.c.y, cz = T.c.z;
  const float abx = bx - ax, aby = by - ay, abz = bz - az;
  const float acx = cx - ax, acy = cy - ay, acz = cz - az;
  const float apx = px - ax, apy = py - ay, apz = pz - az;
  float t;
  t = abx * apx; t = t + aby * apy; const float d1 = t + abz * apz;
  t = acx * apx; t = t + acy * apy; const float d2 = t + acz * apz;
  if (d1 <= 0.0f && d2 <= 0.0f) {
    l1 = 0.0f; l2 = 0.0f; region = 0;
    t = apx * apx; t = t + apy * apy; return t + apz * apz;
  }
  const float bpx = px - bx, bpy = py - by, bpz = pz - bz;
  t = abx * bpx; t = t + aby * bpy; const float d3 = t + abz * bpz;
  t = acx * bpx; t = t + acy * bpy; const float d4 = t + acz * bpz;
  if (d3 >= 0.0f && d4 <= d3) {
    l1 = 1.0f; l2 = 0.0f; region = 1;
    t = bpx * bpx; t = t + bpy * bpy; return t + bpz * bpz;
  }
  const float nx = aby * acz - abz * acy;
  const float ny = abz * acx - abx * acz;
  const float nz = abx * acy - aby * acx;
  float xx = apy * bpz - apz * bpy, xy = apz * bpx - apx * bpz, xz = apx * bpy - apy * bpx;
  t = nx * xx; t = t + ny * xy; const float vc = t + nz * xz;
  if (vc <= 0.0f && d1 >= 0.0f && d3 <= 0.0f) {
    const float v = d1 / (d1 - d3);
    const float ex = px - (ax + v * abx), ey = py - (ay + v * aby), ez = pz - (az + v * abz);
    l1 = v; l2 = 0.0f; region = 2;
    t = ex * ex; t = t + ey * ey; return t + ez * ez;
  }
  const float cpx = px - cx, cpy = py - cy, cpz = pz - cz;
  t = abx * cpx; t = t + aby * cpy; const float d5 = t + abz * cpz;
  t = acx * cpx; t = t + acy * cpy; const float d6 = t + acz * cpz;
  if (d6 >= 0.0f && d5 <= d6) {
    l1 = 0.0f; l2 = 1.0f; region = 3;
    t = cpx * cpx; t = t + cpy * cpy; return t + cpz * cpz;
  }
  xx = cpy * apz - cpz * apy; xy = cpz * apx - cpx * apz; xz = cpx * apy - cpy * apx;
  t = nx * xx; t = t + ny * xy; const float vb = t + nz * xz;
  if (vb <= 0.0f && d2 >= 0.0f && d6 <= 0.0f) {
    const float w = d2 / (d2 - d6);
    const float ex = px - (ax + w * acx), ey = py - (ay + w * acy), ez = pz - (az + w * acz);
    l1 = 0.0f; l2 = w; region = 4;
    t = ex * ex; t = t + ey * ey; return t + ez * ez;
  }
  xx = bpy * cpz - bpz * cpy; xy = bpz * cpx - bpx * cpz; xz = bpx * cpy - bpy * cpx;
  t = nx * xx; t = t + ny * xy; const float va = t + nz * xz;
  const float e43 = d4 - d3, e56 = d5 - d6;
  if (va <= 0.0f && e43 >= 0.0f && e56 >= 0.0f) {
    const float w = e43 / (e43 + e56);
    const float bcx = cx - bx, bcy = cy - by, bcz = cz - bz;
    const float ex = px - (bx + w * bcx), ey = py - (by + w * bcy), ez = pz - (bz + w * bcz);
    l1 = 1.0f - w; l2 = w; region = 5;
    t = ex * ex; t = t + ey * ey; return t + ez * ez;
  }
  const float den = (va + vb) + vc;
  if (den > 0.0f) {
    region = 6;
    t = nx * apx; t = t + ny * apy; const float tn = t + nz * apz;
    t = nx * nx; t = t + ny * ny; const float nn = t + nz * nz;
    const float tt = tn * tn;
    // fl(tt / nn) > reject whenever tt > fl(fl(reject nn)(1 + 2^-20))
    if (tt > (reject * nn) * (1.0f + 0x1p-20f)) return INFINITY;
    l1 = vb; l2 = vc; den_out = den;
    return tt / nn;
  }
  // zero-area triangle: nearest point of the three edges, first strict minimum
  float best = INFINITY, bl1 = 0.0f, bl2 = 0.0f;
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    const float s0x = s == 2 ? bx : ax, s0y = s == 2 ? by : ay, s0z = s == 2 ? bz : az;
    const float s1x = s == 0 ? bx : cx, s1y = s == 0 ? by : cy, s1z = s == 0 ? bz : cz;
    const float ex = s1x - s0x, ey = s1y - s0y, ez = s1z - s0z;
    const float qx = px - s0x, qy = py - s0y, qz = pz - s0z;
    t = ex * ex; t = t + ey * ey; const float ee = t + ez * ez;
    t = qx * ex; t = t + qy * ey; const float qe = t + qz * ez;
    float u = ee > 0.0f ? qe / ee : 0.0f;
    if (u < 0.0f) u = 0.0f;
    if (u > 1.0f) u = 1.0f;
    const float rx = px - (s0x + u * ex), ry = py - (s0y + u * ey), rz = pz - (s0z + u * ez);
    t = rx * rx; t = t + ry * ry; const float dd = t + rz * rz;
    if (dd < best) {
      best = dd;
      bl1 = s == 0 ? u : (s == 1 ? 0.0f : 1.0f - u);
      bl2 = s == 0 ? 0.0f : u;
    }
  }
  l1 = bl1; l2 = bl2; region = 7;
  return best;
}

// ------------------------------------------------------- BVH traversal
// Squared-distance bound above which a box cannot hold a triangle whose FP32
// distance is <= best: the FP32 distance of a triangle is at least
// (d_true - slack)^2 (1 - 8u) with slack = 2^-18 (R + |p|_inf), and the FP32
// box distance at most its true value times (1 + 6u).
__host__ __device__ __forceinline__ float prune_bound(float best, float slack) {
  const float s = sqrtf(best) * (1.0f + 0x1p-20f) + slack;
  return s * s * (1.0f + 0x1p-20f);
}

// l1, l2 are the barycentrics of the nearest point, or for a face-region
// result their numerators over `den` (divided by nearest_bary where used).
struct Nearest {
  float d2;
  int32_t slot;
  int32_t orig;
  float l1, l2;
  float den = 1.0f;
};

__host__ __device__ __forceinline__ void nearest_bary(const Nearest& h, float& l1, float& l2) {
  l1 = h.l1;
  l2 = h.l2;
  if (h.den != 1.0f) {
    l1 = h.l1 / h.den;
    l2 = h.l2 / h.den;
  }
}

// FP32 operations of tri_dist2 up to each exit (vertex a, vertex b, edge ab,
// vertex c, edge ac, edge bc, face, zero-area fallback).
constexpr uint32_t kTriFlops[8] = {24, 37, 71, 73, 98, 117, 114, 175};
template <bool kStats>
__host__ __device__ __forceinline__ void test_tri(const TriRec* __restrict__ tris, int32_t s, float px, float py, float pz,
                                         Nearest& h, TravCount& cnt) {
  const TriRec T = tris[s];
  float l1 = 0.0f, l2 = 0.0f, den = 1.0f;
  int region = 0;
  const float d = tri_dist2(px, py, pz, T, h.d2, l1, l2, den, region);
  if (kStats) {
    ++cnt.tris;
    cnt.flops += kTriFlops[region & 7];
  }
  int32_t orig;
  memcpy(&orig, &T.a.w, 4);
  if (d < h.d2 || (d == h.d2 && orig < h.orig)) {
    h.d2 = d; h.slot = s; h.orig = orig; h.l1 = l1; h.l2 = l2;
    h.den = region == 6 ? den : 1.0f;
  }
}

// Exact nearest triangle: lexicographic minimum of (FP32 squared distance,
// original index). `h.slot` may name a candidate triangle on entry (warm
// start: the previous step's nearest), tested first so that the search starts
// with a finite bound. Each node test sorts the four children by box lower
// bound, tests the leaf children's triangles at once (nearest first), keeps
// the nearest surviving inner child in registers as the next node and pushes
// the other inner children farthest first; entries are popped only when the
// current subtree is done, and skipped when their bound no longer reaches the
// best distance. (Measured on gfx950 against a stack that also holds leaves
// and against a loop that defers leaves until every lane of the wavefront
// holds one: this order is the fastest of the three.)
struct StackEntry {
  int32_t node;
  float lb;
};

template <bool kStats>
__host__ __device__ void bvh_nearest(const Node4* __restrict__ nodes, const TriRec* __restrict__ tris, float px,
                                     float py, float pz, float radius, Nearest& h, TravCount& cnt) {
  const float slack = 0x1p-18f * (radius + fmaxf(fabsf(px), fmaxf(fabsf(py), fabsf(pz))));
  if (h.slot >= 0) {
    const int32_t s = h.slot;
    h.d2 = INFINITY;
    h.orig = INT_MAX;
    h.slot = -1;
    test_tri<kStats>(tris, s, px, py, pz, h, cnt);
  }
  float thr = prune_bound(h.d2, slack);
  StackEntry stk[kStackDepth];
  int sp = 0;
  int32_t node = 0;
  while (true) {
    float4 lox, loy, loz, hix, hiy, hiz;
    int4 ch, ct;
    if (kStats) {
      ++cnt.nodes;
      cnt.flops += 4 * kBoxFlops;
    }
    const float4* N = (const float4*)&nodes[node];
    lox = N[0]; loy = N[1]; loz = N[2]; hix = N[3]; hiy = N[4]; hiz = N[5];
    ch = ((const int4*)N)[6]; ct = ((const int4*)N)[7];
    float lb[4];
    int32_t cc[4], cn[4];
    {
      const float lx[4] = {lox.x, lox.y, lox.z, lox.w}, ly[4] = {loy.x, loy.y, loy.z, loy.w},
                  lz[4] = {loz.x, loz.y, loz.z, loz.w};
      const float hx[4] = {hix.x, hix.y, hix.z, hix.w}, hy[4] = {hiy.x, hiy.y, hiy.z, hiy.w},
                  hz[4] = {hiz.x, hiz.y, hiz.z, hiz.w};
      const int32_t c4[4] = {ch.x, ch.y, ch.z, ch.w}, n4[4] = {ct.x, ct.y, ct.z, ct.w};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float gx = fmaxf(fmaxf(lx[k] - px, px - hx[k]), 0.0f);
        const float gy = fmaxf(fmaxf(ly[k] - py, py - hy[k]), 0.0f);
        const float gz = fmaxf(fmaxf(lz[k] - pz, pz - hz[k]), 0.0f);
        lb[k] = gx * gx + gy * gy + gz * gz;
        cc[k] = c4[k];
        cn[k] = n4[k];
      }
    }
    // sort the four children by lower bound (5 compare-exchanges)
#define MSK_CX(i, j)                                                        \
  if (lb[j] < lb[i]) {                                                      \
    float tl = lb[i]; lb[i] = lb[j]; lb[j] = tl;                            \
    int32_t tc = cc[i]; cc[i] = cc[j]; cc[j] = tc;                          \
    int32_t tn = cn[i]; cn[i] = cn[j]; cn[j] = tn;                          \
  }
    MSK_CX(0, 1) MSK_CX(2, 3) MSK_CX(0, 2) MSK_CX(1, 3) MSK_CX(1, 2)
#undef MSK_CX
    // leaves, nearest first (an unused slot has count 0)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (cc[k] < 0 && cn[k] > 0 && lb[k] <= thr) {
        const int32_t first = (-cc[k] - 1) & ~3;
        const float before = h.d2;
        for (int32_t s = first; s < first + cn[k]; ++s) test_tri<kStats>(tris, s, px, py, pz, h, cnt);
        if (h.d2 != before) {
          thr = prune_bound(h.d2, slack);
        }
      }
    }
    // the nearest surviving inner child is next; the others are pushed
    // farthest first
    int32_t next = -1;
    float next_lb = 0.0f;
#pragma unroll
    for (int k = 3; k >= 0; --k) {
      if (cc[k] >= 0 && lb[k] <= thr) {
        if (next >= 0 && sp < kStackDepth) stk[sp++] = StackEntry{next, next_lb};
        next = cc[k];
        next_lb = lb[k];
      }
    }
    if (next >= 0) {
      node = next;
      continue;
    }
    node = -1;
    while (sp > 0) {
      --sp;
      if (stk[sp].lb <= thr) {
        node = stk[sp].node;
        break;
      }
    }
    if (node < 0) break;
  }
}

// ---- prefilter of the exact triangle test
// Squared distance d2 from p to the triangle (quick_flat) with its error
// margin m = (F + H |p - a|^2) |p - a|^2 + G: the exact test's value D of the
// same triangle satisfies sqrt(D) >= sqrt(max(0, d2 - m)) - delta, and for all
// but nearly degenerate triangles sqrt(D) <= sqrt(d2 + m) + delta, delta =
// 2^-21 R covering the exact test's roundings at the size of the coordinates.
// Where the margin's relative part exceeds a quarter the values bound nothing
// (`always`). The frame and margins are prepared by quick_prepare_kernel, whose
// comment derives them; H stands in the low half of F's word.
__device__ __forceinline__ void quick_dist(float px, float py, float pz, const void* quick, int64_t i, float& d2,
                                           float& m, bool& always) {
  float w2, F, G;
  d2 = quick_flat(px, py, pz, quick, i, w2, F, G);
  const float H = __uint_as_float(__float_as_uint(F) << 16), part = F + H * w2;
  m = part * w2 + G;
  always = part > 0.25f;
}

// Largest squared value d2 - m of a triangle that may still beat or tie a
// query whose bound is m2 = min(d2 + m): sqrt(d2 - m) <= sqrt(m2) + 2 delta
// (two_delta = 2 delta; the square root has one ulp).
__device__ __forceinline__ float keep_bound(float m2, float two_delta) {
  const float s = __builtin_amdgcn_sqrtf(m2) * (1.0f + 0x1p-20f) + two_delta;
  return s * s * (1.0f + 0x1p-20f);
}

// m2 of a squared distance: not below the normal numbers, of which boxes and
// keep_bound take the hardware's square root.
__device__ __forceinline__ float bound_of(float d2) { return fmaxf(d2, 0x1p-126f); }

// Planar triangles as elements of the wavefront-shared search (same result as
// the lane-private bvh_nearest, bit for bit, unless the exact test's products
// underflow: in scenes of radius below about 1e-5 whole neighbourhoods tie at
// distance 0, and the two searches may meet different ones of them). Values are squared distances,
// pt.w = 2 delta; the owner's (squared distance, original index) is kept by a
// 64-bit LDS minimum, which realises the lexicographic order exactly.
struct TriEl {
  static constexpr uint32_t kQuickFlops = 60;  // FP32 operations of quick_dist and the two bounds
  struct Owners {
    const char* base[64];    // owner's mesh (batched meshes differ per lane): its nodes,
    uint32_t off_quick[64];  // and its prefilter records
    uint32_t off_tris[64];   // and triangles, in 256 B from the nodes
    unsigned long long key[64];
    int32_t rec_slot[64];
  };
  static __device__ __forceinline__ float keep(float m2, const float4& q) { return keep_bound(m2, fabsf(q.w)); }
  // Not below keep, and without its square root (a quarter-rate instruction):
  // (x + w)^2 <= x^2 (1 + t) + w^2 (1 + 1/t), t = 2^-12, and 2^-19 for rounding.
  // The tests of listed triangles take it: it gives back what their margins'
  // w^4 costs (soup operator's walks 7.85 -> 7.75 ms).
  static __device__ __forceinline__ float keep_wide(float m2, const float4& q) {
    return m2 * (1.0f + 0x1p-12f + 0x1p-19f) + (q.w * q.w) * (4097.0f * (1.0f + 0x1p-19f));
  }
  // Box bound of a query: no triangle in a box whose squared distance exceeds it
  // beats or ties the bound m2 (prune_bound's argument, with delta more: m2
  // bounds the prefilter's value). Finite, so that an infinite lower bound never
  // passes.
  static __device__ __forceinline__ float boxes(float m2, const float4& q) {
    const float w = fabsf(q.w);  // 2^-20 R
    const float slack = 5.0f * w + 0x1p-18f * fmaxf(fabsf(q.x), fmaxf(fabsf(q.y), fabsf(q.z)));
    const float s = __builtin_amdgcn_sqrtf(m2) * (1.0f + 0x1p-20f) + slack;
    return fminf(s * s * (1.0f + 0x1p-20f), 0x1.fffffep127f);
  }
  template <typename Scratch>
  __device__ __forceinline__ const Node4* nodes(Scratch* W, uint32_t o) const {
    return (const Node4*)W->own.base[o];
  }
  template <typename Scratch>
  __device__ __forceinline__ void quick(Scratch* W, uint32_t o, const float4& p, int64_t i, float& lo, float& up,
                                        bool& always) const {
    float d2, m;
    quick_dist(p.x, p.y, p.z, W->own.base[o] + ((uint64_t)W->own.off_quick[o] << 8), i, d2, m, always);
    lo = d2 - m;
    up = d2 + m;
  }
  template <bool kStats, typename Scratch>
  __device__ __forceinline__ void exact(Scratch* W, uint32_t o, int32_t s, bool now, const float4& q,
                                        TravCount& cnt) const {
    if (!now) return;
    const TriRec T = gload_tri((const TriRec*)(W->own.base[o] + ((uint64_t)W->own.off_tris[o] << 8)), s);
    const float reject = __uint_as_float((uint32_t)(W->own.key[o] >> 32));
    float l1, l2, den;
    int region = 0;
    const float d = tri_dist2(q.x, q.y, q.z, T, reject, l1, l2, den, region);
    if (kStats) cnt.flops += kTriFlops[region & 7];
    if (d <= reject) {
      int32_t orig;
      memcpy(&orig, &T.a.w, 4);
      const unsigned long long key = ((unsigned long long)__float_as_uint(d) << 32) | (uint32_t)orig;
      atomicMin(&W->own.key[o], key);
      atomicMin(&W->m2[o], __float_as_uint(bound_of(d)));
      lds_order();
      if (W->own.key[o] == key) W->own.rec_slot[o] = s;
    }
  }
};

// Sets up owner `lane`'s search at (x, y, z), |p| <= 3 R; search_push puts it
// on the stack. `warm` names a slot whose triangle's upper value is the first
// bound (negative: none).
template <typename Scratch>
__device__ __forceinline__ void search_start(Scratch* W, uint32_t lane, const Node4* nodes, const float4* quick,
                                             const TriRec* tris, float radius, float x, float y, float z,
                                             int32_t warm) {
  float m2 = INFINITY;
  if (warm >= 0) {
    float d2, m;
    bool always;
    quick_dist(x, y, z, quick, quick_index(warm), d2, m, always);
    m2 = fminf(d2 + m, INFINITY);  // (no bound where the value overflowed)
  }
  W->pt[lane] = make_float4(x, y, z, 0x1p-20f * radius);
  W->m2[lane] = __float_as_uint(m2);
  W->own.key[lane] = ((unsigned long long)__float_as_uint(INFINITY) << 32) | (uint32_t)INT_MAX;
  W->own.rec_slot[lane] = -1;
  W->own.base[lane] = (const char*)nodes;
  W->own.off_quick[lane] = (uint32_t)(((const char*)quick - (const char*)nodes) >> 8);
  W->own.off_tris[lane] = (uint32_t)(((const char*)tris - (const char*)nodes) >> 8);
}

// Answer of an owner whose search has ended and whose pending tests are done.
// Returns false if the exact minimum lies above what the prefilter's bound
// promised: the search has been set up to run again (its root is to be
// pushed), from then on on exact values.
template <typename Scratch>
__device__ __forceinline__ bool search_answer(Scratch* W, uint32_t lane, Nearest& h) {
  const unsigned long long k = W->own.key[lane];
  h.d2 = __uint_as_float((uint32_t)(k >> 32));
  h.orig = (int32_t)(uint32_t)k;
  h.slot = W->own.rec_slot[lane];
  const float w = W->pt[lane].w;
  if (w >= 0.0f && h.d2 > keep_bound(__uint_as_float(W->m2[lane]), w)) {
    W->m2[lane] = __float_as_uint(bound_of(h.d2));
    W->pt[lane].w = -w;
    return false;
  }
  return true;
}

// The answer's barycentrics: the exact test of its triangle once more.
__device__ __forceinline__ void answer_bary(const TriRec* tris, float px, float py, float pz, Nearest& h) {
  h.l1 = h.l2 = 0.0f;
  h.den = 1.0f;
  if (h.slot < 0) return;
  float l1 = 0.0f, l2 = 0.0f, den = 1.0f;
  int region = 0;
  (void)tri_dist2(px, py, pz, gload_tri(tris, h.slot), INFINITY, l1, l2, den, region);
  h.l1 = l1;
  h.l2 = l2;
  if (region == 6) h.den = den;
}

// ------------------------------------------------------ walk machinery

// Rows that a launch's walks start from: the instantiations for point rows and
// for the PSD estimator's tangent balls leave the other starts and
// contributions out of the persistent kernel's code.
enum RowKind { kRowsAny, kRowsPoints, kRowsBalls };

struct LaneWalk {
  float x, y, z;
  int32_t row;
  uint32_t walk;
  int32_t mesh;
  int32_t step;
  int32_t queries;
  int32_t slot;  // warm-start triangle slot
  int32_t active;
  int32_t tab;    // wavefront row table of the walk (-1: device atomics)
  uint32_t ux, uy;  // direction uniforms of the current step (drawn before its query)
};

// Orthonormal frame (e1, e2) completing a unit vector n (branchless, after
// Duff et al. 2017).
__device__ __forceinline__ void onb(double nx, double ny, double nz, double e1[3], double e2[3]);

// Calls f(mesh) for each mesh among the lanes with `in`, the lanes of other
// meshes masked (all lanes call it; f gets whether the lane takes part). The
// lanes of a wavefront nearly always share one mesh, whose descriptor then
// comes through scalar loads: read per lane, a dozen dependent global loads
// stood in every walk step.
template <typename F>
__device__ __forceinline__ void wave_meshes(const WalkLaunch& L, bool in, int32_t mesh, F f) {
  for (uint64_t todo = __ballot(in); todo != 0;) {
    const int32_t m = __builtin_amdgcn_readlane(mesh, __ffsll((unsigned long long)todo) - 1);
    const bool mine = in && mesh == m;
    f(((ConstMesh*)L.meshes)[m], mine);
    todo &= ~__ballot(mine);
  }
}

// Start of a walk of the PSD estimator (Sec. 3.2, Alg. 2): a point z on the
// tangent ball of row i's sample s (centre c = s - r n), drawn with density
// proportional to the ball's jump kernel 1 / (2 pi |s - z|^3) outside the cap
// of polar angle theta0 about s: u = sin(theta / 2) has density
// proportional to 1 / u^2 on [sin(theta0 / 2), 1], inverted in closed form,
// and the azimuth is uniform. Walks 2j and 2j + 1 are the antithetic pair j
// (azimuth and azimuth + pi). Returns false if the row has no tangent ball.
template <typename MD>
__device__ bool ball_start(const WalkLaunch& L, const MD& M, LaneWalk& w, int32_t& face) {
  const double r = (double)gload(M.ball_r, w.row);
  if (!(r > 0.0)) return false;
  face = gload(M.tri, w.row);
  const double sx = gload(M.p, 3 * w.row), sy = gload(M.p, 3 * w.row + 1), sz = gload(M.p, 3 * w.row + 2);
  double nx = gload(M.n, 3 * w.row), ny = gload(M.n, 3 * w.row + 1), nz = gload(M.n, 3 * w.row + 2);
  const double nl = sqrt(nx * nx + ny * ny + nz * nz);
  nx /= nl; ny /= nl; nz /= nl;
  const double cx = sx - r * nx, cy = sy - r * ny, cz = sz - r * nz;
  const uint4 u = draw(L, (uint32_t)w.row, w.walk >> 1, 0, kPurposeBall, (uint32_t)M.mesh_id);
  const double xi = unit_f(u.x), eta = unit_f(u.y);
  const double su = 1.0 / (1.0 / M.ball_u0 - xi * (1.0 / M.ball_u0 - 1.0));
  const double ct = 1.0 - 2.0 * su * su, st = 2.0 * su * sqrt(fmax(0.0, 1.0 - su * su));
  double sp, cp;
  sincospi(2.0 * eta + ((w.walk & 1u) ? 1.0 : 0.0), &sp, &cp);
  double e1[3], e2[3];
  onb(nx, ny, nz, e1, e2);
  w.x = (float)(cx + r * (ct * nx + st * (cp * e1[0] + sp * e2[0])));
  w.y = (float)(cy + r * (ct * ny + st * (cp * e1[1] + sp * e2[1])));
  w.z = (float)(cz + r * (ct * nz + st * (cp * e1[2] + sp * e2[2])));
  w.slot = gload(M.slot_of_tri, face);
  w.step = 0;
  w.queries = 0;
  return true;
}

// Start of a walk: sample s (point rows: the fixed sample; hat rows:
// s ~ phi_i / A_i on the vertex's one-ring), inset it along the face normal.
// Returns false if the row is discarded.
template <RowKind kRows, typename MD>
__device__ bool walk_start(const WalkLaunch& L, const MD& M, LaneWalk& w, int32_t& face, double lam[3]) {
  if (kRows == kRowsBalls || (kRows == kRowsAny && M.ball_r)) return ball_start(L, M, w, face);
  const float sgn = M.side ? 1.0f : -1.0f;
  float sx, sy, sz, nx, ny, nz;
  if (kRows == kRowsPoints || M.mode == kRowsPoint) {
    if (gload(M.discarded, w.row)) return false;
    face = gload(M.tri, w.row);
    sx = gload(M.p, 3 * w.row); sy = gload(M.p, 3 * w.row + 1); sz = gload(M.p, 3 * w.row + 2);
    nx = gload(M.n, 3 * w.row); ny = gload(M.n, 3 * w.row + 1); nz = gload(M.n, 3 * w.row + 2);
    lam[0] = gload(M.bary, 3 * w.row); lam[1] = gload(M.bary, 3 * w.row + 1); lam[2] = gload(M.bary, 3 * w.row + 2);
  } else {
    const uint4 u = draw(L, (uint32_t)w.row, w.walk, 0, kPurposeHatStart, (uint32_t)M.mesh_id);
    const uint4 v = draw(L, (uint32_t)w.row, w.walk, 0, kPurposeSplit, (uint32_t)M.mesh_id);
    const int32_t b0 = gload(M.ring_ptr, w.row), b1 = gload(M.ring_ptr, w.row + 1);
    const double target = (double)unit_f(u.x) * gload(M.ring_cum, b1 - 1);
    int32_t e = b0;
    while (e < b1 - 1 && !(gload(M.ring_cum, e) > target)) ++e;
    face = gload(M.ring_tri, e);
    const float m1 = unit_f(u.y), m2 = unit_f(u.z), m3 = unit_f(u.w);
    const float li = fmaxf(fminf(m1, m2), fminf(fmaxf(m1, m2), m3));  // median: Beta(2,2)
    const float sv = unit_f(v.x);
    const int64_t f3 = 3 * (int64_t)face;
    const int32_t f[3] = {gload(M.faces, f3), gload(M.faces, f3 + 1), gload(M.faces, f3 + 2)};
    const int corner = f[0] == w.row ? 0 : (f[1] == w.row ? 1 : 2);
    // products of 24-bit values are exact in FP64: the weights sum to 1
    const double la = (1.0 - (double)li) * (double)sv, lb = (1.0 - (double)li) * (1.0 - (double)sv);
    lam[0] = corner == 0 ? (double)li : la;
    lam[1] = corner == 1 ? (double)li : (corner == 0 ? la : lb);
    lam[2] = corner == 2 ? (double)li : lb;
    const TriRec T = gload_tri(M.tris, gload(M.slot_of_tri, face));
    const float l0 = (float)lam[0], l1 = (float)lam[1], l2 = (float)lam[2];
    sx = l0 * T.a.x + l1 * T.b.x + l2 * T.c.x;
    sy = l0 * T.a.y + l1 * T.b.y + l2 * T.c.y;
    sz = l0 * T.a.z + l1 * T.b.z + l2 * T.c.z;
    nx = gload(M.face_normals, 3 * face); ny = gload(M.face_normals, 3 * face + 1); nz = gload(M.face_normals, 3 * face + 2);
  }
  const float h = M.inset;
  w.x = sx + sgn * h * nx;
  w.y = sy + sgn * h * ny;
  w.z = sz + sgn * h * nz;
  w.slot = gload(M.slot_of_tri, face);
  w.step = 0;
  w.queries = 0;
  return true;
}

// Sparse merge of up to NH sorted table rows with weights: emits each column
// once with sum_h weight_h * value_h (FP64).
template <int NH, typename MD, typename Emit>
__device__ __forceinline__ void merge_rows(const MD& M, const int32_t (&vtx)[NH], const double (&wt)[NH],
                                           Emit emit) {
  int32_t p[NH], e[NH];
#pragma unroll
  for (int k = 0; k < NH; ++k) {
    if (vtx[k] >= 0 && wt[k] != 0.0) {
      p[k] = gload(M.b_rowptr, vtx[k]);
      e[k] = gload(M.b_rowptr, vtx[k] + 1);
    } else {
      p[k] = 0;
      e[k] = 0;
    }
  }
  while (true) {
    int32_t cmin = INT_MAX;
    int32_t col[NH];
#pragma unroll
    for (int k = 0; k < NH; ++k) {
      col[k] = p[k] < e[k] ? gload(M.b_col, p[k]) : INT_MAX;
      cmin = min(cmin, col[k]);
    }
    if (cmin == INT_MAX) break;
    double v = 0.0;
#pragma unroll
    for (int k = 0; k < NH; ++k) {
      if (col[k] == cmin) {
        v += wt[k] * (double)gload(M.b_val, p[k]);
        ++p[k];
      }
    }
    emit(cmin, v);
  }
}

// ---- point basis (point-based k-NN interpolator)
// The k nearest sample points of q, as the k smallest (squared FP32 distance,
// index) pairs, searched ring by ring of grid cells around q's cell: after
// ring R every unvisited point lies outside the block of (2R + 1)^3 cells, so
// the search ends once the k-th distance is below the squared distance from q
// to that block's boundary (with a margin for rounding) or the block covers
// the grid. Weights exp(-d^2 / (2 sigma^2)) exp(-(1 - n_q . n_j) / tau),
// normalised (equal shares if all underflow). Returns the neighbour count.
__device__ __noinline__ int knn_eval(const KnnDev& G, float qx, float qy, float qz, double nqx, double nqy,
                                     double nqz, int32_t idx[kMaxKnn], double w[kMaxKnn]) {
#pragma clang fp contract(off)
  const int k = G.k;
  float bd[kMaxKnn];
  int m = 0;
  const float q[3] = {qx, qy, qz};
  int c[3];
  for (int a = 0; a < 3; ++a) {
    int ci = (int)floorf((q[a] - G.lo[a]) / G.cell);
    c[a] = min(max(ci, 0), G.dim[a] - 1);
  }
  for (int R = 0;; ++R) {
    for (int dz = -R; dz <= R; ++dz) {
      const int z = c[2] + dz;
      if (z < 0 || z >= G.dim[2]) continue;
      for (int dy = -R; dy <= R; ++dy) {
        const int y = c[1] + dy;
        if (y < 0 || y >= G.dim[1]) continue;
        const bool face = (dz == -R || dz == R || dy == -R || dy == R);
        for (int dx = -R; dx <= R; dx += (face ? 1 : 2 * R)) {
          const int x = c[0] + dx;
          if (x >= 0 && x < G.dim[0]) {
            const int64_t cid = ((int64_t)z * G.dim[1] + y) * G.dim[0] + x;
            for (int32_t e = gload(G.cell_start, cid); e < gload(G.cell_start, cid + 1); ++e) {
              const int32_t j = gload(G.cell_pts, e);
              const float4 pj = gload4(G.pts, j);
              const float ex = qx - pj.x, ey = qy - pj.y, ez = qz - pj.z;
              float d2 = ex * ex;
              d2 = d2 + ey * ey;
              d2 = d2 + ez * ez;
              if (m == k && !(d2 < bd[k - 1] || (d2 == bd[k - 1] && j < idx[k - 1]))) continue;
              int pos = m < k ? m++ : k - 1;
              while (pos > 0 && (d2 < bd[pos - 1] || (d2 == bd[pos - 1] && j < idx[pos - 1]))) {
                bd[pos] = bd[pos - 1];
                idx[pos] = idx[pos - 1];
                --pos;
              }
              bd[pos] = d2;
              idx[pos] = j;
            }
          }
          if (R == 0) break;
        }
      }
    }
    bool covers = true;
    float gap = INFINITY;
    for (int a = 0; a < 3; ++a) {
      covers = covers && c[a] - R <= 0 && c[a] + R >= G.dim[a] - 1;
      const float blo = G.lo[a] + (float)(c[a] - R) * G.cell, bhi = G.lo[a] + (float)(c[a] + R + 1) * G.cell;
      gap = fminf(gap, fminf(q[a] - blo, bhi - q[a]));
    }
    if (covers) break;
    if (m == k && gap > 0.0f && bd[k - 1] < (gap * gap) * (1.0f - 0x1p-16f)) break;
  }
  double sum = 0.0;
  for (int a = 0; a < m; ++a) {
    const float4 nj = gload4(G.nrm, idx[a]);
    w[a] = exp(-(double)bd[a] * G.inv2s2) * exp(-(1.0 - (nqx * nj.x + nqy * nj.y + nqz * nj.z)) * G.inv_tau);
    sum += w[a];
  }
  for (int a = 0; a < m; ++a) w[a] = sum > 0.0 ? w[a] / sum : 1.0 / m;
  return m;
}

// Hit point and unit face normal of a walk's nearest triangle (FP64 from the
// FP32 vertices and barycentrics), then the point basis there. Not inlined:
// the walk kernels keep their registers for the walk itself.
__device__ __noinline__ int knn_at_hit(const MeshDev& M, const Nearest& hit, int32_t idx[kMaxKnn],
                                       double w[kMaxKnn]) {
  double t[3], n[3];
  const TriRec T = gload_tri(M.tris, hit.slot);
  float b1, b2;
  nearest_bary(hit, b1, b2);
  const double l1 = b1, l2 = b2, l0 = (1.0 - l1) - l2;
  const double a[3] = {T.a.x, T.a.y, T.a.z}, b[3] = {T.b.x, T.b.y, T.b.z}, c[3] = {T.c.x, T.c.y, T.c.z};
  double e1[3], e2[3];
  for (int k = 0; k < 3; ++k) {
    t[k] = l0 * a[k] + l1 * b[k] + l2 * c[k];
    e1[k] = b[k] - a[k];
    e2[k] = c[k] - a[k];
  }
  n[0] = e1[1] * e2[2] - e1[2] * e2[1];
  n[1] = e1[2] * e2[0] - e1[0] * e2[2];
  n[2] = e1[0] * e2[1] - e1[1] * e2[0];
  const double nl = sqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
  if (nl > 0.0)
    for (int k = 0; k < 3; ++k) n[k] /= nl;
  return knn_eval(M.knn, (float)t[0], (float)t[1], (float)t[2], n[0], n[1], n[2], idx, w);
}

// Contribution of a finished walk to its row, emitted once per column:
// point rows emit b(t) (the start is fixed per row; the finalisation folds
// in b(s)), hat rows emit c = b(s) - b(t). Escaped walks have b(t) = 0.
template <bool kKnn, RowKind kRows, typename MD, typename Emit>
__device__ void walk_contrib(const WalkLaunch& L, const MD& M, const LaneWalk& w, bool has_t, const Nearest& hit,
                             Emit emit) {
  if (kRows == kRowsBalls || (kRows == kRowsAny && M.ball_r)) return;  // PSD walks: the rank-one updates are formed from the walk log
  if constexpr (kKnn) {  // point basis: b(t) from the hit point's k nearest samples (point rows)
    if (M.knn.k > 0) {
      if (has_t) {
        int32_t idx[kMaxKnn];
        double wk[kMaxKnn];
        const int m = knn_at_hit(*(const MeshDev*)&M, hit, idx, wk);
        for (int a = 0; a < m; ++a) emit(idx[a], wk[a]);
      }
      return;
    }
  }
  int32_t tv[3] = {-1, -1, -1};
  double tw[3] = {0.0, 0.0, 0.0};
  if (has_t) {
    const int64_t f3 = 3 * (int64_t)hit.orig;
    const int32_t f[3] = {gload(M.faces, f3), gload(M.faces, f3 + 1), gload(M.faces, f3 + 2)};
    tv[0] = f[0]; tv[1] = f[1]; tv[2] = f[2];
    float b1, b2;
    nearest_bary(hit, b1, b2);
    const double l1 = b1, l2 = b2;
    tw[0] = (1.0 - l1) - l2; tw[1] = l1; tw[2] = l2;
  }
  if (kRows == kRowsPoints || M.mode == kRowsPoint) {
    if (has_t) merge_rows<3>(M, tv, tw, emit);
  } else {
    int32_t face;
    double lam[3];
    LaneWalk tmp = w;
    walk_start<kRows>(L, M, tmp, face, lam);
    const int64_t f3 = 3 * (int64_t)face;
    const int32_t f[3] = {gload(M.faces, f3), gload(M.faces, f3 + 1), gload(M.faces, f3 + 2)};
    const int32_t vv[6] = {f[0], f[1], f[2], tv[0], tv[1], tv[2]};
    const double ww[6] = {lam[0], lam[1], lam[2], -tw[0], -tw[1], -tw[2]};
    merge_rows<6>(M, vv, ww, emit);
  }
}

// Walk log of a finished walk.
template <typename MD>
__device__ void walk_record(const WalkLaunch& L, const MD& M, const LaneWalk& w, int32_t status, bool has_t,
                            const Nearest& hit) {
  if (M.log_status) {
    const int64_t li = (int64_t)w.row * M.walks_per_row + ((int64_t)w.walk - L.walk_offset);
    gstore(M.log_status, li, status);
    gstore(M.log_tri, li, has_t ? hit.orig : -1);
    float b1, b2;
    nearest_bary(hit, b1, b2);
    gstore(M.log_bary, 2 * li, has_t ? b1 : 0.0f);
    gstore(M.log_bary, 2 * li + 1, has_t ? b2 : 0.0f);
    gstore(M.log_queries, li, w.queries);
  }
}

template <typename MD>
__device__ __forceinline__ bool walk_has_t(const MD& M, int32_t status, const Nearest& hit) {
  return status != kEscaped && hit.orig >= 0 && hit.orig < M.n_tris;
}

// Scatter a finished walk straight into its row with FP64 device atomics.
template <bool kKnn = false, typename MD>
__device__ void walk_finish_global(const WalkLaunch& L, const MD& M, const LaneWalk& w, int32_t status,
                                   const Nearest& hit) {
  const bool has_t = walk_has_t(M, status, hit);
  double* a1 = M.acc1 + (int64_t)w.row * M.K;
  double* a2 = M.acc2 + (int64_t)w.row * M.K;
  walk_contrib<kKnn, kRowsAny>(L, M, w, has_t, hit, [&](int32_t j, double v) {
    gadd(a1, j, v);
    gadd(a2, j, v * v);
  });
  gadd(M.row_queries, w.row, (unsigned long long)w.queries);
  if (status == kEscaped) gadd(M.row_escaped, w.row, 1ull);
  if (status == kCapped) gadd(M.row_capped, w.row, 1ull);
  walk_record(L, M, w, status, has_t, hit);
}

// ---- wavefront row tables (persistent form)
// Each wavefront owns two small open-addressing tables in LDS, column ->
// (sum v, sum v^2), plus the row's query / escape / cap counts. The walks of
// one queue chunk (one row) add into one table with LDS atomics; when the
// chunk's last walk has finished, the wavefront flushes the table into the
// FP64 row with one device atomic per distinct column. AccT = double keeps
// the partial sums in FP64; AccT = float keeps them in FP32 (a chunk holds at
// most `chunk` walks) and flushes them into the FP64 rows; AccT = CompF32
// keeps them as compensated FP32 pairs.
// Row-table slots per wavefront table (2^bits) and the occupancy the
// persistent kernels are compiled for: with 64 slots, FP64 tables and four
// search scratches take 40,192 B of the 40,960 that let a CU hold the four
// workgroups which persistent launches count on (kLdsPerBlock).
// The streaming kernel measured fastest on gfx950 at 4 waves per SIMD (128
// VGPRs, few spills) against 3 (no spills) and 5, 6 (many spills); 32-slot
// tables lost to their extra device atomics and 128 slots gained nothing.
#ifndef MSK_TABLE_SLOT_BITS
#define MSK_TABLE_SLOT_BITS 6
#endif
constexpr int kSlotBits = MSK_TABLE_SLOT_BITS, kSlots = 1 << kSlotBits, kProbes = 8, kWaves = 4;
static_assert(kSlots == 64, "record_point_walks harvests one slot per lane");
constexpr size_t kLdsPerBlock = 160 * 1024 / 4;
constexpr int32_t kEmptyKey = -1;

// Compensated FP32 partial sum: the value is hi + lo, a double-float pair.
// An addition of x = xh + xl (the FP64 contribution split into two floats)
// forms s = fl(hi + xh) and its exact rounding error e by Knuth's TwoSum,
// then lo += e + xl; the pair is one 64-bit LDS word replaced by
// compare-and-swap, so concurrent lanes on one slot serialise and none is
// lost. The sum's error is then of order u^2 n max|x| plus u |sum| for the
// final rounding of lo, instead of u n max|x| for a plain FP32 sum (u =
// 2^-24, n terms).
struct CompF32 {
  float hi, lo;
};

template <typename AccT>
__device__ __forceinline__ AccT acc_zero() {
  return (AccT)0;
}
template <>
__device__ __forceinline__ CompF32 acc_zero<CompF32>() {
  return CompF32{0.0f, 0.0f};
}
__device__ __forceinline__ double acc_value(double a) { return a; }
__device__ __forceinline__ double acc_value(float a) { return (double)a; }
__device__ __forceinline__ double acc_value(CompF32 a) { return (double)a.hi + (double)a.lo; }

__device__ __forceinline__ void lds_acc_add(double* p, double v) { atomicAdd(p, v); }
__device__ __forceinline__ void lds_acc_add(float* p, double v) { atomicAdd(p, (float)v); }
__device__ __forceinline__ void lds_acc_add(CompF32* p, double v) {
#pragma clang fp contract(off)
  const float xh = (float)v;
  const float xl = (float)(v - (double)xh);
  unsigned long long* q = reinterpret_cast<unsigned long long*>(p);
  unsigned long long old = __atomic_load_n(q, __ATOMIC_RELAXED), seen;
  do {
    seen = old;
    const float hi = __uint_as_float((uint32_t)seen), lo = __uint_as_float((uint32_t)(seen >> 32));
    const float sum = hi + xh;
    const float bv = sum - hi;
    const float err = (hi - (sum - bv)) + (xh - bv);
    const float nlo = lo + (err + xl);
    const unsigned long long nw =
        (unsigned long long)__float_as_uint(sum) | ((unsigned long long)__float_as_uint(nlo) << 32);
    old = atomicCAS(q, seen, nw);
  } while (old != seen);
}

// The same additions where one lane alone adds to the slot.
__device__ __forceinline__ void slot_add(double* p, double v) { *p += v; }
__device__ __forceinline__ void slot_add(float* p, double v) { *p += (float)v; }
__device__ __forceinline__ void slot_add(CompF32* p, double v) { lds_acc_add(p, v); }

template <typename AccT>
struct WaveTables {
  int32_t key[kWaves][2][kSlots];
  AccT v1[kWaves][2][kSlots];
  AccT v2[kWaves][2][kSlots];
  unsigned long long cnt[kWaves][2][3];
};

template <typename AccT>
__device__ __forceinline__ void table_add(WaveTables<AccT>& T, int wi, int t, int32_t j, double v, double* g1,
                                          double* g2) {
  const uint32_t h = ((uint32_t)j * 2654435761u) >> (32 - kSlotBits);
#pragma unroll 1
  for (int p = 0; p < kProbes; ++p) {
    const uint32_t si = (h + (uint32_t)p) & (kSlots - 1);
    const int32_t old = atomicCAS(&T.key[wi][t][si], kEmptyKey, j);
    if (old == kEmptyKey || old == j) {
      lds_acc_add(&T.v1[wi][t][si], v);
      lds_acc_add(&T.v2[wi][t][si], v * v);
      return;
    }
  }
  gadd(g1, j, v);  // table full along this probe sequence
  gadd(g2, j, v * v);
}

// Records an ended walk: its row's counters and log, and (with `contrib`) its
// contribution, into its row table if it has one, else into the row itself.
template <typename AccT, bool kKnn, RowKind kRows, typename MD>
__device__ void walk_finish(const WalkLaunch& L, const MD& M, const LaneWalk& w, int32_t status, bool contrib,
                            const Nearest& hit, WaveTables<AccT>& T, int wi) {
  const bool has_t = walk_has_t(M, status, hit);
  const bool tab = w.tab >= 0;
  if (contrib) {
    double* a1 = M.acc1 + (int64_t)w.row * M.K;
    double* a2 = M.acc2 + (int64_t)w.row * M.K;
    walk_contrib<kKnn, kRows>(L, M, w, has_t, hit, [&](int32_t j, double v) {
      if (tab) {
        table_add(T, wi, w.tab, j, v, a1, a2);
      } else {
        gadd(a1, j, v);
        gadd(a2, j, v * v);
      }
    });
  }
  if (tab) {
    atomicAdd(&T.cnt[wi][w.tab][0], (unsigned long long)w.queries);
    if (status == kEscaped) atomicAdd(&T.cnt[wi][w.tab][1], 1ull);
    if (status == kCapped) atomicAdd(&T.cnt[wi][w.tab][2], 1ull);
  } else {
    gadd(M.row_queries, w.row, (unsigned long long)w.queries);
    if (status == kEscaped) gadd(M.row_escaped, w.row, 1ull);
    if (status == kCapped) gadd(M.row_capped, w.row, 1ull);
  }
  walk_record(L, M, w, status, has_t, hit);
}

__device__ __forceinline__ double shfl_f64(double v, int src) {
  const int lo = __shfl(__double2loint(v), src), hi = __shfl(__double2hiint(v), src);
  return __hiloint2double(hi, lo);
}

// Contributions of ended point-row walks with a row table and a per-vertex
// basis table, two walks at a time, 32 lanes each (all lanes of the wavefront
// call it; `mine`: this lane's walk is one). The entries of the hit triangle's
// three table rows are read at once, one per lane; equal columns meet in the
// row table's slots, where their FP64 sum v forms before it goes into sum v and
// sum v^2. Merged by one lane per walk, entry by entry, each of up to 24
// columns waited for a load and a chain of LDS atomics: 13% of the soup
// operator's time. Walks whose columns do not fit their row table are left for
// walk_finish: the lanes whose walk is done get true.
template <typename AccT, typename MD>
__device__ __forceinline__ bool record_point_walks(const MD& M, SearchScratch<TriEl>* W, uint32_t lane, bool mine, int32_t tab,
                                                   const Nearest& hit, WaveTables<AccT>& T, int wi) {
  int32_t p[3] = {0, 0, 0}, n[3] = {0, 0, 0};
  double wt[3] = {0.0, 0.0, 0.0};
  if (mine) {
    float b1, b2;
    nearest_bary(hit, b1, b2);
    wt[1] = b1;
    wt[2] = b2;
    wt[0] = (1.0 - wt[1]) - wt[2];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int32_t v = gload(M.faces, 3 * (int64_t)hit.orig + k);
      p[k] = gload(M.b_rowptr, v);
      n[k] = wt[k] != 0.0 ? gload(M.b_rowptr, v + 1) - p[k] : 0;
    }
  }
  W->sum[0][lane] = 0.0;
  W->sum[1][lane] = 0.0;
  lds_order();
  const int half = (int)(lane >> 5);
  bool ok = mine;
  for (uint64_t todo = __ballot(mine); todo != 0;) {
    const int a = __ffsll((unsigned long long)todo) - 1;
    todo &= todo - 1;
    const int b = todo != 0 ? __ffsll((unsigned long long)todo) - 1 : -1;
    todo &= todo - (b >= 0 ? 1 : 0);
    const int src = half ? max(b, 0) : a;
    const bool valid = half == 0 || b >= 0;
    const int32_t n0 = __shfl(n[0], src), n1 = __shfl(n[1], src), n2 = __shfl(n[2], src);
    const int32_t p0 = __shfl(p[0], src), p1 = __shfl(p[1], src), p2 = __shfl(p[2], src);
    const double w0 = shfl_f64(wt[0], src), w1 = shfl_f64(wt[1], src), w2 = shfl_f64(wt[2], src);
    const int32_t t = __shfl(tab, src);
    const int32_t tot = valid ? n0 + n1 + n2 : 0;
    bool fail = false;
    for (int32_t e = (int32_t)(lane & 31u); __ballot(e < tot) != 0; e += 32) {
      if (e < tot) {
        const int32_t i = e < n0 ? p0 + e : (e < n0 + n1 ? p1 + e - n0 : p2 + e - n0 - n1);
        const double wk = e < n0 ? w0 : (e < n0 + n1 ? w1 : w2);
        const int32_t j = gload(M.b_col, i);
        const double v = wk * (double)gload(M.b_val, i);
        const uint32_t h = ((uint32_t)j * 2654435761u) >> (32 - kSlotBits);
        bool placed = false;
        for (int q = 0; q < kProbes && !placed; ++q) {
          const uint32_t si = (h + (uint32_t)q) & (kSlots - 1);
          const int32_t old = atomicCAS(&T.key[wi][t][si], kEmptyKey, j);
          placed = old == kEmptyKey || old == j;
          if (placed) atomicAdd(&W->sum[half][si], v);
        }
        fail |= !placed;
      }
    }
    lds_order();
    const uint64_t bad = __ballot(fail);
    const int32_t ta = __shfl(tab, a), tb = __shfl(tab, max(b, 0));
    const double xa = W->sum[0][lane], xb = W->sum[1][lane];
    if (xa != 0.0 && (uint32_t)bad == 0u) {
      slot_add(&T.v1[wi][ta][lane], xa);
      slot_add(&T.v2[wi][ta][lane], xa * xa);
    }
    if (xb != 0.0 && (uint32_t)(bad >> 32) == 0u) {
      slot_add(&T.v1[wi][tb][lane], xb);
      slot_add(&T.v2[wi][tb][lane], xb * xb);
    }
    W->sum[0][lane] = 0.0;
    W->sum[1][lane] = 0.0;
    if ((uint32_t)bad != 0u && (int)lane == a) ok = false;
    if ((uint32_t)(bad >> 32) != 0u && (int)lane == b) ok = false;
    lds_order();
  }
  return ok;
}

// Wavefront-cooperative flush of table t into row `row` of mesh `mesh`.
template <typename AccT>
__device__ void table_flush(const WalkLaunch& L, WaveTables<AccT>& T, int wi, int t, int32_t mesh, int32_t row) {
  __builtin_amdgcn_wave_barrier();
  ConstMesh& F = ((ConstMesh*)L.meshes)[mesh];
  double* a1 = F.acc1 + (int64_t)row * F.K;
  double* a2 = F.acc2 + (int64_t)row * F.K;
  for (int i = (int)__lane_id(); i < kSlots; i += 64) {
    const int32_t j = T.key[wi][t][i];
    if (j != kEmptyKey) {
      gadd(a1, j, acc_value(T.v1[wi][t][i]));
      gadd(a2, j, acc_value(T.v2[wi][t][i]));
      T.key[wi][t][i] = kEmptyKey;
      T.v1[wi][t][i] = acc_zero<AccT>();
      T.v2[wi][t][i] = acc_zero<AccT>();
    }
  }
  if (__lane_id() == 0) {
    if (T.cnt[wi][t][0]) gadd(F.row_queries, row, T.cnt[wi][t][0]);
    if (T.cnt[wi][t][1]) gadd(F.row_escaped, row, T.cnt[wi][t][1]);
    if (T.cnt[wi][t][2]) gadd(F.row_capped, row, T.cnt[wi][t][2]);
    T.cnt[wi][t][0] = T.cnt[wi][t][1] = T.cnt[wi][t][2] = 0;
  }
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ void onb(double nx, double ny, double nz, double e1[3], double e2[3]) {
  const double sg = nz >= 0 ? 1.0 : -1.0;
  const double a = -1.0 / (sg + nz);
  const double b = nx * ny * a;
  e1[0] = 1.0 + sg * nx * nx * a; e1[1] = sg * b; e1[2] = -sg * nx;
  e2[0] = b; e2[1] = sg + ny * ny * a; e2[2] = -ny;
}

// One step of a live walk. Returns -1 while the walk continues, else its
// final status (hit / escaped / capped) with `hit` set for hits and caps.
// First half of a WoS step (Sec. 2; exterior roulette of Sec. 3.3): the step
// cap, and outside the bounding sphere escape or re-entry. Returns kEscaped
// when the walk ends here, else -1: the walk needs the nearest-triangle
// query at (w.x, w.y, w.z); `capped` marks the query that ends a capped walk.
template <typename MD>
__device__ int32_t walk_begin(const WalkLaunch& L, const MD& M, LaneWalk& w, bool& capped) {
  capped = w.step >= M.max_steps;
  // step cap: the walk ends at the nearest boundary point of its position
  if (capped) return -1;
  const uint4 u = draw(L, (uint32_t)w.row, w.walk, (uint32_t)w.step, kPurposeStep, (uint32_t)M.mesh_id);
  w.ux = u.x;
  w.uy = u.y;
  const float rho2 = w.x * w.x + w.y * w.y + w.z * w.z;
  const double rho = rho2 > M.radius * M.radius * (1.0f - 0x1p-18f)
                         ? sqrt((double)w.x * w.x + (double)w.y * w.y + (double)w.z * w.z)
                         : 0.0;
  if (rho > M.radius_d) {
    // Outside the bounding sphere: escape with probability 1 - R/rho, else
    // jump to the exact first hitting point of the sphere (density ~
    // |x-y|^-3, inverted in closed form).
    const double R = M.radius_d;
    if ((double)unit_f(u.z) < 1.0 - R / rho) return kEscaped;
    const double a = rho * rho + R * R, b = 2.0 * rho * R;
    const double qi = 1.0 / (rho + R) + (double)unit_f(u.w) * (1.0 / (rho - R) - 1.0 / (rho + R));
    const double mu = fmin(1.0, fmax(-1.0, (a - 1.0 / (qi * qi)) / b));
    const uint4 v = draw(L, (uint32_t)w.row, w.walk, (uint32_t)w.step, kPurposeReentry, (uint32_t)M.mesh_id);
    const double phi = 6.283185307179586 * (double)unit_f(v.x);
    const double nx = w.x / rho, ny = w.y / rho, nz = w.z / rho;
    double e1[3], e2[3];
    onb(nx, ny, nz, e1, e2);
    const double st = sqrt(fmax(0.0, 1.0 - mu * mu));
    double sp, cp;
    sincos(phi, &sp, &cp);
    w.x = (float)(R * (mu * nx + st * (cp * e1[0] + sp * e2[0])));
    w.y = (float)(R * (mu * ny + st * (cp * e1[1] + sp * e2[1])));
    w.z = (float)(R * (mu * nz + st * (cp * e1[2] + sp * e2[2])));
    // the walk goes on from the sphere in this same step (u.x, u.y unused so far)
  }
  return -1;
}

// Second half: with the query's answer in `hit`, stop in the eps-shell or
// take the ball step r (shrunk by the conservative guard) along a uniform
// direction. Returns kCapped / kHit when the walk ends, else -1.
template <typename MD>
__device__ int32_t walk_end(const MD& M, LaneWalk& w, bool capped, const Nearest& hit) {
  ++w.queries;
  if (capped) return kCapped;
  w.slot = hit.slot;
  if (hit.d2 < M.eps2) return kHit;
  const float r = sqrtf(hit.d2) * (1.0f - M.kappa) - M.delta;
  const float u0 = unit_f(w.ux), u1 = unit_f(w.uy);
  const float z = 1.0f - 2.0f * u0;
  const float rxy = 2.0f * sqrtf(u0 * (1.0f - u0));
  // v_sin/v_cos take the angle in revolutions: sin(2 pi u1), cos(2 pi u1)
  const float sn = __builtin_amdgcn_sinf(u1), cs = __builtin_amdgcn_cosf(u1);
  w.x += r * rxy * cs;
  w.y += r * rxy * sn;
  w.z += r * z;
  ++w.step;
  return -1;
}

// One whole step with a lane-private query (plain kernel).
template <bool kStats, typename MD>
__device__ int32_t walk_step(const WalkLaunch& L, const MD& M, LaneWalk& w, Nearest& hit, TravCount& cnt) {
  bool capped;
  const int32_t st = walk_begin(L, M, w, capped);
  if (st >= 0) return st;
  hit.d2 = INFINITY;
  hit.orig = INT_MAX;
  hit.slot = w.slot;
  bvh_nearest<kStats>(M.nodes, M.tris, w.x, w.y, w.z, M.radius, hit, cnt);
  return walk_end(M, w, capped, hit);
}

__device__ __forceinline__ void decode_walk(const WalkLaunch& L, uint64_t g, LaneWalk& w) {
  const uint64_t slot = g / (uint64_t)L.walks_per_slot;
  const auto& rs = ((const MSK_GLOBAL RowSlot*)L.slots)[slot];
  w.mesh = rs.mesh;
  w.row = rs.row;
  w.walk = (uint32_t)((int64_t)(g - slot * (uint64_t)L.walks_per_slot) + L.walk_offset + rs.walk0);
}

// ------------------------------------------------------------- kernels

// Plain form: one thread per walk, run to completion.
template <bool kStats, bool kKnn = false>
__global__ void __launch_bounds__(256) walk_plain_kernel(WalkLaunch L) {
  const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= (uint64_t)L.n_slots * (uint64_t)L.walks_per_slot) return;
  LaneWalk w;
  decode_walk(L, g, w);
  ConstMesh& M = ((ConstMesh*)L.meshes)[w.mesh];
  int32_t face;
  double lam[3];
  if (!walk_start<kRowsAny>(L, M, w, face, lam)) return;
  Nearest hit;
  TravCount cnt;
  int32_t st;
  do {
    st = walk_step<kStats>(L, M, w, hit, cnt);
  } while (st < 0);
  walk_finish_global<kKnn>(L, M, w, st, hit);
  if (kStats && L.stats) {
    atomicAdd(L.stats, (unsigned long long)cnt.nodes);
    atomicAdd(L.stats + 1, (unsigned long long)cnt.tris);
    atomicAdd(L.stats + 2, (unsigned long long)cnt.flops);
  }
}

__device__ __forceinline__ uint32_t lane_id() { return __lane_id(); }

#ifndef MSK_PERSISTENT_WAVES_PER_EU
#define MSK_PERSISTENT_WAVES_PER_EU 4
#endif
#if MSK_PERSISTENT_WAVES_PER_EU > 0
#define MSK_PERSISTENT_OCCUPANCY __attribute__((amdgpu_waves_per_eu(MSK_PERSISTENT_WAVES_PER_EU)))
#else
#define MSK_PERSISTENT_OCCUPANCY
#endif
// lanes with an answered query that trigger the step continuation (8, 12, 24
// and 32 measured the same)
#ifndef MSK_STEP_MIN
#define MSK_STEP_MIN 16
#endif
constexpr int kStepMin = MSK_STEP_MIN;
// Optional per-phase cycle counts of the streaming kernel (a measurement
// build only: -DMSK_PHASE_TIMING=1); phases are timed by the wavefront's
// shader clock at points every lane passes together.
#ifndef MSK_PHASE_TIMING
#define MSK_PHASE_TIMING 0
#endif
#if MSK_PHASE_TIMING
__device__ unsigned long long g_phase_cycles[16];
#define MSK_TICK(var) const uint64_t var = (uint64_t)__builtin_amdgcn_s_memtime()
#define MSK_ACC(i, a, b) ph[i] += (b) - (a)
#else
#define MSK_TICK(var)
#define MSK_ACC(i, a, b)
#endif

// Streaming form of the persistent kernel: the queries of a wavefront's walks
// run on its shared search (search_pass), so a walk whose query is long does
// not hold the others: walks whose query is answered wait until enough of them
// do (kStepMin), then finish their step and start the next query together;
// ended walks and idle lanes wait for the next bookkeeping pass (L.regen_min).
// At most L.max_owners lanes of a wavefront carry a walk: a launch of few
// walks spreads them over all wavefronts. The walks, their queries and their
// results are those of the other forms.
//   Bound by vector issue (0.79 of the issue rate over a batch's launch),
// with few walks by the longest walk's chain of queries, about 5 us each. Walk
// kernel with a stack per lane and exact tests of every listed triangle, and
// now: 2.0M walks among 53,000 triangles of the soup 15.4 -> 7.8 ms, 4.1M walks
// on a 500,000-face sphere 64.3 -> 27.6 ms, 41,472 walks on 320 faces 3.0 -> 1.0
// ms, a batch of 12 meshes 33.8 -> 20 ms.
template <bool kStats, typename AccT, bool kKnn, RowKind kRows>
__global__ void __launch_bounds__(256) MSK_PERSISTENT_OCCUPANCY walk_stream_kernel(WalkLaunch L) {
  __shared__ WaveTables<AccT> T;
  __shared__ SearchScratch<TriEl> coop[kWaves];
  static_assert(sizeof(T) + sizeof(coop) <= kLdsPerBlock, "four workgroups per CU");
  const int wi = (int)uniform(threadIdx.x >> 6);
  SearchScratch<TriEl>* W = &coop[wi];
  for (int i = threadIdx.x; i < kWaves * 2 * kSlots; i += blockDim.x) {
    (&T.key[0][0][0])[i] = kEmptyKey;
    (&T.v1[0][0][0])[i] = acc_zero<AccT>();
    (&T.v2[0][0][0])[i] = acc_zero<AccT>();
  }
  for (int i = threadIdx.x; i < kWaves * 2 * 3; i += blockDim.x) (&T.cnt[0][0][0])[i] = 0;
  __syncthreads();
  const uint32_t lane = __lane_id();
  const bool owner = lane < (uint32_t)L.max_owners;
  const int qhome = blockIdx.x & 7;
  // the wavefront's first chunk has its place in the home queue; the counters
  // hand out those after the first chunks of all (4096 atomics on 8 counters
  // at once took as long as a launch of few walks)
  const auto queue_first = [&](int q) {
    return (uint64_t)((gridDim.x + 7u - (uint32_t)q) >> 3) * kWaves * (uint64_t)L.chunk;
  };
  uint64_t cur = gload(L.queue_end, 8 + qhome) + (uint64_t)((blockIdx.x >> 3) * kWaves + wi) * (uint64_t)L.chunk;
  uint64_t cend = min(cur + (uint64_t)L.chunk, (uint64_t)gload(L.queue_end, qhome));
  cur = uniform64(min(cur, cend));
  cend = uniform64(cend);
  bool fresh_chunk = cur < cend;  // cur .. cend is a chunk whose table is not chosen yet
  // wave-uniform table bookkeeping
  int32_t t_used[2] = {0, 0}, t_mesh[2] = {0, 0}, t_row[2] = {0, 0}, t_out[2] = {0, 0};
  int32_t c_tab = -1, c_mesh = -1, c_row = -1;  // current chunk's row and table
  LaneWalk w;
  w.active = 0;
  w.tab = -1;
  // lane's state: mode 0 no walk, 1 searching, 2 search ended, 3 walk ended
  // (its answer stays in the wavefront's scratch until the next bookkeeping
  // pass records it), 4 at its start
  int32_t mode = 0, fin_status = -1;
  bool capped = false;
  uint32_t npend = 0, size = 0;  // pending exact tests and stack items of the wavefront (uniform)
  TravCount cnt;                 // statistics kernels: this lane's share of the work
  bool drained = false;
#if MSK_PHASE_TIMING
  uint64_t ph[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#endif
  while (true) {
    MSK_TICK(tk0);
    if (mode == 1 && W->open[lane] == 0) mode = 2;
    // (uniform by construction; said again so that all control flow below is
    // scalar)
    size = uniform(size);
    drained = uniform(drained ? 1u : 0u) != 0;
    // ---- what this pass does: `step` finishes the steps whose search has
    // ended and starts the next ones, once kStepMin lanes wait (a quarter of
    // the wavefront's walks if that is less) or the stack is empty; `book`
    // records ended walks and hands out new ones, once L.regen_min lanes wait
    // (those of ended walks no longer count when the queues are empty: they
    // wait for the last one) or no search is left; else a trip of the search
    const uint64_t pend = __ballot(mode == 2 || mode == 4), busy = __ballot(mode == 1) | pend;
    const bool step = pend != 0 && size <= (uint32_t)kRootLimit &&
                      (size == 0 || (int)__popcll(pend) >= min(kStepMin, (int)(__popcll(busy) + 3) >> 2));
    const bool book =
        !step && (size == 0 || (!drained && (int)__popcll(__ballot(mode == 3 || (mode == 0 && owner))) >= L.regen_min));
    search_pass<kStats>(TriEl{}, W, lane, !step && !book, step ? pend : ~0ull, size, npend, cnt);
    MSK_TICK(tk1);
    MSK_ACC(1, tk0, tk1);
#if MSK_PHASE_TIMING
    ph[6] += !step && !book;
    ph[7] += book;
#endif
    if (step) {
      bool fresh = false;
      int32_t entry = 1;
      wave_meshes(L, mode == 2 || mode == 4, w.mesh, [&](ConstMesh& M, bool mine) {
        if (!mine) return;
        int32_t st = -1;
        bool go = mode == 4;
        if (mode == 2) {
          Nearest hit;
          if (search_answer(W, lane, hit)) {
            st = walk_end(M, w, capped, hit);
            go = st < 0;
          } else {
            fresh = true;
            mode = 1;
          }
        }
        if (go) {
          st = walk_begin(L, M, w, capped);
          if (st < 0) {
            search_start(W, lane, M.nodes, M.quick, M.tris, M.radius, w.x, w.y, w.z, w.slot);
            fresh = true;
            mode = 1;
          }
        }
        if (st >= 0) {
          fin_status = st;
          mode = 3;
        }
        entry = M.entry;
      });
      search_push(W, lane, fresh, entry, size);
      MSK_TICK(tk2);
      MSK_ACC(5, tk1, tk2);
    }
    if (book) {
      MSK_TICK(tb0);
      const bool fin = mode == 3;
      const int32_t fin_tab = fin ? w.tab : -1;
      wave_meshes(L, fin, w.mesh, [&](ConstMesh& M, bool mine) {
        Nearest hit;
        hit.d2 = INFINITY;
        hit.orig = INT_MAX;
        hit.slot = -1;
        hit.l1 = hit.l2 = 0.0f;
        if (mine && fin_status != kEscaped) {
          const unsigned long long k = W->own.key[lane];
          hit.d2 = __uint_as_float((uint32_t)(k >> 32));
          hit.orig = (int32_t)(uint32_t)k;
          hit.slot = W->own.rec_slot[lane];
          const float4 q = W->pt[lane];
          answer_bary(M.tris, q.x, q.y, q.z, hit);
        }
        bool done = false;
        if constexpr (kRows == kRowsPoints && !kKnn)
          done = record_point_walks(M, W, lane, mine && w.tab >= 0 && walk_has_t(M, fin_status, hit), w.tab, hit, T, wi);
        if (mine) walk_finish<AccT, kKnn, kRows>(L, M, w, fin_status, !done, hit, T, wi);
      });
      if (fin) {
        w.active = 0;
        w.tab = -1;
        mode = 0;
      }
      MSK_TICK(tb1);
      MSK_ACC(2, tb0, tb1);
      for (int t2 = 0; t2 < 2; ++t2) {
        t_out[t2] -= (int32_t)__popcll(__ballot(fin && fin_tab == t2));
        // flush once the table's walks are done and its chunk hands out no more
        if (t_used[t2] && t_out[t2] == 0 && !(t2 == c_tab && cur < cend)) {
          table_flush(L, T, wi, t2, t_mesh[t2], t_row[t2]);
          t_used[t2] = 0;
          if (c_tab == t2) c_tab = -1;
        }
      }
      MSK_TICK(tb2);
      MSK_ACC(3, tb1, tb2);
      // refill idle lanes from the queue chunks
      uint64_t idle = __ballot(owner && !w.active);
      while (idle != 0 && !drained) {
        if (cur >= cend) {
          // the first queue from the home queue on that is not empty: all
          // counters are read at once, so that a wavefront takes its end from
          // one load instead of an atomic on each queue
          bool left = false;
          if (lane < 8u) {
            const int q = (qhome + (int)lane) & 7;
            left = __hip_atomic_load((MSK_GLOBAL unsigned long long*)L.queue_next + kQueueStride * q, __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT) + queue_first(q) < gload(L.queue_end, q);
          }
          const uint64_t some = __ballot(left);
          if (some == 0) {
            drained = true;
            continue;
          }
          const int q = (qhome + __ffsll((unsigned long long)some) - 1) & 7;
          uint64_t start = 0;
          if (lane == 0)
            start = __hip_atomic_fetch_add((MSK_GLOBAL unsigned long long*)L.queue_next + kQueueStride * q,
                                           (unsigned long long)L.chunk, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          start = uniform64(start) + queue_first(q);  // the first lane's
          const uint64_t qend = uniform64(gload(L.queue_end, q));
          if (start >= qend) continue;  // another wavefront took the last chunk
          cur = start;
          cend = min(start + (uint64_t)L.chunk, qend);
          fresh_chunk = true;
        }
        if (fresh_chunk) {
          fresh_chunk = false;
          // the chunk's row takes the table it already has, else a free one
          const auto& rs = ((const MSK_GLOBAL RowSlot*)L.slots)[cur / (uint64_t)L.walks_per_slot];
          c_mesh = (int32_t)uniform((uint32_t)rs.mesh);
          c_row = (int32_t)uniform((uint32_t)rs.row);
          c_tab = -1;
          for (int t2 = 0; t2 < 2; ++t2)
            if (t_used[t2] && t_mesh[t2] == c_mesh && t_row[t2] == c_row) c_tab = t2;
          if (c_tab < 0) {
            for (int t2 = 0; t2 < 2; ++t2)
              if (!t_used[t2] && c_tab < 0) {
                c_tab = t2;
                t_used[t2] = 1;
                t_mesh[t2] = c_mesh;
                t_row[t2] = c_row;
              }
          }
        }
        const uint32_t rank = __popcll(idle & ((1ull << lane) - 1ull));
        const uint64_t avail = cend - cur;
        const uint32_t take = (uint32_t)min(avail, (uint64_t)__popcll(idle));
        bool fresh = false;
        const bool start = owner && !w.active && rank < take;
        if (start) decode_walk(L, cur + rank, w);
        wave_meshes(L, start, w.mesh, [&](ConstMesh& M, bool mine) {
          if (!mine) return;
          int32_t face;
          double lam[3];
          w.active = walk_start<kRows>(L, M, w, face, lam) ? 1 : 0;
          w.tab = (w.active && c_tab >= 0 && w.mesh == c_mesh && w.row == c_row) ? c_tab : -1;
          mode = w.active ? 4 : 0;
          fresh = w.tab >= 0;
        });
        if (c_tab >= 0) t_out[c_tab] += (int32_t)__popcll(__ballot(fresh));
        cur += take;
        idle = __ballot(owner && !w.active);
        // lanes whose row was discarded stay idle
      }
      MSK_TICK(tb3);
      MSK_ACC(4, tb2, tb3);
      MSK_ACC(0, tb0, tb3);
      if (drained && __ballot(w.active) == 0) {
        for (int t2 = 0; t2 < 2; ++t2)
          if (t_used[t2]) {
            table_flush(L, T, wi, t2, t_mesh[t2], t_row[t2]);
            t_used[t2] = 0;
          }
        break;
      }
    }
  }
  if (kStats && L.stats) {
    atomicAdd(L.stats, (unsigned long long)cnt.nodes);
    atomicAdd(L.stats + 1, (unsigned long long)cnt.tris);
    atomicAdd(L.stats + 2, (unsigned long long)cnt.flops);
  }
#if MSK_PHASE_TIMING
  if (lane == 0)
    for (int i = 0; i < 8; ++i) atomicAdd(&g_phase_cycles[i], (unsigned long long)ph[i]);
#endif
}

__global__ void init_queues_kernel(unsigned long long* next, unsigned long long* end, QueueInit q) {
  const int i = threadIdx.x;
  if (i < 8) {
    next[kQueueStride * i] = q.begin[i];
    end[i] = q.end[i];
    end[8 + i] = q.begin[i];
  }
}

__global__ void fill_u64_kernel(unsigned long long* p, int64_t n, unsigned long long v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

__global__ void fill_u32_kernel(uint32_t* p, int64_t n, uint32_t v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// Largest ball inside the domain tangent at each point row's sample s, centre
// c = s - r n (Sec. 3.2; Alg. 2, LargestTangentBall): bisection over
// [0, r_max]; a radius is accepted when c's nearest surface point is at
// least t = r - min(tol, 2^-10 r) away and the ball lies inside the scene's
// bounding sphere. 0 = no radius accepted. Each step needs only whether some
// triangle lies closer than t, so its query starts from the bound
// B = t^2 (1 + 2^-20) instead of +inf (when a triangle has sqrt(d2) < t then
// d2 < B) and stops at the first triangle found with sqrt(d2) < t; when none
// lies below B the ball is accepted. Same decisions as comparing the exact
// nearest distance with t, with only the boxes near the ball visited.
//
// The bisection takes three levels per round: the eight lanes of a row take
// the (up to) seven midpoints of the next three levels at once (lane k heap
// node k of that subtree: node 1 the current midpoint, node 2k and 2k + 1 the
// midpoints of its lower and upper halves), then all follow the path the
// sequential bisection takes through them. Every midpoint is formed by the
// same float operations as in the sequential loop, so the radius is the same.
// The midpoints' queries run on the wavefront-shared search: a large ball deep
// inside the shape meets thousands of boxes, which all 64 lanes share. (On a
// lane each: 6.2 ms for 4,096 rows on 80,000 faces; now 0.4 ms, bound by vector
// issue.) rows_per_wave (1, 2, 4 or
// 8) is as low as still gives every resident wavefront rows. row_queries
// counts the bounded queries that the lanes issue (up to seven per round of
// three levels, so more than the iters decisions they serve).
__global__ void __launch_bounds__(256) MSK_PERSISTENT_OCCUPANCY
    tangent_ball_kernel(MeshDev M, int64_t n_rows, int32_t rows_per_wave, float r_max, int32_t iters, float tol,
                        float* radius) {
  __shared__ SearchScratch<TriEl, true> coop[kWaves];
  const int wi = (int)uniform(threadIdx.x >> 6);
  SearchScratch<TriEl, true>* W = &coop[wi];
  const uint32_t lane = __lane_id();
  const int sub = (int)(lane & 7u), gbase = (int)(lane & ~7u);
  TravCount cnt;
  uint32_t size = 0, npend = 0;
  const int64_t waves = (int64_t)gridDim.x * kWaves;
  for (int64_t base = ((int64_t)blockIdx.x * kWaves + wi) * rows_per_wave; base < n_rows;
       base += waves * rows_per_wave) {
    const int64_t i = base + (lane >> 3);
    const bool valid = (int32_t)(lane >> 3) < rows_per_wave && i < n_rows;
    float sx = 0.f, sy = 0.f, sz = 0.f;
    double nx = 0.0, ny = 0.0, nz = 1.0;
    if (valid) {
      sx = M.p[3 * i]; sy = M.p[3 * i + 1]; sz = M.p[3 * i + 2];
      nx = M.n[3 * i]; ny = M.n[3 * i + 1]; nz = M.n[3 * i + 2];
      const double nl = sqrt(nx * nx + ny * ny + nz * nz);
      nx /= nl; ny /= nl; nz /= nl;
    }
    float lo = 0.0f, hi = r_max;
    uint32_t issued = 0;
    for (int32_t done = 0; done < iters;) {
      const int levels = min(3, iters - done);
      // the lane's midpoint: whether its ball lies inside the bounding sphere,
      // and the bounded query for a triangle closer than t
      bool inside = false, fresh = false;
      float t = 0.0f;
      if (valid && sub >= 1 && sub < (1 << levels)) {
        float a = lo, b = hi;
        const int depth = 31 - __clz(sub);  // bits of the node index below its leading one
        for (int j = depth - 1; j >= 0; --j) {
          const float m = 0.5f * (a + b);
          if ((sub >> j) & 1)
            a = m;
          else
            b = m;
        }
        const float mid = 0.5f * (a + b);
        const double cxd = sx - mid * nx, cyd = sy - mid * ny, czd = sz - mid * nz;
        t = mid - fminf(tol, mid * 0x1p-10f);
        inside = sqrt(cxd * cxd + cyd * cyd + czd * czd) + mid <= M.radius_d;
        if (t > 0.0f) {
          ++issued;
          // a ball that leaves the bounding sphere is refused whatever the query says
          if (inside) {
            search_start(W, lane, M.nodes, M.quick, M.tris, M.radius, (float)cxd, (float)cyd, (float)czd, -1);
            const float bound = (t * t) * (1.0f + 0x1p-20f);
            W->m2[lane] = __float_as_uint(bound_of(bound));
            W->own.key[lane] = ((unsigned long long)__float_as_uint(bound) << 32) | (uint32_t)INT_MAX;
            // an upper value below `stop` means sqrt(exact value) < t
            const float ts = t - W->pt[lane].w;
            W->stop[lane] = ts > 0.0f ? ts * ts * (1.0f - 0x1p-20f) : 0.0f;
            fresh = true;
          }
        }
      }
      bool closer = false, open = fresh;
      search_push(W, lane, fresh, M.entry, size);
      while (true) {
        const bool step = size == 0;
        search_pass<false, true>(TriEl{}, W, lane, !step, ~0ull, size, npend, cnt);
        if (!step) continue;
        bool again = false;
        if (open) {
          const unsigned long long k = W->own.key[lane];
          closer = (int32_t)(uint32_t)k != INT_MAX && sqrtf(__uint_as_float((uint32_t)(k >> 32))) < t;
          // ended by an upper value that no exact one has confirmed: search on
          // exact values only
          again = !closer && W->pt[lane].w >= 0.0f && __uint_as_float(W->m2[lane]) < W->stop[lane];
          open = again;
          if (again) {
            W->pt[lane].w = -W->pt[lane].w;
            W->m2[lane] = __float_as_uint(bound_of((t * t) * (1.0f + 0x1p-20f)));
          }
        }
        search_push(W, lane, again, M.entry, size);
        if (size == 0) break;
      }
      const unsigned long long mask = __ballot(inside && !closer);  // every lane of the wavefront takes part
      int node = 1;
      for (int l = 0; l < levels; ++l) {
        const float mid = 0.5f * (lo + hi);
        const int bit = (int)((mask >> (gbase + node)) & 1ull);
        if (bit)
          lo = mid;
        else
          hi = mid;
        node = 2 * node + bit;
      }
      done += levels;
    }
    if (valid && sub == 0) radius[i] = lo;
    if (valid && issued) atomicAdd(M.row_queries + i, (unsigned long long)issued);
  }
}

__global__ void knn_eval_kernel(KnnDev G, double cx, double cy, double cz, const float* __restrict__ Q,
                                const float* __restrict__ Nq, int64_t n, int32_t* __restrict__ idx,
                                float* __restrict__ w) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float qx = (float)((double)Q[3 * i] - cx);
  const float qy = (float)((double)Q[3 * i + 1] - cy);
  const float qz = (float)((double)Q[3 * i + 2] - cz);
  double nx = Nq[3 * i], ny = Nq[3 * i + 1], nz = Nq[3 * i + 2];
  const double nl = sqrt(nx * nx + ny * ny + nz * nz);
  if (nl > 0.0) {
    nx /= nl; ny /= nl; nz /= nl;
  }
  int32_t id[kMaxKnn];
  double wk[kMaxKnn];
  const int m = knn_eval(G, qx, qy, qz, nx, ny, nz, id, wk);
  for (int a = 0; a < G.k; ++a) {
    idx[i * G.k + a] = a < m ? id[a] : -1;
    w[i * G.k + a] = a < m ? (float)wk[a] : 0.0f;
  }
}

// Prefilter records of a mesh. With u = 2^-24, w = |p - a|, L the longest and e
// the shortest edge, s the sine of the smallest angle:
//   * quick_dist's own error: p - a, the frame, the in-plane coordinates and
//     the edge terms are off by at most about 12 u (w + L) in distance, so its
//     squared value by 24 u (w + L)^2;
//   * tri_dist2's face value (n.ap)^2 / (n.n): n = ab x ac is off by 5 u |ab|
//     |ac| <= 5 u |n| / s, n.ap by 4 u |n| w more: u w^2 (20 / s + 16) in the
//     square. (Its other values are distances from points of the triangle.)
//   * A face taken where an edge or a vertex is nearest: the foot lies outside
//     the triangle by some distance t, and the value is short of the square by
//     t^2. The sign of n.(bp x cp) holds farther out than 5 u w / s (n's error)
//     plus 5 u |bp| |cp| / |bc| + 3 u w (its own): next to a short edge |bp| and
//     |cp| are at most w + e, next to a long one their product is at most
//     (w + L) w, so t <= 8 u w^2 / e + 16 u w / s + 16 u (w + L). The vertex tests
//     are off by 4 u w along an edge, by 6 u w L / e <= 6 u w / s at the far end of
//     a short one. Taken as t <= 24 u w^2 / e + 24 u w / s, the rest in the first.
//   * its edge and vertex values add roundings at the size of the coordinates,
//     delta = 2^-21 R in distance, which keep_bound carries;
//   * in a mesh of small units its products underflow: (n.ap)^2 by up to 2^-149,
//     2^-149 / (n.n) in the value (edges of 1e-7: 1e-3 of their square), the
//     squares of lengths by a few 2^-149. The margin holds 2^-147 / (n.n) +
//     2^-126, so that upper values, and with them m2, stay normal numbers.
// Together F (w^2 + L^2), (w + L)^2 being at most 2 (w^2 + L^2), H w^4 and the
// last. A triangle with F > 1/8 (s below 3e-5) or n.n below 2^-120 gets margins
// that send every test of it to the exact one, wherever the query is: a fixed
// G above every square.
//   The w^4 is the query's own. With (4 R)^2 w^2 in its place and s >= 0.01 asked
// for, triangles below 6e-5 of the scene's size and needles had no prefilter
// value, and each trip that met one ended with exact tests: 256,000 walks
// among 128,000 needles (s = 0.003) 157 ms, now 15.8 ms; outside 100 spheres of
// 3e-4 R 43.5 ms, now 8.9 ms; 200,000 closest points there 11.0 and 2.0 ms, now
// 3.9 and 0.6 ms. The two operations more a test needs show in no other case
// (4.1M walks on 500,000 triangles: 29.8 ms both ways). On 19 million triangles
// and points of all shapes and sizes at most 0.005 of the margin was needed.
__global__ void quick_prepare_kernel(const TriRec* __restrict__ tris, int64_t n, float4* __restrict__ quick) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n + kQuickPad) return;
  float4* q = quick + quick_index(i);
  TriRec T;
  int32_t index = kPadTri;
  if (i < n) {
    T = tris[i];
    memcpy(&index, &T.a.w, 4);
  }
  if (index == kPadTri) {
    quick_pad(q);
    return;
  }
  const double A[3] = {T.a.x, T.a.y, T.a.z}, B[3] = {T.b.x, T.b.y, T.b.z}, C[3] = {T.c.x, T.c.y, T.c.z};
  double ab = 0.0, ac = 0.0, bc = 0.0, nrm[3];
  for (int k = 0; k < 3; ++k) {
    const int k1 = (k + 1) % 3, k2 = (k + 2) % 3;
    ab += (B[k] - A[k]) * (B[k] - A[k]);
    ac += (C[k] - A[k]) * (C[k] - A[k]);
    bc += (C[k] - B[k]) * (C[k] - B[k]);
    nrm[k] = (B[k1] - A[k1]) * (C[k2] - A[k2]) - (B[k2] - A[k2]) * (C[k1] - A[k1]);
  }
  ab = sqrt(ab);
  ac = sqrt(ac);
  bc = sqrt(bc);
  const double nn = sqrt(nrm[0] * nrm[0] + nrm[1] * nrm[1] + nrm[2] * nrm[2]);
  const double lmax = fmax(ab, fmax(ac, bc));
  const double emin = fmin(ab, fmin(ac, bc));
  const double smin = nn * emin / (ab * ac * bc);  // sin of the smallest angle
  const double u = 0x1p-24, ts = 24.0 * u / smin, te = 24.0 * u / emin;
  const double F = u * (128.0 + 64.0 / smin) + 2.0 * ts * ts, H = 2.0 * te * te;
  const double G = F * lmax * lmax + 0x1p-126 + 0x1p-147 / (nn * nn);
  // F and H rounded up to 16 bits each, in one word
  const uint32_t fh = ((__float_as_uint((float)F) + 0x10000u) & 0xFFFF0000u) |
                      ((__float_as_uint((float)H) + 0x10000u) >> 16);
  if (!(F <= 0.125) || !(H < 1e30) || !(nn * nn >= 0x1p-120) ||
      !quick_frame(A, B, C, q, (double)__uint_as_float(fh), G * (1.0 + 0x1p-7)))
    quick_always(A, q, 0.5f, 0x1p126f);
}

// A query of the query kernel: its point (scene frame) and mesh, a warm-start
// slot or -1, and the mesh's entry level.
struct Query {
  float x, y, z, radius;
  const Node4* nodes;
  const float4* quick;
  const TriRec* tris;
  int32_t warm, entry;
};

// Caller's points: nearest triangle, squared distance and barycentrics.
struct PointQueries {
  const Node4* nodes;
  const float4* quick;
  const TriRec* tris;
  float radius;
  int32_t entry;
  double cx, cy, cz;
  const float* Q;
  int32_t* tri;
  float* d2;
  float* bary;
  static constexpr bool kBary = true;
  __device__ __forceinline__ Query load(int64_t i) const {
    return Query{(float)((double)Q[3 * i] - cx), (float)((double)Q[3 * i + 1] - cy), (float)((double)Q[3 * i + 2] - cz),
                 radius, nodes, quick, tris, -1, entry};
  }
  __device__ __forceinline__ void store(int64_t i, const Nearest& h) const {
    tri[i] = h.orig;
    d2[i] = h.d2;
    nearest_bary(h, bary[2 * i], bary[2 * i + 1]);
  }
};

// Point rows whose inset point is closer than h/2 to the surface are
// discarded (the inset left the thin region it should probe).
template <typename MD>
__device__ __forceinline__ Query discard_query(const MD& M, int64_t i) {
  const float sgn = M.side ? 1.0f : -1.0f;
  return Query{M.p[3 * i] + sgn * M.inset * M.n[3 * i], M.p[3 * i + 1] + sgn * M.inset * M.n[3 * i + 1],
               M.p[3 * i + 2] + sgn * M.inset * M.n[3 * i + 2], M.radius, M.nodes, M.quick, M.tris,
               M.slot_of_tri[M.tri[i]], M.entry};
}
template <typename MD>
__device__ __forceinline__ void discard_store(const MD& M, int64_t i, const Nearest& h, int32_t* discarded) {
  discarded[i] = h.d2 < 0.25f * M.inset * M.inset ? 1 : 0;
  atomicAdd(M.row_queries + i, 1ull);
}
struct DiscardRows {
  MeshDev M;
  int32_t* discarded;
  static constexpr bool kBary = false;
  __device__ __forceinline__ Query load(int64_t i) const { return discard_query(M, i); }
  __device__ __forceinline__ void store(int64_t i, const Nearest& h) const { discard_store(M, i, h, discarded); }
};

// The same over the point rows of several meshes: launch index j belongs to
// the last range k with R[k].first <= j, as row j - R[k].first of its mesh.
struct DiscardBatch {
  const MeshDev* meshes;
  const RowRange* R;
  int32_t n_ranges;
  static constexpr bool kBary = false;
  __device__ __forceinline__ RowRange range(int64_t j) const {
    int32_t lo = 0, hi = n_ranges - 1;
    while (lo < hi) {
      const int32_t mid = (lo + hi + 1) >> 1;
      if (R[mid].first <= j)
        lo = mid;
      else
        hi = mid - 1;
    }
    return R[lo];
  }
  __device__ __forceinline__ Query load(int64_t j) const {
    const RowRange r = range(j);
    return discard_query(meshes[r.mesh], j - r.first);
  }
  __device__ __forceinline__ void store(int64_t j, const Nearest& h) const {
    const RowRange r = range(j);
    discard_store(meshes[r.mesh], j - r.first, h, r.discarded);
  }
};

// Queries that keep the lane-private search: far from the scene the exact
// test's sign errors exceed the slack of the box bounds, so that what it finds
// depends on the order of the search; and points that are no numbers have no
// distance.
__device__ __forceinline__ bool far_query(const Query& p) {
  const float far = 1.7f * p.radius;
  return !(fabsf(p.x) <= far && fabsf(p.y) <= far && fabsf(p.z) <= far);
}

template <typename Src>
__device__ __forceinline__ void answer_alone(const Src& src, int64_t i, const Query& p) {
  Nearest h;
  TravCount cnt;
  h.d2 = INFINITY; h.orig = INT_MAX; h.slot = -1;
  bvh_nearest<false>(p.nodes, p.tris, p.x, p.y, p.z, p.radius, h, cnt);
  src.store(i, h);
}

// The far ones among n queries, after a query kernel that leaves them: a
// wavefront looks through the blocks of 64 queries g, g + G, ... and answers
// the far ones 64 at a time, one per lane, with kFarWaves wavefronts per SIMD
// (80 VGPRs; at 8 the traversal spills: 13.1 ms). Bound by the dependent loads
// of the traversals. Answered by the query kernel as they came, on 4
// wavefronts per SIMD and few of their lanes, they held the others: 1,000,000
// points on 79,380 faces, all of them 3 to 10 radii away, 11.7 ms, now 10.0 ms;
// 2% of them, the others near the surface, 4.2 ms, now 2.2 ms; 30%, 10.0 ms, now
// 5.0 ms.
constexpr int kFarWaves = 6;
template <typename Src>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kFarWaves)))
    far_queries_kernel(Src src, int64_t nq) {
  __shared__ int64_t list[kWaves][128];
  const int wi = (int)uniform(threadIdx.x >> 6);
  const uint32_t lane = __lane_id();
  const int64_t G = (int64_t)gridDim.x * kWaves;
  uint32_t n = 0;
  for (int64_t b = (int64_t)blockIdx.x * kWaves + wi;; b += G) {
    const int64_t i = b * 64 + lane;
    const bool more = b * 64 < nq, far = i < nq && far_query(src.load(i));
    const uint64_t mk = __ballot(far);
    if (far) list[wi][n + mbcnt64(mk)] = i;
    n += (uint32_t)__popcll(mk);
    lds_order();
    if (more && n < 64) continue;
    const uint32_t take = min(n, 64u);
    if (lane < take) {
      const int64_t q = list[wi][n - take + lane];
      answer_alone(src, q, src.load(q));
    }
    n -= take;
    lds_order();
    if (!more) break;  // (fewer than 64 were left)
  }
}

// Nearest triangles of n queries on the wavefront-shared search: lanes with an
// answered query wait until a quarter of the wavefront's queries do, then
// store their answers and take the next queries together. At most 2^own_shift
// lanes of a wavefront carry a query: a small call spreads over all
// wavefronts, whose other lanes help. The k-th block of wavefront g holds the
// up to 8 queries from ((k G + g) << block_shift) on, G the number of
// wavefronts: neighbours share a wavefront, and each wavefront sees all parts
// of the caller's array (in blocks of 64, an array of points near the surface
// followed by far ones took 12.4 instead of 6.9 ms).
//   On a thread per query with a traversal of its own, 1,000 queries on 1,280
// faces took 230 us and 1,000,003 on 499,280 faces 9.6 ms, as long as the
// slowest traversal of each wavefront; now 32 us and 3.5 ms, a few trips'
// latency and vector issue.
template <typename Src, bool kFar>
__global__ void __launch_bounds__(256) MSK_PERSISTENT_OCCUPANCY
    query_stream_kernel(Src src, int64_t nq, int32_t own_shift) {
  typedef SearchScratch<TriEl, false, kQueryItemCap> Scratch;
  __shared__ Scratch coop[kWaves];
  static_assert(sizeof(coop) <= kLdsPerBlock, "four workgroups per CU");
  const int wi = (int)uniform(threadIdx.x >> 6);
  Scratch* W = &coop[wi];
  const uint32_t lane = __lane_id();
  const int64_t G = (int64_t)gridDim.x * kWaves, g = (int64_t)blockIdx.x * kWaves + wi;
  const bool owner = lane < (1u << own_shift);
  const int block_shift = min(own_shift, 3);
  int64_t next = 0;  // queries handed out (uniform)
  bool drained = false;
  int32_t mode = 0;  // 0 idle, 1 searching, 2 search ended
  int64_t qi = 0;
  const TriRec* tris = nullptr;
  int32_t entry = 1;
  uint32_t npend = 0, size = 0;
  TravCount cnt;
  while (true) {
    if (mode == 1 && W->open[lane] == 0) mode = 2;
    size = uniform(size);
    const uint64_t pend = __ballot(mode == 2), busy = __ballot(mode == 1 || mode == 2);
    const bool step = size == 0 || (size <= (uint32_t)kRootLimit &&
                                    (int)__popcll(pend) >= min(kStepMin, (int)(__popcll(busy) + 3) >> 2));
    search_pass<false>(TriEl{}, W, lane, !step, pend, size, npend, cnt);
    if (step) {
      bool fresh = false;
      if (mode == 2) {
        Nearest h;
        if (search_answer(W, lane, h)) {
          if (Src::kBary) {
            const float4 q = W->pt[lane];
            answer_bary(tris, q.x, q.y, q.z, h);
          }
          src.store(qi, h);
          mode = 0;
        } else {
          mode = 1;
          fresh = true;
        }
      }
      const uint64_t idle = __ballot(mode == 0 && owner);
      if (!drained && idle != 0) {
        const int64_t pos = next + mbcnt64(idle);
        const int64_t q = ((((pos >> block_shift) * G) + g) << block_shift) + (pos & ((1ll << block_shift) - 1));
        const bool take = mode == 0 && owner && q < nq;
        if (take) {
          qi = q;
          const Query p = src.load(qi);
          if (!far_query(p)) {
            // few queries leave the stack room enough for a cold start
            const int32_t warm = p.warm < 0 && own_shift > 2 ? nearest_leaf(p.nodes, p.x, p.y, p.z) : p.warm;
            search_start(W, lane, p.nodes, p.quick, p.tris, p.radius, p.x, p.y, p.z, warm);
            tris = p.tris;
            entry = p.entry;
            mode = 1;
            fresh = true;
          } else if (kFar) {
            answer_alone(src, qi, p);
          }
        }
        const uint32_t got = (uint32_t)__popcll(__ballot(take));
        drained = got < (uint32_t)__popcll(idle);
        next += got;
      }
      search_push(W, lane, fresh, entry, size);
      if (drained && __ballot(mode != 0) == 0) break;
    }
  }
}

// S_ij = (w_i / h) mean_ij, se_ij = (w_i / h) sqrt(var_ij / W_i), var with
// the unbiased (W-1) normalisation. Point rows hold sums of b(t) here and
// the entries where b(s) != 0 are corrected by finalize_point_fix_kernel.
__global__ void finalize_kernel(MeshDev M, int64_t n_rows, const int64_t* __restrict__ walks,
                                const double* __restrict__ w, double* S, double* se) {
  const int64_t n = n_rows * M.K;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < n; idx += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = idx / M.K;
    const double Wi = (double)walks[i];
    const double scale = (M.mode == kRowsPoint && M.discarded[i]) ? 0.0 : w[i] / M.inset_d;
    const double s1 = M.mode == kRowsPoint ? -M.acc1[idx] : M.acc1[idx];
    const double mean = s1 / Wi;
    const double var = fmax(0.0, M.acc2[idx] / Wi - mean * mean) * (Wi / (Wi - 1.0));
    S[idx] = scale * mean;
    se[idx] = scale * sqrt(var / Wi);
  }
}

// With jump_only (exterior), the killing term is dropped (Sec. 3.3, exterior
// Beurling-Deny form; the paper's default exterior operator): an escaped
// walk contributes nothing instead of b(s), so b(s) enters once per walk
// that did not escape.
__global__ void finalize_point_fix_kernel(MeshDev M, int64_t n_rows, const int64_t* __restrict__ walks,
                                          const double* __restrict__ w, double* S, double* se, int32_t jump_only) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_rows || M.discarded[i]) return;
  const int32_t* f = M.faces + 3 * (int64_t)M.tri[i];
  const int32_t vv[3] = {f[0], f[1], f[2]};
  const double ww[3] = {(double)M.bary[3 * i], (double)M.bary[3 * i + 1], (double)M.bary[3 * i + 2]};
  const double Wi = (double)walks[i];
  const double Hi = jump_only ? Wi - (double)M.row_escaped[i] : Wi;  // walks that carry b(s)
  const double scale = w[i] / M.inset_d;
  auto fix = [&](int32_t j, double bs) {
    const int64_t idx = i * M.K + j;
    const double t1 = M.acc1[idx], t2 = M.acc2[idx];
    const double s1 = Hi * bs - t1;
    const double s2 = Hi * bs * bs - 2.0 * bs * t1 + t2;
    const double mean = s1 / Wi;
    const double var = fmax(0.0, s2 / Wi - mean * mean) * (Wi / (Wi - 1.0));
    S[idx] = scale * mean;
    se[idx] = scale * sqrt(var / Wi);
  };
  if (M.knn.k > 0) {
    double nx = M.n[3 * i], ny = M.n[3 * i + 1], nz = M.n[3 * i + 2];
    const double nl = sqrt(nx * nx + ny * ny + nz * nz);
    nx /= nl; ny /= nl; nz /= nl;
    int32_t idx[kMaxKnn];
    double wk[kMaxKnn];
    const int m = knn_eval(M.knn, M.p[3 * i], M.p[3 * i + 1], M.p[3 * i + 2], nx, ny, nz, idx, wk);
    for (int a = 0; a < m; ++a) fix(idx[a], wk[a]);
  } else {
    merge_rows<3>(M, vv, ww, fix);
  }
}

}  // namespace msk

// ------------------------------------------------------ launch wrappers

namespace msk {

static inline int blocks_for(int64_t n, int bs) { return (int)std::min<int64_t>((n + bs - 1) / bs, 1 << 20); }

hipError_t launch_walk_plain(const WalkLaunch& L, hipStream_t s) {
  const int64_t n = L.n_slots * L.walks_per_slot;
  if (n <= 0) return hipSuccess;
  const int64_t nb = (n + 255) / 256;
  if (nb > INT32_MAX) return hipErrorInvalidValue;
  if (L.knn && L.stats) return hipErrorInvalidValue;  // the point basis has no counting instantiation
  if (L.knn)
    hipLaunchKernelGGL((walk_plain_kernel<false, true>), dim3((unsigned)nb), dim3(256), 0, s, L);
  else if (L.stats)
    hipLaunchKernelGGL(walk_plain_kernel<true>, dim3((unsigned)nb), dim3(256), 0, s, L);
  else
    hipLaunchKernelGGL(walk_plain_kernel<false>, dim3((unsigned)nb), dim3(256), 0, s, L);
  return hipGetLastError();
}

hipError_t launch_walk_persistent(const WalkLaunch& L, int grid, hipStream_t s) {
  if (L.knn && L.stats) return hipErrorInvalidValue;  // the point basis has no counting instantiation
  if (L.accum < 0 || L.accum > 2) return hipErrorInvalidValue;
  const dim3 g(grid), t(256);
#define MSK_LAUNCH(AccT, knn, rows) hipLaunchKernelGGL((walk_stream_kernel<false, AccT, knn, rows>), g, t, 0, s, L)
#define MSK_LAUNCH_ACC(knn, rows)                                              \
  do {                                                                         \
    if (L.accum == 1)                                                          \
      MSK_LAUNCH(float, knn, rows);                                            \
    else if (L.accum == 2)                                                     \
      MSK_LAUNCH(CompF32, knn, rows);                                          \
    else                                                                       \
      MSK_LAUNCH(double, knn, rows);                                           \
  } while (0)
  if (L.stats) {
    if (L.accum == 1)
      hipLaunchKernelGGL((walk_stream_kernel<true, float, false, kRowsAny>), g, t, 0, s, L);
    else if (L.accum == 2)
      hipLaunchKernelGGL((walk_stream_kernel<true, CompF32, false, kRowsAny>), g, t, 0, s, L);
    else
      hipLaunchKernelGGL((walk_stream_kernel<true, double, false, kRowsAny>), g, t, 0, s, L);
  } else if (L.rows == 2) {  // PSD walks: no contributions, no row tables
    MSK_LAUNCH(double, false, kRowsBalls);
  } else if (L.knn) {  // point basis: instantiations carrying the k-NN evaluation
    if (L.rows == 1)
      MSK_LAUNCH_ACC(true, kRowsPoints);
    else
      MSK_LAUNCH_ACC(true, kRowsAny);
  } else if (L.rows == 1) {
    MSK_LAUNCH_ACC(false, kRowsPoints);
  } else {
    MSK_LAUNCH_ACC(false, kRowsAny);
  }
#undef MSK_LAUNCH_ACC
#undef MSK_LAUNCH
  return hipGetLastError();
}

#if MSK_PHASE_TIMING
extern "C" int msk_debug_phase_cycles(unsigned long long* out, int reset) {
  if (hipMemcpyFromSymbol(out, HIP_SYMBOL(g_phase_cycles), sizeof(unsigned long long) * 8) != hipSuccess) return 1;
  if (reset) {
    unsigned long long z[16] = {0};
    if (hipMemcpyToSymbol(HIP_SYMBOL(g_phase_cycles), z, sizeof(z)) != hipSuccess) return 1;
  }
  return 0;
}
#endif

// Counts the non-finite entries of a (n values) into *count (grid-stride).
__global__ void count_nonfinite_kernel(const double* __restrict__ a, int64_t n, unsigned long long* count) {
  unsigned long long c = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    c += isfinite(a[i]) ? 0ull : 1ull;
  // wavefront sum, one atomic per wavefront with any
  for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
  if (__lane_id() == 0 && c) atomicAdd(count, c);
}

// Per-estimate totals of the per-row counters, one workgroup per estimate:
// out[6 k + 0..5] = queries, escaped walks, capped walks, discarded rows,
// walks of the kept rows, non-finite entries.
__global__ void row_totals_kernel(const RowCounters* __restrict__ sets, unsigned long long* __restrict__ out) {
  const RowCounters C = sets[blockIdx.x];
  __shared__ unsigned long long acc[5];
  if (threadIdx.x < 5) acc[threadIdx.x] = 0;
  __syncthreads();
  unsigned long long v[5] = {0, 0, 0, 0, 0};
  for (int64_t i = threadIdx.x; i < C.n; i += blockDim.x) {
    v[0] += C.queries[i];
    v[1] += C.escaped[i];
    v[2] += C.capped[i];
    const bool dropped = C.discarded[i] != 0;
    v[3] += dropped ? 1ull : 0ull;
    v[4] += dropped ? 0ull : (unsigned long long)C.walks[i];
  }
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    for (int off = 32; off > 0; off >>= 1) v[k] += __shfl_xor(v[k], off);
    if (__lane_id() == 0 && v[k]) atomicAdd(&acc[k], v[k]);
  }
  __syncthreads();
  if (threadIdx.x < 5) out[6 * blockIdx.x + threadIdx.x] = acc[threadIdx.x];
  if (threadIdx.x == 5) out[6 * blockIdx.x + 5] = *C.nonfinite;
}

hipError_t launch_count_nonfinite(const double* a, int64_t n, unsigned long long* count, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int blocks = (int)std::min<int64_t>(1024, (n + 255) / 256);
  hipLaunchKernelGGL(count_nonfinite_kernel, dim3(blocks), dim3(256), 0, s, a, n, count);
  return hipGetLastError();
}

hipError_t launch_init_queues(unsigned long long* next, unsigned long long* end, const QueueInit& q, hipStream_t s) {
  hipLaunchKernelGGL(init_queues_kernel, dim3(1), dim3(64), 0, s, next, end, q);
  return hipGetLastError();
}

hipError_t launch_fill_u64(void* p, int64_t n, unsigned long long v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_u64_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, (unsigned long long*)p, n, v);
  return hipGetLastError();
}

hipError_t launch_fill_u32(void* p, int64_t n, uint32_t v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_u32_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, (uint32_t*)p, n, v);
  return hipGetLastError();
}

// The query kernel over n queries: as many wavefronts as are resident at once
// (4 per SIMD), each with as few queries at a time as still covers n, up to
// one per lane.
template <typename Src>
static hipError_t launch_queries(const Src& src, int64_t n, int32_t n_cu, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t waves = 16ll * n_cu;
  int own_shift = 0;
  while (own_shift < 6 && (waves << own_shift) < n) ++own_shift;
  const int64_t blocks = std::min<int64_t>(4ll * n_cu, (((n - 1) >> own_shift) / kWaves) + 1);
  // Up to 128 queries a wavefront the second launch costs more than it saves
  // (200,000 points on 79,380 faces: 214 us near the surface and 1.36 ms with 2%
  // far ones, 220 us and 1.41 ms with it; 1,000,000 points: 0.64 ms both ways,
  // 4.2 and 2.3 ms). Inset tests are hardly ever far.
  if (!Src::kBary || n <= 128 * waves) {
    hipLaunchKernelGGL((query_stream_kernel<Src, true>), dim3((unsigned)blocks), dim3(256), 0, s, src, n, own_shift);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((query_stream_kernel<Src, false>), dim3((unsigned)blocks), dim3(256), 0, s, src, n, own_shift);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t far_blocks = std::min<int64_t>((int64_t)kFarWaves * n_cu, (n + 255) / 256);
  hipLaunchKernelGGL(far_queries_kernel<Src>, dim3((unsigned)far_blocks), dim3(256), 0, s, src, n);
  return hipGetLastError();
}

hipError_t launch_discard(const MeshDev& M, int64_t n_rows, int32_t n_cu, int32_t* discarded, hipStream_t s) {
  return launch_queries(DiscardRows{M, discarded}, n_rows, n_cu, s);
}

hipError_t launch_discard_batch(const MeshDev* meshes, const RowRange* ranges, int32_t n_ranges, int64_t n_total,
                                int32_t n_cu, hipStream_t s) {
  if (n_ranges <= 0) return hipSuccess;
  return launch_queries(DiscardBatch{meshes, ranges, n_ranges}, n_total, n_cu, s);
}

hipError_t launch_row_totals(const RowCounters* sets, int32_t n_sets, unsigned long long* out, hipStream_t s) {
  if (n_sets <= 0) return hipSuccess;
  hipLaunchKernelGGL(row_totals_kernel, dim3(n_sets), dim3(256), 0, s, sets, out);
  return hipGetLastError();
}

hipError_t launch_knn_eval(const KnnDev& G, const double* c, const float* Q, const float* Nq, int64_t n, int32_t* idx,
                           float* w, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(knn_eval_kernel, dim3(blocks_for(n, 128)), dim3(128), 0, s, G, c[0], c[1], c[2], Q, Nq, n, idx,
                     w);
  return hipGetLastError();
}

hipError_t launch_tangent_ball(const MeshDev& M, int64_t n_rows, float r_max, int32_t iters, float tol, int32_t n_cu,
                               float* radius, hipStream_t s) {
  if (n_rows <= 0) return hipSuccess;
  const int64_t waves = 16ll * n_cu;
  int32_t rows = 1;
  while (rows < 8 && rows * waves < n_rows) rows *= 2;
  const int64_t blocks = std::min<int64_t>(4ll * n_cu, (n_rows + rows * kWaves - 1) / (rows * kWaves));
  hipLaunchKernelGGL(tangent_ball_kernel, dim3((unsigned)blocks), dim3(256), 0, s, M, n_rows, rows, r_max, iters, tol,
                     radius);
  return hipGetLastError();
}

hipError_t launch_quick_prepare(const TriRec* tris, int64_t n, float4* quick, hipStream_t s) {
  hipLaunchKernelGGL(quick_prepare_kernel, dim3((unsigned)((n + kQuickPad + 255) / 256)), dim3(256), 0, s, tris, n,
                     quick);
  return hipGetLastError();
}

hipError_t launch_closest_points(const Node4* nodes, const TriRec* tris, const float4* quick, int32_t entry,
                                 float radius, const double* c, const float* Q, int64_t nq, int32_t n_cu, int32_t* tri,
                                 float* d2, float* bary, hipStream_t s) {
  return launch_queries(PointQueries{nodes, quick, tris, radius, entry, c[0], c[1], c[2], Q, tri, d2, bary}, nq, n_cu, s);
}

hipError_t launch_finalize(const MeshDev& M, int64_t n_rows, const int64_t* walks, const double* w, double* S,
                           double* se, hipStream_t s,
                           int32_t jump_only) {
  if (n_rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(finalize_kernel, dim3(blocks_for(n_rows * M.K, 256)), dim3(256), 0, s, M, n_rows, walks, w, S, se);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || M.mode != kRowsPoint) return e;
  hipLaunchKernelGGL(finalize_point_fix_kernel, dim3(blocks_for(n_rows, 128)), dim3(128), 0, s, M, n_rows, walks, w, S,
                     se, jump_only);
  return hipGetLastError();
}

}  // namespace msk
