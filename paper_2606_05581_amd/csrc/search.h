// The exact nearest-element search that the wavefronts of the walk, query and
// Kelvin kernels share, and the device helpers it stands on.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <climits>

#include "msk_internal.h"

namespace msk {

// Device memory behind a pointer that was itself read from memory: such a
// pointer is generic to the compiler, and its flat accesses count as LDS
// accesses too, so that every wait for LDS data would wait for them.
#define MSK_GLOBAL __attribute__((address_space(1)))

template <typename T>
__device__ __forceinline__ T gload(const T* p, int64_t i) {
  return ((const MSK_GLOBAL T*)p)[i];
}
__device__ __forceinline__ float4 gload4(const void* p, int64_t i) {
  typedef float V __attribute__((ext_vector_type(4)));
  const V v = ((const MSK_GLOBAL V*)p)[i];
  return make_float4(v.x, v.y, v.z, v.w);
}
template <typename T>
__device__ __forceinline__ void gstore(T* p, int64_t i, T v) {
  ((MSK_GLOBAL T*)p)[i] = v;
}
template <typename T>
__device__ __forceinline__ void gadd(T* p, int64_t i, T v) {
  (void)__hip_atomic_fetch_add((MSK_GLOBAL T*)p + i, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Squared distance from p to the flat triangle of the quick record at i (see
// msk_internal.h), in the triangle's own frame: a branch-free handful of fused
// operations. Also |p - a|^2 and the record's F and G.
__device__ __forceinline__ float quick_flat(float px, float py, float pz, const void* quick, int64_t i, float& w2,
                                            float& F, float& G) {
  const float4 r0 = gload4(quick, i), r1 = gload4(quick, i + 4), r2 = gload4(quick, i + 8),
               r3 = gload4(quick, i + 12), r4 = gload4(quick, i + 16);
  const float gx = px - r0.x, gy = py - r0.y, gz = pz - r0.z;
  const float x = r1.x * gx + r1.y * gy + r1.z * gz;
  const float y = r2.x * gx + r2.y * gy + r2.z * gz;
  const float z = r3.x * gx + r3.y * gy + r3.z * gz;
  const float c1 = r0.w, s1 = r1.w, l1 = r2.w, c2 = r3.w, s2 = r4.x, l2 = r4.y;
  const float b = c1 * l1 - c2 * l2;  // vertex b lies at (b, 0), vertex c at l1 (c1, s1)
  const float t0 = x - __builtin_amdgcn_fmed3f(x, 0.0f, b);
  const float q1 = x * c1 + y * s1, h1 = x * s1 - y * c1;
  const float t1 = q1 - __builtin_amdgcn_fmed3f(q1, 0.0f, l1);
  const float xb = x - b;
  const float q2 = xb * c2 + y * s2, h2 = y * c2 - xb * s2;
  const float t2 = q2 - __builtin_amdgcn_fmed3f(q2, 0.0f, l2);
  const float e = fminf(fminf(y * y + t0 * t0, h1 * h1 + t1 * t1), h2 * h2 + t2 * t2);
  const float in = fminf(fminf(y, h1), h2);
  w2 = gx * gx + gy * gy + gz * gz;
  F = r4.z;
  G = r4.w;
  return z * z + (in >= 0.0f ? 0.0f : e);
}

// The record of triangle (a, b, c) (FP64; F and G given), field by field 4
// float4 apart; false if it has no frame (no area).
__device__ __forceinline__ bool quick_frame(const double a[3], const double b[3], const double c[3], float4* q,
                                            double F, double G) {
  double ab[3], ac[3], n[3];
  for (int k = 0; k < 3; ++k) {
    ab[k] = b[k] - a[k];
    ac[k] = c[k] - a[k];
  }
  n[0] = ab[1] * ac[2] - ab[2] * ac[1];
  n[1] = ab[2] * ac[0] - ab[0] * ac[2];
  n[2] = ab[0] * ac[1] - ab[1] * ac[0];
  const double lab = sqrt(ab[0] * ab[0] + ab[1] * ab[1] + ab[2] * ab[2]);
  const double lac = sqrt(ac[0] * ac[0] + ac[1] * ac[1] + ac[2] * ac[2]);
  const double nn = sqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
  const double bx = ac[0] - ab[0], by = ac[1] - ab[1], bz = ac[2] - ab[2];
  const double lbc = sqrt(bx * bx + by * by + bz * bz);
  if (!(nn > 0.0) || !(lab > 0.0) || !(lac > 0.0) || !(lbc > 0.0)) return false;
  double u[3], m[3], v[3];
  for (int k = 0; k < 3; ++k) {
    u[k] = ab[k] / lab;
    m[k] = n[k] / nn;
  }
  v[0] = m[1] * u[2] - m[2] * u[1];
  v[1] = m[2] * u[0] - m[0] * u[2];
  v[2] = m[0] * u[1] - m[1] * u[0];
  const double cx = ac[0] * u[0] + ac[1] * u[1] + ac[2] * u[2], cy = ac[0] * v[0] + ac[1] * v[1] + ac[2] * v[2];
  q[0] = make_float4((float)a[0], (float)a[1], (float)a[2], (float)(cx / lac));
  q[4] = make_float4((float)u[0], (float)u[1], (float)u[2], (float)(cy / lac));
  q[8] = make_float4((float)v[0], (float)v[1], (float)v[2], (float)lac);
  q[12] = make_float4((float)m[0], (float)m[1], (float)m[2], (float)((cx - lab) / lbc));
  q[16] = make_float4((float)(cy / lbc), (float)lbc, (float)F, (float)G);
  return true;
}

// The records of a pad (no query accepts it) and of an element without a
// frame (every query sends it to the exact test: without a frame the flat
// value is 0, so F and G alone have to make the element's lower value the
// smallest and stay finite themselves. The search keeps a slot number in the
// low bits of a lower value, where those of an infinity would make it NaN).
__device__ __forceinline__ void quick_pad(float4* q) {
  q[0] = make_float4(INFINITY, INFINITY, INFINITY, 0.0f);
  for (int k = 1; k < 5; ++k) q[4 * k] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
}
__device__ __forceinline__ void quick_always(const double a[3], float4* q, float F, float G) {
  q[0] = make_float4((float)a[0], (float)a[1], (float)a[2], 0.0f);
  for (int k = 1; k < 4; ++k) q[4 * k] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  q[16] = make_float4(0.0f, 0.0f, F, G);
}

// Work counted by the statistics kernels; a box lower bound costs 17 FP32
// operations (6 subtractions, 6 maxima, 3 products, 2 sums).
constexpr uint32_t kBoxFlops = 17;
struct TravCount {
  uint64_t nodes = 0, tris = 0, flops = 0;
};

// A value that all lanes of the wavefront share, in a scalar register.
__device__ __forceinline__ uint32_t uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
  return (uint64_t)uniform((uint32_t)(v >> 32)) << 32 | uniform((uint32_t)v);
}

__device__ __forceinline__ uint32_t mbcnt64(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Orders LDS accesses of a wavefront as written: the hardware executes one
// wavefront's LDS instructions in issue order, so only the compiler must
// not move them (a fence would also wait for all outstanding global and
// scratch accesses).
__device__ __forceinline__ void lds_order() { __asm__ __volatile__("" ::: "memory"); }

// Exclusive prefix sum over the wavefront of a count below 8 (bit-sliced
// ballots); `total` receives the wavefront's sum.
__device__ __forceinline__ uint32_t wave_prefix_small(uint32_t v, uint32_t& total) {
  uint32_t pre = 0, tot = 0;
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    const uint64_t m = __ballot((v >> b) & 1u);
    pre += mbcnt64(m) << b;
    tot += (uint32_t)__popcll(m) << b;
  }
  total = tot;
  return pre;
}

// Wavefront-shared nearest-element search: the exact search of an element kind
// El (planar triangles, walk.hip; images of triangles under the Kelvin
// transform, kelvin.hip). Up to 64 queries of a wavefront, one per owner
// lane, share one stack of (node, owner) items in LDS. A trip takes up to 64
// items from its top, one per lane whoever their owners are, tests the four
// child boxes, lists the leaf children's triangles, tests those 64 at a time
// with the whole wavefront, and pushes the inner children that still reach
// their owner's bound, the nearest ones of all lanes on top. A query ends when
// none of its items is left (`open`).
//   The search of a point far from every surface visits hundreds to thousands
// of nodes. On a stack per lane it held its wavefront for that many trips
// with one lane busy: 256,000 walks on a 500,000-face sphere took 15.6 ms,
// 16.4M walks 153 ms, so that 17 of the 51 ms of 4.1M walks were such tails.
// Here all lanes share its nodes, and the 4.1M walks take 29 ms.
//
// Elements are listed in units of one block of 4 slots of one owner, one
// lane each (one word: block << 6 | owner lane; leaves start at a block and
// hold at least one element, so meshes have fewer than 2^26). The
// lanes past a shorter leaf meet pads. A leaf wider than 4 lists its second
// block once the first ones are done.
//
// A listed element takes a prefilter only: FP32 values lo and up of its
// distance with lo <= exact value <= up (El::quick; in El's own measure). up
// lowers the owner's bound m2 through an LDS minimum; if lo still reaches that
// bound the element goes to the wavefront's pending list, and the exact test
// runs on the pending elements that are left once their owner's search has
// ended (or the list is full): one to three per query instead of all of them.
// The exact minimum is the lexicographic one of (value, original index).
// Should it lie above what m2 promised (possible only where an element breaks
// its upper value: nearly degenerate triangles), the owner's search runs again
// with m2 at that minimum and lowered by exact values only (negative pt.w), so
// no result rests on the upper values. Elements without an upper value
// (`always`) are tested as soon as they are listed.
//   Exact tests of all listed triangles were bound by VALU issue: about 190
// wavefront instructions per round of 64 tests, every region's path among
// them. The prefilter of triangles takes about 75.
//
// The stack holds kCap items. A trip's lanes whose children would raise it over
// the limit, 64 below, put their item back instead (lanes in order from the
// top), and a trip within 12 items of the limit takes one item only, whose
// subtree adds at most 3 items a level (3 x depth + 5 <= kStackDepth). The units
// of a trip lie above the stack's top; lanes whose units do not fit there put
// their item back as well. (A trip that took only as many items as the room
// could hold four children of crept along with a few items once 64 far queries
// had filled the stack.)
//   A full stack is slow: searches whose elements are about equally far (the
// inside of a sphere) then advance an item at a time. So new queries start only
// while at most kRootLimit items wait, less than a trip takes: the more items
// each search has, the fewer run at once. Walk kernel with 32 instead of 256:
// 4.1M walks on 500,000 triangles 36 -> 30 ms, a batch of 12 meshes 23.4 -> 20.8
// ms (64: 31.4 and 21.9 ms, 16: as 32). And the query kernel, which keeps no
// row tables in LDS, has 960 items where the others have 512: 1,000,003 points
// 6.6 -> 3.5 ms, 200,000 points halfway to the centre of a sphere of 327,680
// triangles 12.8 -> 3.1 ms (384 items: 23 ms; a stack per lane 6.2 ms).
constexpr int kItemCap = 512, kQueryItemCap = 960, kRootLimit = 32;
constexpr int kPendCap = 128;
// `kStop`: queries that only ask whether an element lies below a value end
// once m2 is below `stop`.
template <typename El, bool kStop = false, int kCap = kItemCap>
struct SearchScratch {
  static constexpr int cap = kCap, limit = kCap - 64;
  static_assert(limit + kStackDepth <= cap, "one item's subtree must fit above the limit");
  static_assert(kRootLimit + 64 <= limit, "new queries must fit below the limit");
  uint32_t item[kCap];   // node << 6 | owner; above the top: units, block << 6 | owner
  uint16_t lb[kCap];     // item's box lower bound, FP32 cut to 16 bits
  float4 pt[64];             // owner's query point; w: El's absolute allowance, negative: m2 lowered by exact values only
  uint32_t m2[64];           // bound on the owner's minimum, in El's measure (float bits)
  uint32_t open[64];         // owner's items on the stack
  typename El::Owners own;   // what El keeps per owner
  float stop[kStop ? 64 : 1];
  union {
    struct {
      uint32_t pend[kPendCap];
      float pend_lo[kPendCap];
    };
    double sum[2][64];  // free for the kernel while nothing is pending
  };
};

// Exact tests of the pending elements whose owner is in `done` (all lanes
// call it); those of other owners stay listed, those that no longer reach
// their owner's bound are dropped. Returns the new list length.
template <bool kStats, typename El, typename Scratch>
__device__ __forceinline__ uint32_t flush_pending(const El& el, Scratch* W, uint32_t lane, uint32_t n, uint64_t done,
                                                  TravCount& cnt) {
  uint32_t kept = 0;
  n = uniform(n);
  for (uint32_t b = 0; b < n; b += 64) {
    const bool in = b + lane < n;
    const uint32_t word = in ? W->pend[b + lane] : 0u;
    const float lo = in ? W->pend_lo[b + lane] : INFINITY;
    const uint32_t o = word & 63u;
    const float4 q = W->pt[o];
    const bool live = in && lo <= El::keep(__uint_as_float(W->m2[o]), q);
    const bool now = live && ((done >> o) & 1ull);
    const bool later = live && !now;
    const uint64_t mk = __ballot(later);
    lds_order();
    if (later) {  // at most b + lane: never over an entry that is still to be read
      const uint32_t p = kept + mbcnt64(mk);
      W->pend[p] = word;
      W->pend_lo[p] = lo;
    }
    kept = uniform(kept + (uint32_t)__popcll(mk));
    // the slot within its block stands in the low bits of the lower value
    el.template exact<kStats>(W, o, (int32_t)(word >> 6 << 2 | (__float_as_uint(lo) & 3u)), now, q, cnt);
    lds_order();
  }
  return kept;
}

// Pushes the searches of the lanes with `fresh` (all lanes of the wavefront
// call it, with size <= kRootLimit): the root, or, while the stack has fewer
// items than the wavefront lanes, all nodes of the deepest full level of the
// tree (`entry` = 1, 4, 16 or 64 of them, consecutive in breadth-first order)
// that still fits: the levels above cost a trip each and answer nothing.
template <typename Scratch>
__device__ __forceinline__ void search_push(Scratch* W, uint32_t lane, bool fresh, int32_t entry, uint32_t& size) {
  const uint64_t m = __ballot(fresh);
  const uint32_t nf = (uint32_t)__popcll(m);
  uint32_t es = 0;
#pragma unroll
  for (uint32_t e = 2; e <= 6; e += 2)
    if (size + (nf << e) <= 64u && __ballot(fresh && entry < (1 << e)) == 0) es = e;
  if (fresh) {
    W->lb[Scratch::limit + mbcnt64(m)] = (uint16_t)lane;  // above any item of such a pass
    W->open[lane] = 1u << es;
  }
  lds_order();
  const uint32_t first = ((1u << es) - 1u) / 3u;
  if (lane < nf << es) {
    const uint32_t o = W->lb[Scratch::limit + (lane >> es)];
    W->item[size + lane] = (first + (lane & ((1u << es) - 1u))) << 6 | o;
    W->lb[size + lane] = 0;
  }
  lds_order();
  size += nf << es;
}

// One pass of the wavefront (all lanes call it). With `trip` it is a trip of
// the search; without, it only runs the pending exact tests of the owners in
// `done`. Both kinds share one copy of the exact test: the walk kernel's loop
// is long enough to miss the instruction cache.
template <bool kStats, bool kStop = false, typename El, typename Scratch>
__device__ __forceinline__ void search_pass(const El& el, Scratch* W, uint32_t lane, bool trip, uint64_t done, uint32_t& size,
                                            uint32_t& npend, TravCount& cnt) {
  size = uniform(size);
  npend = uniform(npend);
  const int32_t room = (int32_t)Scratch::limit - (int32_t)size;  // for more items than are taken
  const uint32_t n = trip ? min(room >= 12 ? 64u : 1u, size) : 0u;
  const bool tr = lane < n;
  float lb[4] = {INFINITY, INFINITY, INFINITY, INFINITY};
  int32_t cc[4] = {0, 0, 0, 0};
  // leaf children within the bound: unit words, and whether a second block follows
  uint32_t uw[4] = {~0u, ~0u, ~0u, ~0u};
  uint32_t nu = 0, n2 = 0, o = 0, word = 0;
  float l0 = 0.0f;
  float4 q = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  bool live = false, back = false;
  if (tr) {
    word = W->item[size - 1u - lane];
    l0 = __uint_as_float((uint32_t)W->lb[size - 1u - lane] << 16);
    o = word & 63u;
    q = W->pt[o];
    const float m2 = __uint_as_float(W->m2[o]);
    const float thr = El::boxes(m2, q);
    live = l0 <= thr && !(kStop && m2 < W->stop[o]);
    if (live) {
      if (kStats) {
        ++cnt.nodes;
        cnt.flops += 4 * kBoxFlops;
      }
      const char* N = (const char*)el.nodes(W, o) + ((uint64_t)(word >> 6) << 7);
      const float4 lox = gload4(N, 0), loy = gload4(N, 1), loz = gload4(N, 2), hix = gload4(N, 3), hiy = gload4(N, 4),
                   hiz = gload4(N, 5), ch = gload4(N, 6);
      const float lx[4] = {lox.x, lox.y, lox.z, lox.w}, ly[4] = {loy.x, loy.y, loy.z, loy.w},
                  lz[4] = {loz.x, loz.y, loz.z, loz.w};
      const float hx[4] = {hix.x, hix.y, hix.z, hix.w}, hy[4] = {hiy.x, hiy.y, hiy.z, hiy.w},
                  hz[4] = {hiz.x, hiz.y, hiz.z, hiz.w};
      const int32_t c4[4] = {__float_as_int(ch.x), __float_as_int(ch.y), __float_as_int(ch.z), __float_as_int(ch.w)};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float gx = fmaxf(fmaxf(lx[k] - q.x, q.x - hx[k]), 0.0f);
        const float gy = fmaxf(fmaxf(ly[k] - q.y, q.y - hy[k]), 0.0f);
        const float gz = fmaxf(fmaxf(lz[k] - q.z, q.z - hz[k]), 0.0f);
        const float l = gx * gx + gy * gy + gz * gz;
        // an unused slot has child < 0 and an empty box (l = inf > thr)
        const bool leaf = c4[k] < 0, hit = leaf && l <= thr;
        lb[k] = leaf ? INFINITY : l;
        cc[k] = c4[k];
        uw[k] = hit ? (((uint32_t)~c4[k] >> 2) << 6) | o : ~0u;
        nu += hit ? 1u : 0u;
        n2 += hit ? (uint32_t)~c4[k] & 1u : 0u;
      }
    }
  }
  size -= n;
  uint32_t total = 0;
  bool force = false;
  if (trip) {
    done = ~0ull;
    const uint32_t before = wave_prefix_small(nu, total);
    if (total > (uint32_t)Scratch::cap - size) {
      back = nu > 0 && before + nu > (uint32_t)Scratch::cap - size;
      total = (uint32_t)__builtin_amdgcn_readlane((int)before, __ffsll((unsigned long long)__ballot(back)) - 1);
      if (back) {
        uw[0] = uw[1] = uw[2] = uw[3] = ~0u;
        n2 = 0;
        live = false;
      }
    }
    uint32_t pos = size + before;
    lds_order();
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (uw[k] != ~0u) W->item[pos++] = uw[k];
    if (kStats && nu > 0) {
      cnt.tris += El::kQuickFlops > 0 ? (nu + n2) << 2 : 0u;
      cnt.flops += ((nu + n2) << 2) * El::kQuickFlops;
    }
    lds_order();
  }
  bool flush = !trip && npend != 0;
  uint32_t u0 = 0;
  while (true) {
    if (flush || (npend > (uint32_t)(kPendCap - 64) && u0 < total)) {
      npend = flush_pending<kStats>(el, W, lane, npend, done, cnt);
      flush = false;
    } else if (u0 < total) {
      const uint32_t u = u0 + (lane >> 2);
      bool cand = false;
      uint32_t entry = 0;
      float lo = 0.0f;
      if (u < total) {
        const uint32_t pk = W->item[size + u];
        const uint32_t uo = pk & 63u;
        const uint32_t bl = pk >> 6;
        const float4 p = W->pt[uo];
        const float m2 = __uint_as_float(W->m2[uo]);
        float up;
        bool always;
        el.quick(W, uo, p, (int64_t)bl * 20 + (lane & 3u), lo, up, always);
        // (most upper values lie above the bound: without the look at it the
        // PSD estimator's walks take 4.75 instead of 4.5 ms)
        if (p.w >= 0.0f && up < m2) atomicMin(&W->m2[uo], __float_as_uint(up));
        lds_order();
        cand = lo <= El::keep_wide(__uint_as_float(W->m2[uo]), p);  // (flush_pending takes El::keep)
        force |= cand && (always || p.w < 0.0f);
        entry = pk;
        // the slot within its block goes into the low bits of the lower value,
        // which grows by at most 3 * 2^-23 of it: El::keep allows for 2^-20
        lo = __uint_as_float((__float_as_uint(lo) & ~3u) | (lane & 3u));
      }
      const uint64_t mk = __ballot(cand);
      if (cand) {
        const uint32_t p = npend + mbcnt64(mk);
        W->pend[p] = entry;
        W->pend_lo[p] = lo;
      }
      npend += (uint32_t)__popcll(mk);
      lds_order();
      u0 += 16;
      // elements without an upper value bound nothing until they are tested
      flush = u0 >= total && __ballot(force) != 0;
    } else if (__ballot(n2 > 0) != 0) {  // the second blocks of wide leaves
      uint32_t pos = size + wave_prefix_small(n2, total);
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (uw[k] != ~0u && ((uint32_t)~cc[k] & 1u)) W->item[pos++] = uw[k] + 64u;
      lds_order();
      n2 = 0;
      u0 = 0;
    } else {
      break;
    }
  }
  if (!trip) return;
  uint32_t pushed = 0;
  bool put[4] = {false, false, false, false};
  if (live) {
    const float thr = El::boxes(__uint_as_float(W->m2[o]), q);
#define MSK_CX(i, j)                                                        \
  if (lb[j] < lb[i]) {                                                      \
    float tl = lb[i]; lb[i] = lb[j]; lb[j] = tl;                            \
    int32_t tc = cc[i]; cc[i] = cc[j]; cc[j] = tc;                          \
  }
    MSK_CX(0, 1) MSK_CX(2, 3) MSK_CX(0, 2) MSK_CX(1, 3) MSK_CX(1, 2)
#undef MSK_CX
#pragma unroll
    for (int k = 0; k < 4; ++k) {  // leaf children and unused slots carry lb = inf
      put[k] = lb[k] <= thr;
      pushed += put[k] ? 1u : 0u;
    }
  }
  lds_order();
  uint64_t mp[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) mp[k] = __ballot(put[k]);
  const int32_t more = (int32_t)(__popcll(mp[0]) + __popcll(mp[1]) + __popcll(mp[2]) + __popcll(mp[3]));
  if (n > 1u && (more > room + (int32_t)n || __ballot(back) != 0)) {
    // no room for all children: lanes in order while their extra items fit
    uint32_t extra = pushed > 1u ? pushed - 1u : 0u, all;
    extra += wave_prefix_small(extra, all);
    if (extra > (uint32_t)room && pushed > 1u) {
      back = true;
      pushed = 0;
      put[0] = put[1] = put[2] = put[3] = false;
    }
    const uint64_t m = __ballot(back);
    if (back) {
      const uint32_t p = size + mbcnt64(m);
      W->item[p] = word;
      W->lb[p] = (uint16_t)(__float_as_uint(l0) >> 16);
      pushed = 1;
    }
    size += (uint32_t)__popcll(m);
#pragma unroll
    for (int k = 0; k < 4; ++k) mp[k] = __ballot(put[k]);
  }
#pragma unroll
  for (int k = 3; k >= 0; --k) {
    if (put[k]) {
      const uint32_t p = size + mbcnt64(mp[k]);
      W->item[p] = ((uint32_t)cc[k] << 6) | o;
      W->lb[p] = (uint16_t)(__float_as_uint(lb[k]) >> 16);
    }
    size += (uint32_t)__popcll(mp[k]);
  }
  if (tr && pushed != 1u) atomicAdd(&W->open[o], pushed - 1u);
  lds_order();
}

// First slot of the leaf that a descent by the boxes' farthest corners
// reaches: the warm start of a query without one. (Searches without a first
// bound push every child they meet: 64 of them filled the stack, and 1,000,003
// cold queries on 499,280 faces took 40 ms. A descent by the nearest box picks
// at random among the boxes that hold the point.)
__device__ __forceinline__ int32_t nearest_leaf(const Node4* nodes, float x, float y, float z) {
  int32_t c = 0;
  do {
    const Node4* N = nodes + c;
    float best = INFINITY;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float gx = fmaxf(fabsf(N->lox[k] - x), fabsf(N->hix[k] - x));
      const float gy = fmaxf(fabsf(N->loy[k] - y), fabsf(N->hiy[k] - y));
      const float gz = fmaxf(fabsf(N->loz[k] - z), fabsf(N->hiz[k] - z));
      const float l = gx * gx + gy * gy + gz * gz;
      if (l < best) {  // an unused slot has an empty box: l = inf
        best = l;
        c = N->child[k];
      }
    }
    if (!(best < INFINITY)) return -1;
  } while (c >= 0);
  return ~c & ~3;
}

}  // namespace msk
