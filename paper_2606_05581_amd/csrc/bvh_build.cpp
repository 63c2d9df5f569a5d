// Host construction of the walk geometry: scene frame, binned-SAH binary
// tree, collapse to 4-wide nodes, breadth-first node order and leaf-order
// triangle records.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <exception>
#include <limits>
#include <mutex>
#include <thread>

#include "msk_internal.h"

namespace msk {
namespace {

struct Box {
  float lo[3], hi[3];
  double area() const {
    double d[3];
    for (int k = 0; k < 3; ++k) d[k] = std::max(0.0, (double)hi[k] - (double)lo[k]);
    return 2.0 * (d[0] * d[1] + d[1] * d[2] + d[2] * d[0]);
  }
};

struct BNode {  // binary node
  Box box;
  int32_t left = -1, right = -1;  // children (inner)
  int32_t first = 0, count = 0;   // leaf range in the triangle order
};

typedef float f4 __attribute__((vector_size(16)));

// An element's box and centroid, a vector register each (the fourth lane unused).
struct Elem {
  f4 lo, hi, c;
};

// std::min / std::max of a and b, lane by lane.
inline f4 vmin(f4 a, f4 b) { return b < a ? b : a; }
inline f4 vmax(f4 a, f4 b) { return a < b ? b : a; }

struct VBox {
  f4 lo, hi;
  void reset() {
    const float inf = std::numeric_limits<float>::infinity();
    lo = f4{inf, inf, inf, inf};
    hi = -lo;
  }
  void grow(const VBox& b) {
    lo = vmin(lo, b.lo);
    hi = vmax(hi, b.hi);
  }
  double area() const {
    double d[3];
    for (int k = 0; k < 3; ++k) d[k] = std::max(0.0, (double)hi[k] - (double)lo[k]);
    return 2.0 * (d[0] * d[1] + d[1] * d[2] + d[2] * d[0]);
  }
};

// The binary tree over `order`, split by split. A range's tree depends on that
// range alone, so once the top of the tree has cut it into ranges of at most
// n / 16 elements, threads take the ranges one by one and their nodes are
// appended afterwards; the tree is the one a single thread builds. One pass
// over a range bins all three axes, boxes as vectors. A 30,000-triangle mesh
// is built and uploaded in 3.4 ms on eight threads (9.9 ms element by element
// and axis by axis on one). Below kThreadElems the work of a millisecond or
// less is not worth the threads' start.
#ifndef MSK_BVH_THREAD_ELEMS
#define MSK_BVH_THREAD_ELEMS 8192
#endif
constexpr int32_t kThreadElems = MSK_BVH_THREAD_ELEMS;

struct Builder {
  const std::vector<Elem>& el;
  std::vector<int32_t>& order;
  std::vector<BNode> nodes;
  int leaf_size;

  struct Item { int32_t first, count, parent; bool is_left; };

  Builder(const std::vector<Elem>& el_, std::vector<int32_t>& order_, int leaf)
      : el(el_), order(order_), leaf_size(leaf) {}

  // Nodes of the items on `stack` and below into `out`; items of at most
  // `defer` elements go to `later` instead.
  void grow(std::vector<Item>& stack, std::vector<BNode>& out, int32_t defer, std::vector<Item>* later) const {
    constexpr int kBins = 16;
    while (!stack.empty()) {
      const Item it = stack.back();
      stack.pop_back();
      if (it.count <= defer) {
        later->push_back(it);
        continue;
      }
      VBox b, cb;
      b.reset();
      cb.reset();
      for (int32_t i = it.first; i < it.first + it.count; ++i) {
        const Elem& e = el[order[i]];
        b.grow({e.lo, e.hi});
        cb.grow({e.c, e.c});
      }
      const bool split = it.count > leaf_size;
      int best_axis = -1, best_bin = -1;
      double best_cost = std::numeric_limits<double>::infinity();
      double scale[3] = {0.0, 0.0, 0.0};  // 0: no extent, not binned
      if (split) {
        VBox bins[3][kBins];
        int32_t cnt[3][kBins] = {{0}};
        for (int ax = 0; ax < 3; ++ax) {
          const double ext = (double)cb.hi[ax] - (double)cb.lo[ax];
          if (ext > 0) scale[ax] = kBins / ext;
          for (auto& x : bins[ax]) x.reset();
        }
        for (int32_t i = it.first; i < it.first + it.count; ++i) {
          const Elem& e = el[order[i]];
          const f4 off = e.c - cb.lo;
          for (int ax = 0; ax < 3; ++ax) {
            const int bi = std::min(kBins - 1, (int)(off[ax] * scale[ax]));
            cnt[ax][bi]++;
            bins[ax][bi].grow({e.lo, e.hi});
          }
        }
        for (int ax = 0; ax < 3; ++ax) {
          if (!(scale[ax] > 0)) continue;
          VBox lb[kBins];
          int32_t lc[kBins];
          VBox acc;
          acc.reset();
          int32_t c = 0;
          for (int i = 0; i < kBins; ++i) {
            acc.grow(bins[ax][i]);
            c += cnt[ax][i];
            lb[i] = acc;
            lc[i] = c;
          }
          acc.reset();
          c = 0;
          for (int i = kBins - 1; i > 0; --i) {
            if (cnt[ax][i] == 0) continue;  // the cut above this bin is the one already priced
            acc.grow(bins[ax][i]);
            c += cnt[ax][i];
            if (lc[i - 1] == 0) continue;
            const double cost = lb[i - 1].area() * lc[i - 1] + acc.area() * c;
            if (cost < best_cost) {
              best_cost = cost;
              best_axis = ax;
              best_bin = i;
            }
          }
        }
      }
      int32_t mid = -1;
      if (split && best_axis >= 0) {
        const float lo = cb.lo[best_axis];
        const double sc = scale[best_axis];
        auto part = std::partition(order.begin() + it.first, order.begin() + it.first + it.count, [&](int32_t t) {
          return std::min(kBins - 1, (int)((el[t].c[best_axis] - lo) * sc)) < best_bin;
        });
        mid = (int32_t)(part - order.begin());
        if (mid == it.first || mid == it.first + it.count) mid = -1;
      }
      if (split && mid < 0) {  // coincident centroids: split the range in half
        mid = it.first + it.count / 2;
      }
      BNode nd;
      for (int k = 0; k < 3; ++k) {
        nd.box.lo[k] = b.lo[k];
        nd.box.hi[k] = b.hi[k];
      }
      const int32_t id = (int32_t)out.size();
      if (!split) {
        nd.first = it.first;
        nd.count = it.count;
      }
      out.push_back(nd);
      if (split) {
        stack.push_back({mid, it.first + it.count - mid, id, false});
        stack.push_back({it.first, mid - it.first, id, true});
      }
      if (it.parent >= 0) (it.is_left ? out[it.parent].left : out[it.parent].right) = id;
    }
  }

  void build(int32_t n) {
    std::vector<Item> stack, later;
    stack.push_back({0, n, -1, false});
    grow(stack, nodes, n >= kThreadElems ? n / 16 : 0, &later);
    std::vector<std::vector<BNode>> sub(later.size());
    std::atomic<size_t> next{0};
    std::exception_ptr failed;
    std::mutex m;
    auto work = [&] {
      try {
        for (size_t i; (i = next.fetch_add(1)) < later.size();) {
          std::vector<Item> own{{later[i].first, later[i].count, -1, false}};
          sub[i].reserve((size_t)(2 * later[i].count / std::max(1, leaf_size) + 8));
          grow(own, sub[i], 0, nullptr);
        }
      } catch (...) {
        std::lock_guard<std::mutex> lk(m);
        failed = std::current_exception();
      }
    };
    std::vector<std::thread> threads;
    const unsigned hc = std::min(std::max(1u, std::thread::hardware_concurrency()), 8u);
    try {
      for (unsigned i = 1; i < hc && i < later.size(); ++i) threads.emplace_back(work);
    } catch (const std::exception&) {  // no more threads: those there are do the work
    }
    work();
    for (auto& t : threads) t.join();
    if (failed) std::rethrow_exception(failed);
    for (size_t i = 0; i < later.size(); ++i) {
      const int32_t base = (int32_t)nodes.size();
      for (BNode nd : sub[i]) {
        if (nd.left >= 0) {
          nd.left += base;
          nd.right += base;
        }
        nodes.push_back(nd);
      }
      const Item& it = later[i];
      (it.is_left ? nodes[it.parent].left : nodes[it.parent].right) = base;
    }
  }
};

}  // namespace

std::string build_bvh_boxes(const std::vector<Box3f>& boxes, const std::vector<float>& cen, int leaf_size,
                            std::vector<Node4>& nodes_out, std::vector<int32_t>& leaf_order, int& depth) {
  if (boxes.empty()) return "no elements";
  if (leaf_size < 1 || leaf_size > 8) return "leaf_size must be in 1..8";
  const int64_t nf = (int64_t)boxes.size();
  std::vector<Elem> el((size_t)nf);
  for (int64_t i = 0; i < nf; ++i) {
    const Box3f& b = boxes[i];
    el[i] = {f4{b.lo[0], b.lo[1], b.lo[2], 0.f}, f4{b.hi[0], b.hi[1], b.hi[2], 0.f},
             f4{cen[3 * i], cen[3 * i + 1], cen[3 * i + 2], 0.f}};
  }
  std::vector<int32_t> order((size_t)nf);
  for (int64_t i = 0; i < nf; ++i) order[i] = (int32_t)i;
  Builder bld(el, order, leaf_size);
  bld.nodes.reserve((size_t)(2 * nf / std::max(1, leaf_size) + 8));
  bld.build((int32_t)nf);
  const std::vector<BNode>& bn = bld.nodes;

  // Collapse to 4-wide nodes, breadth first. Each wide node gathers up to
  // four binary descendants by repeatedly opening the largest inner child.
  struct WItem { int32_t bin; int32_t depth; };
  std::vector<WItem> queue;
  nodes_out.clear();
  std::vector<int32_t> wide_of;  // queue index == wide node index
  queue.push_back({0, 1});
  size_t head = 0;
  int maxdepth = 0;
  std::vector<int32_t> leaf_first, leaf_count;
  // leaf order assigned in BFS order of leaves
  leaf_order.clear();
  leaf_order.reserve((size_t)nf);
  while (head < queue.size()) {
    WItem it = queue[head++];
    maxdepth = std::max(maxdepth, it.depth);
    Node4 w;
    for (int k = 0; k < 4; ++k) {
      w.lox[k] = w.loy[k] = w.loz[k] = INFINITY;
      w.hix[k] = w.hiy[k] = w.hiz[k] = -INFINITY;
      w.child[k] = INT32_MIN;
      w.count[k] = 0;
    }
    int32_t kids[4];
    int nk = 0;
    const BNode& root = bn[it.bin];
    if (root.left < 0) {
      kids[nk++] = it.bin;  // whole tree is a single leaf
    } else {
      kids[nk++] = root.left;
      kids[nk++] = root.right;
      while (nk < 4) {
        int best = -1;
        double ba = -1;
        for (int k = 0; k < nk; ++k)
          if (bn[kids[k]].left >= 0 && bn[kids[k]].box.area() > ba) {
            ba = bn[kids[k]].box.area();
            best = k;
          }
        if (best < 0) break;
        int32_t b = kids[best];
        kids[best] = bn[b].left;
        kids[nk++] = bn[b].right;
      }
    }
    for (int k = 0; k < nk; ++k) {
      const BNode& c = bn[kids[k]];
      w.lox[k] = c.box.lo[0]; w.loy[k] = c.box.lo[1]; w.loz[k] = c.box.lo[2];
      w.hix[k] = c.box.hi[0]; w.hiy[k] = c.box.hi[1]; w.hiz[k] = c.box.hi[2];
      if (c.left < 0) {
        int32_t first = (int32_t)leaf_order.size();
        for (int32_t i = c.first; i < c.first + c.count; ++i) leaf_order.push_back(order[i]);
        w.child[k] = -first - 1;
        w.count[k] = c.count;
      } else {
        w.child[k] = (int32_t)queue.size();
        queue.push_back({kids[k], it.depth + 1});
      }
    }
    nodes_out.push_back(w);
  }
  depth = maxdepth;
  if ((int64_t)leaf_order.size() != nf) return "internal error: element count mismatch";
  // traversal stack: at most 3 pending siblings per level (with margin)
  if (3 * maxdepth + 5 > kStackDepth) return "BVH too deep for the traversal stack";
  return "";
}

std::string build_bvh_host(const float* V, int64_t nv, const int32_t* F, int64_t nf, int leaf_size, HostBvh& out) {
  if (nv < 3 || nf < 1) return "mesh needs at least 3 vertices and 1 triangle";
  // the walk kernel packs a triangle slot and a lane into one 32-bit word
  if (nf >= (int64_t)1 << 26) return "too many triangles (a mesh holds at most 2^26 - 1)";
  if (leaf_size < 1 || leaf_size > 8) return "leaf_size must be in 1..8";
  out.leaf_size = leaf_size;
  double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int64_t i = 0; i < nv; ++i)
    for (int k = 0; k < 3; ++k) {
      double x = V[3 * i + k];
      if (!std::isfinite(x)) return "vertex coordinates must be finite";
      lo[k] = std::min(lo[k], x);
      hi[k] = std::max(hi[k], x);
    }
  for (int k = 0; k < 3; ++k) out.centre[k] = 0.5 * (lo[k] + hi[k]);
  double r2 = 0;
  for (int64_t i = 0; i < nv; ++i) {
    double d0 = V[3 * i] - out.centre[0], d1 = V[3 * i + 1] - out.centre[1], d2 = V[3 * i + 2] - out.centre[2];
    r2 = std::max(r2, d0 * d0 + d1 * d1 + d2 * d2);
  }
  out.radius = (1.0 + std::ldexp(1.0, -20)) * std::sqrt(r2);
  std::vector<float> Vr((size_t)nv * 3);
  for (int64_t i = 0; i < nv; ++i)
    for (int k = 0; k < 3; ++k) Vr[3 * i + k] = (float)((double)V[3 * i + k] - out.centre[k]);

  std::vector<Box3f> tb((size_t)nf);
  std::vector<float> cen((size_t)nf * 3);
  double area = 0;
  for (int64_t t = 0; t < nf; ++t) {
    for (int k = 0; k < 3; ++k) {
      tb[t].lo[k] = std::numeric_limits<float>::infinity();
      tb[t].hi[k] = -std::numeric_limits<float>::infinity();
    }
    double c[3] = {0, 0, 0}, P[3][3];
    for (int j = 0; j < 3; ++j) {
      int64_t v = F[3 * t + j];
      if (v < 0 || v >= nv) return "face index out of range";
      for (int k = 0; k < 3; ++k) {
        float x = Vr[3 * v + k];
        tb[t].lo[k] = std::min(tb[t].lo[k], x);
        tb[t].hi[k] = std::max(tb[t].hi[k], x);
        c[k] += x;
        P[j][k] = V[3 * v + k];
      }
    }
    for (int k = 0; k < 3; ++k) cen[3 * t + k] = (float)(c[k] / 3.0);
    double e1[3], e2[3];
    for (int k = 0; k < 3; ++k) {
      e1[k] = P[1][k] - P[0][k];
      e2[k] = P[2][k] - P[0][k];
    }
    double cx = e1[1] * e2[2] - e1[2] * e2[1], cy = e1[2] * e2[0] - e1[0] * e2[2], cz = e1[0] * e2[1] - e1[1] * e2[0];
    area += 0.5 * std::sqrt(cx * cx + cy * cy + cz * cz);
  }
  if (!(area > 0)) return "mesh has zero total area";
  out.area = area;

  std::vector<int32_t> leaf_order;
  std::string err = build_bvh_boxes(tb, cen, leaf_size, out.nodes, leaf_order, out.depth);
  if (!err.empty()) return err;
  std::vector<TriRec> tris(leaf_order.size());
  out.slot_of_tri.assign((size_t)nf, -1);
  for (size_t slot = 0; slot < leaf_order.size(); ++slot) {
    const int32_t t = leaf_order[slot];
    TriRec r;
    const int32_t* f = F + 3 * (int64_t)t;
    r.a = make_float4(Vr[3 * f[0]], Vr[3 * f[0] + 1], Vr[3 * f[0] + 2], 0.f);
    r.b = make_float4(Vr[3 * f[1]], Vr[3 * f[1] + 1], Vr[3 * f[1] + 2], 0.f);
    r.c = make_float4(Vr[3 * f[2]], Vr[3 * f[2] + 1], Vr[3 * f[2] + 2], 0.f);
    int32_t ti = t;
    std::memcpy(&r.a.w, &ti, 4);
    out.slot_of_tri[t] = (int32_t)slot;
    tris[slot] = r;
  }
  out.tris.swap(tris);
  if ((int64_t)out.tris.size() != nf) return "internal error: triangle count mismatch";
  return "";
}

std::vector<int32_t> align_leaf_order(std::vector<Node4>& nodes, int64_t n, int& entry) {
  std::vector<int32_t> from;
  from.reserve((size_t)n * 3 / 2 + 8);
  for (Node4& w : nodes)
    for (int k = 0; k < 4; ++k) {
      if (w.child[k] >= 0 || w.count[k] == 0) continue;
      const int32_t first = -w.child[k] - 1;
      w.child[k] = -((int32_t)from.size() + (w.count[k] - 1) / 4) - 1;
      for (int32_t i = first; i < first + w.count[k]; ++i) from.push_back(i);
      while (from.size() % 4) from.push_back(-1);
    }
  // levels 0, 1, 2 (nodes 0; 1-4; 5-20) with four inner children each
  entry = 1;
  for (size_t level = 1, i = 0; level <= 16; level *= 4) {
    bool full = i + level <= nodes.size();
    for (size_t j = i; full && j < i + level; ++j)
      for (int k = 0; k < 4; ++k) full = full && nodes[j].child[k] >= 0;
    if (!full) break;
    entry = (int)(4 * level);
    i += level;
  }
  return from;
}

void align_leaves(HostBvh& b) {
  const std::vector<int32_t> from = align_leaf_order(b.nodes, (int64_t)b.tris.size(), b.entry);
  TriRec pad;
  pad.a = pad.b = pad.c = make_float4(0.f, 0.f, 0.f, 0.f);
  std::memcpy(&pad.a.w, &kPadTri, 4);
  std::vector<TriRec> tris(from.size(), pad);
  for (size_t s = 0; s < from.size(); ++s) {
    if (from[s] < 0) continue;
    tris[s] = b.tris[from[s]];
    int32_t t;
    std::memcpy(&t, &tris[s].a.w, 4);
    b.slot_of_tri[t] = (int32_t)s;
  }
  b.tris.swap(tris);
}

}  // namespace msk
