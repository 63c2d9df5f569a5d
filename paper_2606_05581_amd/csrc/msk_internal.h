// Internal layouts shared by the host code and the HIP kernels of libmsk.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <vector>

namespace msk {

// 4-wide BVH node, one 128-byte line. Child k's box is
// [lo{x,y,z}[k], hi{x,y,z}[k]]; child[k] >= 0 is an inner node index,
// child[k] < 0 a leaf of count[k] triangles. As the tree is built, ~child[k] is
// the leaf's first slot; once align_leaf_order has laid the leaves out in
// blocks of 4 slots (every tree on the device), the first slot is ~child[k] & ~3
// and the low two bits hold the number of blocks less one.
// An unused slot has an empty box (lo = +inf, hi = -inf) and count 0.
struct alignas(128) Node4 {
  float lox[4], loy[4], loz[4];
  float hix[4], hiy[4], hiz[4];
  int32_t child[4];
  int32_t count[4];
};
static_assert(sizeof(Node4) == 128, "node must be one 128-byte line");

// Triangle in BVH leaf order: vertices as float offsets from the scene
// centre; a.w holds the original triangle index (bit pattern of an int32).
struct alignas(16) TriRec {
  float4 a, b, c;
};
static_assert(sizeof(TriRec) == 48, "triangle record must be 48 bytes");

// A slot past the end of a leaf holds a record with this index; no query
// accepts it.
constexpr int32_t kPadTri = -1;

// Prefilter record of a triangle (quick_prepare_kernel): the triangle in its
// own frame and the margins of the squared distance computed from it, as five
// float4: vertex a, c1; x axis (along ab), s1; y axis (towards c), l1; normal,
// c2; s2, l2, F, G. (c1, s1) and (c2, s2) are the unit directions of ac and bc
// in the plane, l1 and l2 their lengths; the margin is (F + H |p - a|^2) |p - a|^2
// + G, the upper 16 bits of H in the low half of F's word.
// Records lie in blocks of 4 slots, field by field (20 float4 a block: field j
// of slot s is float4 4 j + s % 4 of block s / 4), so that the 4 lanes of a
// unit read 64 contiguous bytes per field. kQuickPad pad records follow the
// last slot.
constexpr int kQuickPad = 8;
__host__ __device__ inline int64_t quick_index(int64_t slot) { return (slot >> 2) * 20 + (slot & 3); }

constexpr int kStackDepth = 64;     // traversal stack entries per lane
constexpr int kMaxTableNnz = 32;    // basis entries per vertex
constexpr int kMaxTop = 85;         // largest accepted msk_bvh_opts.top_nodes

// Host-side BVH build result.
struct HostBvh {
  double centre[3];
  double radius;
  double area;
  std::vector<Node4> nodes;
  std::vector<TriRec> tris;
  std::vector<int32_t> slot_of_tri;  // original triangle -> leaf-order slot
  int depth = 0;                     // levels of 4-wide nodes
  int leaf_size = 4;
  int entry = 1;                     // align_leaves
};

// Builds the scene frame and a 4-wide BVH over float offsets from the
// centre. Returns an empty string on success, else an error message.
std::string build_bvh_host(const float* V, int64_t nv, const int32_t* F, int64_t nf, int leaf_size, HostBvh& out);

// Lets every leaf start at a slot that is a multiple of 4, pads filling the
// slots past a shorter leaf: a leaf's prefilter records, which lie in blocks of
// 4 slots, then fill whole cache lines. Leaf references change to -child - 1 =
// first slot + (blocks - 1). Returns the former slot of each slot (-1: a pad)
// and finds `entry`, the nodes of the deepest level whose levels above are
// full (1, 4, 16 or 64).
std::vector<int32_t> align_leaf_order(std::vector<Node4>& nodes, int64_t n, int& entry);
// The same for a mesh's tree and triangles.
void align_leaves(HostBvh& b);

// The same binned-SAH build and 4-wide collapse over any elements given by
// their boxes and centroids (n x 3 floats): the nodes in breadth-first order
// and the element order of the leaf slots.
struct Box3f {
  float lo[3], hi[3];
};
std::string build_bvh_boxes(const std::vector<Box3f>& boxes, const std::vector<float>& cen, int leaf_size,
                            std::vector<Node4>& nodes_out, std::vector<int32_t>& leaf_order, int& depth);

// ------------------------------------------------------------ kernel ABI

enum RowMode : int32_t { kRowsPoint = 0, kRowsHatRing = 1 };
enum WalkStatus : int32_t { kHit = 0, kEscaped = 1, kCapped = 2 };

// Everything a walk needs about one mesh (device pointers).
// Point basis (point-based k-NN interpolator): the k nearest sample points
// of a query, found on a uniform grid, with bilateral weights. k = 0: the
// basis is the per-vertex table instead.
constexpr int kMaxKnn = 16;
struct KnnDev {
  const float4* pts;          // scene-frame positions (w unused)
  const float4* nrm;          // unit normals (w unused)
  const int32_t* cell_start;  // n_cells + 1 offsets into cell_pts
  const int32_t* cell_pts;    // point indices, by cell
  float lo[3];                // grid origin (scene frame)
  float cell;                 // cell edge
  int32_t dim[3];
  int32_t k;
  double inv2s2;              // 1 / (2 sigma^2)
  double inv_tau;             // 1 / tau_n
};

struct MeshDev {
  const Node4* nodes;
  const TriRec* tris;
  const float4* quick;         // prefilter records
  const int32_t* slot_of_tri;  // original face -> slot
  const int32_t* faces;        // original faces (n_tris x 3)
  int64_t n_tris;
  int32_t entry;               // nodes of the deepest full level of the tree: 1, 4, 16 or 64 (HostBvh)
  int32_t mode;                // RowMode
  float radius;                // bounding-sphere radius (float)
  double radius_d;
  float eps2;                  // eps^2
  float inset;                 // h (walk geometry)
  double inset_d;              // h (scaling of the estimate)
  float kappa;                 // relative step shrink
  float delta;                 // absolute step shrink (delta_rel * radius)
  float slack;                 // absolute error allowance of the FP32 distance
  int32_t side;                // 0 interior, 1 exterior
  int32_t mesh_id;             // low 24 bits of the fourth Philox counter word
  int32_t walks_per_row;       // W
  int64_t max_steps;
  // rows (original order)
  const float* p;              // point rows: scene-frame float positions (n x 3)
  const float* n;              // point rows: unit normals (n x 3)
  const int32_t* tri;          // point rows: face
  const float* bary;           // point rows: barycentrics (n x 3)
  const int32_t* ring_ptr;     // hat rows
  const int32_t* ring_tri;
  const double* ring_cum;
  const float* face_normals;
  const int32_t* discarded;    // per row (point rows)
  const float* ball_r;         // PSD estimator: per-row tangent-ball radius (0 = dropped); null otherwise
  double ball_u0;              // PSD estimator: sin(theta0 / 2) of the cap left out about s
  // basis table
  const int32_t* b_rowptr;
  const int32_t* b_col;
  const float* b_val;
  int64_t K;
  KnnDev knn;                  // point basis (knn.k > 0) instead of the table
  // accumulators (original row order)
  double* acc1;                // point rows: sum b(t); hat rows: sum c
  double* acc2;                // point rows: sum b(t)^2; hat rows: sum c^2
  unsigned long long* row_queries;
  unsigned long long* row_escaped;
  unsigned long long* row_capped;
  // optional walk log, (row, walk) -> row * W + walk - walk_offset
  int32_t* log_status;
  int32_t* log_tri;
  float* log_bary;
  int32_t* log_queries;
};

// A unit of queued work: one row of one mesh; walk ids are slot * W + w.
struct RowSlot {
  int32_t mesh;
  int32_t row;
  uint32_t walk0;  // the slot's first walk, after the launch's walk_offset
};

// A queue counter has a cache line of its own.
constexpr int kQueueStride = 16;

struct WalkLaunch {
  const MeshDev* meshes;       // device array
  const RowSlot* slots;        // device array, n_slots
  int64_t n_slots;
  int64_t walks_per_slot;      // W
  int64_t walk_offset;         // first walk index
  uint32_t seed_lo, seed_hi;
  // persistent form: 8 queues over contiguous slot ranges
  unsigned long long* queue_next;  // 8 counters (walk ids), kQueueStride apart
  const unsigned long long* queue_end;  // 8 ends, then 8 beginnings
  int32_t chunk;
  int32_t regen_min;
  int32_t max_owners;          // persistent form: lanes of a wavefront that carry a walk (1..64)
  int32_t rows;                // persistent form: 1 all meshes have point rows, 2 tangent balls (PSD), else 0
  unsigned long long* stats;   // optional: [nodes visited, triangles tested, FP32 operations]
  int32_t accum;               // persistent form, wavefront row-table partial sums:
                               // 0 FP64, 1 FP32, 2 compensated FP32 (double-float pairs)
  int32_t knn;                 // some mesh uses the point basis: launch the k-NN instantiations
};

// One mesh's point rows in a discard pass over the rows of several meshes.
struct RowRange {
  int64_t first;         // launch index of the mesh's row 0 (ascending over the ranges)
  int32_t mesh;          // index into the launch's MeshDev array
  int32_t* discarded;    // the mesh's discard flags (written)
};

// The per-row counters of one estimate, summed by launch_row_totals.
struct RowCounters {
  const unsigned long long* queries;
  const unsigned long long* escaped;
  const unsigned long long* capped;
  const int32_t* discarded;
  const int64_t* walks;
  const unsigned long long* nonfinite;  // one count
  int64_t n;
};

}  // namespace msk

namespace msk {
// kernel launch wrappers (walk.hip)
hipError_t launch_walk_plain(const WalkLaunch& L, hipStream_t s);
hipError_t launch_walk_persistent(const WalkLaunch& L, int grid, hipStream_t s);
struct QueueInit {
  unsigned long long begin[8], end[8];
};
hipError_t launch_count_nonfinite(const double* a, int64_t n, unsigned long long* count, hipStream_t s);
hipError_t launch_init_queues(unsigned long long* next, unsigned long long* end, const QueueInit& q, hipStream_t s);
hipError_t launch_fill_u64(void* p, int64_t n, unsigned long long v, hipStream_t s);
hipError_t launch_fill_u32(void* p, int64_t n, uint32_t v, hipStream_t s);
hipError_t launch_tangent_ball(const MeshDev& M, int64_t n_rows, float r_max, int32_t iters, float tol, int32_t n_cu,
                               float* radius, hipStream_t s);
hipError_t launch_discard(const MeshDev& M, int64_t n_rows, int32_t n_cu, int32_t* discarded, hipStream_t s);
hipError_t launch_discard_batch(const MeshDev* meshes, const RowRange* ranges, int32_t n_ranges, int64_t n_total,
                                int32_t n_cu, hipStream_t s);
// out: 6 x n_sets counts (queries, escaped, capped, discarded rows, walks of kept rows, non-finite entries)
hipError_t launch_row_totals(const RowCounters* sets, int32_t n_sets, unsigned long long* out, hipStream_t s);
hipError_t launch_knn_eval(const KnnDev& G, const double* c, const float* Q, const float* Nq, int64_t n, int32_t* idx,
                           float* w, hipStream_t s);
// n slots (a multiple of 4); quick: 5 (n + kQuickPad) float4
hipError_t launch_quick_prepare(const TriRec* tris, int64_t n, float4* quick, hipStream_t s);
hipError_t launch_closest_points(const Node4* nodes, const TriRec* tris, const float4* quick, int32_t entry,
                                 float radius, const double* c, const float* Q, int64_t nq, int32_t n_cu, int32_t* tri,
                                 float* d2, float* bary, hipStream_t s);
hipError_t launch_finalize(const MeshDev& M, int64_t n_rows, const int64_t* walks, const double* w, double* S,
                           double* se, hipStream_t s, int32_t jump_only = 0);

// Blocked symmetric products shared by the PSD estimator and the mesh basis
// (psd.hip):
int64_t psd_blocks(int64_t Kp);
// Partial 64 x 64 upper blocks of A^T A (A: m x Kp row-major) into P: slices x 4 slots of psd_blocks(Kp) blocks
hipError_t launch_psd_syrk(const double* A, int64_t m, int64_t Kp, int64_t slices, double* P, hipStream_t s);
hipError_t launch_psd_reduce(const double* P, int64_t n_slots, int64_t K, int64_t Kp, double* C, hipStream_t s);

// Fixed workspace of the allocation-free estimate (noalloc.hip): 64 MiB per
// device, and the padding of the 8 queue counters to cache lines of their own.
// noalloc_scratch_init looks its address up on `device` (which must be current)
// once; noalloc_scratch returns it (nullptr if the lookup failed or was not
// made, with the HIP error in *err).
constexpr size_t kNoallocScratchBytes = (size_t(64) << 20) + 768;
hipError_t noalloc_scratch_init(int device);
void* noalloc_scratch(int device, hipError_t* err);

}  // namespace msk
