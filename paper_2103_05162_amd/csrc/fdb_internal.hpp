// Host-side internals of libfdbscan: the workspace plan, the device views the
// kernels receive, and the launch helpers each kernel file exports.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

struct fdb_handle;

namespace fdb {

// Keys per thread in a radix pass, by key width (measured: 64-bit keys fit two
// 6144-key tiles per CU in LDS; 32-bit keys do best at 5632, two rounds of the 768
// tiles resident at once for 8M of them). Small inputs take fewer (k_sort.hip). The
// workspace sizes the look-back status for the tile taken (sort_status_words).
template <typename K>
constexpr int sort_items() { return sizeof(K) == 8 ? 24 : 22; }
constexpr int kScanItems = 16;                 // items per thread in the device scan
constexpr int kScanTile = 256 * kScanItems;
constexpr int64_t kMaxPoints = (int64_t(1) << 30) - 1;
constexpr uint8_t kCliqueCore = 2, kInClique = 3;  // core flags of points in FDbscan's cliques (TravArgs::core)
constexpr int kRecNb = 8;  // neighbouring primitives recorded per non-core point
constexpr int kBorderCounters = 32 * 17;  // words of TravArgs::border_n (they fit the digit histograms)

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Byte offsets of every buffer inside the caller's (or the handle's) workspace.
// Sizes depend on (n, dim, algo) only, never on eps or minPts: the footprint is
// linear in n (Section 3.2).
struct Plan {
  int64_t n = 0;
  int dim = 3;
  int algo = 0;
  size_t bytes = 0;
  // common
  size_t bounds, misc, gplan, keys0, keys1, vals0, vals1, hist, pass_plan, tilectr, status;
  size_t xs;                       // dim * n floats, sorted SoA
  size_t node_a, node_b, rope, leaf_rope, ends, other, gamma, cut;
  size_t labels, core, lone, qborder, brec_i, brec_nb;
  int64_t brec_cap = 0;
  size_t minorig, lflag, rank, bsums, cid, border;
  // DenseBox
  size_t cell_id, cell_start, cand, cell_dense, cell_lo, cell_hi, pflag, prim_start, prim_cnt,
      prim_lo, prim_hi, prim_key, dense_list;
  // batches
  int num_clouds = 0;
  size_t cl_lo, cl_scale, cl_eps2, cl_minpts, cl_root, cl_end, cl_flags, cl_ord;
  int64_t scan_blocks = 0;
  int64_t super_cap = 0;  // DenseBox: supers that the node records' buffer holds
};

// FDbscan's curve over a scene too wide for its keys: floats of a sample per axis, sorted,
// and where the curve has each (6 kCurveKnots, in the place of TreeView's cut, which FDbscan
// has no use for).
constexpr int kCurveKnots = 1024;

Plan make_plan(int64_t n, int dim, int algo, int num_clouds = 0);

// Small device-side scalars kept in the workspace's misc block.
enum MiscSlot : int {
  kMiscNumClusters = 0,  // K after the scan
  kMiscNumCells = 1,     // DenseBox: number of non-empty cells
  kMiscNumCand = 2,      // DenseBox: cells with >= minPts points
  kMiscNumPrims = 3,     // DenseBox: m = dense cells + points outside them
  kMiscNumDense = 4,     // DenseBox: dense cells
  kMiscCut = 7,          // entries of the hierarchy's cut (TreeView::cut)
  kMiscNumBricks = 8,    // DenseBox: occupied bricks
  kMiscNumCliques = 9,   // FDbscan: listed cliques
  kMiscNumBoxes = 10,    // FDbscan: listed boxes of fewer than minPts points
  kMiscCount = 16
};

// DenseBox grid of one cloud (Section 4.2: cells of side eps/sqrt(d)), sized on
// the device from the scene bounds by k_grid_plan, so no value goes back to the
// host mid-call. The key, sort and dense-cell kernels and the walks read it.
// When the eps/sqrt(d) grid needs more cells per axis than a 64-bit key holds
// (21 bits per axis in 3D, 31 in 2D), the cells are widened to fit (coarse = 1,
// FDB_INFO_DENSEBOX_FALLBACK): density is still decided by the exact guard, so
// labels stay exact; only fewer cells come out dense.
struct GridPlan {
  float inv_h[4];      // 1 / cell side, per axis
  uint32_t ncell[4];   // cells per axis (>= 1)
  int32_t bits;        // key bits per axis
  int32_t key64;       // 1: d * bits > 32, keys are stored as 64-bit words, else 32-bit
  int32_t passes;      // 8-bit radix passes over the d * bits key bits
  int32_t start;       // key buffer (0/1) the key kernel fills: the sort then ends in buffer 1
  int32_t coarse;      // cells widened to fit 64-bit keys
  int32_t grid_on;     // neighbours are searched through the grid (CellIndex), else through the hierarchy
  float reach;         // eps / side plus rounding slack, in cell units
  float lo[3];         // the scene's low corner
  int32_t axis_bits[3];  // key bits of each axis (FDbscan's curve: its own for each)
  int32_t curve_sampled;  // the curve's cells follow a sample of the points (kCurveKnots)
  int32_t sets;          // a batch: some cloud's minPts is worth TravArgs::cell_sets
  double curve_inv[3];   // FDbscan's curve: 1 / cell side of each axis
  uint64_t supers;     // supers of the grid (a batch: of all its grids)
};

// The occupied cells as a three-level index (fdb_cells.hpp): supers (16 bytes each:
// occupancy word, first brick), bricks (occupancy word, first cell) and each cell's
// first primitive. A batch has a grid per cloud: its corner in cl_lo, 1 / side and
// reach in cl_scale (x, w), and in cl_grid[2 c] its cells per axis and first super.
struct CellIndex {
  const GridPlan* plan;
  uint4* supers;
  uint4* bricks;
  int* cell_prim;   // first primitive of each cell, complemented for a dense cell; then the number of primitives
  int* brick_base;  // first cell of each brick (while the index is built)
  uint8_t* cell_code;  // low 6 key bits of each cell (while the index is built)
  int64_t super_cap;   // supers the table holds
  const float4* cl_lo;
  const float4* cl_scale;
  const int4* cl_grid;
};

// Node records are interleaved: node k's two halves sit at node_a[kNodeStride * k]
// and node_b[kNodeStride * k] with node_b = node_a + 1, so a node is 32
// contiguous bytes (one cache line) rather than two lines in two arrays.
constexpr int kNodeStride = 2;

// Device view of an LBVH over m primitives. Internal node k: node_a[k] =
// (lo.xyz, other end of its leaf range as int bits), node_b[k] = (hi.xyz, split
// position gamma as int bits); its leaves are [min(k,other), max(k,other)], its
// children cover [first,gamma] and [gamma+1,last]. rope[k] / leaf_rope[l] give
// the next node in depth-first pre-order after that subtree (kEnd at the end).
struct TreeView {
  const float4* node_a;
  const float4* node_b;
  const int* rope;
  const int* leaf_rope;
  int m_cap;       // number of primitives, or an upper bound when d_m is set
  const int* d_m;  // device-side primitive count (DenseBox), or null
  int leaf_size;   // subtrees of at most this many primitives are scanned linearly
  // A cut through the hierarchy (single-cloud trees): the maximal subtrees of at
  // most cut_span(m) primitives, as pairs {lo.xyz, node ref} {hi.xyz, last
  // primitive}, *cut_n of them; a box walk over the whole tree tests these at once
  // instead of descending from the root. Null, or a count above kCutMax: no cut.
  const float4* cut = nullptr;
  const int* cut_n = nullptr;
};

constexpr int kCutMax = 8192;
constexpr int kCutDiv = 256;      // the cut holds about kCutDiv to 2 kCutDiv subtrees
constexpr int kCutUnroll = 4;     // cut entries a lane loads at once
__host__ __device__ inline int cut_span(int m) {
  const int span = (m + kCutDiv - 1) / kCutDiv;
  return span > 64 ? span : 64;
}

// ---- launch helpers (stream-ordered, asynchronous) --------------------------
void fill_u32(uint32_t* p, uint32_t v, int64_t n, hipStream_t s);
void fill_u8(uint8_t* p, uint8_t v, int64_t n, hipStream_t s);
// Up to 8 fills of 32-bit words in one launch (a call's counters and flags).
struct FillSeg {
  uint32_t* p;
  uint32_t v;
  int64_t n;
};
struct FillList {
  FillSeg seg[8];
  int count = 0;
  void add(void* p, uint32_t v, int64_t n) {
    if (n > 0) seg[count++] = FillSeg{static_cast<uint32_t*>(p), v, n};
  }
};
void fill_multi(const FillList& L, hipStream_t s);

// k_prep.hip
void launch_bounds(const float* pts, int64_t n, int dim, uint32_t* bounds, uint32_t* info, hipStream_t s);
// DenseBox of one cloud: k_grid_plan writes *plan from the bounds (after
// launch_bounds; eps is the caller's), then the cell keys go to key buffer
// plan->start as 32- or 64-bit words with the identity permutation, and their
// digits are counted for the sort (hist: 8 x 256 words, cleared by the caller). The key kernel also clears the super table that
// the grid's index is built into (plan->supers entries, when plan->grid_on).
// knots: FDbscan (its keys are a curve's, and no cells are searched), null for DenseBox.
void launch_grid_plan(const float* pts, int64_t n, const uint32_t* bounds, int dim, float eps, int64_t super_cap,
                      float* knots, GridPlan* plan, uint32_t* info, hipStream_t s);
void launch_gridkeys(const float* pts, int64_t n, int dim, const uint32_t* bounds, const GridPlan* plan,
                     void* keys0, void* keys1, uint32_t* vals0, uint32_t* vals1, uint32_t* hist, uint4* supers,
                     const float* knots, hipStream_t s);
void launch_permute(const float* pts, int64_t n, int dim, const uint32_t* perm, float* xs, uint32_t* info,
                    hipStream_t s);

// k_sort.hip: LSD radix sort of (64-bit key, index) pairs over the low `bits` bits (a
// batch's). hist holds the digit counts of every pass, from the key kernel. pass_plan: 8
// words (which passes run: one over a constant digit need not). The tile counters (16
// words) and look-back words (sort_status_words) are cleared here. Returns which of the
// two buffers holds the result (0 or 1).
int radix_sort(uint64_t* keys0, uint64_t* keys1, uint32_t* vals0, uint32_t* vals1, int64_t n, int bits,
               const uint32_t* hist, uint32_t* pass_plan, uint32_t* tilectr, uint64_t* status, uint32_t* info,
               hipStream_t s);
int64_t sort_status_words(int64_t n, bool key64);
// The same with key width and pass count taken from a GridPlan on the device:
// passes for both widths are launched and those the plan does not call for exit
// at once. The keys start in buffer plan->start and end in buffer 1; hist holds
// every pass's digit counts (from the key kernel). The caller has cleared the tile
// counters (16 words) and the look-back words (planned_status_words(n)).
void radix_sort_planned(void* keys0, void* keys1, uint32_t* vals0, uint32_t* vals1, int64_t n, const GridPlan* plan,
                        const uint32_t* hist, uint32_t* tilectr, uint64_t* status, uint32_t* info, hipStream_t s);
int64_t planned_status_words(int64_t n);

// k_tree.hip
// prim_lo / prim_hi: DenseBox leaf records (null for FDbscan, whose leaves are
// the sorted points); see TravArgs. ends: m words of scratch; other / gamma:
// each internal node's other range end and split (m - 1 words each). cut / cut_n:
// the cut of TreeView (kCutMax pairs, and a counter the caller zeroed), or null.
// keys: 64-bit words, or where d_key64 is given and *d_key64 on the device is 0, 32-bit.
// d_skip (device, optional): nonzero = no hierarchy is needed, the kernels leave.
void build_lbvh(const void* keys, const int* d_key64, int m, int dim, const float* xs, int64_t n_pts,
                const float4* prim_lo, const float4* prim_hi, float4* node_a, float4* node_b, int* rope,
                int* leaf_rope, int* ends, int* other, int* gamma, const int* d_m, uint32_t* info, hipStream_t s,
                float4* cut = nullptr, int* cut_n = nullptr, bool ends_ready = false, const int* d_skip = nullptr);

// k_dense.hip
// sorted_keys are 64-bit words when key64 (or, with d_key64 set, when *d_key64 on
// the device says so), else 32-bit; prim_key receives each primitive's key as a
// 64-bit word. ends / minorig (optional): set to -1 per primitive and to INT_MAX
// per point, the starting values of build_lbvh's exchange words (pass
// ends_ready) and of launch_finalize's minorig; border_n (optional): the core pass'
// counters, cleared. The grid's index ix is built over
// the cells (its words and bricks only when ix.plan->grid_on).
void densebox_cells(const void* sorted_keys, bool key64, const int* d_key64, int64_t n, int dim, const float* xs,
                    float eps2, int min_pts, int* cell_id, int* cell_start, int* cand, uint8_t* cell_dense,
                    float4* cell_lo, float4* cell_hi, int* pflag, int* prim_start, int* prim_cnt, float4* prim_lo,
                    float4* prim_hi, uint64_t* prim_key, int* dense_list, int* labels, uint8_t* core, int* misc,
                    int* bsums, hipStream_t s, const CellIndex& ix, int key_shift = 0,
                    const int* cl_minpts = nullptr, const float* cl_eps2 = nullptr, int num_clouds = 0,
                    int* ends = nullptr, int* minorig = nullptr, int* border_n = nullptr);

// k_trav.hip
// With minPts up to this a cell that is not dense has too few points for TravArgs::
// cell_sets to be worth it.
constexpr int kSetMinPts = 16;

struct TravArgs {
  TreeView t;
  const float* xs;  // sorted SoA coordinates: x[n], y[n], z[n]
  int64_t n;
  float eps2;
  int packet_leaf;    // bucket size of the cliques' walks (a bucket is loaded one point per lane)
  int min_pts;
  int* labels;
  // nonzero = core; FDbscan: kInClique for a point of a listed clique, kCliqueCore for one
  // of a smaller clique, 0 elsewhere before the core pass
  uint8_t* core;
  int* cliques;      // FDbscan: the nodes (kLeaf | point) that are listed cliques, *num_cliques of them
  int* num_cliques;
  int* boxes;        // FDbscan: boxes that are no cliques before the core pass, *num_boxes of them
  int* num_boxes;
  uint8_t* lone;  // set by the core pass: 1 = not core and no
                  // neighbour but itself (noise); NULL if no core pass
  // Border work left by the core pass for non-core points with some neighbour
  // other than themselves. Up to kRecNb neighbouring primitives of such a point (the
  // point itself, or a dense cell's first point) are recorded, so the border pass
  // needs no walk: record k of shard x (of kNumXcd), at r = x * brec_cap + k, is point
  // brec_i[r] with neighbours brec_nb[r * kRecNb + t] (-1 = none); the first brec_cap
  // asked for in a shard are stored. Points with more neighbouring primitives, or past
  // the capacity, are listed in qborder per XCD (DenseBox: their primitive indices;
  // XCD x's list starts at its share of the queries) and walk again. border_n holds
  // the counts (kBorderCounters words, zero before the core pass).
  int* brec_i;
  int* brec_nb;
  int brec_cap;
  int* qborder;
  int* border_n;
  const int* cid;
  int* border;
  // DenseBox primitives (null for FDbscan). Primitive r covers sorted points
  // [prim_start[r], prim_start[r] + |prim_cnt[r]|); prim_cnt > 0: a single
  // point, < 0: a dense cell. prim_lo[r] is the leaf record a walk loads: a
  // point's coordinates with its sorted index as int bits in w (>= 0), or a
  // dense cell's low corner with w = -2 - its first point; prim_hi[r] is a
  // dense cell's high corner.
  const int* prim_start;
  const int* prim_cnt;
  const float4* prim_lo;
  const float4* prim_hi;
  const int* dense_list;  // dense-cell primitive indices
  const int* d_ndense;    // their number (device)
  CellIndex ix;           // DenseBox: the grid's cells; ix.plan->grid_on says whether the walks go through it
  // DenseBox, or null: of each cell of kSetCell points or more that is not dense, once the
  // core pass is done: its first core point, all of them being in one set (kSetWhole added
  // where all its points are core), -2: it has none, -1: unknown
  const int* cell_sets;
  // batches (null pkeys = one cloud): cloud of sorted point i = pkeys[i] >> key_shift;
  // per cloud: first node and last primitive of its subtree, eps^2, minPts
  const uint64_t* pkeys;
  int key_shift;
  int num_clouds;
  const int* cloud_root;
  const int* cloud_end;
  const float* cloud_eps2;
  const int* cloud_minpts;
  uint32_t* info;  // FDB_INFO_* bits; kernels raise FDB_INFO_INTERNAL on a broken walk
  int block;
};
void launch_core(const TravArgs& a, int dim, bool densebox, hipStream_t s);
// Fills cell_sets (its memory: sets) where minPts makes it worth it, after the core pass.
void launch_cell_sets(TravArgs& a, int dim, const int* cell_start, const uint8_t* cell_dense, const int* d_cells,
                      int* sets, hipStream_t s);
// FDbscan's cliques (subtrees of core points pairwise within eps): found, marked in labels
// and core, listed in cliques, before the core pass and, of fewer than minPts points each,
// after it; then joined to what is within reach of them.
void launch_cliques(const TravArgs& a, int dim, hipStream_t s);
void launch_core_boxes(const TravArgs& a, hipStream_t s);
void launch_main_cliques(const TravArgs& a, int dim, bool all_core, hipStream_t s);
void launch_main(const TravArgs& a, int dim, bool densebox, bool all_core, bool first_border, int part,
                 hipStream_t s);
void launch_border(const TravArgs& a, int dim, bool densebox, hipStream_t s);
void launch_debug_walk(const TreeView& t, int m, int mask, int* out_leaves, int* out_count, int cap,
                       uint32_t* info, hipStream_t s);

// k_label.hip
// labels[i] = i; with ends / minorig / border_n, also those starting values (see densebox_cells);
// with core, no point is core yet.
void launch_init_labels(int* labels, int64_t n, hipStream_t s, int* ends = nullptr, int* minorig = nullptr,
                        int* border_n = nullptr, uint8_t* core = nullptr);
// With minorig (core flags final): also the smallest input index (perm) of each
// root's core points, in minorig[root] (INT_MAX beforehand, unless minorig_init:
// then filled here first), and the leader words `bits` (ceil(n/32)) cleared.
void launch_finalize(int* labels, int64_t n, uint32_t* info, hipStream_t s, const uint8_t* core = nullptr,
                     const uint32_t* perm = nullptr, int* minorig = nullptr, uint32_t* bits = nullptr,
                     bool minorig_init = true);
void launch_core_from_sets(const int* labels, uint8_t* core, int64_t n, int min_pts, hipStream_t s);
void launch_check_forest(const int* labels, const uint8_t* core, int64_t n, uint32_t* bad, uint32_t* info,
                         hipStream_t s);
// Canonical cluster ids (ids 0..K-1 in increasing order of each cluster's
// smallest core input index). bits: ceil(n/32) leader words; wpre: ceil(n/32) ints.
// minorig_ready: launch_finalize already filled minorig and cleared the leader words.
void canonical_ids(const int* labels, const uint8_t* core, const uint32_t* perm, int64_t n, int* minorig,
                   uint32_t* bits, int* wpre, int* bsums, int* cid, int* d_k, hipStream_t s,
                   bool ids = true, bool minorig_ready = false);

// k_batch.hip
void batch_prep(const float* pts, const int64_t* off, int num_clouds, int64_t n, int dim, const float* eps,
                const int32_t* min_pts, int bpd, bool densebox, uint32_t* cl_ord, float4* cl_lo, float4* cl_scale,
                float* cl_eps2, int* cl_minpts, int* cl_flags, uint32_t* info, GridPlan* plan, int64_t super_cap,
                hipStream_t s);
void batch_keys(const float* pts, const int64_t* off, int num_clouds, int64_t n, int dim, const float4* cl_lo,
                const float4* cl_scale, int bpd, int shift, uint64_t* keys, uint32_t* vals, int sort_bits,
                uint32_t* hist, uint4* supers, const GridPlan* plan, hipStream_t s);
void batch_roots(const int64_t* off, int num_clouds, int64_t n, const int* pidx, const int* d_m, const int* other,
                 int* root, int* end, uint32_t* info, const int* d_skip, hipStream_t s);
void batch_cluster_ids(const int* labels, const uint8_t* core, const int* minorig, const uint32_t* bits,
                       const int* wpre, const uint64_t* pkeys, int shift, const int64_t* off, int num_clouds,
                       int64_t n, const int* total, const int* cl_flags, int* cid, int32_t* num_clusters,
                       hipStream_t s);
void launch_scatter(const int* labels, const uint8_t* core, const uint32_t* perm, const int* cid,
                    const int* border, bool first_border, bool have_border, int64_t n, int32_t* out_labels,
                    uint8_t* out_core, uint32_t* info, hipStream_t s);
// The device word of FDB_INFO_* bits that a handle's calls raise (for copies
// ordered on a stream; the server reads its batches' bits this way).
const uint32_t* handle_info(const fdb_handle* h);

// Exclusive scan of two arrays of int32 counts in place.
void scan_block_sums(int* a, int* b, int64_t blocks, hipStream_t s);

// k_serve.hip: one job of a served batch - its own buffers and its place in the
// batch (first point off; first workgroup gblk of the gather and sblk of the
// scatter, each workgroup moving kSegVec * 256 elements).
constexpr int kSegVec = 4;
struct JobSeg {
  const float* points;
  int32_t* labels;
  uint8_t* core;
  int64_t n;
  int64_t off;
  int32_t gblk, sblk;
};
int64_t seg_blocks(int64_t elems);
void launch_gather(const JobSeg* seg, int num, int64_t total_blocks, int dim, float* dst, hipStream_t s);
void launch_scatter_jobs(const JobSeg* seg, int num, int64_t total_blocks, const int32_t* labels,
                         const uint8_t* core, hipStream_t s);

}  // namespace fdb
