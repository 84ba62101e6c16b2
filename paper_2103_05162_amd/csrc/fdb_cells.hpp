// Neighbour search over the DenseBox grid itself (cells of side eps/sqrt(d), so
// everything within eps of a point lies within 2 cells of its own per axis).
//
// The occupied cells come sorted along the Morton curve, so a cell is found by
// counting the occupied cells before it, in three levels of 64-bit occupancy words:
//   super  64 bricks (16^3 cells in 3D, 64^2 in 2D), a dense table over the grid
//   brick  64 cells (4^3 or 8^2), only occupied ones, in curve order
//   cell   only occupied ones, in curve order: cell_prim[c] = its first primitive
// A word's bits follow the curve (the 6 low key bits of the child), and its entry
// holds the index of its first child, so child k is first + popcount(bits below k).
// A query's cells lie in at most 2 bricks per axis: it loads every brick's super
// entry at once, then every brick entry at once, and then walks the cells' bits,
// three dependent loads from a query to a candidate. A walk down the hierarchy is a
// chain of ~80 dependent loads for the same candidates (~1.1 us each), and the
// hierarchy need not be built. Where the grid has more supers than the table holds
// (a scene of far outliers, or an eps tiny against the extent), its cell
// coordinates round too coarsely, or eps^2 leaves the range of fp32 (grid_eps), the plan
// leaves grid_on clear and the walks go through the hierarchy. Measured, hierarchy -> grid: uniform 2M-point set (4
// neighbours expected) core pass 0.93 -> 0.27, point main phase 1.06 -> 0.67, border
// pass 0.79 -> 0.13 ms; 8M dense-clump set core pass (with a filter for isolated points
// before it) 0.30 -> 0.15, point main phase 0.20 -> 0.12 ms; 370k-point mixture core
// pass 0.20 -> 0.08, point main phase 0.39 -> 0.16 ms; building the hierarchy took
// 0.15 ms on the 8M set, 1.9 ms in the batch of 4,096 clouds, and the index takes
// 0.04 and 0.39 ms.
#pragma once

#include "fdb_device.hpp"
#include "fdb_internal.hpp"

namespace fdb {

// Coordinate bits per level and axis: a brick is kSide cells wide.
template <int D>
constexpr int kLevelShift = D == 3 ? 2 : 3;
template <int D>
constexpr int kMaxBricks = D == 3 ? 8 : 4;  // bricks that can hold cells within 2 per axis

template <int D>
constexpr int kSuperSide = 1 << (2 * kLevelShift<D>);  // cells a super is wide
// Cells within reach of a query lie within two of its own per axis while reach is
// below this (a reach is sqrt(d) plus the slack of the largest cell coordinate).
constexpr double kMaxReach = 1.999;
// The range of eps in which a pair that passes the test s <= fl32(eps * eps) is at most
// eps (1 + 2^-16) apart, so that a reach holds all of them: every rounding is then
// relative (eps^2 in [2^-120, 2^126]; a square that underflows is below 2^-30 of it).
// Outside it the test passes pairs at other distances (eps = 1e-23: squares and eps^2 are
// 0 up to 2.6e-23 apart; eps above 1.8e19: all are infinite, every pair passes), and the
// hierarchy, whose box bounds round as the test does, finds the neighbours.
__device__ __forceinline__ bool grid_eps(float eps) { return eps >= 0x1p-60f && eps <= 0x1p63f; }

// Empties the super table (a grid-stride share of every thread of the launch).
__device__ __forceinline__ void clear_supers(uint4* __restrict__ supers, uint64_t count) {
  const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
  for (uint64_t k = blockIdx.x * uint64_t(blockDim.x) + threadIdx.x; k < count; k += stride)
    supers[k] = make_uint4(0, 0, 0, 0);
}

// Morton code (6 bits) of a child from the low kLevelShift bits of its coordinates,
// axis 0 highest, as the keys interleave them.
template <int D>
__device__ __forceinline__ uint32_t child_code(const int* c) {
  if constexpr (D == 3) {
    const uint32_t x = c[0] & 3, y = c[1] & 3, z = c[2] & 3;
    return ((x & 1) << 2 | (x & 2) << 4) | ((y & 1) << 1 | (y & 2) << 3) | ((z & 1) | (z & 2) << 2);
  } else {
    const uint32_t x = c[0] & 7, y = c[1] & 7;
    return ((x & 1) << 1 | (x & 2) << 2 | (x & 4) << 3) | ((y & 1) | (y & 2) << 1 | (y & 4) << 2);
  }
}

// Local coordinate (axis a) of the child with this code.
template <int D>
__device__ __forceinline__ int code_coord(uint32_t code, int a) {
  const uint32_t v = code >> (D - 1 - a);
  if constexpr (D == 3) return static_cast<int>((v & 1u) | ((v >> 2) & 2u));
  else return static_cast<int>((v & 1u) | ((v >> 1) & 2u) | ((v >> 2) & 4u));
}

// Codes whose coordinate on axis a is at least v, and at most v (v a local coordinate):
// compared bit by bit from the lowest, the words holding the codes with that bit of
// the axis set. No branches: a switch over v cost more than the walk's steps.
template <int D>
__device__ __forceinline__ uint64_t axis_word(int a, int bit) {
  if constexpr (D == 3) {
    constexpr uint64_t w[3][2] = {{0xf0f0f0f0f0f0f0f0ull, 0xffffffff00000000ull},
                                  {0xccccccccccccccccull, 0xffff0000ffff0000ull},
                                  {0xaaaaaaaaaaaaaaaaull, 0xff00ff00ff00ff00ull}};
    return w[a][bit];
  } else {
    constexpr uint64_t w[2][3] = {{0xccccccccccccccccull, 0xff00ff00ff00ff00ull, 0xffffffff00000000ull},
                                  {0xaaaaaaaaaaaaaaaaull, 0xf0f0f0f0f0f0f0f0ull, 0xffff0000ffff0000ull}};
    return w[a][bit];
  }
}
template <int D>
__device__ __forceinline__ uint64_t codes_from(int a, int v) {
  uint64_t m = ~0ull;
#pragma unroll
  for (int k = 0; k < kLevelShift<D>; ++k) {
    const uint64_t w = axis_word<D>(a, k), t = 0ull - static_cast<uint64_t>((v >> k) & 1);
    m = (w & m) | (~t & (w | m));  // bit set: both, clear: either
  }
  return m;
}
template <int D>
__device__ __forceinline__ uint64_t codes_upto(int a, int v) {
  uint64_t m = ~0ull;
#pragma unroll
  for (int k = 0; k < kLevelShift<D>; ++k) {
    const uint64_t w = ~axis_word<D>(a, k), t = 0ull - static_cast<uint64_t>((v >> k) & 1);
    m = (w & m) | (t & (w | m));  // bit set: either, clear: both
  }
  return m;
}
// The codes of the brick with coordinate br on axis a whose cells lie in [lo, hi].
template <int D>
__device__ __forceinline__ uint64_t codes_in(int a, int br, int lo, int hi) {
  const int base = br << kLevelShift<D>, top = (1 << kLevelShift<D>) - 1;
  uint64_t m = codes_from<D>(a, max(lo - base, 0)) & codes_upto<D>(a, min(hi - base, top));
  return lo - base <= top && hi >= base ? m : 0ull;
}

// One query's grid: cell coordinates are t = (x - lo) * inv_h, computed as the key
// kernel computes them.
struct CellGrid {
  float lo[3];
  float inv_h;
  float reach;    // eps in cells plus rounding slack (< 2)
  int ncell[3];   // cells per axis; 0 = no grid (a batch's cloud with bad input)
  int off;        // the grid's first super
};

template <int D, bool B>
__device__ __forceinline__ CellGrid query_grid(const CellIndex& ix, int cloud) {
  CellGrid g;
  if (B) {
    const float4 l = ix.cl_lo[cloud], s = ix.cl_scale[cloud];
    const int4 c = ix.cl_grid[2 * cloud];  // the cloud's record is two int4
    g.lo[0] = l.x; g.lo[1] = l.y; g.lo[2] = l.z;
    g.inv_h = s.x;
    g.reach = s.w;
    g.ncell[0] = c.x; g.ncell[1] = c.y; g.ncell[2] = c.z;
    g.off = c.w;
  } else {
    const GridPlan& p = *ix.plan;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      g.lo[k] = p.lo[k];
      g.ncell[k] = static_cast<int>(p.ncell[k]);
    }
    g.inv_h = p.inv_h[0];
    g.reach = p.reach;
    g.off = 0;
  }
  return g;
}

// Supers per axis, and the table index of the super holding brick coordinates br.
template <int D>
__device__ __forceinline__ int supers_on(int ncell) {
  return (ncell + kSuperSide<D> - 1) / kSuperSide<D>;
}
template <int D>
__device__ __forceinline__ int super_index(const CellGrid& g, const int* br) {
  int s = br[0] >> kLevelShift<D>;
  s = s * supers_on<D>(g.ncell[1]) + (br[1] >> kLevelShift<D>);
  if (D == 3) s = s * supers_on<D>(g.ncell[2]) + (br[2] >> kLevelShift<D>);
  return g.off + s;
}

__device__ __forceinline__ uint64_t word_of(uint4 e) { return uint64_t(e.x) | uint64_t(e.y) << 32; }

// A query box in cell units ([tlo, thi] per axis, a point when equal) and the range
// of cells within reach of it. `own` is the query's own cell, which all of it lies in.
template <int D>
struct CellRange {
  float tlo[3], thi[3];
  int own[3], lo[3], hi[3];
  float r2;
};

__device__ __forceinline__ float cell_t(float v, float lo, float inv_h) { return fmaxf((v - lo) * inv_h, 0.0f); }

template <int D>
__device__ __forceinline__ void cell_range(CellRange<D>& cr, const CellGrid& g, const float* qlo, const float* qhi) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    cr.tlo[a] = cr.thi[a] = 0.0f;
    cr.own[a] = cr.lo[a] = cr.hi[a] = 0;
  }
#pragma unroll
  for (int a = 0; a < D; ++a) {
    cr.tlo[a] = cell_t(qlo[a], g.lo[a], g.inv_h);
    cr.thi[a] = cell_t(qhi[a], g.lo[a], g.inv_h);
    const int top = g.ncell[a] - 1;
    const float ftop = static_cast<float>(top);
    cr.own[a] = cr.tlo[a] >= ftop ? top : static_cast<int>(cr.tlo[a]);  // as the key kernel clamps it
    const float l = floorf(cr.tlo[a] - g.reach), h = floorf(cr.thi[a] + g.reach);
    // the clamps keep the own cell in the range and the range within 2 cells of it
    cr.lo[a] = max(max(l > 0.0f ? (l >= ftop ? top : static_cast<int>(l)) : 0, cr.own[a] - 2), 0);
    cr.lo[a] = min(cr.lo[a], cr.own[a]);
    cr.hi[a] = min(min(h >= ftop ? top : static_cast<int>(h), cr.own[a] + 2), top);
    cr.hi[a] = max(cr.hi[a], cr.own[a]);
  }
  cr.r2 = g.reach * g.reach;
}

// Brick n of the range (bit a of n, highest axis first, picks the second brick on an
// axis): its coordinates, or false when the range does not reach it.
template <int D>
__device__ __forceinline__ bool range_brick(const CellRange<D>& cr, int n, int* br) {
  bool use = true;
  br[2] = 0;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    br[a] = (cr.lo[a] >> kLevelShift<D>) + ((n >> (D - 1 - a)) & 1);
    use = use && br[a] <= (cr.hi[a] >> kLevelShift<D>);
  }
  return use;
}

// The codes of brick br's cells inside the range; with MASKED, those of the own brick
// only from the own cell on.
template <int D, bool MASKED>
__device__ __forceinline__ uint64_t range_codes(const CellRange<D>& cr, const int* br) {
  uint64_t m = ~0ull;
  if (MASKED) {
    bool own = true;
#pragma unroll
    for (int a = 0; a < D; ++a) own = own && br[a] == (cr.own[a] >> kLevelShift<D>);
    if (own) m = ~0ull << child_code<D>(cr.own);
  }
#pragma unroll
  for (int a = 0; a < D; ++a) {
    m &= codes_in<D>(a, br[a], cr.lo[a], cr.hi[a]);
  }
  return m;
}

// Is the cell with this code in brick br within reach of the query box? Per axis
// the gap between the box and the cell's interval, zero on the own cell's axis
// coordinate (whatever its rounding). Never false for a cell that holds a neighbour:
// the reach covers the rounding of both coordinates.
template <int D>
__device__ __forceinline__ bool cell_in_reach(const CellRange<D>& cr, const int* br, uint32_t code) {
  float s = 0.0f;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    const int c = (br[a] << kLevelShift<D>) + code_coord<D>(code, a);
    const float f = static_cast<float>(c);
    const float gap = c == cr.own[a] ? 0.0f : fmaxf(fmaxf(f - cr.thi[a], cr.tlo[a] - (f + 1.0f)), 0.0f);
    s += gap * gap;
  }
  return s <= cr.r2;
}

// The codes of the range's cells in each of its bricks, as what a brick's coordinate
// on an axis (side 0 or 1) allows.
template <int D>
struct BrickSides {
  uint64_t in[D][2], from_own;
  int n_own;  // the query's own brick
  template <bool MASKED>
  __device__ __forceinline__ uint64_t cells(int n) const {
    uint64_t m = ~0ull;
#pragma unroll
    for (int a = 0; a < D; ++a) {  // a select by mask: indexing would put the array in memory
      const uint64_t t = 0ull - static_cast<uint64_t>((n >> (D - 1 - a)) & 1);
      m &= (in[a][0] & ~t) | (in[a][1] & t);
    }
    if (MASKED && n == n_own) m &= from_own;
    return m;
  }
};

// Looks up the range's bricks and hands each occupied one with cells in the range
// (with MASKED, from the query's own cell on) to put(word, n, first cell), its cells in
// the range being word & bs.cells(n). Brick n takes one or the other of the range's
// brick coordinates on each axis, so what a coordinate adds to the child code, the
// super index and the range's codes is computed per axis and side, not per brick; the
// loads of a level are all in flight together. NEAR: the query's own brick first, else
// the lower coordinates. The core pass stops at minPts neighbours, so it looks near
// first (batch of 4,096 clouds: 6.0 -> 4.1 ms, though the points that stop early have
// met fewer dense cells to join, and the dense-cell main phase takes 6.7 for 5.7 ms).
template <int D, bool MASKED, bool NEAR, typename F>
__device__ __forceinline__ void lookup_bricks(const CellIndex& ix, const CellGrid& g, const CellRange<D>& cr, bool on,
                                              BrickSides<D>& bs, F&& put) {
  constexpr int S = kLevelShift<D>, NB = kMaxBricks<D>;
  uint32_t code[D][2];
  int sup[D][2];
  bool two[D];
  int stride = 1, n_own = 0;
#pragma unroll
  for (int a = D - 1; a >= 0; --a) {
    const int own = cr.own[a] >> S, lo = cr.lo[a] >> S, hi = cr.hi[a] >> S;
    two[a] = lo != hi;
    if (!NEAR) n_own |= (own - lo) << (D - 1 - a);
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      int br[3] = {0, 0, 0};
      br[a] = !NEAR ? lo + o : (o == 0 ? own : own + (hi > own ? 1 : -1));
      code[a][o] = child_code<D>(br);
      sup[a][o] = (br[a] >> S) * stride;
      bs.in[a][o] = codes_in<D>(a, br[a], cr.lo[a], cr.hi[a]);
    }
    stride *= supers_on<D>(g.ncell[a]);
  }
  uint4 e[NB];
  int b[NB];
  bool use[NB];
  bs.n_own = n_own;
  bs.from_own = MASKED ? ~0ull << child_code<D>(cr.own) : ~0ull;
  auto side = [](int n, int a) { return (n >> (D - 1 - a)) & 1; };
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    use[n] = on;
    int s = g.off;
#pragma unroll
    for (int a = 0; a < D; ++a) {
      use[n] = use[n] && (!side(n, a) || two[a]);
      s += sup[a][side(n, a)];
    }
    e[n] = make_uint4(0, 0, 0, 0);
    if (use[n]) e[n] = ix.supers[s];
  }
  int b_own = -1;
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    uint32_t c = 0;
#pragma unroll
    for (int a = 0; a < D; ++a) c |= code[a][side(n, a)];
    const uint64_t w = word_of(e[n]);
    use[n] = (w >> c) & 1;
    b[n] = static_cast<int>(e[n].z) + __popcll(w & ((1ull << c) - 1));
    if (MASKED && n == n_own && use[n]) b_own = b[n];
  }
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    if (MASKED && b[n] < b_own) use[n] = false;
    e[n] = make_uint4(0, 0, 0, 0);
    if (use[n]) e[n] = ix.bricks[b[n]];
  }
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    const uint64_t w = word_of(e[n]);
    if (w & bs.template cells<MASKED>(n)) put(w, n, static_cast<int>(e[n].z));
  }
}

// Cells outside dense ones of this many points or more are looked up as sets (TravArgs::
// cell_sets).
constexpr int kSetCell = 8;

// The primitives [first, last) of cell c, and whether it is a dense cell (one
// primitive). cell_prim holds a dense cell's primitive as its complement; the entry
// after the last cell is the number of primitives.
__device__ __forceinline__ void cell_prims(const CellIndex& ix, int c, int& first, int& last, bool& dense) {
  const int a = ix.cell_prim[c], b = ix.cell_prim[c + 1];
  dense = a < 0;
  first = a < 0 ? ~a : a;
  last = b < 0 ? ~b : b;
}

// ---- packets: a run of lanes searched together ----------------------------------------
// Queries next to each other on the curve share most of their neighbourhood. A packet
// takes the box of cells within reach of any of its queries: the wavefront looks up
// the box's bricks a lane each, lists the occupied cells inside the box in LDS, and
// hands their primitives to the caller 64 at a time, a primitive per lane, to be
// broadcast to the queries. So a candidate is loaded once for all of them, in
// coalesced loads, where a walk per lane loads it for each (64 cache lines per load
// instruction).
constexpr int kBoxBricks = 256;  // a packet's box spans at most this many bricks

template <int D>
struct CellBox {
  int lo[3], hi[3];  // cells
  int bricks;        // bricks it spans; above kBoxBricks: too spread out for a packet
};

// The cells within reach of the box [qlo, qhi].
template <int D>
__device__ __forceinline__ CellBox<D> cell_box(const CellGrid& g, const float* qlo, const float* qhi) {
  CellBox<D> b;
  float bricks = 1.0f;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    const int top = g.ncell[a] - 1;
    const float ftop = static_cast<float>(top);
    const float l = floorf(cell_t(qlo[a], g.lo[a], g.inv_h) - g.reach);
    const float h = floorf(cell_t(qhi[a], g.lo[a], g.inv_h) + g.reach);
    b.lo[a] = l >= ftop ? top : (l > 0.0f ? static_cast<int>(l) : 0);
    b.hi[a] = h >= ftop ? top : (h > 0.0f ? static_cast<int>(h) : 0);
    bricks *= static_cast<float>((b.hi[a] >> kLevelShift<D>) - (b.lo[a] >> kLevelShift<D>) + 1);
  }
  b.bricks = bricks > static_cast<float>(kBoxBricks) ? kBoxBricks + 1 : static_cast<int>(bricks);
  return b;
}

__device__ __forceinline__ float readlane_float(float v, int k) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k));
}

__device__ __forceinline__ uint64_t readlane64(uint64_t v, int k) {
  return uint64_t(static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v >> 32), k))) << 32 |
         static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), k));
}

// Hands each lane's primitives [cur, end) to visit_lanes(r), called on the whole wavefront
// with a primitive per lane (-1: none); true when visit_lanes said (uniformly) to stop.
// Lanes step through kStepRange of their own, and what is left of a range goes over all
// lanes: a cell that is not dense can hold thousands of points (a large minPts, or a scene
// so wide that the rounding of its cells' edges puts a box past the guard), and the other
// lanes would wait for it. Dense-cell and point main phases of 500,000 points in 2D, scales
// log-uniform over six decades, us: 2091 + 2196 by steps alone, 174 + 289 so. (One call
// of visit_lanes: a second copy of its code cost 2 to 3% of calls that never take it.)
constexpr int kStepRange = 64;
template <typename F>
__device__ __forceinline__ bool visit_ranges(int cur, int end, F&& visit_lanes) {
  for (int step = 0;; ++step) {
    const uint64_t left = ballot(cur < end);
    if (!left) return false;
    int r = cur < end ? cur : -1;
    if (step < kStepRange) {
      ++cur;
    } else {
      const int L = __ffsll(static_cast<unsigned long long>(left)) - 1;
      const int first = __builtin_amdgcn_readlane(cur, L);
      if (cur == first) cur += 64;  // (lane L alone: ranges are apart)
      r = first + lane_id();
      if (r >= __builtin_amdgcn_readlane(end, L)) r = -1;
    }
    if (visit_lanes(r)) return true;
  }
}

// Hands the primitives above `mask` in the box's cells to visit_lanes(r), called on
// the whole wavefront with a primitive per lane (-1: none); visit_lanes returns true
// (uniformly) to stop. pass(c), called for a cell of kSetCell primitives or more, says
// that all of them can be left out. list: kBoxList ints of the wavefront's LDS.
constexpr int kBoxList = 512;

template <int D, typename F, typename P>
__device__ __forceinline__ void box_candidates(const CellIndex& ix, const CellGrid& g, const CellBox<D>& b, int mask,
                                               int* list, F&& visit_lanes, P&& pass) {
  constexpr int S = kLevelShift<D>;
  const int lane = lane_id();
  int b0[3] = {0, 0, 0}, nb[3] = {1, 1, 1};
#pragma unroll
  for (int a = 0; a < D; ++a) {
    b0[a] = b.lo[a] >> S;
    nb[a] = (b.hi[a] >> S) - b0[a] + 1;
  }
  int cnt = 0;
  for (int c = 0; c < b.bricks; c += 64) {
    const int k = c + lane;
    int br[3] = {0, 0, 0};
    if (D == 3) {
      const int t = k / nb[2];
      br[0] = b0[0] + t / nb[1];
      br[1] = b0[1] + t % nb[1];
      br[2] = b0[2] + k % nb[2];
    } else {
      br[0] = b0[0] + k / nb[1];
      br[1] = b0[1] + k % nb[1];
    }
    const uint32_t code = child_code<D>(br);
    uint4 e = make_uint4(0, 0, 0, 0);
    if (k < b.bricks) e = ix.supers[super_index<D>(g, br)];
    const uint64_t sw = word_of(e);
    const bool use = (sw >> code) & 1;
    const int bi = static_cast<int>(e.z) + __popcll(sw & ((1ull << code) - 1));
    e = make_uint4(0, 0, 0, 0);
    if (use) e = ix.bricks[bi];
    uint64_t m = word_of(e);
#pragma unroll
    for (int a = 0; a < D; ++a) m &= codes_in<D>(a, br[a], b.lo[a], b.hi[a]);
    for (uint64_t todo = ballot(m != 0);;) {
      // list the cells of as many bricks as fit, a lane per cell code
      for (; todo && cnt <= kBoxList - 64; todo &= todo - 1) {
        const int n = __ffsll(static_cast<unsigned long long>(todo)) - 1;
        const uint64_t wn = readlane64(word_of(e), n), mn = readlane64(m, n);
        const int base = __builtin_amdgcn_readlane(static_cast<int>(e.z), n);
        if ((mn >> lane) & 1) list[cnt + __popcll(mn & lanemask_lt())] = base + __popcll(wn & lanemask_lt());
        cnt += __popcll(mn);
      }
      if (!todo && c + 64 < b.bricks && cnt <= kBoxList - 64) break;  // more bricks first
      for (int q = 0; q < cnt; q += 64) {
        int cur = 0, end = 0;
        bool dense;
        if (q + lane < cnt) {
          cell_prims(ix, list[q + lane], cur, end, dense);
          if (end - cur >= kSetCell && pass(list[q + lane])) cur = end;
        }
        if (visit_ranges(max(cur, mask + 1), end, visit_lanes)) return;
      }
      cnt = 0;
      if (!todo) break;
    }
  }
}

// Runs the wavefront's queries (lanes of `todo`, each the box [qlo, qhi] in its
// cloud's grid) as packets: packet(lanes, grid, cells, lo, hi) for aligned runs of 64,
// 32, 16 or 8 lanes of one cloud, the largest whose box [lo, hi] reaches at most a
// brick a query and kBoxExtra more. Returns the lanes left, to walk on their own. One
// ascending butterfly gives the boxes of all the runs.
constexpr int kBoxExtra = 8;

template <int D, bool B, typename F>
__device__ __forceinline__ uint64_t for_packets(const CellIndex& ix, int cloud, const float* qlo, const float* qhi,
                                                uint64_t todo, F&& packet) {
  const int lane = lane_id();
  const bool on = (todo >> lane) & 1;
  const CellGrid own = query_grid<D, B>(ix, B ? cloud : 0);
  float lo[3] = {0.0f, 0.0f, 0.0f}, hi[3] = {0.0f, 0.0f, 0.0f}, blo[3] = {0.0f, 0.0f, 0.0f}, bhi[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int a = 0; a < D; ++a) {
    lo[a] = on ? qlo[a] : INFINITY;
    hi[a] = on ? qhi[a] : -INFINITY;
  }
  int c_lo = on ? cloud : 0x7fffffff, c_hi = on ? cloud : -1;
  int size = 0;  // the run this lane is taken in (0: none)
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
#pragma unroll
    for (int a = 0; a < D; ++a) {
      lo[a] = fminf(lo[a], __shfl_xor(lo[a], off));
      hi[a] = fmaxf(hi[a], __shfl_xor(hi[a], off));
    }
    if (B) {
      c_lo = min(c_lo, __shfl_xor(c_lo, off));
      c_hi = max(c_hi, __shfl_xor(c_hi, off));
    }
    if (off < 4) continue;
    const int run = 2 * off;
    const uint64_t lanes = todo & ((run == 64 ? ~0ull : (1ull << run) - 1) << (lane & ~(run - 1)));
    // (a lane that is no query may lie in another cloud: its answer is not used)
    const int bricks = cell_box<D>(own, lo, hi).bricks;
    if (on && (!B || c_lo == c_hi) && bricks <= kBoxBricks && bricks <= __popcll(lanes) + kBoxExtra) {
      size = run;
#pragma unroll
      for (int a = 0; a < D; ++a) {
        blo[a] = lo[a];
        bhi[a] = hi[a];
      }
    }
  }
  if (own.ncell[0] <= 0) size = 0;
  uint64_t left = ballot(on && size > 0);
  const uint64_t alone = ballot(on && size == 0);
  while (left) {
    const int fl = __ffsll(static_cast<unsigned long long>(left)) - 1;
    const int run = __builtin_amdgcn_readlane(size, fl);
    const uint64_t lanes = todo & ((run == 64 ? ~0ull : (1ull << run) - 1) << (fl & ~(run - 1)));
    float plo[3] = {0.0f, 0.0f, 0.0f}, phi[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int a = 0; a < D; ++a) {
      plo[a] = readlane_float(blo[a], fl);
      phi[a] = readlane_float(bhi[a], fl);
    }
    const CellGrid g = query_grid<D, B>(ix, B ? __builtin_amdgcn_readlane(cloud, fl) : 0);
    CellBox<D> box = cell_box<D>(g, plo, phi);
    box.bricks = __builtin_amdgcn_readfirstlane(box.bricks);
#pragma unroll
    for (int a = 0; a < D; ++a) {  // the same on every lane
      box.lo[a] = __builtin_amdgcn_readfirstlane(box.lo[a]);
      box.hi[a] = __builtin_amdgcn_readfirstlane(box.hi[a]);
    }
    packet(lanes, g, box, plo, phi);
    left &= ~lanes;
  }
  return alone;
}

// A lane's walk over the primitives in the cells within reach of its query; with
// MASKED only primitives above `mask`. The bricks it found wait in the wavefront's
// LDS, a column per lane, kMaxBricks rows: their words and first cells (12 bytes a
// row: at 20, with the cells to visit beside them, LDS left 14 wavefronts a CU and the
// walks, which wait for loads, took a third longer). A step is straight-line code (a
// walk that skipped empty bricks and cells out of reach in nested loops took 16,000
// vector instructions a wavefront on the uniform 2M-point set, where lanes wait for
// each other's inner loops).
template <int D>
struct CellWalk {
  BrickSides<D> bs;
  uint64_t word, left;  // current brick's cells, and those still to visit
  int base;             // its first cell
  int next, bricks;     // the next row, the rows in use
  uint32_t rows;        // brick number n of each row, 4 bits each, the next row's lowest
  int cur, end;         // pending primitives [cur, end)
};

template <int D>
constexpr int kWalkWaveBytes = kMaxBricks<D> * 12 * 64;  // LDS of a wavefront's walks

template <int D, bool MASKED, bool NEAR>
__device__ __forceinline__ void cell_walk_init(CellWalk<D>& w, const CellIndex& ix, const CellGrid& g,
                                               const CellRange<D>& cr, bool on, char* lds) {
  uint64_t* s_word = reinterpret_cast<uint64_t*>(lds) + lane_id();
  int* s_base = reinterpret_cast<int*>(lds + kMaxBricks<D> * 64 * 8) + lane_id();
  int k = 0;
  w.rows = 0;
  lookup_bricks<D, MASKED, NEAR>(ix, g, cr, on, w.bs, [&](uint64_t word, int n, int base) {
    s_word[64 * k] = word;
    s_base[64 * k] = base;
    w.rows |= static_cast<uint32_t>(n) << (4 * k);
    ++k;
  });
  w.word = w.left = 0;
  w.base = 0;
  w.next = 0;
  w.bricks = k;
  w.cur = w.end = 0;
}

template <int D>
__device__ __forceinline__ bool cell_walk_done(const CellWalk<D>& w) {
  return w.cur >= w.end && w.left == 0 && w.next >= w.bricks;
}

// The next primitive of the walk, or -1 (also where a cell has none above the mask, or
// pass(c) has it left out, as in box_candidates).
template <int D, bool MASKED, typename P>
__device__ __forceinline__ int cell_walk_step(CellWalk<D>& w, const CellIndex& ix, int mask, char* lds, P&& pass) {
  if (w.cur >= w.end) {
    if (w.left == 0 && w.next < w.bricks) {
      w.word = (reinterpret_cast<const uint64_t*>(lds) + lane_id())[64 * w.next];
      w.base = (reinterpret_cast<const int*>(lds + kMaxBricks<D> * 64 * 8) + lane_id())[64 * w.next];
      w.left = w.word & w.bs.template cells<MASKED>(static_cast<int>(w.rows & 15u));
      w.rows >>= 4;
      ++w.next;
    }
    if (w.left) {
      const uint64_t below = w.left ^ (w.left - 1);  // the lowest bit left and those under it
      w.left &= w.left - 1;
      bool dense;
      const int c = w.base + __popcll(w.word & (below >> 1));
      cell_prims(ix, c, w.cur, w.end, dense);
      if (w.end - w.cur >= kSetCell && pass(c)) w.cur = w.end;
      if (MASKED) w.cur = max(w.cur, mask + 1);
    }
  }
  return w.cur < w.end ? w.cur++ : -1;
}

}  // namespace fdb
