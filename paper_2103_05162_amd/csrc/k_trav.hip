// Traversal kernels: one query per lane in Morton order (Section 4.1),
// stack-less top-down walks over the LBVH using escape links.
//   core   - preprocessing: count neighbours, stop at minPts (Section 3.2).
//   main   - the fused phase: union (or claim) on discovery, nothing stored
//            (Algorithm 3); the walk is masked so query i only reaches
//            primitives above its own, handling every pair once (Section 4.1,
//            Figure 1).
//   border - canonical labels: a non-core point takes the smallest cluster id
//            among its core neighbours.
// FDbscan takes subtrees of points pairwise within eps (cliques) as one set at once.
// DenseBox variants (Section 4.2) search the grid's cells, or a tree over dense-cell
// boxes plus the points outside dense cells; a box hit scans the cell's points.
//
// Every walk has a scope: the subtree it starts from, the last primitive of
// that subtree, eps^2 and minPts. A single cloud's scope is the whole tree; in
// a batch the keys carry the cloud id above the Morton bits, so each cloud is
// one subtree, and a query's scope is its cloud's (with its own eps, minPts).
#include <algorithm>
#include <type_traits>

#include "fdb_cells.hpp"
#include "fdb_device.hpp"
#include "fdb_internal.hpp"

namespace fdb {

namespace {

struct Query {
  float x, y, z;
};

struct Scope {
  uint32_t start;  // first node of the walk (internal node, or kLeaf | leaf)
  int end;         // last primitive of the subtree
  float eps2;
  int min_pts;
};

template <int D>
__device__ __forceinline__ Query load_point(const float* __restrict__ xs, int64_t n, int64_t i) {
  Query q;
  q.x = xs[i];
  q.y = xs[n + i];
  q.z = D == 3 ? xs[2 * n + i] : 0.0f;
  return q;
}

__device__ __forceinline__ int tree_m(const TreeView& t) { return t.d_m ? *t.d_m : t.m_cap; }

__device__ __forceinline__ int cloud_of(const TravArgs& a, int i) {
  return min(static_cast<int>(a.pkeys[i] >> a.key_shift), a.num_clouds - 1);
}

// Scope of the query at sorted point index i.
template <bool BATCHED>
__device__ __forceinline__ Scope scope_of(const TravArgs& a, int m, int i) {
  Scope s;
  if (BATCHED) {
    const int c = cloud_of(a, i);
    s.start = static_cast<uint32_t>(a.cloud_root[c]);
    s.end = a.cloud_end[c];
    s.eps2 = a.cloud_eps2[c];
    s.min_pts = a.cloud_minpts[c];
  } else {
    s.start = m == 1 ? kLeaf : 0u;
    s.end = m - 1;
    s.eps2 = a.eps2;
    s.min_pts = a.min_pts;
  }
  return s;
}

// A box query (every point of [lo, hi]); the walks take it or a point.
struct BoxQ {
  float lo[3], hi[3];
};

template <int D>
__device__ __forceinline__ float node_gap2(const Query& q, float4 a, float4 b) {
  return box_dist2<D>(q.x, q.y, q.z, a.x, a.y, a.z, b.x, b.y, b.z);
}
template <int D>
__device__ __forceinline__ float node_gap2(const BoxQ& q, float4 a, float4 b) {
  return boxbox_dist2<D>(q.lo, q.hi, a.x, a.y, a.z, b.x, b.y, b.z);
}

// Walk the subtree of sc, calling visit(first, last) for every bucket (at most
// leaf_size primitives) and single leaf the walk reaches; visit returns true to stop.
// With MASKED, only the primitives above the mask (>= 0) are walked: the escape links
// from leaf `mask` on lead to the subtrees right of it, so no node above them is looked
// at. The walk ends where an escape link would leave the subtree (past primitive sc.end).
// subtree(first, last, lo, hi), called for a node within reach, says what to do with
// it: 0 walk it, 1 pass over it, 2 stop.
//
// A pre-order walk reaches each node at most once, so more than 2m steps, or a
// reference outside the tree, means the tree is broken: the walk then stops and
// raises the internal-error bit instead of looping or reading out of bounds.
struct EverySubtree {
  __device__ __forceinline__ int operator()(int, int, const float4&, const float4&) const { return 0; }
};

template <int D, bool MASKED, typename QT, typename F, typename S = EverySubtree>
__device__ __forceinline__ void traverse(const TreeView& t, int m, const Scope& sc, const QT& q, int mask,
                                         uint32_t* info, F&& visit, S&& subtree = S{}) {
  if (m <= 0) return;
  if (MASKED && mask >= sc.end) return;
  uint32_t node = MASKED ? static_cast<uint32_t>(t.leaf_rope[mask]) : sc.start;
  int64_t steps = 0;
  const int64_t max_steps = 2 * int64_t(m) + 2;
  while (node != kEnd) {
    if (++steps > max_steps) {
      atomicOr(info, kInternalBit);
      return;
    }
    if (node & kLeaf) {
      int l = static_cast<int>(node & ~kLeaf);
      if (l >= m) {
        atomicOr(info, kInternalBit);
        return;
      }
      if (visit(l, l) || l >= sc.end) return;
      node = static_cast<uint32_t>(t.leaf_rope[l]);
      continue;
    }
    if (node >= static_cast<uint32_t>(m - 1)) {
      atomicOr(info, kInternalBit);
      return;
    }
    // the escape link is loaded with the node, not after its box test fails
    const float4 a = t.node_a[kNodeStride * size_t(node)];
    const float4 b = t.node_b[kNodeStride * size_t(node)];
    const uint32_t esc = static_cast<uint32_t>(t.rope[node]);
    const int k = static_cast<int>(node);
    const int o = __float_as_int(a.w), g = __float_as_int(b.w);
    const int first = o < k ? o : k, last = o > k ? o : k;
    if (node_gap2<D>(q, a, b) > sc.eps2) {
      if (last >= sc.end) return;
      node = esc;
      continue;
    }
    if (first < 0 || last >= m || g < first || g >= last) {
      atomicOr(info, kInternalBit);
      return;
    }
    const int whole = subtree(first, last, a, b);
    if (whole == 2) return;
    if (whole == 1) {
      if (last >= sc.end) return;
      node = esc;
      continue;
    }
    if (last - first < t.leaf_size) {
      if (visit(first, last) || last >= sc.end) return;
      node = esc;
      continue;
    }
    node = first == g ? (kLeaf | static_cast<uint32_t>(g)) : static_cast<uint32_t>(g);
  }
}

// Which of the points s .. min(s + 3, e) are within eps of q, as bits: a lane's loads of
// all four are in flight together.
template <int D>
__device__ __forceinline__ unsigned near_bits(const float* __restrict__ xs, int64_t n, int s, int e, const Query& q,
                                              float eps2) {
  float v[4][3];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int64_t k = min(s + u, e);
    v[u][0] = xs[k];
    v[u][1] = xs[n + k];
    v[u][2] = D == 3 ? xs[2 * n + k] : 0.0f;
  }
  unsigned bits = 0;
#pragma unroll
  for (int u = 0; u < 4; ++u)
    bits |= s + u <= e && dist2v<D>(v[u][0], v[u][1], v[u][2], q.x, q.y, q.z) <= eps2 ? 1u << u : 0u;
  return bits;
}

// FDbscan's boxes: nodes [first, last] of kCliqueMin points or more in a box of diagonal
// at most eps. Their points are pairwise within eps, as the point-by-point test would
// decide: rounded subtraction, squaring and addition are monotone, so the test of the
// box's corners bounds every pair's. So are those of every node inside a box. A box of
// minPts points or more is a clique: all its points are core and in one set, whatever part
// of the tree a walk meets them in (k_cliques says so beforehand). In any other box the
// core points are in one set, which k_core_boxes says once the core pass knows them.
constexpr int kCliqueMin = 4;
// Cliques of this many points search for themselves, a wavefront each; the points of
// smaller ones search each for itself, as points outside cliques do (but are in one set
// and known to be core). Main phase with 8 / 12 / 16, us: 2M-point friends-of-friends
// set 1812 / 1825 / 1829, 8M-point set 853 / 670 / 743, 16,384 points in 2D 169 / 174 /
// 175. kCliqueMin 2, 4: alike; 16: 160 us more on the friends-of-friends set.
constexpr int kCliqueWave = 12;
// A clique of more points than this (or minPts, if larger) searches as the largest nodes
// in it that have no more: one wavefront takes a clique, and tests its points against every
// 64 candidates. Two bodies of 30,000 points, each a clique, whose boxes are within eps
// though no pair is, took 249 ms as one search each (3.5 when queries walked as packets).
// With 64 / 128 / 256 / 512 / 1024 at most, call, us: those bodies in 2D 490 / 730 / 920 /
// 1350 / 1350, in 3D 293 / 570 / 590 / 900 / 7660; 8M-point set 4124 / 3593 / 3306 / 3179 /
// 3125 (any size: 3343).
constexpr int kCliqueMost = 512;
template <int D>
__device__ __forceinline__ bool is_box(int first, int last, const float4& lo, const float4& hi, float eps2) {
  return last - first + 1 >= kCliqueMin && dist2v<D>(hi.x, hi.y, hi.z, lo.x, lo.y, lo.z) <= eps2;
}
// A core point of the box [first, last], to stand for them all, or -1 (unknown: neither
// its first point nor its last is one).
__device__ __forceinline__ int box_core(const uint8_t* core, int first, int last, int min_pts) {
  if (last - first + 1 >= min_pts || core[first]) return first;
  return core[last] ? last : -1;
}

// Wave-uniform walk for a box query (every point of box [lo,hi]), masked like
// traverse(): visit(first, last) is called with the same primitive range on
// every lane, for each bucket (a subtree of at most leaf_size primitives, cut
// to primitives above the mask) and each single leaf the walk reaches.
template <int D, typename F>
__device__ __forceinline__ bool traverse_box(const TreeView& t, int m, const Scope& sc, const float* lo,
                                             const float* hi, int mask, int leaf_size, uint32_t* info, F&& visit) {
  if (m <= 0 || mask >= sc.end) return false;
  uint32_t node = sc.start;
  int64_t steps = 0;
  const int64_t max_steps = 2 * int64_t(m) + 2;
  while (node != kEnd) {
    node = __builtin_amdgcn_readfirstlane(node);
    if (++steps > max_steps) {
      atomicOr(info, kInternalBit);
      return false;
    }
    if (node & kLeaf) {
      int l = static_cast<int>(node & ~kLeaf);
      if (l >= m) {
        atomicOr(info, kInternalBit);
        return false;
      }
      if (visit(l, l)) return true;
      if (l >= sc.end) return false;
      node = static_cast<uint32_t>(t.leaf_rope[l]);
      continue;
    }
    if (node >= static_cast<uint32_t>(m - 1)) {
      atomicOr(info, kInternalBit);
      return false;
    }
    const float4 na = t.node_a[kNodeStride * size_t(node)];
    const float4 nb = t.node_b[kNodeStride * size_t(node)];
    const uint32_t esc = static_cast<uint32_t>(t.rope[node]);
    const int k = static_cast<int>(node);
    const int o = __float_as_int(na.w), g = __float_as_int(nb.w);
    const int first = o < k ? o : k, last = o > k ? o : k;
    if (boxbox_dist2<D>(lo, hi, na.x, na.y, na.z, nb.x, nb.y, nb.z) > sc.eps2) {
      if (last >= sc.end) return false;
      node = esc;
      continue;
    }
    if (first < 0 || last >= m || g < first || g >= last) {
      atomicOr(info, kInternalBit);
      return false;
    }
    if (last - first < leaf_size) {
      int s = first <= mask ? mask + 1 : first;
      if (s <= last && visit(s, last)) return true;
      if (last >= sc.end) return false;
      node = esc;
      continue;
    }
    if (g <= mask)
      node = last == g + 1 ? (kLeaf | static_cast<uint32_t>(g + 1)) : static_cast<uint32_t>(g + 1);
    else
      node = first == g ? (kLeaf | static_cast<uint32_t>(g)) : static_cast<uint32_t>(g);
  }
  return false;
}

// An ancestor of x close to its root: labels followed for up to 16 hops, all
// lanes of a bucket at once. Equal to a query's root means the two are already
// in one set (sets only grow); anything else only means "unknown". When the chain
// had two links or more to spare, x is re-pointed straight at the ancestor found (an
// ancestor stays an ancestor, whichever store comes last): points are visited by many
// walks, and the next visit takes one load.
//
// The store is an agent-scope one, as every store to labels is whose word another XCD may
// store to in the same kernel. Plain ones (up to here the case) left XCDs with different
// values of the word in the kernels that followed: an XCD whose own L2 had the root passed
// the word over in the finalisation, the others read a parent of it in the border pass,
// and border points took ids from slots that hold none (500k points in the plane, minPts
// 140, FDbscan: 5 calls of 6). Agent-scope stores go to memory, so they are made for longer
// chains only. Calls with plain stores / none / agent-scope ones for every chain / for
// longer ones, us: 16,384 points FDbscan 444 / 461 / 465 / 451, 2M friends-of-friends
// FDbscan 2531 / 2715 / 2728 / 2727, DenseBox 1530 / 1564 / 1597 / 1562, 370k mixture 632 /
// 658 / 657 / 650, batch of 4,096 clouds 25,591 / 26,369 / 25,986 / 26,085.
__device__ __forceinline__ int ancestor_compress(int* labels, int x) {
  const int x0 = x;
  int p = labels[x];
  int h = 0;
#pragma unroll 1
  for (; h < 16 && p != x; ++h) {
    x = p;
    p = labels[x];
  }
  if (h > 2) st_agent(labels + x0, p);
  return p;
}

// Wavefront-cooperative form of traverse_box: the wavefront expands up to 64
// tree nodes per step (one per lane) from its own stack in LDS, newest first,
// so a walk takes about as many steps as the tree is deep instead of one step
// per node. Every bucket and leaf that one step reaches is handed out a
// primitive per lane, visit_lanes(r) being called on the whole wavefront with
// each lane's own primitive (-1 for none), so the visitor loads all of them at
// once. It visits the same buckets and leaves as traverse_box (in another order:
// callers only union, which does not depend on it). Children that do not fit on
// the stack have their subtrees walked with traverse_box instead. SKIP (FDbscan's
// unions): the walk starts from the escape links above the mask (>= 0), and boxes whose
// core points (skip_core) are already in the set of root skip_root (labels skip_labels;
// the visitor may advance it) are not walked.
constexpr int kWideStack = 512;  // entries per wavefront

template <int D, bool SKIP, typename F>
__device__ __forceinline__ void traverse_box_wide_lanes(const TreeView& t, int m, const Scope& sc, const float* lo,
                                                        const float* hi, int mask, int leaf_size, uint32_t* info,
                                                        uint32_t* stack, F&& visit_lanes,
                                                        int* skip_labels, const uint8_t* skip_core,
                                                        const int& skip_root) {
  if (m <= 0 || mask >= sc.end) return;
  const int lane = lane_id();
  // is the node a box whose core points are in the set of skip_root?
  auto known = [&](int first, int last, const float4& na, const float4& nb) {
    if (!SKIP || skip_root < 0 || !is_box<D>(first, last, na, nb, sc.eps2)) return false;
    const int c = box_core(skip_core, first, last, sc.min_pts);
    return c >= 0 && ancestor_compress(skip_labels, c) == skip_root;
  };
  // a range [s, e] of one lane (wave-uniform arguments), 64 primitives per call
  auto range = [&](int s, int e) {
    for (int b = s; b <= e; b += 64)
      if (visit_lanes(b + lane <= e ? b + lane : -1)) return true;
    return false;
  };
  int top = 0;
  if (SKIP) {
    // the subtrees above the mask, as the escape links have them, left to right
    uint32_t x = static_cast<uint32_t>(t.leaf_rope[mask]);
    for (int last = mask; last < sc.end && x != kEnd;) {
      if (top == kWideStack || (x & ~kLeaf) >= static_cast<uint32_t>(m)) {
        if (lane == 0) atomicOr(info, kInternalBit);
        return;
      }
      if (lane == 0) stack[top] = x;
      ++top;
      const int k = static_cast<int>(x & ~kLeaf);
      if (x & kLeaf) {
        last = k;
        x = static_cast<uint32_t>(t.leaf_rope[k]);
      } else {
        last = max(k, __float_as_int(t.node_a[kNodeStride * size_t(k)].w));
        x = static_cast<uint32_t>(t.rope[k]);
      }
    }
  }
  // a walk over the whole tree starts from the cut: its boxes are tested 64 at a
  // time and the ones within reach pushed, instead of descending from the root
  const int nc = !SKIP && t.cut && sc.start == 0 && sc.end == m - 1 ? *t.cut_n : 0;
  if (nc > 0 && nc <= kCutMax) {
    for (int b = 0; b < nc && top >= 0; b += 64 * kCutUnroll) {
      float4 ca[kCutUnroll], cb[kCutUnroll];
#pragma unroll
      for (int u = 0; u < kCutUnroll; ++u) {  // the loads of kCutUnroll chunks in flight together
        const int c = min(b + u * 64 + lane, nc - 1);
        ca[u] = t.cut[2 * c];
        cb[u] = t.cut[2 * c + 1];
      }
#pragma unroll
      for (int u = 0; u < kCutUnroll; ++u) {
        const bool hit = b + u * 64 + lane < nc && __float_as_int(cb[u].w) > mask &&
                   boxbox_dist2<D>(lo, hi, ca[u].x, ca[u].y, ca[u].z, cb[u].x, cb[u].y, cb[u].z) <= sc.eps2;
        const uint64_t hm = ballot(hit);
        if (top < 0 || top + __popcll(hm) > kWideStack) {
          top = -1;  // more than the stack holds: start from the root instead
        } else {
          if (hit) stack[top + __popcll(hm & lanemask_lt())] = __float_as_uint(ca[u].w);
          top += __popcll(hm);
        }
      }
    }
  }
  if (!SKIP && (nc <= 0 || nc > kCutMax || top < 0)) {
    if (lane == 0) stack[0] = sc.start;
    top = 1;
  }
  int64_t guard = 0;
  const int64_t max_rounds = 2 * int64_t(m) + 2;
  while (top > 0) {
    if (++guard > max_rounds) {
      atomicOr(info, kInternalBit);
      return;
    }
    const int take = top < 64 ? top : 64;
    top -= take;
    const uint32_t node = lane < take ? stack[top + lane] : kEnd;
    int bs = -1, be = -1;
    uint32_t c0 = kEnd, c1 = kEnd;
    if (node != kEnd) {
      if (node & kLeaf) {
        const int l = static_cast<int>(node & ~kLeaf);
        if (l >= m) atomicOr(info, kInternalBit);
        else if (l > mask) bs = be = l;
      } else if (node >= static_cast<uint32_t>(m - 1)) {
        atomicOr(info, kInternalBit);
      } else {
        const float4 na = t.node_a[kNodeStride * size_t(node)];
        const float4 nb = t.node_b[kNodeStride * size_t(node)];
        const int k = static_cast<int>(node);
        const int o = __float_as_int(na.w), g = __float_as_int(nb.w);
        const int first = o < k ? o : k, last = o > k ? o : k;
        if (last > mask && boxbox_dist2<D>(lo, hi, na.x, na.y, na.z, nb.x, nb.y, nb.z) <= sc.eps2) {
          if (first < 0 || last >= m || g < first || g >= last) {
            atomicOr(info, kInternalBit);
          } else if (known(first, last, na, nb)) {
            // nothing to join
          } else if (last - first < leaf_size) {
            bs = first <= mask ? mask + 1 : first;
            be = last;
          } else {
            if (g > mask) c0 = first == g ? (kLeaf | static_cast<uint32_t>(g)) : static_cast<uint32_t>(g);
            c1 = last == g + 1 ? (kLeaf | static_cast<uint32_t>(g + 1)) : static_cast<uint32_t>(g + 1);
          }
        }
      }
    }
    // this step's buckets laid end to end over the lanes: slot k of round q is
    // primitive q*64 + lane of the concatenation, found by a binary search over the
    // lanes' exclusive prefix sums (the last lane starting at or before it)
    const int len = bs >= 0 ? be - bs + 1 : 0;
    int incl = len;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int y = __shfl_up(incl, off);
      if (lane >= off) incl += y;
    }
    const int excl = incl - len;
    const int total = __shfl(incl, 63);
    for (int q = 0; q < total; q += 64) {  // every lane takes part in the shuffles
      const int slot = q + lane;
      const int sl = slot < total ? slot : total - 1;
      int lo = 0;
#pragma unroll
      for (int step = 32; step > 0; step >>= 1)
        if (__shfl(excl, lo + step) <= sl) lo += step;
      const int first = __shfl(bs, lo), ex = __shfl(excl, lo);
      if (visit_lanes(slot < total ? first + (sl - ex) : -1)) return;
    }
    const uint64_t m0 = ballot(c0 != kEnd), m1 = ballot(c1 != kEnd);
    const int n0 = __popcll(m0), n1 = __popcll(m1);
    if (top + n0 + n1 <= kWideStack) {
      const uint64_t lt = lanemask_lt();
      if (c0 != kEnd) stack[top + __popcll(m0 & lt)] = c0;
      if (c1 != kEnd) stack[top + n0 + __popcll(m1 & lt)] = c1;
      top += n0 + n1;
    } else {
      // stack full: walk each child's subtree on its own
      for (uint64_t cm = m0 | m1; cm; cm &= cm - 1) {
        const int L = __ffsll(static_cast<unsigned long long>(cm)) - 1;
        for (int side = 0; side < 2; ++side) {
          const uint32_t c = static_cast<uint32_t>(__shfl(static_cast<int>(side ? c1 : c0), L));
          if (c == kEnd) continue;
          int end;
          if (c & kLeaf) {
            end = static_cast<int>(c & ~kLeaf);
          } else {
            const int oc = __float_as_int(t.node_a[kNodeStride * size_t(c)].w);
            end = oc > static_cast<int>(c) ? oc : static_cast<int>(c);
          }
          const Scope sub{c, end, sc.eps2, sc.min_pts};
          if (traverse_box<D>(t, m, sub, lo, hi, mask, leaf_size, info, range)) return;
        }
      }
    }
  }
}

template <int D, typename F>
__device__ __forceinline__ void traverse_box_wide_lanes(const TreeView& t, int m, const Scope& sc, const float* lo,
                                                        const float* hi, int mask, int leaf_size, uint32_t* info,
                                                        uint32_t* stack, F&& visit_lanes) {
  const int none = -1;
  traverse_box_wide_lanes<D, false>(t, m, sc, lo, hi, mask, leaf_size, info, stack, visit_lanes, nullptr, nullptr, none);
}

// True only if `root` is an ancestor of x within a few plain-load hops (then x
// already is in root's set: sets only grow). False means "unknown". When the
// chain had two intermediate links or more, x is re-pointed straight at root (see
// ancestor_compress) and the next check is one load.
__device__ __forceinline__ bool known_same_set(int* labels, int x, int root) {
  const int x0 = x;
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    int p = labels[x];
    if (p == root) {
      if (h > 1) st_agent(labels + x0, root);
      return true;
    }
    if (p == x) return false;
    x = p;
  }
  return false;
}

// Slot in a list (counter *n) for every thread where pred holds, -1 elsewhere:
// one atomic per workgroup, threads in order within it. Every thread of the
// workgroup must call it (it synchronises the workgroup); s_w holds 17 ints.
__device__ __forceinline__ int block_reserve(int* n, bool pred, int* s_w) {
  const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const uint64_t b = ballot(pred);
  if (lane_id() == 0) s_w[w] = __popcll(b);
  __syncthreads();
  if (threadIdx.x == 0) {
    int tot = 0;
    for (int k = 0; k < nw; ++k) {
      const int c = s_w[k];
      s_w[k] = tot;
      tot += c;
    }
    s_w[16] = tot ? atomicAdd(n, tot) : 0;
  }
  __syncthreads();
  const int slot = s_w[16] + s_w[w] + __popcll(b & lanemask_lt());
  __syncthreads();
  return pred ? slot : -1;
}

// Up to kRecNb neighbouring primitives of one query, kept in LDS: row t of the
// workgroup's table (kRecNb x blockDim ints, dynamic shared memory) holds every
// thread's t-th neighbour, so a neighbour costs one store.
struct NbRec {
  int* col;  // &table[0][threadIdx.x]; entry t at col[t * blockDim.x]
  int nn;
};

__device__ __forceinline__ void rec_init(NbRec& r, int* table) {
  r.col = table + threadIdx.x;
  r.nn = 0;
}

__device__ __forceinline__ void rec_add(NbRec& r, int j) {
  if (r.nn < kRecNb) r.col[r.nn * blockDim.x] = j;
  ++r.nn;
}

__device__ __forceinline__ int rec_get(const NbRec& r, int t) { return r.col[t * blockDim.x]; }

// Records tell a dense cell (stored as -2 - its first point) from a point.
__device__ __forceinline__ int cell_ref(int s) { return -2 - s; }
__device__ __forceinline__ bool is_cell_ref(int v) { return v < -1; }
__device__ __forceinline__ int ref_point(int v) { return v < -1 ? -2 - v : v; }

// Where the border pass finds its work: counts of records (in kNumXcd shards, which
// the workgroups of each XCD take in turn, so that a region of many non-core points
// fills all of them alike) and of listed walks per XCD, and the queries per XCD of the
// core pass, each on a memory line of its own (a
// counter that every workgroup of the chip adds to passes them one at a time: with
// one for all, the core pass of the uniform 2M-point set took 0.69 ms in workgroups
// of 64, 0.39 of 128 and 0.29 of 256).
__device__ __forceinline__ constexpr int kRecCount(int shard) { return 32 * shard; }
__device__ __forceinline__ constexpr int kWalkCount(int xcd) { return 32 * (kNumXcd + xcd); }
constexpr int kWalkShare = 32 * 2 * kNumXcd;

// End of a core pass for query point i (primitive p): core and lone flags, and
// what the border pass will need: nothing (core, or lone: border -1 now), a
// neighbour record, or a walk. Called by every thread of the workgroup.
// first: the first query of this XCD's share (which its walk list starts at).
__device__ __forceinline__ void core_epilogue(const TravArgs& a, bool mine, int i, int p, int cnt, int min_pts,
                                              const NbRec& rec, int* s_w, int64_t first) {
  const bool core = mine && cnt >= min_pts;
  const bool lone = mine && cnt <= 1 && !core;
  if (mine) {
    a.core[i] = core ? 1 : 0;
    a.lone[i] = lone ? 1 : 0;
    if (lone) a.border[i] = -1;
  }
  if (core) {
    // A core point and a dense cell it reaches are a core pair: join them now,
    // so the main phase finds them in one set and skips the cell scan.
    const int nr = rec.nn < kRecNb ? rec.nn : kRecNb;
    int root = i;
    for (int t = 0; t < nr; ++t) {
      const int v = rec_get(rec, t);
      if (is_cell_ref(v)) root = uf_union(a.labels, root, ref_point(v), a.info);
    }
  }
  const bool want = mine && !core && !lone;
  const bool fits = want && rec.nn <= kRecNb;
  const int xcd = static_cast<int>(blockIdx.x % kNumXcd);
  const int shard = static_cast<int>(blockIdx.x / kNumXcd % kNumXcd);
  const int slot = block_reserve(a.border_n + kRecCount(shard), fits, s_w);
  const bool stored = fits && slot < a.brec_cap;
  if (stored) {
    const int64_t k = int64_t(shard) * a.brec_cap + slot;
    a.brec_i[k] = i;
#pragma unroll
    for (int t = 0; t < kRecNb; ++t) a.brec_nb[k * kRecNb + t] = t < rec.nn ? ref_point(rec_get(rec, t)) : -1;
  }
  if (__syncthreads_or(want && !stored)) {
    const int wslot = block_reserve(a.border_n + kWalkCount(xcd), want && !stored, s_w);
    if (wslot >= 0) a.qborder[first + wslot] = p;
  }
}

// A non-core point with no neighbour but itself (known once the core pass has
// run) is noise: nothing to claim, no cluster to join.
__device__ __forceinline__ bool is_lone(const TravArgs& a, int i) { return a.lone && a.lone[i]; }

__device__ __forceinline__ float readlane_f(float v, int k) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k));
}

// Is every point in the box [lo, hi] within eps of q, as the
// point-by-point test would decide? Per axis the corner farther from q (by the
// rounded difference) bounds every point's rounded difference, since rounded
// subtraction, squaring and addition are monotone; so the test at that corner,
// made with the same operations in the same order, holds for all of them.
template <int D>
__device__ __forceinline__ bool cell_within(float4 lo, float4 hi, const Query& q, float eps2) {
  const float cx = fabsf(lo.x - q.x) > fabsf(hi.x - q.x) ? lo.x : hi.x;
  const float cy = fabsf(lo.y - q.y) > fabsf(hi.y - q.y) ? lo.y : hi.y;
  const float cz = fabsf(lo.z - q.z) > fabsf(hi.z - q.z) ? lo.z : hi.z;
  return dist2v<D>(cx, cy, cz, q.x, q.y, q.z) <= eps2;
}

// ---------------------------------------------------------------- FDbscan ----

template <int D, bool B>
__global__ void k_core_fdb(TravArgs a) {
  __shared__ int s_w[17];
  extern __shared__ int s_rec[];  // kRecNb * blockDim.x
  const int64_t i64 = xcd_spread(blockIdx.x, blockDim.x, threadIdx.x, a.n);
  const bool mine = i64 >= 0 && i64 < a.n && a.core[i64] < kCliqueCore;
  const int i = mine ? static_cast<int>(i64) : 0;
  const int m = tree_m(a.t);
  const Scope sc = scope_of<B>(a, m, i);
  const Query q = load_point<D>(a.xs, a.n, i);
  int cnt = 0;
  NbRec rec;
  rec_init(rec, s_rec);
  if (mine)
    traverse<D, false>(a.t, m, sc, q, 0, a.info, [&](int s, int e) {
      for (int j = s; j <= e && cnt < sc.min_pts; j += 4)
        for (unsigned nb = near_bits<D>(a.xs, a.n, j, e, q, sc.eps2); nb; nb &= nb - 1) {
          const int k = j + __ffs(nb) - 1;
          if (k != i) rec_add(rec, k);
          ++cnt;
        }
      return cnt >= sc.min_pts;
    }, [&](int first, int last, const float4& lo, const float4& hi) {
      // enough points in a box all within eps: core, whichever they are
      if (cnt + (last - first + 1) < sc.min_pts || !cell_within<D>(lo, hi, q, sc.eps2)) return 0;
      cnt = sc.min_pts;
      return 2;
    });
  const int64_t share = xcd_share(a.n, blockDim.x);
  if (blockIdx.x == 0 && threadIdx.x == 0) a.border_n[kWalkShare] = static_cast<int>(share);
  core_epilogue(a, mine, i, i, cnt, sc.min_pts, rec, s_w, (blockIdx.x % kNumXcd) * share);
}

// The queries of a kernel whose number `total` only the device knows: a
// workgroup takes chunks of kLanes queries a wavefront, blockIdx.x, + gridDim.x, ...
// (gridDim.x a multiple of kNumXcd), laid out over the XCDs as xcd_spread has them.
// The grid is capped (query_grid_blocks): with a workgroup for each of the n points
// the queries could be, 65,536 workgroups without work took 15 us a launch (8M set).
// Few queries take fewer lanes a wavefront, down to 8, so that kWaves wavefronts or
// more share them: a wavefront's time is its lanes' loads, scans and unions one after the
// other, and 44k queries (370k-point mixture) fill only 700 wavefronts of 64.
constexpr int kWaves = 4096;

struct Chunks {
  int64_t chunk, off;  // queries per XCD; this workgroup's first within its XCD's
  int lanes, step, slot, xcd;

  __device__ __forceinline__ Chunks(int64_t total, bool spread) {
    lanes = 64;
    while (spread && lanes > 8 && total < int64_t(kWaves) * (lanes / 2)) lanes >>= 1;
    const int per = lanes * static_cast<int>(blockDim.x >> 6);  // queries a workgroup and chunk
    chunk = xcd_share(total, per);
    xcd = static_cast<int>(blockIdx.x % kNumXcd);
    off = int64_t(blockIdx.x / kNumXcd) * per;
    step = static_cast<int>(gridDim.x / kNumXcd) * per;
    slot = lane_id() < lanes ? static_cast<int>(threadIdx.x >> 6) * lanes + lane_id() : -1;
  }
  __device__ __forceinline__ bool in() const { return off < chunk; }
  __device__ __forceinline__ void next() { off += step; }
  // this lane's query (at or above the total where the chunk runs past it), -1: none
  __device__ __forceinline__ int query() const { return slot < 0 ? -1 : static_cast<int>(xcd * chunk + off + slot); }
};

// Cliques, before the core pass: a thread takes kCliqueItems nodes in turn and looks at the
// two children of each (their records lie side by side). Cliques in no larger one, and of
// larger ones than `most` the largest nodes that are not, get their points marked: core
// (kInClique where the node searches for itself, which kCliqueWave points in it or a clique
// above it are worth, else kCliqueCore) and one set, their first point's. A node above them
// hangs its right child's first point under its own, so a clique of any size is one set and
// no wavefront marks more than `most` points. Boxes of fewer than minPts points in no
// larger one are listed for k_core_boxes. A workgroup lists through LDS and reserves once.
// Bound by the node records: 8M points (80% of them in cliques) 120 us for 268 MB of nodes
// read up to three times.
constexpr int kCliqueItems = 8;

template <int D, bool B>
__global__ __launch_bounds__(256) void k_cliques(TravArgs a) {
  constexpr int kList = 2 * 256 * kCliqueItems;
  __shared__ int s_list[kList];  // nodes that search from the front, boxes from the back
  __shared__ int s_n, s_b, s_at, s_bat;
  const int m = tree_m(a.t);
  const int lane = lane_id();
  if (threadIdx.x == 0) s_n = s_b = 0;
  __syncthreads();
  struct Node {
    int first = 0, last = -1, g = -1;
    bool box = false;
  };
  auto load = [&](int k) {
    const float4 lo = a.t.node_a[kNodeStride * size_t(k)], hi = a.t.node_b[kNodeStride * size_t(k)];
    const int o = __float_as_int(lo.w);
    Node v;
    v.first = o < k ? o : k;
    v.last = o > k ? o : k;
    v.g = __float_as_int(hi.w);
    if (v.first < 0 || v.last >= m || v.g < v.first || v.g >= v.last) {  // not a node: the walks report it
      v.g = -1;
      return v;
    }
    if (B && cloud_of(a, v.first) != cloud_of(a, v.last)) return v;
    v.box = is_box<D>(v.first, v.last, lo, hi, B ? a.cloud_eps2[cloud_of(a, v.first)] : a.eps2);
    return v;
  };
  const int64_t base = blockIdx.x * int64_t(256 * kCliqueItems) + threadIdx.x;
  for (int t = 0; t < kCliqueItems; ++t) {
    const int64_t k64 = base + t * 256;
    int lo[2] = {0, 0}, hi[2] = {-1, -1};  // ranges to mark
    bool search[2] = {false, false};
    if (k64 < m - 1) {
      const int k = static_cast<int>(k64);
      const Node v = load(k);
      const int min_pts = v.box ? (B ? a.cloud_minpts[cloud_of(a, v.first)] : a.min_pts) : 0;
      const int most = max(kCliqueMost, min_pts);
      const bool large = v.box && v.last - v.first + 1 > most;
      if (large) a.labels[v.g + 1] = v.first;
      // node c (a child, or the root) is a box in no larger one, or in a large one
      auto take = [&](int slot, uint32_t ref, int first, int last, int cloud_minpts, bool inside) {
        const int size = last - first + 1;
        if (!inside && size < cloud_minpts) {
          s_list[kList - 1 - atomicAdd(&s_b, 1)] = static_cast<int>(ref);
          return;
        }
        if (size > max(kCliqueMost, cloud_minpts)) return;
        lo[slot] = first;
        hi[slot] = last;
        search[slot] = inside || size >= kCliqueWave;
        if (search[slot]) s_list[atomicAdd(&s_n, 1)] = static_cast<int>(ref);
      };
      if (k == 0 && v.box && !large) take(0, 0u, v.first, v.last, min_pts, false);
      if (v.g >= 0 && (!v.box || large)) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const int x = v.g + c;
          const bool leaf = c ? v.last == x : v.first == x;
          if (leaf) {
            if (large) take(c, kLeaf | static_cast<uint32_t>(x), x, x, min_pts, true);
            continue;
          }
          const Node w = load(x);
          if (w.g < 0 || !w.box) {
            // (a child of a large clique is a box unless it is smaller than one)
            if (large && w.g >= 0) take(c, static_cast<uint32_t>(x), w.first, w.last, min_pts, true);
            continue;
          }
          const int mp = large ? min_pts : (B ? a.cloud_minpts[cloud_of(a, w.first)] : a.min_pts);
          take(c, static_cast<uint32_t>(x), w.first, w.last, mp, large);
        }
      }
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int how = search[c] ? kInClique : kCliqueCore;
      for (uint64_t fm = ballot(hi[c] >= lo[c]); fm; fm &= fm - 1) {
        const int L = __ffsll(static_cast<unsigned long long>(fm)) - 1;
        const int first = __builtin_amdgcn_readlane(lo[c], L), last = __builtin_amdgcn_readlane(hi[c], L);
        const int flag = __builtin_amdgcn_readlane(how, L);
        for (int i = first + lane; i <= last; i += 64) {
          if (i > first) a.labels[i] = first;  // (the first point's is its own, or a node's above)
          a.core[i] = static_cast<uint8_t>(flag);
        }
      }
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    s_at = s_n ? atomicAdd(a.num_cliques, s_n) : 0;
    s_bat = s_b ? atomicAdd(a.num_boxes, s_b) : 0;
  }
  __syncthreads();
  for (int k = threadIdx.x; k < s_n; k += 256) a.cliques[s_at + k] = s_list[k];
  for (int k = threadIdx.x; k < s_b; k += 256) a.boxes[s_bat + k] = s_list[kList - 1 - k];
}

// The boxes of fewer than minPts points, once the core pass is done, eight lanes each: their
// core points become one set, and a box of nothing else is a clique from now on. Where an
// eps-ball holds several times minPts points and a box of diagonal eps fewer than that (it
// has 1/22 of the ball in three dimensions), there are no other boxes, and the main phase
// tests every pair without these: 200,000 points in 3D, FDbscan, us, without / with: minPts
// 100 of 1700 neighbours 7842 / 1227, 1000 of 4000 14,360 / 3690; in 2D 1000 of 4000 9906 /
// 2155 (walking as packets past whole sets of the hierarchy's cut: 2727, 7842, 3737).
__global__ __launch_bounds__(256) void k_core_boxes(TravArgs a) {
  constexpr int G = 8;
  const int nb = *a.num_boxes;
  const int sub = threadIdx.x & (G - 1);
  for (int64_t b0 = blockIdx.x * int64_t(256 / G); b0 < nb; b0 += int64_t(gridDim.x) * (256 / G)) {
    const int64_t b = b0 + threadIdx.x / G;
    const int k = b < nb ? a.boxes[b] : 0;
    const int o = b < nb ? __float_as_int(a.t.node_a[kNodeStride * size_t(k)].w) : 0;
    const int first = o < k ? o : k, last = b < nb ? (o > k ? o : k) : -1;
    int rep = 0x7fffffff, cnt = 0;
    for (int i = first + sub; i <= last; i += G)
      if (a.core[i]) {
        rep = min(rep, i);
        ++cnt;
      }
#pragma unroll
    for (int off = G / 2; off > 0; off >>= 1) {
      rep = min(rep, __shfl_xor(rep, off));
      cnt += __shfl_xor(cnt, off);
    }
    const int size = last - first + 1;
    const bool all = cnt == size && cnt > 0, search = all && size >= kCliqueWave;
    const uint8_t flag = search ? kInClique : kCliqueCore;
    if (cnt > 1)
      for (int i = first + sub; i <= last; i += G)
        if (a.core[i]) {
          a.labels[i] = rep;
          if (all) a.core[i] = flag;
        }
    const uint64_t sm = ballot(search && sub == 0);
    if (sm) {
      const int leader = __ffsll(static_cast<unsigned long long>(sm)) - 1;
      int at = 0;
      if (lane_id() == leader) at = atomicAdd(a.num_cliques, __popcll(sm));
      at = __shfl(at, leader);
      if (search && sub == 0) a.cliques[at + __popcll(sm & lanemask_lt())] = k;
    }
  }
}

// First-claim main phase (the paper's border rule), a lane per point. A core point
// passes over boxes already in its set, if all of their points are core (with packets of
// near queries instead 1M dense clumps took 23.7 ms a call, with lanes 1.3).
__device__ __forceinline__ void main_pair_first(const TravArgs& a, int i, bool ci, int j, bool cj, int& root,
                                                bool& done) {
  int* labels = a.labels;
  if (ci && cj) {
    if (!known_same_set(labels, j, root)) root = uf_union(labels, root, j, a.info);
  } else if (ci) {
    uf_claim(labels, j, i);
  } else if (cj) {
    uf_claim(labels, i, j);
    done = true;  // i is a member now (by this or an earlier claim)
  }
}

template <int D, bool B>
__global__ void k_main_fdb_first(TravArgs a) {
  const int64_t i64 = xcd_spread(blockIdx.x, blockDim.x, threadIdx.x, a.n);
  if (i64 < 0 || i64 >= a.n) return;
  const int i = static_cast<int>(i64);
  const bool ci = a.core[i] != 0;
  if (!ci && is_lone(a, i)) return;
  const int m = tree_m(a.t);
  const Scope sc = scope_of<B>(a, m, i);
  const Query q = load_point<D>(a.xs, a.n, i);
  int* labels = a.labels;
  int root = i;
  bool done = false;
  traverse<D, true>(a.t, m, sc, q, i, a.info, [&](int s, int e) {
    for (int j = s; j <= e && !done; j += 4)
      for (unsigned nb = near_bits<D>(a.xs, a.n, j, e, q, sc.eps2); nb && !done; nb &= nb - 1) {
        const int k = j + __ffs(nb) - 1;
        main_pair_first(a, i, ci, k, a.core[k] != 0, root, done);
      }
    return done;
  }, [&](int first, int last, const float4& lo, const float4& hi) {
    return ci && is_box<D>(first, last, lo, hi, sc.eps2) &&
                   (last - first + 1 >= sc.min_pts || a.core[first] >= kCliqueCore) &&
                   known_same_set(labels, first, root)
               ? 1 : 0;
  });
}

// Canonical (and minPts <= 2) main phase of the points outside the cliques of
// k_main_cliques: a lane each, walking over the points above its own and passing over
// cliques that already are in its set, so a dense clump costs a look at each of its
// cliques. Bound by each lane's chain of dependent loads and, in sparse sets, by unions.
// Before there were cliques, wavefronts of 64 near queries walked as packets, to share
// the clumps' candidates; with them walks of their own are faster everywhere (main phase
// with the packets / without: 8M-point set 1124 / 256 us, 16,384 points 430 / 123,
// friends-of-friends set 1629 / 1673), and a packet of spread-out queries, which took
// them one by one, no longer exists (1.5M uniform points, minPts 5: 18.0 -> 2.4 ms a call).
template <int D, bool ALL_CORE, bool B>
__global__ void k_main_fdb(TravArgs a) {
  const int64_t i64 = xcd_spread(blockIdx.x, blockDim.x, threadIdx.x, a.n);
  if (i64 < 0 || i64 >= a.n) return;
  const int i = static_cast<int>(i64);
  const int f = a.core[i];
  if (f == kInClique || !(ALL_CORE || f)) return;
  const int m = tree_m(a.t);
  const Scope sc = scope_of<B>(a, m, i);
  const Query q = load_point<D>(a.xs, a.n, i);
  int* labels = a.labels;
  int root = i;
  traverse<D, true>(a.t, m, sc, q, i, a.info, [&](int s, int e) {
    for (int j = s; j <= e; j += 4)
      for (unsigned nb = near_bits<D>(a.xs, a.n, j, e, q, sc.eps2); nb; nb &= nb - 1) {
        const int k = j + __ffs(nb) - 1;
        if ((ALL_CORE || a.core[k]) && !known_same_set(labels, k, root)) root = uf_union(labels, root, k, a.info);
      }
    return false;
  }, [&](int first, int last, const float4& lo, const float4& hi) {
    if (!is_box<D>(first, last, lo, hi, sc.eps2)) return 0;
    const int c = ALL_CORE ? first : box_core(a.core, first, last, sc.min_pts);
    return c >= 0 && known_same_set(labels, c, root) ? 1 : 0;
  });
}

// Main phase of the cliques that search for themselves: one wavefront per clique A (a node,
// or kLeaf | a point of a large one) walks the tree once with A's box over the points above A. A candidate is a core point within eps of A's box that is
// not known to be in A's set, one per lane; it joins the set if some point of A is
// within eps (the points below A look for A themselves: other points in k_main_fdb,
// points of cliques here). A wavefront's time is its rounds, each a chain of
// dependent loads; starting from the cut's 8192 boxes instead of the escape links cost
// 128 rounds of box tests a clique (friends-of-friends set, cliques of 4 and more: 1426
// us, 896 us from the links). One lane per clique was slower (1222 us, and on 16,384
// points 190 us instead of 40).
template <int D, bool ALL_CORE, bool B>
__global__ __launch_bounds__(256) void k_main_cliques(TravArgs a) {
  __shared__ uint32_t s_stack[4 * kWideStack];
  uint32_t* stack = s_stack + (threadIdx.x >> 6) * kWideStack;
  const int m = tree_m(a.t), nq = *a.num_cliques;
  const int lane = lane_id();
  const int nwaves = (gridDim.x * blockDim.x) >> 6;
  int* labels = a.labels;
  for (int w = (xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x) >> 6; w < nq; w += nwaves) {
    const uint32_t ref = static_cast<uint32_t>(a.cliques[w]);
    const int k = static_cast<int>(ref & ~kLeaf);
    int sa = k, ea = k;
    float4 na, nb;
    if (ref & kLeaf) {
      const Query q = load_point<D>(a.xs, a.n, k);
      na = nb = make_float4(q.x, q.y, q.z, 0.0f);
    } else {
      na = a.t.node_a[kNodeStride * size_t(k)];
      nb = a.t.node_b[kNodeStride * size_t(k)];
      const int o = __float_as_int(na.w);
      sa = o < k ? o : k;
      ea = o > k ? o : k;
    }
    const float alo[3] = {na.x, na.y, na.z}, ahi[3] = {nb.x, nb.y, nb.z};
    const Scope sc = scope_of<B>(a, m, sa);
    const float eps2 = sc.eps2;
    int r = uf_find(labels, sa, a.info);
    traverse_box_wide_lanes<D, true>(a.t, m, sc, alo, ahi, ea, a.packet_leaf, a.info, stack, [&](int jl) {
      float cx = 0.0f, cy = 0.0f, cz = 0.0f;
      int cl = -1;
      bool need = false;
      if (jl >= 0 && (ALL_CORE || a.core[jl])) {
        cx = a.xs[jl];
        cy = a.xs[a.n + jl];
        cz = D == 3 ? a.xs[2 * a.n + jl] : 0.0f;
        need = box_dist2<D>(cx, cy, cz, alo[0], alo[1], alo[2], ahi[0], ahi[1], ahi[2]) <= eps2;
        if (need) cl = ancestor_compress(labels, jl);
        need = need && cl != r;
      }
      bool reach = false;
      for (int base = sa; base <= ea && ballot(need && !reach); base += 64) {
        const int at = min(base + lane, ea);
        const float px = a.xs[at], py = a.xs[a.n + at], pz = D == 3 ? a.xs[2 * a.n + at] : 0.0f;
        const int cnt = min(64, ea - base + 1);
        for (int u = 0; u < cnt; ++u)
          reach |= need && dist2v<D>(cx, cy, cz, readlane_f(px, u), readlane_f(py, u), readlane_f(pz, u)) <= eps2;
      }
      if (ballot(reach)) {
        // one union for all candidates of a set
        bool joins = false;
        for (uint64_t rm = ballot(reach); rm;) {
          const int L = __ffsll(static_cast<unsigned long long>(rm)) - 1;
          const int c = __builtin_amdgcn_readlane(cl, L);
          if (lane == L) joins = true;
          rm &= ~ballot(reach && cl == c);
        }
        if (joins) uf_union(labels, r, jl, a.info);
        int nr = 0;
        if (lane == 0) nr = uf_find(labels, r, a.info);
        r = __builtin_amdgcn_readfirstlane(nr);
      }
      return false;
    }, labels, a.core, r);
  }
}

// Border pass from the core pass's neighbour records (no walk): the smallest
// cluster id among the recorded core neighbours.
__global__ void k_border_rec(TravArgs a) {
  const int shard = static_cast<int>(blockIdx.x % kNumXcd);
  const int64_t slot = int64_t(blockIdx.x / kNumXcd) * blockDim.x + threadIdx.x;
  if (slot >= min(a.border_n[kRecCount(shard)], a.brec_cap)) return;
  const int64_t k = int64_t(shard) * a.brec_cap + slot;
  const int i = a.brec_i[k];
  int best = 0x7fffffff;
#pragma unroll
  for (int t = 0; t < kRecNb; ++t) {
    const int j = a.brec_nb[k * kRecNb + t];
    if (j >= 0 && a.core[j]) {
      const int c = a.cid[a.labels[j]];
      best = c < best ? c : best;
    }
  }
  a.border[i] = best == 0x7fffffff ? -1 : best;
}

// Border pass over the listed queries: non-core points whose neighbours were
// not all recorded (the core pass wrote -1 for lone points, and the records
// cover the rest).
template <int D, bool B>
__global__ void k_border_fdb(TravArgs a) {
  const int xcd = static_cast<int>(blockIdx.x % kNumXcd);
  const int64_t slot = int64_t(blockIdx.x / kNumXcd) * blockDim.x + threadIdx.x;
  if (slot >= a.border_n[kWalkCount(xcd)]) return;
  const int i = a.qborder[int64_t(xcd) * a.border_n[kWalkShare] + slot];
  const int m = tree_m(a.t);
  const Scope sc = scope_of<B>(a, m, static_cast<int>(i));
  const Query q = load_point<D>(a.xs, a.n, i);
  int best = 0x7fffffff;
  traverse<D, false>(a.t, m, sc, q, 0, a.info, [&](int s, int e) {
    for (int j = s; j <= e && best > 0; j += 4)
      for (unsigned nb = near_bits<D>(a.xs, a.n, j, e, q, sc.eps2); nb; nb &= nb - 1) {
        const int k = j + __ffs(nb) - 1;
        if (!a.core[k]) continue;
        const int c = a.cid[a.labels[k]];
        best = c < best ? c : best;
      }
    return best == 0;
  });
  a.border[i] = best == 0x7fffffff ? -1 : best;
}

// --------------------------------------------------------------- DenseBox ----
// Primitive p covers sorted points [prim_start[p], prim_start[p] + |cnt|):
// cnt > 0 is a single point, cnt < 0 a dense cell (all core, one cluster).
// Points outside dense cells query one lane per point primitive (so
// wavefronts are full and in Morton order); a dense cell queries once, one
// wavefront per cell, whose 64 lanes test the cell's points together.

// A walk reads primitive r through its leaf record prim_lo[r] (see TravArgs):
// one 16-byte load gives a point primitive's coordinates and sorted index, or a
// dense cell's low corner and first point.
__device__ __forceinline__ int rec_index(float4 lr) { return __float_as_int(lr.w); }

template <int D>
__device__ __forceinline__ bool rec_point_near(float4 lr, const Query& q, float eps2) {
  return dist2v<D>(lr.x, lr.y, lr.z, q.x, q.y, q.z) <= eps2;
}

template <int D>
__device__ __forceinline__ bool cell_box_near(const TravArgs& a, int r, float4 lo, const Query& q, float eps2) {
  const float4 hi = a.prim_hi[r];
  return box_dist2<D>(q.x, q.y, q.z, lo.x, lo.y, lo.z, hi.x, hi.y, hi.z) <= eps2;
}

// The query of point primitive p (its record), or an idle lane's (mine false).
__device__ __forceinline__ void own_record(const TravArgs& a, int p, int m, bool& mine, int& i, Query& q) {
  const float4 lr = p >= 0 && p < m ? a.prim_lo[p] : make_float4(0.0f, 0.0f, 0.0f, __int_as_float(-1));
  mine = rec_index(lr) >= 0;
  i = mine ? rec_index(lr) : 0;
  q.x = lr.x;
  q.y = lr.y;
  q.z = lr.z;
}

// Is some point of the cell [sa, sa+na) within eps of p? (whole wavefront)
template <int D>
__device__ __forceinline__ bool cell_reaches_point(const float* __restrict__ xs, int64_t n, int sa, int na, float px,
                                                   float py, float pz, float eps2) {
  const int lane = lane_id();
  for (int base = 0; base < na; base += 64) {
    bool h = false;
    if (base + lane < na) {
      const int64_t j = sa + base + lane;
      h = dist2v<D>(xs[j], xs[n + j], D == 3 ? xs[2 * n + j] : 0.0f, px, py, pz) <= eps2;
    }
    if (ballot(h)) return true;
  }
  return false;
}

// Is some pair (a in cell A, b in cell B) within eps? (whole wavefront.) A's
// points are taken 64 at a time, keeping those within eps of B's box; B's
// points are loaded 64 at a time too, keeping those within eps of the box of
// the kept A points (box gaps never exceed point distances, so nothing that
// could pass is dropped), and each kept B point is tested against all kept A
// points at once.
template <int D>
__device__ __forceinline__ bool cells_touch(const float* __restrict__ xs, int64_t n, int sa, int na, int sb, int nb,
                                           float4 blo, float4 bhi, float eps2) {
  const int lane = lane_id();
  for (int base = 0; base < na; base += 64) {
    bool act = base + lane < na;
    float ax = 0.0f, ay = 0.0f, az = 0.0f;
    if (act) {
      const int64_t j = sa + base + lane;
      ax = xs[j];
      ay = xs[n + j];
      az = D == 3 ? xs[2 * n + j] : 0.0f;
      act = box_dist2<D>(ax, ay, az, blo.x, blo.y, blo.z, bhi.x, bhi.y, bhi.z) <= eps2;
    }
    if (!ballot(act)) continue;
    // an A point whose eps-ball holds B's whole tight box pairs with every B point
    if (ballot(act && cell_within<D>(blo, bhi, Query{ax, ay, az}, eps2))) return true;
    float lo[3] = {act ? ax : INFINITY, act ? ay : INFINITY, act ? az : INFINITY};
    float hi[3] = {act ? ax : -INFINITY, act ? ay : -INFINITY, act ? az : -INFINITY};
#pragma unroll
    for (int k = 0; k < D; ++k)
      for (int off = 32; off > 0; off >>= 1) {
        lo[k] = fminf(lo[k], __shfl_xor(lo[k], off));
        hi[k] = fmaxf(hi[k], __shfl_xor(hi[k], off));
      }
    if (D == 2) lo[2] = hi[2] = 0.0f;
    for (int bb = 0; bb < nb; bb += 64) {
      bool near_b = bb + lane < nb;
      float bx = 0.0f, by = 0.0f, bz = 0.0f;
      if (near_b) {
        const int64_t j = sb + bb + lane;
        bx = xs[j];
        by = xs[n + j];
        bz = D == 3 ? xs[2 * n + j] : 0.0f;
        near_b = box_dist2<D>(bx, by, bz, lo[0], lo[1], lo[2], hi[0], hi[1], hi[2]) <= eps2;
      }
      for (uint64_t bm = ballot(near_b); bm; bm &= bm - 1) {
        const int k = __ffsll(static_cast<unsigned long long>(bm)) - 1;
        const float px = readlane_f(bx, k), py = readlane_f(by, k), pz = readlane_f(bz, k);
        if (ballot(act && dist2v<D>(ax, ay, az, px, py, pz) <= eps2)) return true;
      }
    }
  }
  return false;
}

// Number of points of the cell [s, s+c) within eps of p, counted 64 at a time
// until at least `want` (whole wavefront).
template <int D>
__device__ __forceinline__ int cell_count_near(const float* __restrict__ xs, int64_t n, int s, int c, float px,
                                               float py, float pz, float eps2, int want) {
  const int lane = lane_id();
  int found = 0;
  for (int base = 0; base < c && found < want; base += 64) {
    bool h = false;
    if (base + lane < c) {
      const int64_t j = s + base + lane;
      h = dist2v<D>(xs[j], xs[n + j], D == 3 ? xs[2 * n + j] : 0.0f, px, py, pz) <= eps2;
    }
    found += __popcll(ballot(h));
  }
  return found;
}

// Resumable per-lane walk, one primitive (or one internal node) per step, so
// that a wavefront can pause between steps: the sparse-point kernels below run
// their lanes in lock-step and, whenever some lanes have reached a dense cell,
// scan each such cell with the whole wavefront (64 points per ballot) instead
// of one lane looping over hundreds of points.
struct Walk {
  uint32_t node;  // next node to examine, kEnd when finished
  int cur, end;   // pending bucket primitives [cur, end]; empty when cur > end
  int last;       // last primitive of the scope
  uint32_t steps;  // remaining step budget (see traverse()); 2m + 2 <= 2^31
};

template <bool MASKED>
__device__ __forceinline__ void walk_init(Walk& w, int m, const Scope& sc, int mask, bool on) {
  w.cur = 1;
  w.end = 0;
  w.last = sc.end;
  w.steps = 2u * static_cast<uint32_t>(m) + 2u;
  if (!on || m <= 0 || (MASKED && mask >= sc.end)) w.node = kEnd;
  else w.node = sc.start;
}

__device__ __forceinline__ bool walk_done(const Walk& w) { return w.node == kEnd && w.cur > w.end; }

template <int D, bool MASKED, typename QT>
__device__ __forceinline__ int walk_step(Walk& w, const TreeView& t, int m, const QT& q, float eps2, int mask,
                                         uint32_t* info) {
  if (w.cur <= w.end) return w.cur++;
  const uint32_t node = w.node;
  if (node == kEnd) return -1;
  if (w.steps-- == 0) {
    atomicOr(info, kInternalBit);
    w.node = kEnd;
    return -1;
  }
  if (node & kLeaf) {
    const int l = static_cast<int>(node & ~kLeaf);
    if (l >= m) {
      atomicOr(info, kInternalBit);
      w.node = kEnd;
      return -1;
    }
    w.node = l >= w.last ? kEnd : static_cast<uint32_t>(t.leaf_rope[l]);
    return l;
  }
  if (node >= static_cast<uint32_t>(m - 1)) {
    atomicOr(info, kInternalBit);
    w.node = kEnd;
    return -1;
  }
  const float4 a = t.node_a[kNodeStride * size_t(node)];
  const float4 b = t.node_b[kNodeStride * size_t(node)];
  const uint32_t esc = static_cast<uint32_t>(t.rope[node]);  // loaded with the node
  const int k = static_cast<int>(node);
  const int o = __float_as_int(a.w), g = __float_as_int(b.w);
  const int first = o < k ? o : k, last = o > k ? o : k;
  if (node_gap2<D>(q, a, b) > eps2) {
    w.node = last >= w.last ? kEnd : esc;
    return -1;
  }
  if (first < 0 || last >= m || g < first || g >= last) {
    atomicOr(info, kInternalBit);
    w.node = kEnd;
    return -1;
  }
  if (last - first < t.leaf_size) {
    w.cur = (MASKED && first <= mask) ? mask + 1 : first;
    w.end = last;
    w.node = last >= w.last ? kEnd : esc;
    return w.cur <= w.end ? w.cur++ : -1;
  }
  if (MASKED && g <= mask)
    w.node = last == g + 1 ? (kLeaf | static_cast<uint32_t>(g + 1)) : static_cast<uint32_t>(g + 1);
  else
    w.node = first == g ? (kLeaf | static_cast<uint32_t>(g)) : static_cast<uint32_t>(g);
  return -1;
}

// ---- grid or hierarchy ------------------------------------------------------------
// The DenseBox kernels walk the grid's cells (G, fdb_cells.hpp) or the hierarchy (!G), as
// the plan on the device says. Each is built for either walk alone, and both are
// launched, the other leaving at once: the hierarchy's walks then keep the occupancy
// that the grid's LDS would take. Up to kEitherMax points a call's time is its launches
// (3 to 4.5 us each), and one kernel holds both (1,000 points 192 -> 180 us, 370k 636 ->
// 616 us; a 300k set through the hierarchy, one far outlier, 9.5 -> 9.6 ms). A walker yields one primitive per step, so
// that a wavefront can pause its lanes between steps and scan a large dense cell together.
enum Walks { kHierarchy, kGrid, kEither };
constexpr int64_t kEitherMax = int64_t(1) << 19;

template <int W, typename F>
__device__ __forceinline__ void with_walk(const TravArgs& a, F&& f) {
  const bool grid = a.ix.plan->grid_on != 0;
  if constexpr (W != kHierarchy)
    if (grid) f(std::true_type{});
  if constexpr (W != kGrid)
    if (!grid) f(std::false_type{});
}

// LDS of a wavefront's search through the grid: a packet's cell list or the columns
// of its lanes' walks (dynamic shared memory).
template <int D, bool G>
constexpr int kSearchLds = G ? kWalkWaveBytes<D> : 0;
static_assert(kWalkWaveBytes<2> >= kBoxList * 4 && kWalkWaveBytes<3> >= kBoxList * 4, "a packet's list fits too");
template <int D, bool G>
__device__ __forceinline__ char* search_lds(char* base) {
  return base + (threadIdx.x >> 6) * kSearchLds<D, G>;
}

struct EveryCell {
  __device__ __forceinline__ bool operator()(int) const { return false; }
};

template <int D, bool B, bool MASKED, bool G, bool NEAR = false>
struct Walker {
  using State = std::conditional_t<G, CellWalk<D>, Walk>;
  State w;
  char* lds;

  // wave_lds: search_lds of the wavefront. The query is the box [lo, hi] (a point
  // when they are equal) at sorted point i.
  __device__ __forceinline__ void init(const TravArgs& a, int m, const Scope& sc, int i, const float* lo,
                                       const float* hi, int mask, bool on, char* wave_lds) {
    lds = wave_lds;
    if constexpr (G) {
      const CellGrid g = query_grid<D, B>(a.ix, B ? cloud_of(a, i) : 0);
      CellRange<D> cr;
      cell_range<D>(cr, g, lo, hi);
      cell_walk_init<D, MASKED, NEAR>(w, a.ix, g, cr, on && g.ncell[0] > 0, lds);
    } else {
      walk_init<MASKED>(w, m, sc, mask, on);
    }
  }
  __device__ __forceinline__ bool done() const {
    if constexpr (G) return cell_walk_done(w);
    else return walk_done(w);
  }
  template <typename QT, typename P = EveryCell>
  __device__ __forceinline__ int step(const TravArgs& a, int m, const QT& q, float eps2, int mask, P&& pass = P{}) {
    if constexpr (G) return cell_walk_step<D, MASKED>(w, a.ix, mask, lds, pass);
    else return walk_step<D, MASKED>(w, a.t, m, q, eps2, mask, a.info);
  }
};

// Neighbours that a lane has to join to its query's set, put off until some lane has
// kHits of them: a union is a chain of several round trips for which the whole
// wavefront waits, so lanes do theirs together (a column per lane in the wavefront's
// LDS). Uniform 2M-point set: point main phase 0.72 -> 0.66 ms. (The dense-cell main
// phase keeps joining at once: its pair tests are what costs, and the set they skip
// by has to be up to date; put off, the batch's 5.0 ms became 9.5.)
constexpr int kHits = 8;
constexpr int kHitBytes = kHits * 64 * 4;

struct Hits {
  int* col;
  int n;
};

__device__ __forceinline__ void hits_init(Hits& h, char* lds) {
  h.col = reinterpret_cast<int*>(lds) + lane_id();
  h.n = 0;
}

__device__ __forceinline__ void hits_add(Hits& h, int j) { h.col[64 * h.n++] = j; }

__device__ __forceinline__ bool hits_full(const Hits& h) { return ballot(h.n >= kHits) != 0; }

__device__ __forceinline__ void hits_join(Hits& h, int* labels, int& root, uint32_t* info) {
  for (int t = 0; ballot(t < h.n); ++t) {
    if (t < h.n) {
      const int j = h.col[64 * t];
      if (!known_same_set(labels, j, root)) root = uf_union(labels, root, j, info);
    }
  }
  h.n = 0;
}

// Cells and pairs this small are tested by the lane that reached them (all lanes at
// once) instead of by the wavefront one lane after another.
constexpr int kLaneScan = 16;    // points of a dense cell against one point
constexpr int kLanePairs = 128;  // pairs of two dense cells

// Number of points of the cell [s, s+c) within eps of q (this lane alone).
template <int D>
__device__ __forceinline__ int lane_count_near(const float* __restrict__ xs, int64_t n, int s, int c, const Query& q,
                                               float eps2) {
  int found = 0;
  for (int j = 0; j < c; j += 4) {
    float v[4][3];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t k = s + min(j + u, c - 1);
      v[u][0] = xs[k];
      v[u][1] = xs[n + k];
      v[u][2] = D == 3 ? xs[2 * n + k] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (j + u < c && dist2v<D>(v[u][0], v[u][1], v[u][2], q.x, q.y, q.z) <= eps2) ++found;
  }
  return found;
}

// Is some pair of a point of cell [sa, sa+na) and one of [sb, sb+nb), whose tight box
// is [blo, bhi], within eps? (this lane alone)
template <int D>
__device__ __forceinline__ bool lane_cells_touch(const float* __restrict__ xs, int64_t n, int sa, int na, int sb,
                                                 int nb, float4 blo, float4 bhi, float eps2) {
  int hits = 0;
  for (int j = 0; j < na && hits == 0; ++j) {
    const Query q = load_point<D>(xs, n, sa + j);
    if (box_dist2<D>(q.x, q.y, q.z, blo.x, blo.y, blo.z, bhi.x, bhi.y, bhi.z) <= eps2)
      hits = cell_within<D>(blo, bhi, q, eps2) ? 1 : lane_count_near<D>(xs, n, sb, nb, q, eps2);
  }
  return hits != 0;
}

// Core pass for points outside dense cells, one lane per point primitive p (called by
// every thread of the workgroup).
template <int D, bool B, bool G>
__device__ __forceinline__ void core_query(const TravArgs& a, int m, int p, int64_t first, char* s_dyn, int* s_w) {
  const int lane = lane_id();
  bool mine;
  int i;
  Query q;
  own_record(a, p, m, mine, i, q);  // dense cells are core by construction
  const Scope sc = scope_of<B>(a, m, i);
  int cnt = 0;
  NbRec rec;
  rec_init(rec, reinterpret_cast<int*>(s_dyn + size_t(kSearchLds<D, G>) * (blockDim.x >> 6)));
  const float qv[3] = {q.x, q.y, q.z};
  Walker<D, B, false, G, true> w;
  w.init(a, m, sc, i, qv, qv, 0, mine, search_lds<D, G>(s_dyn));
  bool active = mine && !w.done();
  while (ballot(active)) {
    int pend = -1, pcnt = 0;  // a dense cell to scan: its first point and its size
    if (active) {
      const int r = w.step(a, m, q, sc.eps2, 0);
      if (r >= 0) {
        const float4 lr = a.prim_lo[r];
        const int s = rec_index(lr);
        if (s >= 0) {
          if (rec_point_near<D>(lr, q, sc.eps2)) {
            ++cnt;
            if (s != i) rec_add(rec, s);
          }
        } else {
          const float4 hr = a.prim_hi[r];
          if (box_dist2<D>(q.x, q.y, q.z, lr.x, lr.y, lr.z, hr.x, hr.y, hr.z) <= sc.eps2) {
            const int np = __float_as_int(hr.w);
            if (cell_within<D>(lr, hr, q, sc.eps2)) {  // counted whole, no scan
              cnt += np;
              rec_add(rec, s);  // s == cell_ref(first point)
            } else if (G && np <= kLaneScan) {
              const int found = lane_count_near<D>(a.xs, a.n, ref_point(s), np, q, sc.eps2);
              cnt += found;
              if (found) rec_add(rec, s);
            } else {  // both from the records already loaded: the scan starts with the points
              pend = ref_point(s);
              pcnt = np;
            }
          }
        }
      }
    }
    for (uint64_t pm = ballot(pend >= 0); pm; pm &= pm - 1) {
      const int L = __ffsll(static_cast<unsigned long long>(pm)) - 1;
      const int s = __shfl(pend, L);
      const int want = __shfl(sc.min_pts - cnt, L);
      const int found = cell_count_near<D>(a.xs, a.n, s, __shfl(pcnt, L), __shfl(q.x, L), __shfl(q.y, L),
                                           __shfl(q.z, L), readlane_f(sc.eps2, L), want);
      if (lane == L && found > 0) {
        cnt += found;
        rec_add(rec, cell_ref(s));  // a dense cell: all core, one cluster; its first point stands for it
      }
    }
    if (active && (cnt >= sc.min_pts || w.done())) active = false;
  }
  core_epilogue(a, mine, i, p, cnt, sc.min_pts, rec, s_w, first);
}

// (The hierarchy's walks at eight wavefronts a SIMD; seven, which the scalar registers that the
// compiler takes when left alone allow, took 804 us for 734 on 2M points with a far one.)
template <int D, bool B, int W>
__global__ __launch_bounds__(W == kHierarchy ? 1024 : 256, W == kHierarchy ? 8 : 1) void k_core_dbx(TravArgs a) {
  __shared__ int s_w[17];
  extern __shared__ __align__(16) char s_dyn[];  // the walk's columns, then neighbour records
  with_walk<W>(a, [&](auto grid) {
    constexpr bool G = decltype(grid)::value;
    const int m = tree_m(a.t);
    Chunks c(m, G);
    if (blockIdx.x == 0 && threadIdx.x == 0) a.border_n[kWalkShare] = static_cast<int>(c.chunk);
    for (; c.in(); c.next()) core_query<D, B, G>(a, m, c.query(), c.xcd * c.chunk, s_dyn, s_w);
  });
}

// The core points of a cell are within eps of each other (their tight box passes the test, as
// a dense cell's does), so they are one set: with a large minPts cells that are not dense
// hold many, all of which a walk would meet and look up, query by query. Eight lanes a cell.
// Main
// phases of 200,000 evenly spread points, us, walked point by point / with sets (as packets
// through the hierarchy): 3D, minPts 300 of 1500 neighbours 4660 / 1080 (4550), 1000 of 4000
// 10,910 / 2660 (10,730); 1,000 places of 300 equal points in 2D, minPts 2000, 1580 / 720
// (348).
constexpr int kSetWhole = 1 << 30;

template <int D, bool B>
__global__ __launch_bounds__(256) void k_cell_sets(TravArgs a, const int* __restrict__ cell_start,
                                                   const uint8_t* __restrict__ dense, const int* __restrict__ d_cells,
                                                   int* __restrict__ sets) {
  constexpr int G = 8;
  if (!a.ix.plan->grid_on || (B && !a.ix.plan->sets)) return;
  const int ncells = *d_cells;
  const int sub = threadIdx.x & (G - 1);
  for (int64_t c0 = blockIdx.x * int64_t(256 / G); c0 < ncells; c0 += int64_t(gridDim.x) * (256 / G)) {
    const int64_t c = c0 + threadIdx.x / G;
    const int s = c < ncells ? cell_start[c] : 0, e = c < ncells ? cell_start[c + 1] : 0;
    if (e - s < kSetCell || dense[c]) continue;  // (a cell's lanes go together)
    int rep = 0x7fffffff, cnt = 0;
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int i = s + sub; i < e; i += G) {
      if (!a.core[i]) continue;
      rep = min(rep, i);
      ++cnt;
#pragma unroll
      for (int k = 0; k < D; ++k) {
        const float v = a.xs[k * a.n + i];
        lo[k] = fminf(lo[k], v);
        hi[k] = fmaxf(hi[k], v);
      }
    }
#pragma unroll
    for (int off = G / 2; off > 0; off >>= 1) {
      rep = min(rep, __shfl_xor(rep, off));
      cnt += __shfl_xor(cnt, off);
#pragma unroll
      for (int k = 0; k < D; ++k) {
        lo[k] = fminf(lo[k], __shfl_xor(lo[k], off));
        hi[k] = fmaxf(hi[k], __shfl_xor(hi[k], off));
      }
    }
    if (D == 2) lo[2] = hi[2] = 0.0f;
    const float eps2 = B ? a.cloud_eps2[cloud_of(a, s)] : a.eps2;
    const bool one = cnt > 0 && dist2v<D>(hi[0], hi[1], hi[2], lo[0], lo[1], lo[2]) <= eps2;
    if (one)
      for (int i = s + sub; i < e; i += G)
        // (a root hangs under the first core point whether that is a root or not)
        if (i != rep && a.core[i] && cas_agent(a.labels + i, i, rep) != i) uf_union(a.labels, rep, i, a.info);
    if (sub == 0) sets[c] = cnt == 0 ? -2 : one ? rep + (cnt == e - s ? kSetWhole : 0) : -1;
  }
}

// May a core query in the set of root pass over cell c, all of whose core points are in its
// set (or which has none)? First claim: and which has no others to claim.
template <bool FIRST, bool B>
__device__ __forceinline__ bool cell_known(const TravArgs& a, int c, int root) {
  if (!a.cell_sets || (B && !a.ix.plan->sets)) return false;
  const int v = a.cell_sets[c];
  if (v < 0) return !FIRST && v == -2;
  return !(FIRST && v < kSetWhole) && known_same_set(a.labels, v & (kSetWhole - 1), root);
}

// Do the dense cells hold kLargeCell points or more on average (m primitives, nd dense
// cells)? Then packets and brick summaries pay in the point main phase: a query's
// candidates are mostly large cells of few sets, met by its neighbours too.
constexpr int kLargeCell = 16;
__device__ __forceinline__ bool large_cells(const TravArgs& a, int m) {
  const int64_t nd = *a.d_ndense;
  return nd > 0 && a.n - (m - nd) >= kLargeCell * nd;
}

// Main phase, points outside dense cells: pairs with primitives above their own.
// One lane per point primitive; lanes whose point is not a query stay idle.
// (Compacting the few core queries into full wavefronts was slower: their
// wavefront-wide cell scans then run on too few wavefronts to fill the chip.)
// Canonical labels: when a wavefront's core queries lie in a box at most
// kPointsPacketExt eps wide (and, in a batch, in one cloud), they walk as one
// packet: one lane-parallel wide walk over the box reaches every primitive above
// the smallest query within eps of any query; each candidate is broadcast and
// every lane keeps the pairs above its own primitive, so the unions are those of
// the per-lane walks. Queries around a dense clump otherwise each walk most of
// the clump's subtree one node per step.
constexpr float kPointsPacketExt = 8.0f;
constexpr int kPointsFewQueries = 32;   // at most this many queries ...
constexpr float kPointsFewExt = 32.0f;  // ... form a packet up to this many eps wide

template <int D, bool ALL_CORE, bool FIRST, bool B, bool G>
__device__ __forceinline__ void points_query(const TravArgs& a, int m, int p, char* s_dyn) {
  // G: the walk's columns; else packet walks, kWideStack entries per wavefront
  uint32_t* s_pstack = reinterpret_cast<uint32_t*>(s_dyn);
  constexpr int kWaveLds = kSearchLds<D, G> + (G ? kHitBytes : 0);
  char* lds = s_dyn + (threadIdx.x >> 6) * kWaveLds;
  const int lane = lane_id();
  bool pt;
  int i;
  Query q;
  own_record(a, p, m, pt, i, q);
  const bool ci = pt && (ALL_CORE || a.core[i]);
  const bool mine = pt && (ci || (FIRST && !is_lone(a, i)));
  const Scope sc = scope_of<B>(a, m, i);
  int* labels = a.labels;
  // the core pass may already have joined i to dense cells it reaches
  int root = mine && ci ? uf_find(labels, i, a.info) : i;
  // A packet of queries (lanes mm, in the box [lo, hi]): their own pairs, then the
  // candidates that walk() brings, above the first of them. Point primitives up to
  // plast are the packet's own.
  auto packet = [&](uint64_t mm, const float* lo, const float* hi, float eps2, int plast, auto&& walk) {
    const bool on = (mm >> lane) & 1;
    const int fl = __ffsll(static_cast<unsigned long long>(mm)) - 1;
    // Phase A: pairs of this wavefront's own queries (every core point primitive
    // in its range is a query), each joined from its lower primitive.
    for (uint64_t km = mm; km; km &= km - 1) {
      const int kl = __ffsll(static_cast<unsigned long long>(km)) - 1;
      const int jk = __shfl(i, kl);
      const float px = readlane_f(q.x, kl), py = readlane_f(q.y, kl), pz = readlane_f(q.z, kl);
      if (on && lane < kl && dist2v<D>(px, py, pz, q.x, q.y, q.z) <= eps2 && !known_same_set(labels, jk, root))
        root = uf_union(labels, root, jk, a.info);
    }
    if (on) root = uf_find(labels, root, a.info);
    int r = __shfl(root, fl);
    bool common = !ballot(on && root != r);
    walk([&](int rr) {
      float4 lr = make_float4(0.0f, 0.0f, 0.0f, 0.0f), hr = lr;
      bool hit = false;
      int anc = -1;
      if (rr >= 0) {
        lr = a.prim_lo[rr];
        const int v = rec_index(lr);
        if (v >= 0) {
          hit = rr > plast && (ALL_CORE || a.core[v]) &&
                box_dist2<D>(lr.x, lr.y, lr.z, lo[0], lo[1], lo[2], hi[0], hi[1], hi[2]) <= eps2;
        } else {
          hr = a.prim_hi[rr];
          hit = boxbox_dist2<D>(lo, hi, lr.x, lr.y, lr.z, hr.x, hr.y, hr.z) <= eps2;
        }
        if (hit) anc = ancestor_compress(labels, ref_point(v));
      }
      const bool is_pt = rec_index(lr) >= 0;
      if (common) {
        // Points, all at once: every lane tests its own candidate against all
        // queries (register broadcasts), then the lanes that reach one join
        // the packet's set in parallel.
        const bool cand = hit && is_pt && anc != r;
        if (ballot(cand)) {
          bool reach = false;
          for (uint64_t qm = mm; qm; qm &= qm - 1) {
            const int kl = __ffsll(static_cast<unsigned long long>(qm)) - 1;
            reach |= cand && dist2v<D>(lr.x, lr.y, lr.z, readlane_f(q.x, kl), readlane_f(q.y, kl),
                                       readlane_f(q.z, kl)) <= eps2;
          }
          if (ballot(reach)) {
            if (reach && !known_same_set(labels, rec_index(lr), r)) uf_union(labels, r, rec_index(lr), a.info);
            int nr = 0;
            if (lane == fl) nr = uf_find(labels, r, a.info);
            r = __shfl(nr, fl);
            if (on) root = r;
          }
        }
      }
      // cells, and points when the queries are in several sets: one at a time
      for (uint64_t vm = ballot(hit && !(common && (is_pt || anc == r))); vm; vm &= vm - 1) {
        const int k = __ffsll(static_cast<unsigned long long>(vm)) - 1;
        const int rk = __builtin_amdgcn_readlane(rr, k);
        const int v = __builtin_amdgcn_readlane(rec_index(lr), k);
        const int j = ref_point(v);
        const int ak = __builtin_amdgcn_readlane(anc, k);
        const float px = readlane_f(lr.x, k), py = readlane_f(lr.y, k), pz = readlane_f(lr.z, k);
        if (common && ak == r) continue;  // joined by an earlier candidate of this walk
        if (v >= 0) {  // a core point above every query of the wavefront (queries in several sets)
          if (on && ak != root && dist2v<D>(px, py, pz, q.x, q.y, q.z) <= eps2 && !known_same_set(labels, j, root))
            root = uf_union(labels, root, j, a.info);
          continue;
        }
        // a dense cell: one of its points within eps of a query suffices
        const float ux = readlane_f(hr.x, k), uy = readlane_f(hr.y, k), uz = readlane_f(hr.z, k);
        const int nk = __builtin_amdgcn_readlane(__float_as_int(hr.w), k);  // the cell's size
        const bool nb = on && rk > p && (common || ak != root) &&
                        box_dist2<D>(q.x, q.y, q.z, px, py, pz, ux, uy, uz) <= eps2 &&
                        (common || !known_same_set(labels, j, root));
        if (common && ballot(nb) && known_same_set(labels, j, r)) continue;
        // a query whose eps-ball holds the whole cell reaches it without a scan
        const bool full = nb && cell_within<D>(make_float4(px, py, pz, 0.0f), make_float4(ux, uy, uz, 0.0f), q, eps2);
        if (common) {
          const uint64_t fm = ballot(full);
          if (fm) {
            const int L = __ffsll(static_cast<unsigned long long>(fm)) - 1;
            int nr = 0;
            if (lane == L) nr = uf_union(labels, r, j, a.info);
            r = __shfl(nr, L);
            if (on) root = r;
            continue;  // the whole packet is in one set with the cell now
          }
        } else if (full) {
          root = uf_union(labels, root, j, a.info);
        }
        if (G && nk <= kLaneScan) {
          const bool reach = nb && !full && lane_count_near<D>(a.xs, a.n, j, nk, q, eps2) > 0;
          const uint64_t rm = ballot(reach);
          if (common && rm) {
            const int L = __ffsll(static_cast<unsigned long long>(rm)) - 1;
            int nr = 0;
            if (lane == L) nr = uf_union(labels, r, j, a.info);
            r = __shfl(nr, L);
            if (on) root = r;
          } else if (reach) {
            root = uf_union(labels, root, j, a.info);
          }
          continue;
        }
        for (uint64_t lm = ballot(nb && !full); lm; lm &= lm - 1) {
          const int L = __ffsll(static_cast<unsigned long long>(lm)) - 1;
          const bool reach = cell_reaches_point<D>(a.xs, a.n, j, nk, readlane_f(q.x, L),
                                                   readlane_f(q.y, L), readlane_f(q.z, L), eps2);
          if (common) {
            if (!reach) continue;
            int nr = 0;
            if (lane == L) nr = uf_union(labels, r, j, a.info);
            r = __shfl(nr, L);
            if (on) root = r;
            break;  // the whole packet is in one set with the cell now
          }
          if (lane == L && reach) root = uf_union(labels, root, j, a.info);
        }
      }
      return false;
    }, [&](int c) { return common && cell_known<FIRST, B>(a, c, r); });
  };
  const uint64_t mm = ballot(mine);
  if (!mm) return;
  const float qv[3] = {q.x, q.y, q.z};
  bool single = mine;
  if (!FIRST && G && large_cells(a, m)) {
    single = (for_packets<D, B>(a.ix, B ? cloud_of(a, i) : 0, qv, qv, mm,
                                [&](uint64_t lanes, const CellGrid& g, const CellBox<D>& box, const float* lo,
                                    const float* hi) {
                                  const int fl = __ffsll(static_cast<unsigned long long>(lanes)) - 1;
                                  const int ll = 63 - __clzll(static_cast<unsigned long long>(lanes));
                                  const int pmin = __builtin_amdgcn_readlane(p, fl);
                                  packet(lanes, lo, hi, readlane_f(sc.eps2, fl), __builtin_amdgcn_readlane(p, ll),
                                         [&](auto&& visit, auto&& pass) {
                                           box_candidates<D>(a.ix, g, box, pmin, reinterpret_cast<int*>(lds), visit,
                                                             pass);
                                         });
                                }) >> lane) & 1;
  } else if constexpr (!FIRST && !G) {
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    if (mine) {
      lo[0] = hi[0] = q.x;
      lo[1] = hi[1] = q.y;
      lo[2] = hi[2] = q.z;
    }
#pragma unroll
    for (int d = 0; d < 3; ++d)
      for (int off = 32; off > 0; off >>= 1) {
        lo[d] = fminf(lo[d], __shfl_xor(lo[d], off));
        hi[d] = fmaxf(hi[d], __shfl_xor(hi[d], off));
      }
    const int fl = __ffsll(static_cast<unsigned long long>(mm)) - 1;
    const int i0 = __shfl(i, fl), pmin = __shfl(p, fl);  // primitives rise with the lanes
    const Scope ps = scope_of<B>(a, m, i0);
    const bool other_cloud = B && mine && cloud_of(a, i) != cloud_of(a, i0);
    float ext = fmaxf(hi[0] - lo[0], hi[1] - lo[1]);
    if (D == 3) ext = fmaxf(ext, hi[2] - lo[2]);
    // a few queries spread wider still walk as one packet: their per-lane walks
    // would each cross the clumps in between on their own
    const float ext_max = __popcll(mm) <= kPointsFewQueries ? kPointsFewExt : kPointsPacketExt;
    if (!ballot(other_cloud) && ext * ext <= ext_max * ext_max * ps.eps2) {
      uint32_t* stack = s_pstack + (threadIdx.x >> 6) * kWideStack;
      packet(mm, lo, hi, ps.eps2, __shfl(p, 63), [&](auto&& visit, auto&&) {
        traverse_box_wide_lanes<D>(a.t, m, ps, lo, hi, pmin, a.t.leaf_size, a.info, stack, visit);
      });
      return;
    }
  }
  Walker<D, B, true, G> w;
  w.init(a, m, sc, i, qv, qv, p, single, lds);
  Hits hits;
  hits_init(hits, lds + kSearchLds<D, G>);
  bool active = single && !w.done();
  while (ballot(active)) {
    int pend = -1, pcnt = 0;  // a dense cell to scan: its first point and its size
    if (active) {
      const int r = w.step(a, m, q, sc.eps2, p, [&](int c) { return ci && cell_known<FIRST, B>(a, c, root); });
      if (r >= 0) {
        const float4 lr = a.prim_lo[r];
        const int s = rec_index(lr);
        if (s >= 0) {
          if (rec_point_near<D>(lr, q, sc.eps2)) {
            const bool cj = ALL_CORE || a.core[s];
            if (ci && cj) {
              if (G) {
                if (labels[s] != root) hits_add(hits, s);
              } else if (!known_same_set(labels, s, root)) {
                root = uf_union(labels, root, s, a.info);
              }
            } else if (FIRST && ci) {
              uf_claim(labels, s, i);
            } else if (FIRST && cj) {
              uf_claim(labels, i, s);
              active = false;  // i is a member now (by this or an earlier claim)
            }
          }
        } else {
          const float4 hr = a.prim_hi[r];
          if (box_dist2<D>(q.x, q.y, q.z, lr.x, lr.y, lr.z, hr.x, hr.y, hr.z) <= sc.eps2 &&
              !(ci && known_same_set(labels, ref_point(s), root))) {
            pend = ref_point(s);
            pcnt = __float_as_int(hr.w);
            if (G && (pcnt <= kLaneScan || cell_within<D>(lr, hr, q, sc.eps2))) {
              if (cell_within<D>(lr, hr, q, sc.eps2) ||
                  lane_count_near<D>(a.xs, a.n, pend, pcnt, q, sc.eps2) > 0) {
                if (ci) {
                  hits_add(hits, pend);
                } else if (FIRST) {
                  uf_claim(labels, i, pend);
                  active = false;
                }
              }
              pend = -1;
            }
          }
        }
      }
    }
    // a dense cell: one of its points within eps suffices
    for (uint64_t pm = ballot(pend >= 0); pm; pm &= pm - 1) {
      const int L = __ffsll(static_cast<unsigned long long>(pm)) - 1;
      const int s = __shfl(pend, L);
      const bool hit = cell_reaches_point<D>(a.xs, a.n, s, __shfl(pcnt, L), __shfl(q.x, L), __shfl(q.y, L),
                                             __shfl(q.z, L), readlane_f(sc.eps2, L));
      if (lane == L && hit) {
        if (ci) {
          root = uf_union(labels, root, s, a.info);
        } else if (FIRST) {
          uf_claim(labels, i, s);
          active = false;
        }
      }
    }
    if (G && hits_full(hits)) hits_join(hits, labels, root, a.info);
    if (active && w.done()) active = false;
  }
  if (G) hits_join(hits, labels, root, a.info);
}

// (In 2D the grid's walks fit six wavefronts a SIMD with 80 registers; 81, which the compiler
// takes when left alone, cost 1% of 1M points.)
template <int D, bool ALL_CORE, bool FIRST, bool B, int W>
__global__ __launch_bounds__(W == kHierarchy ? 1024 : 256, D == 2 && W == kGrid && !B ? 6 : 1) void k_main_dbx_points(
    TravArgs a) {
  extern __shared__ __align__(16) char s_dyn[];
  with_walk<W>(a, [&](auto grid) {
    constexpr bool G = decltype(grid)::value;
    const int m = tree_m(a.t);
    for (Chunks c(m, G); c.in(); c.next()) points_query<D, ALL_CORE, FIRST, B, G>(a, m, c.query(), s_dyn);
  });
}

// Main phase, dense cells, when they are few (see cells_lane_mode):
// one wavefront per cell A walks the tree once with A's box,
// over primitives above A; a dense neighbour B joins A's set if some pair is
// within eps, a core point if some point of A reaches it, and (first-claim
// mode) a non-core point is claimed the same way. Many cells go to
// k_main_dbx_cells_lane instead (the two kernels are launched together and each
// leaves the other's case alone).
constexpr int kCellsPerWaveMax = 65536;

// More than 65,536 dense cells (8 per wavefront of the 8192 below) go to the
// lane-per-cell kernel: measured faster there, for small cells (a batch of 4,096
// clouds: 13 vs 62 ms) and for large ones (a batch of 50 clouds of up to 2M
// points: 3 vs 8 ms); with fewer cells a wavefront per cell keeps more
// wavefronts busy (8M-point set, 20k cells: 0.3 vs 0.96 ms). Both kernels read
// the count.
__device__ __forceinline__ bool cells_lane_mode(const TravArgs& a) { return *a.d_ndense > kCellsPerWaveMax; }

// The whole wavefront hands the primitives above A in the cells within reach of A's
// box to visit_lanes, a primitive per lane (-1: none). The lanes first look up a
// brick each, then take the cells of a brick by its bits, lane = code, and list those
// within reach in LDS (at most 5^D).
constexpr int kCellList = 128;

template <int D, typename F>
__device__ __forceinline__ void cells_near_box_lanes(const CellIndex& ix, const CellGrid& g, const float* lo,
                                                     const float* hi, int A, int* list, F&& visit_lanes) {
  if (g.ncell[0] <= 0) return;
  const int lane = lane_id();
  CellRange<D> cr;
  cell_range<D>(cr, g, lo, hi);
  int br[3] = {0, 0, 0};
  bool use = range_brick<D>(cr, lane, br) && lane < kMaxBricks<D>;
  const uint32_t code = child_code<D>(br);
  uint4 e = make_uint4(0, 0, 0, 0);
  if (use) e = ix.supers[super_index<D>(g, br)];
  const uint64_t sw = word_of(e);
  use = use && ((sw >> code) & 1);
  const int b = static_cast<int>(e.z) + __popcll(sw & ((1ull << code) - 1));
  bool own = use;
#pragma unroll
  for (int a = 0; a < D; ++a) own = own && br[a] == (cr.own[a] >> kLevelShift<D>);
  const uint64_t om = ballot(own);
  const int b_own = om ? __shfl(b, __ffsll(static_cast<unsigned long long>(om)) - 1) : -1;
  e = make_uint4(0, 0, 0, 0);
  if (use && b >= b_own) e = ix.bricks[b];
  const uint64_t mask = word_of(e) & range_codes<D, true>(cr, br);
  int cnt = 0;
  for (uint64_t bm = ballot(mask != 0); bm; bm &= bm - 1) {
    const int n = __ffsll(static_cast<unsigned long long>(bm)) - 1;
    const uint64_t wn = uint64_t(static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(e.y), n))) << 32 |
                        static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(e.x), n));
    const uint64_t mn = uint64_t(static_cast<uint32_t>(
                            __builtin_amdgcn_readlane(static_cast<int>(mask >> 32), n))) << 32 |
                        static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(mask), n));
    const int base = __builtin_amdgcn_readlane(static_cast<int>(e.z), n);
    int bn[3];
    range_brick<D>(cr, n, bn);
    const bool in = ((mn >> lane) & 1) && cell_in_reach<D>(cr, bn, static_cast<uint32_t>(lane));
    const uint64_t im = ballot(in);
    if (in) list[cnt + __popcll(im & lanemask_lt())] = base + __popcll(wn & lanemask_lt());
    cnt += __popcll(im);
  }
  for (int q = 0; q < cnt; q += 64) {
    int cur = 0, end = 0;
    bool dense;
    if (q + lane < cnt) cell_prims(ix, list[q + lane], cur, end, dense);
    visit_ranges(max(cur, A + 1), end, visit_lanes);
  }
}

template <int D, bool ALL_CORE, bool FIRST, bool B, bool G>
__device__ __forceinline__ void cells_wave(const TravArgs& a, int nd, uint32_t* stack) {
  const int m = tree_m(a.t);
  const int lane = lane_id();
  const int wave = (xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x) >> 6;
  const int nwaves = (gridDim.x * blockDim.x) >> 6;
  int* labels = a.labels;
  // wavefront w takes a contiguous slice of the dense-cell list (filled in
  // roughly increasing key order), so neighbouring cells share an XCD's L2
  const int per = (nd + nwaves - 1) / nwaves;
  const int dbeg = wave * per, dend = min(nd, dbeg + per);
  for (int w = dbeg; w < dend; ++w) {
    const int A = a.dense_list[w];
    const int sa = a.prim_start[A], na = -a.prim_cnt[A];
    const Scope sc = scope_of<B>(a, m, sa);
    const float eps2 = sc.eps2;
    const float4 alo4 = a.prim_lo[A], ahi4 = a.prim_hi[A];
    const float alo[3] = {alo4.x, alo4.y, alo4.z}, ahi[3] = {ahi4.x, ahi4.y, ahi4.z};
    // the core pass may already have joined A to other sets
    int root = uf_find(labels, sa, a.info);
    auto visit = [&](int r) {
      // every lane loads its primitive's record and what decides a skip (core
      // flag, an ancestor near the root); candidates then go one after another
      float4 lr = make_float4(0.0f, 0.0f, 0.0f, 0.0f), hr = lr;
      bool hit = false, cj = false;
      int anc = -1;
      if (r >= 0) {
        lr = a.prim_lo[r];
        const int v = rec_index(lr);
        if (v >= 0) {
          hit = box_dist2<D>(lr.x, lr.y, lr.z, alo[0], alo[1], alo[2], ahi[0], ahi[1], ahi[2]) <= eps2;
        } else {
          hr = a.prim_hi[r];
          hit = boxbox_dist2<D>(alo, ahi, lr.x, lr.y, lr.z, hr.x, hr.y, hr.z) <= eps2;
        }
        if (hit) {
          const int j = ref_point(v);
          cj = v < 0 || ALL_CORE || a.core[j];  // dense cells are core
          anc = cj ? ancestor_compress(labels, j) : labels[j];
        }
      }
      for (uint64_t vm = ballot(hit && !(cj && anc == root)); vm; vm &= vm - 1) {
        const int k = __ffsll(static_cast<unsigned long long>(vm)) - 1;
        const int v = __builtin_amdgcn_readlane(rec_index(lr), k);
        const int j = ref_point(v);
        const int ak = __builtin_amdgcn_readlane(anc, k);
        const float px = readlane_f(lr.x, k), py = readlane_f(lr.y, k), pz = readlane_f(lr.z, k);
        if (v >= 0) {
          if (__builtin_amdgcn_readlane(static_cast<int>(cj), k)) {
            if (ak == root || known_same_set(labels, j, root)) continue;
            if (cell_reaches_point<D>(a.xs, a.n, sa, na, px, py, pz, eps2)) {
              int nr = 0;
              if (lane == 0) nr = uf_union(labels, root, j, a.info);
              root = __shfl(nr, 0);
            }
          } else if (FIRST) {
            if (ak != j || labels[j] != j) continue;  // claimed already (claims are final)
            if (cell_reaches_point<D>(a.xs, a.n, sa, na, px, py, pz, eps2) && lane == 0) uf_claim(labels, j, sa);
          }
          continue;
        }
        if (ak == root || known_same_set(labels, j, root)) continue;
        const float4 blo = make_float4(px, py, pz, 0.0f);
        const float4 bhi = make_float4(readlane_f(hr.x, k), readlane_f(hr.y, k), readlane_f(hr.z, k), 0.0f);
        if (cells_touch<D>(a.xs, a.n, sa, na, j, -a.prim_cnt[__builtin_amdgcn_readlane(r, k)], blo, bhi, eps2)) {
          int nr = 0;
          if (lane == 0) nr = uf_union(labels, root, j, a.info);
          root = __shfl(nr, 0);
        }
      }
      return false;
    };
    if constexpr (G)
      cells_near_box_lanes<D>(a.ix, query_grid<D, B>(a.ix, B ? cloud_of(a, sa) : 0), alo, ahi, A,
                              reinterpret_cast<int*>(stack), visit);
    else
      traverse_box_wide_lanes<D>(a.t, m, sc, alo, ahi, A, a.t.leaf_size, a.info, stack, visit);
  }
}

template <int D, bool ALL_CORE, bool FIRST, bool B, int W>
__global__ __launch_bounds__(256) void k_main_dbx_cells_wave(TravArgs a) {
  constexpr int kPerWave = W == kGrid ? kCellList : kWideStack;
  static_assert(kPerWave >= kCellList, "a list of cells fits");
  __shared__ uint32_t s_stack[4 * kPerWave];  // 256-thread workgroups
  if (cells_lane_mode(a)) return;
  with_walk<W>(a, [&](auto grid) {
    cells_wave<D, ALL_CORE, FIRST, B, decltype(grid)::value>(a, *a.d_ndense, s_stack + (threadIdx.x >> 6) * kPerWave);
  });
}

// Main phase, dense cells, when they are many (e.g. a batch of many clouds;
// see cells_lane_mode): one lane per dense cell A, walking (in
// lock-step with the other lanes of its wavefront) with A's box over the
// primitives above A, with the same rules as above; each pair test runs on the
// whole wavefront (64 points per ballot), one pending lane after another.
template <int D, bool ALL_CORE, bool FIRST, bool B, bool G>
__device__ __forceinline__ void cells_query(const TravArgs& a, int m, int nd, int k, char* s_dyn) {
  const int lane = lane_id();
  const bool mine = k >= 0 && k < nd;
  const int A = mine ? a.dense_list[k] : 0;
  const float4 alo = mine ? a.prim_lo[A] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  const float4 ahi = mine ? a.prim_hi[A] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  const int sa = mine ? ref_point(rec_index(alo)) : 0;
  const int na = mine ? __float_as_int(ahi.w) : 0;
  const Scope sc = scope_of<B>(a, m, sa);
  BoxQ qa;
  qa.lo[0] = alo.x; qa.lo[1] = alo.y; qa.lo[2] = alo.z;
  qa.hi[0] = ahi.x; qa.hi[1] = ahi.y; qa.hi[2] = ahi.z;
  int* labels = a.labels;
  int root = sa;
  Walker<D, B, true, G> w;
  w.init(a, m, sc, sa, qa.lo, qa.hi, A, mine, search_lds<D, G>(s_dyn));
  bool active = mine && !w.done();
  while (ballot(active)) {
    int pend = -1;
    if (active) {
      const int r = w.step(a, m, qa, sc.eps2, A);
      if (r >= 0) {
        const float4 lr = a.prim_lo[r];
        const int s = ref_point(rec_index(lr));
        bool hit = false;  // settled by this lane alone
        if (rec_index(lr) >= 0) {
          const float px = lr.x, py = lr.y, pz = lr.z;
          if (box_dist2<D>(px, py, pz, qa.lo[0], qa.lo[1], qa.lo[2], qa.hi[0], qa.hi[1], qa.hi[2]) <= sc.eps2) {
            if (ALL_CORE || a.core[s]) {
              if (!known_same_set(labels, s, root)) pend = r;
            } else if (FIRST && labels[s] == s) {
              pend = r;
            }
          }
          if (G && pend >= 0 && na <= kLaneScan) {
            hit = lane_count_near<D>(a.xs, a.n, sa, na, Query{px, py, pz}, sc.eps2) > 0;
            pend = -1;
          }
          if (hit && !(ALL_CORE || a.core[s])) {
            uf_claim(labels, s, sa);  // first-claim mode: a non-core neighbour joins A's cluster
            hit = false;
          }
        } else {
          const float4 blo = lr, bhi = a.prim_hi[r];
          if (boxbox_dist2<D>(qa.lo, qa.hi, blo.x, blo.y, blo.z, bhi.x, bhi.y, bhi.z) <= sc.eps2 &&
              !known_same_set(labels, s, root))
            pend = r;
          const int nb = __float_as_int(bhi.w);
          if (G && pend >= 0 && int64_t(na) * nb <= kLanePairs) {
            hit = lane_cells_touch<D>(a.xs, a.n, sa, na, s, nb, blo, bhi, sc.eps2);
            pend = -1;
          }
        }
        if (hit) root = uf_union(labels, root, s, a.info);
      }
    }
    for (uint64_t pm = ballot(pend >= 0); pm; pm &= pm - 1) {
      const int L = __ffsll(static_cast<unsigned long long>(pm)) - 1;
      const int r = __shfl(pend, L);
      const int sA = __shfl(sa, L), nA = __shfl(na, L);
      const float e2 = readlane_f(sc.eps2, L);
      const int c = a.prim_cnt[r], s = a.prim_start[r];
      bool hit;
      if (c > 0) {
        const float px = a.xs[s], py = a.xs[a.n + s], pz = D == 3 ? a.xs[2 * a.n + s] : 0.0f;
        hit = cell_reaches_point<D>(a.xs, a.n, sA, nA, px, py, pz, e2);
      } else {
        hit = cells_touch<D>(a.xs, a.n, sA, nA, s, -c, a.prim_lo[r], a.prim_hi[r], e2);
      }
      if (lane == L && hit) {
        if (c > 0 && !(ALL_CORE || a.core[s]))
          uf_claim(labels, s, sA);  // first-claim mode: a non-core neighbour joins A's cluster
        else
          root = uf_union(labels, root, s, a.info);
      }
    }
    if (active && w.done()) active = false;
  }
}

template <int D, bool ALL_CORE, bool FIRST, bool B, int W>
__global__ __launch_bounds__(W == kHierarchy ? 1024 : 256) void k_main_dbx_cells_lane(TravArgs a) {
  extern __shared__ __align__(16) char s_dyn[];  // the walk's columns
  const int nd = *a.d_ndense;
  if (!cells_lane_mode(a)) return;
  with_walk<W>(a, [&](auto grid) {
    constexpr bool G = decltype(grid)::value;
    const int m = tree_m(a.t);
    for (Chunks c(nd, G); c.in(); c.next()) cells_query<D, ALL_CORE, FIRST, B, G>(a, m, nd, c.query(), s_dyn);
  });
}

// Canonical border pass for non-core points (all outside dense cells).
// Queries: the listed non-core points whose neighbours were not all recorded
// by the core pass (which wrote -1 for lone points; the records cover the rest).
template <int D, bool B, bool G>
__device__ __forceinline__ void border_query(const TravArgs& a, int m, bool mine, int p, char* s_dyn) {
  const int lane = lane_id();
  const float4 own = mine ? a.prim_lo[p] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  const int i = mine ? rec_index(own) : 0;
  const Scope sc = scope_of<B>(a, m, i);
  const Query q{own.x, own.y, own.z};
  int best = 0x7fffffff;
  const float qv[3] = {q.x, q.y, q.z};
  Walker<D, B, false, G> w;
  w.init(a, m, sc, i, qv, qv, 0, mine, search_lds<D, G>(s_dyn));
  bool active = mine && !w.done();
  while (ballot(active)) {
    int pend = -1;
    if (active) {
      const int r = w.step(a, m, q, sc.eps2, 0);
      if (r >= 0) {
        const float4 lr = a.prim_lo[r];
        const int s = rec_index(lr);
        if (s >= 0) {
          if (rec_point_near<D>(lr, q, sc.eps2) && a.core[s]) {
            const int id = a.cid[a.labels[s]];
            best = id < best ? id : best;
          }
        } else if (cell_box_near<D>(a, r, lr, q, sc.eps2) && a.cid[a.labels[ref_point(s)]] < best) {
          pend = r;
        }
      }
    }
    for (uint64_t pm = ballot(pend >= 0); pm; pm &= pm - 1) {
      const int L = __ffsll(static_cast<unsigned long long>(pm)) - 1;
      const int r = __shfl(pend, L);
      const int s = a.prim_start[r];
      const bool hit = cell_reaches_point<D>(a.xs, a.n, s, -a.prim_cnt[r], __shfl(q.x, L), __shfl(q.y, L),
                                             __shfl(q.z, L), readlane_f(sc.eps2, L));
      if (lane == L && hit) {
        const int id = a.cid[a.labels[s]];
        best = id < best ? id : best;
      }
    }
    if (active && (best == 0 || w.done())) active = false;
  }
  if (mine) a.border[i] = best == 0x7fffffff ? -1 : best;
}

template <int D, bool B, int W>
__global__ __launch_bounds__(W == kHierarchy ? 1024 : 256) void k_border_dbx(TravArgs a) {
  extern __shared__ __align__(16) char s_dyn[];  // the walk's columns
  with_walk<W>(a, [&](auto grid) {
    const int m = tree_m(a.t);
    const int xcd = static_cast<int>(blockIdx.x % kNumXcd), nq = a.border_n[kWalkCount(xcd)];
    const int* list = a.qborder + int64_t(xcd) * a.border_n[kWalkShare];
    for (int64_t k0 = int64_t(blockIdx.x / kNumXcd) * blockDim.x; k0 < nq;
         k0 += int64_t(gridDim.x / kNumXcd) * blockDim.x) {
      const int64_t k = k0 + threadIdx.x;
      const bool mine = k < nq;
      if (ballot(mine)) border_query<D, B, decltype(grid)::value>(a, m, mine, mine ? list[k] : 0, s_dyn);
    }
  });
}

// Test hook: one lane walks the tree with an always-true box test and records,
// in order, the leaves a walk masked at `mask` reaches (mask = -1: unmasked).
__global__ void k_debug_walk(TreeView t, int m, int mask, int* out_leaves, int* out_count, int cap,
                             uint32_t* info) {
  if (blockIdx.x != 0 || threadIdx.x != 0) return;
  const Query q{0.0f, 0.0f, 0.0f};
  const Scope sc{m == 1 ? kLeaf : 0u, m - 1, INFINITY, 0};
  int cnt = 0;
  auto visit = [&](int s, int e) {
    for (int l = s; l <= e; ++l, ++cnt)
      if (cnt < cap) out_leaves[cnt] = l;
    return false;
  };
  if (mask < 0) traverse<3, false>(t, m, sc, q, 0, info, visit);
  else traverse<3, true>(t, m, sc, q, mask, info, visit);
  *out_count = cnt;
}

// Kernels indexed with xcd_spread(): every XCD needs ceil(ceil(n/8)/block)
// workgroups of its own, so the grid is 8 times that.
inline dim3 grid_of(int64_t n, int block) {
  return dim3(static_cast<unsigned>(kNumXcd * ceil_div(ceil_div(n, kNumXcd), block)));
}

// Threads per workgroup of the grid walks: the caller's block_size up to the 256
// that their LDS columns are sized for.
inline int grid_block(const TravArgs& a) { return a.block < 256 ? a.block : 256; }
// Workgroups of a DenseBox kernel of up to n queries (see Chunks), in a multiple of
// kNumXcd; fewer lanes a wavefront make more of them.
inline dim3 query_grid_blocks(int64_t n, int block) {
  constexpr int64_t kMost = 16384;
  const int64_t need = std::max<int64_t>(grid_of(n, block).x, grid_of(std::min<int64_t>(n, kWaves * 64), block / 8).x);
  return dim3(static_cast<unsigned>(std::min<int64_t>(need, kMost)));
}
// Do the DenseBox kernels of this call hold both walks (see Walks)?
template <bool B>
constexpr bool one_kernel(const TravArgs& a) { return !B && a.n <= kEitherMax; }
template <int D>
size_t walk_lds(int block, int more = 0) {  // LDS of a workgroup's searches, and `more` bytes a wavefront
  return size_t(kSearchLds<D, true> + more) * (block / 64);
}

template <int D, bool B>
void core_t(const TravArgs& a, bool densebox, hipStream_t s) {
  const size_t rec = sizeof(int) * kRecNb;  // neighbour records, per thread
  const dim3 g = grid_of(a.n, a.block), b(a.block);
  if (densebox) {
    const int gb = grid_block(a);
    const dim3 gg = query_grid_blocks(a.n, gb);
    const size_t lds = walk_lds<D>(gb) + rec * gb;
    if (one_kernel<B>(a)) {
      hipLaunchKernelGGL((k_core_dbx<D, B, kEither>), gg, dim3(gb), lds, s, a);
    } else {
      hipLaunchKernelGGL((k_core_dbx<D, B, kGrid>), gg, dim3(gb), lds, s, a);
      hipLaunchKernelGGL((k_core_dbx<D, B, kHierarchy>), query_grid_blocks(a.n, a.block), b, rec * a.block, s, a);
    }
  } else {
    hipLaunchKernelGGL((k_core_fdb<D, B>), g, b, rec * a.block, s, a);
  }
}

// part: 0 = everything, 1 = dense-cell queries only, 2 = point queries only (DenseBox)
template <int D, bool ALL, bool FIRST, bool B>
void main_t(const TravArgs& a, bool densebox, int part, hipStream_t s) {
  const dim3 g = grid_of(a.n, a.block), b(a.block);
  const int gb = grid_block(a);
  if (densebox) {
    if (part != 2) {
      // dense cells hold >= minPts points each, so there are at most n / minPts
      const int64_t max_cells = a.min_pts > 1 ? a.n / a.min_pts + 1 : a.n;
      // a batch's many cells usually go to the lane kernel, where this one exits at once
      const dim3 gw(static_cast<unsigned>(std::min<int64_t>(kNumXcd * ceil_div(max_cells, kNumXcd * 4), B ? 2048 : 4096)));
      if (one_kernel<B>(a)) {
        hipLaunchKernelGGL((k_main_dbx_cells_wave<D, ALL, FIRST, B, kEither>), gw, dim3(256), 0, s, a);
      } else {
        hipLaunchKernelGGL((k_main_dbx_cells_wave<D, ALL, FIRST, B, kGrid>), gw, dim3(256), 0, s, a);
        hipLaunchKernelGGL((k_main_dbx_cells_wave<D, ALL, FIRST, B, kHierarchy>), gw, dim3(256), 0, s, a);
      }
      if (max_cells > kCellsPerWaveMax) {
        const dim3 gg = query_grid_blocks(max_cells, gb);
        if (one_kernel<B>(a)) {
          hipLaunchKernelGGL((k_main_dbx_cells_lane<D, ALL, FIRST, B, kEither>), gg, dim3(gb), walk_lds<D>(gb), s, a);
        } else {
          hipLaunchKernelGGL((k_main_dbx_cells_lane<D, ALL, FIRST, B, kGrid>), gg, dim3(gb), walk_lds<D>(gb), s, a);
          hipLaunchKernelGGL((k_main_dbx_cells_lane<D, ALL, FIRST, B, kHierarchy>), query_grid_blocks(max_cells, a.block),
                             b, 0, s, a);
        }
      }
    }
    if (part != 1) {
      const dim3 gg = query_grid_blocks(a.n, gb);
      const size_t lds = walk_lds<D>(gb, kHitBytes), wide = sizeof(uint32_t) * kWideStack;
      if (one_kernel<B>(a)) {
        hipLaunchKernelGGL((k_main_dbx_points<D, ALL, FIRST, B, kEither>), gg, dim3(gb), std::max(lds, wide * (gb / 64)),
                           s, a);
      } else {
        hipLaunchKernelGGL((k_main_dbx_points<D, ALL, FIRST, B, kGrid>), gg, dim3(gb), lds, s, a);
        hipLaunchKernelGGL((k_main_dbx_points<D, ALL, FIRST, B, kHierarchy>), query_grid_blocks(a.n, a.block), b,
                           wide * (a.block / 64), s, a);
      }
    }
  } else if (FIRST) {
    hipLaunchKernelGGL((k_main_fdb_first<D, B>), g, b, 0, s, a);
  } else {
    hipLaunchKernelGGL((k_main_fdb<D, ALL, B>), g, b, 0, s, a);
  }
}

template <int D, bool B>
void border_t(const TravArgs& a, bool densebox, hipStream_t s) {
  const dim3 g = grid_of(a.n, a.block), b(a.block);
  hipLaunchKernelGGL(k_border_rec, dim3(static_cast<unsigned>(kNumXcd * ceil_div(a.brec_cap, 256))), dim3(256), 0, s, a);
  if (densebox) {
    const int gb = grid_block(a);
    const dim3 gg = query_grid_blocks(a.n, gb);
    if (one_kernel<B>(a)) {
      hipLaunchKernelGGL((k_border_dbx<D, B, kEither>), gg, dim3(gb), walk_lds<D>(gb), s, a);
    } else {
      hipLaunchKernelGGL((k_border_dbx<D, B, kGrid>), gg, dim3(gb), walk_lds<D>(gb), s, a);
      hipLaunchKernelGGL((k_border_dbx<D, B, kHierarchy>), query_grid_blocks(a.n, a.block), b, 0, s, a);
    }
  } else hipLaunchKernelGGL((k_border_fdb<D, B>), g, b, 0, s, a);
}

template <int D>
void main_dispatch(const TravArgs& a, bool densebox, bool all_core, bool first_border, int part, hipStream_t s) {
  if (a.pkeys != nullptr) {  // batches always run the core pass
    if (first_border) main_t<D, false, true, true>(a, densebox, part, s);
    else main_t<D, false, false, true>(a, densebox, part, s);
  } else if (all_core) {
    main_t<D, true, false, false>(a, densebox, part, s);
  } else if (first_border) {
    main_t<D, false, true, false>(a, densebox, part, s);
  } else {
    main_t<D, false, false, false>(a, densebox, part, s);
  }
}

}  // namespace

void launch_core(const TravArgs& a, int dim, bool densebox, hipStream_t s) {
  if (a.n <= 0) return;
  const bool B = a.pkeys != nullptr;
  if (dim == 3) {
    if (B) core_t<3, true>(a, densebox, s);
    else core_t<3, false>(a, densebox, s);
  } else {
    if (B) core_t<2, true>(a, densebox, s);
    else core_t<2, false>(a, densebox, s);
  }
}

void launch_cell_sets(TravArgs& a, int dim, const int* cell_start, const uint8_t* cell_dense, const int* d_cells,
                      int* sets, hipStream_t s) {
  a.cell_sets = nullptr;
  const bool B = a.pkeys != nullptr;
  if (a.n < kSetCell || (!B && a.min_pts <= kSetMinPts)) return;
  const dim3 g(static_cast<unsigned>(std::min<int64_t>(4096, ceil_div(a.n, 256 / 8)))), b(256);
  if (dim == 3) {
    if (B) hipLaunchKernelGGL((k_cell_sets<3, true>), g, b, 0, s, a, cell_start, cell_dense, d_cells, sets);
    else hipLaunchKernelGGL((k_cell_sets<3, false>), g, b, 0, s, a, cell_start, cell_dense, d_cells, sets);
  } else {
    if (B) hipLaunchKernelGGL((k_cell_sets<2, true>), g, b, 0, s, a, cell_start, cell_dense, d_cells, sets);
    else hipLaunchKernelGGL((k_cell_sets<2, false>), g, b, 0, s, a, cell_start, cell_dense, d_cells, sets);
  }
  a.cell_sets = sets;
}

void launch_main(const TravArgs& a, int dim, bool densebox, bool all_core, bool first_border, int part,
                 hipStream_t s) {
  if (a.n <= 0) return;
  if (dim == 3) main_dispatch<3>(a, densebox, all_core, first_border, part, s);
  else main_dispatch<2>(a, densebox, all_core, first_border, part, s);
}

void launch_cliques(const TravArgs& a, int dim, hipStream_t s) {
  if (a.n <= 1) return;
  const dim3 g(static_cast<unsigned>(ceil_div(a.n - 1, 256 * kCliqueItems))), b(256);
  if (dim == 3) {
    if (a.pkeys) hipLaunchKernelGGL((k_cliques<3, true>), g, b, 0, s, a);
    else hipLaunchKernelGGL((k_cliques<3, false>), g, b, 0, s, a);
  } else {
    if (a.pkeys) hipLaunchKernelGGL((k_cliques<2, true>), g, b, 0, s, a);
    else hipLaunchKernelGGL((k_cliques<2, false>), g, b, 0, s, a);
  }
}

template <int D>
static void main_cliques_t(const TravArgs& a, bool all_core, hipStream_t s) {
  // a wavefront per clique of kCliqueWave points or more, up to what is resident at once
  const dim3 g(static_cast<unsigned>(std::min<int64_t>(2048, kNumXcd * ceil_div(a.n, kNumXcd * 4 * kCliqueWave)))), b(256);
  if (a.pkeys) hipLaunchKernelGGL((k_main_cliques<D, false, true>), g, b, 0, s, a);
  else if (all_core) hipLaunchKernelGGL((k_main_cliques<D, true, false>), g, b, 0, s, a);
  else hipLaunchKernelGGL((k_main_cliques<D, false, false>), g, b, 0, s, a);
}

void launch_core_boxes(const TravArgs& a, hipStream_t s) {
  if (a.n < kCliqueMin || (!a.pkeys && a.min_pts <= kCliqueMin)) return;  // every box is a clique
  const dim3 g(static_cast<unsigned>(std::min<int64_t>(2048, ceil_div(a.n, 32 * kCliqueMin)))), b(256);
  hipLaunchKernelGGL(k_core_boxes, g, b, 0, s, a);
}

void launch_main_cliques(const TravArgs& a, int dim, bool all_core, hipStream_t s) {
  if (a.n < kCliqueMin) return;
  if (dim == 3) main_cliques_t<3>(a, all_core, s);
  else main_cliques_t<2>(a, all_core, s);
}

void launch_debug_walk(const TreeView& t, int m, int mask, int* out_leaves, int* out_count, int cap,
                       uint32_t* info, hipStream_t s) {
  hipLaunchKernelGGL(k_debug_walk, dim3(1), dim3(64), 0, s, t, m, mask, out_leaves, out_count, cap, info);
}

void launch_border(const TravArgs& a, int dim, bool densebox, hipStream_t s) {
  if (a.n <= 0) return;
  const bool B = a.pkeys != nullptr;
  if (dim == 3) {
    if (B) border_t<3, true>(a, densebox, s);
    else border_t<3, false>(a, densebox, s);
  } else {
    if (B) border_t<2, true>(a, densebox, s);
    else border_t<2, false>(a, densebox, s);
  }
}

}  // namespace fdb
