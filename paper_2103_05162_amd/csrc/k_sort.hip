// LSD radix sort of (key, index) pairs, 8-bit digits, stable. Section 4.1 sorts
// queries and primitives along a space-filling curve; Karras' hierarchy needs
// the keys sorted with equal keys left in index order, which a stable LSD sort
// started from the identity permutation gives.
//
// Design (after Merrill & Adinets' "onesweep"): the key kernels count the digits of
// every pass at once; then in each pass a workgroup ranks a tile (5632 32-bit
// or 6144 64-bit keys) with wavefront ballots and scatters it through LDS, so that
// writes are contiguous per digit. A tile learns its global offsets in one of two
// ways. Look-back: a decoupled look-back over earlier tiles (four status words per
// round trip), tiles numbered in the order workgroups start (an atomic ticket), so
// a tile only waits on tiles already running. Reduce-then-scan (the 32-bit passes
// of the sort planned on the device): a count kernel stores every tile's digit
// counts and a scan turns them into offsets before the pass, which then waits on
// nothing. With ~770 tiles in flight at once on 256 CUs, the look-back's walks over
// earlier tiles' uncached status words cost more than the count kernel's extra
// read of the keys (per-tile clocks: ~10 of a tile's ~24 us went to the look-back).
// Small inputs, where launches cost the most, run all passes in one (k_sort_all).
#include "fdb_device.hpp"
#include "fdb_internal.hpp"

namespace fdb {

namespace {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;
constexpr int kRadix = 256;

// Look-back status word: [epoch:30][flag:2][count:32]. flag 1 = this tile's own
// count, flag 2 = inclusive prefix through this tile. epoch = pass + 1 tells a
// word of this pass from one left by an earlier pass.
constexpr uint64_t kFlagAgg = 1, kFlagIncl = 2;
__device__ __forceinline__ uint64_t pack_status(uint32_t epoch, uint64_t flag, uint32_t count) {
  return (uint64_t(epoch) << 34) | (flag << 32) | count;
}

template <typename K>
__device__ __forceinline__ uint32_t digit_of(K key, int shift) {
  return static_cast<uint32_t>(key >> shift) & 0xffu;
}

// Passes of a host-sequenced sort that need not run, as a bit mask: a pass whose digit
// is the same for every key is the identity permutation. Left out two at a time, so the
// number of passes run keeps its parity and the result ends where the host expects it.
// Called by a whole workgroup (kBlock threads).
__device__ __forceinline__ uint32_t skipped_passes(const uint32_t* hist, int64_t n, int passes) {
  uint32_t constant = 0, skip = 0;
  for (int p = 0; p < passes; ++p)
    constant |= __syncthreads_or(hist[p * kRadix + threadIdx.x] == static_cast<uint32_t>(n)) ? 1u << p : 0u;
  for (int p = 0; p + 1 < passes; ++p)
    if ((constant >> p & 3u) == 3u) skip |= 3u << p++;
  return skip;
}

// Pass plan of a host-sequenced sort (one workgroup), passes[p]: bit 1 = skip, bit 0 =
// source buffer.
__global__ __launch_bounds__(kBlock) void k_pass_plan(const uint32_t* __restrict__ hist, int64_t n, int passes,
                                                      uint32_t* __restrict__ pass_plan) {
  const uint32_t skip = skipped_passes(hist, n, passes);
  if (threadIdx.x) return;
  uint32_t cur = 0;
  for (int p = 0; p < passes; ++p) {
    const uint32_t left_out = skip >> p & 1u;
    pass_plan[p] = left_out << 1 | cur;
    if (!left_out) cur ^= 1u;
  }
}

// Block-wide exclusive scan of one value per thread (kBlock threads).
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* s_wsum) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    uint32_t y = __shfl_up(x, off);
    if (lane >= off) x += y;
  }
  if (lane == 63) s_wsum[w] = x;
  __syncthreads();
  uint32_t add = 0;
  for (int j = 0; j < w; ++j) add += s_wsum[j];
  __syncthreads();
  return x - v + add;
}

// Does pass p run, and which buffer does it read (`from`; it writes the other)?
// With a plan (a DenseBox grid sized on the device), the pass runs only if the
// plan's key width is K's and p is below its pass count, and `from` follows the
// plan's start buffer. Without one, the pass plan of k_pass_plan decides: a pass
// whose digit is the same for every key is the identity permutation and is
// skipped (in pairs, so the result still ends in the buffer the host expects).
template <typename K>
__device__ __forceinline__ bool pass_source(int p, const GridPlan* plan, const uint32_t* pass_plan, int& from) {
  if (plan) {
    if (plan->key64 != (sizeof(K) == 8 ? 1 : 0) || p >= plan->passes) return false;
    from = (plan->start ^ p) & 1;
    return true;
  }
  const uint32_t f = pass_plan[p];
  if (f & 2u) return false;
  from = static_cast<int>(f & 1u);
  return true;
}

// Reduce step of a pass without look-back: every digit's count in every tile,
// digit-major (counts[d * tiles + tile]) for the scan. Tiles are the pass's.
template <typename K>
__global__ __launch_bounds__(kBlock) void k_tile_counts(const K* __restrict__ k0, const K* __restrict__ k1,
                                                        int64_t n, int p, const GridPlan* __restrict__ plan,
                                                        uint32_t* __restrict__ counts, int64_t tiles) {
  int from = 0;
  if (!pass_source<K>(p, plan, nullptr, from)) return;  // the whole grid leaves
  const K* __restrict__ kin = from ? k1 : k0;
  constexpr int kItems = sort_items<K>();
  constexpr int kTile = 256 * kItems;
  __shared__ uint32_t s_h[kRadix];
  const int tid = threadIdx.x;
  s_h[tid] = 0;
  __syncthreads();
  const int tile = xcd_block(blockIdx.x, gridDim.x);  // the pass's mapping: it re-reads these keys from L2
  const int64_t base = int64_t(tile) * kTile;
  const int shift = 8 * p;
  K key[kItems];
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    const int64_t pos = base + k * kBlock + tid;
    key[k] = pos < n ? kin[pos] : K(0);
  }
  // counts only (no ranks): one LDS atomic per wavefront when its lanes share the
  // digit, else one per lane; the ranking pass's eight-ballot digit match made
  // this kernel VALU-bound (24 us a pass on 8M keys)
#pragma unroll
  for (int k = 0; k < kItems; ++k) hist_add(static_cast<K>(key[k] >> shift), base + k * kBlock + tid < n, 1, s_h);
  __syncthreads();
  counts[int64_t(tid) * tiles + tile] = s_h[tid];
}

// Scan step: for digit d (workgroup d), the digit's global offset (from the pass'
// digit counts) plus the running sum of its counts in earlier tiles, in place: where each tile's keys of
// digit d start in the output.
template <typename K>
__global__ __launch_bounds__(kBlock) void k_tile_scan(uint32_t* __restrict__ counts, int64_t tiles, int p,
                                                      const GridPlan* __restrict__ plan,
                                                      const uint32_t* __restrict__ hist) {
  int from = 0;
  if (!pass_source<K>(p, plan, nullptr, from)) return;
  constexpr int kPer = 8;
  __shared__ uint32_t s_wsum[kWaves];
  __shared__ uint32_t s_tot;
  const int d = blockIdx.x, tid = threadIdx.x;
  uint32_t* __restrict__ c = counts + int64_t(d) * tiles;
  // where digit d starts: the keys of smaller digits
  const uint32_t ex = block_exclusive_scan(hist[p * kRadix + tid], s_wsum);
  if (tid == d) s_tot = ex;
  __syncthreads();
  uint32_t run = s_tot;
  __syncthreads();
  for (int64_t c0 = 0; c0 < tiles; c0 += kBlock * kPer) {
    uint32_t v[kPer];
    uint32_t sum = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int64_t i = c0 + int64_t(tid) * kPer + k;
      v[k] = i < tiles ? c[i] : 0u;
      sum += v[k];
    }
    const uint32_t ex = block_exclusive_scan(sum, s_wsum);
    if (tid == kBlock - 1) s_tot = ex + sum;
    uint32_t r = run + ex;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int64_t i = c0 + int64_t(tid) * kPer + k;
      if (i < tiles) c[i] = r;
      r += v[k];
    }
    __syncthreads();
    run += s_tot;
    __syncthreads();
  }
}

template <typename K, int ITEMS>
struct SortLds {
  uint32_t tile;
  uint32_t wcnt[kWaves][kRadix];  // per-wave digit counts, then per-wave prefixes
  uint32_t dstart[kRadix];        // tile-local start of each digit
  uint32_t gbase[kRadix];         // global start of this tile's run of each digit
  uint32_t wsum[kWaves];
  K keys[256 * ITEMS];
  uint32_t vals[256 * ITEMS];
};

// The tiles of one pass that this workgroup takes, from (kin, vin) to (kout, vout).
// OFFS: one tile, which follows from the workgroup's index, its offsets coming from
// k_tile_scan (offs). Otherwise tiles by ticket until none is left, so the grid is what
// is resident at once rather than a workgroup per tile, with the look-back; digit0 is
// where digit threadIdx.x starts. iota: the values are the identity permutation (the
// planned sort's first pass: the key kernel writes none). Returns the tiles taken.
template <typename K, int ITEMS, bool OFFS>
__device__ __forceinline__ int sort_pass(SortLds<K, ITEMS>& s, const K* kin, const uint32_t* vin, K* kout,
                                         uint32_t* vout, int64_t n, int p, bool iota, uint32_t digit0,
                                         uint32_t* tilectr, uint64_t* status, const uint32_t* offs, int64_t otiles,
                                         uint32_t* info) {
  const int shift = 8 * p;
  const uint32_t epoch = static_cast<uint32_t>(p + 1);
  constexpr int kItems = ITEMS;
  constexpr int kTile = 256 * kItems;
  constexpr int kWaveTile = 64 * kItems;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int64_t ntiles = (n + kTile - 1) / kTile;
  for (int taken = 0;; ++taken) {
    if (!OFFS && tid == 0) s.tile = atomicAdd(tilectr, 1u);
    for (int i = tid; i < kWaves * kRadix; i += kBlock) (&s.wcnt[0][0])[i] = 0;
    __syncthreads();
    // OFFS: tiles laid contiguously per XCD (as in k_tile_counts), so the partial
    // output lines where one tile's run of a digit meets the next tile's are
    // completed in one L2 instead of being written to memory from two
    const int64_t tile = OFFS ? int64_t(xcd_block(blockIdx.x, gridDim.x)) : int64_t(s.tile);
    if (tile >= ntiles) return taken;  // uniform: s.tile is shared
    const int64_t wbase = tile * kTile + int64_t(w) * kWaveTile;

    K key[kItems];
    uint32_t val[kItems];
    uint32_t rank[kItems];
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      int64_t pos = wbase + k * 64 + lane;
      bool valid = pos < n;
      key[k] = valid ? kin[pos] : K(0);
      val[k] = valid ? (iota ? static_cast<uint32_t>(pos) : vin[pos]) : 0u;
    }
    // Rank within the wavefront: positions run wave-major, then item, then lane,
    // so processing items in order keeps the sort stable. Items past the end (small
    // inputs) are left out, for the whole wavefront alike.
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      rank[k] = 0;
      if (wbase + k * 64 >= n) continue;
      bool valid = wbase + k * 64 + lane < n;
      uint32_t d = digit_of(key[k], shift);
      uint64_t m = match_digit(d, valid);
      int leader = __ffsll(static_cast<unsigned long long>(m)) - 1;
      uint32_t before = 0;
      if (valid && lane == leader) {  // leaders of distinct digits touch distinct words
        before = s.wcnt[w][d];
        s.wcnt[w][d] = before + static_cast<uint32_t>(__popcll(m));
      }
      before = __shfl(before, leader < 0 ? 0 : leader);
      rank[k] = before + static_cast<uint32_t>(__popcll(m & lanemask_lt()));
    }
    __syncthreads();

    // Thread d: prefix over wavefronts and tile total of digit d.
    const uint32_t d = tid;
    uint32_t total = 0;
#pragma unroll
    for (int j = 0; j < kWaves; ++j) {
      uint32_t c = s.wcnt[j][d];
      s.wcnt[j][d] = total;
      total += c;
    }
    // Thread d: its tile's global start for digit d.
    if constexpr (OFFS) {
      s.gbase[d] = offs[int64_t(d) * otiles + tile];
    } else {
      uint64_t* st = status + tile * kRadix + d;
      uint32_t excl = 0;
      if (tile == 0) {
        st_agent64(st, pack_status(epoch, kFlagIncl, total));
      } else {
        st_agent64(st, pack_status(epoch, kFlagAgg, total));
        int spins = 0;
        for (int64_t j = tile - 1; j >= 0;) {
          // four predecessors per round trip (16: slower, every word read comes from memory)
          uint64_t v[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) v[u] = j - u >= 0 ? ld_agent64(status + (j - u) * kRadix + d) : 0;
          bool done = false, wait = false;
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if (done || wait || j < 0) continue;
            if (static_cast<uint32_t>(v[u] >> 34) != epoch) {
              wait = true;
              continue;
            }
            excl += static_cast<uint32_t>(v[u]);
            if (((v[u] >> 32) & 3u) == kFlagIncl) done = true;
            else --j;
          }
          if (done) break;
          if (wait) {
            if (++spins > (1 << 24)) {
              atomicOr(info, kInternalBit);
              break;
            }
            __builtin_amdgcn_s_sleep(1);
          }
        }
        st_agent64(st, pack_status(epoch, kFlagIncl, excl + total));
      }
      s.gbase[d] = digit0 + excl;
    }
    uint32_t ds = block_exclusive_scan(total, s.wsum);
    s.dstart[d] = ds;
    __syncthreads();

    // Local scatter into LDS in sorted order.
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      if (wbase + k * 64 + lane < n) {
        uint32_t dk = digit_of(key[k], shift);
        uint32_t pos = s.dstart[dk] + s.wcnt[w][dk] + rank[k];
        s.keys[pos] = key[k];
        s.vals[pos] = val[k];
      }
    }
    __syncthreads();
    const int64_t tile_n = n - tile * kTile < kTile ? n - tile * kTile : kTile;
    for (int i = tid; i < tile_n; i += kBlock) {
      K kk = s.keys[i];
      uint32_t dk = digit_of(kk, shift);
      uint32_t dest = s.gbase[dk] + (i - s.dstart[dk]);
      if (dest >= n) {  // only after a failed look-back
        atomicOr(info, kInternalBit);
        continue;
      }
      kout[dest] = kk;
      vout[dest] = s.vals[i];
    }
    if (OFFS) return 1;
    __syncthreads();  // the next tile reuses the LDS
  }
}

// One pass per launch (see sort_pass): the passes whose tile offsets are scanned
// beforehand, and the look-back passes of large inputs. Digit offsets come from the
// histograms.
template <typename K, bool OFFS>
__global__ __launch_bounds__(kBlock) void k_onesweep(K* __restrict__ k0, K* __restrict__ k1,
                                                     uint32_t* __restrict__ v0, uint32_t* __restrict__ v1, int64_t n,
                                                     int p, const GridPlan* __restrict__ plan,
                                                     const uint32_t* __restrict__ pass_plan,
                                                     const uint32_t* __restrict__ hist,
                                                     uint32_t* __restrict__ tilectr_all, uint64_t* __restrict__ status,
                                                     const uint32_t* __restrict__ offs, int64_t otiles,
                                                     uint32_t* __restrict__ info) {
  __shared__ SortLds<K, sort_items<K>()> s;
  int from = 0;
  if (!pass_source<K>(p, plan, pass_plan, from)) return;  // the whole grid leaves
  const uint32_t digit0 = OFFS ? 0u : block_exclusive_scan(hist[p * kRadix + threadIdx.x], s.wsum);
  sort_pass<K, sort_items<K>(), OFFS>(s, from ? k1 : k0, from ? v1 : v0, from ? k0 : k1, from ? v0 : v1, n, p,
                                      plan && p == 0, digit0, tilectr_all + p, status, offs, otiles, info);
}

// Every look-back pass in one launch. A workgroup that finds no tile left of a pass
// publishes what it wrote, counts its tiles as done, waits until all of the pass' are,
// and takes tiles of the next. It only ever waits for tiles that workgroups already
// running have taken, so no workgroup need be resident for another's sake. Digit
// offsets come straight from the histograms, passes over constant digits are skipped
// in pairs (as k_pass_plan has it). With a plan: nothing for the other key width.
// done: a counter per pass, zero beforehand.
template <typename K, int ITEMS>
__device__ __forceinline__ void sort_all(SortLds<K, ITEMS>& s, K* k0, K* k1, uint32_t* v0, uint32_t* v1, int64_t n,
                                         int passes, const GridPlan* plan, const uint32_t* hist, uint32_t* tilectr,
                                         uint32_t* done, uint64_t* status, uint32_t* info) {
  int cur = 0;
  if (plan) {
    passes = plan->passes;
    cur = plan->start;
  }
  const int64_t ntiles = (n + 256 * ITEMS - 1) / (256 * ITEMS);
  const uint32_t skip = plan ? 0u : skipped_passes(hist, n, passes);
  int last = -1;  // the pass before, which has to be complete
  for (int p = 0; p < passes; ++p) {
    if (skip >> p & 1u) continue;
    if (last >= 0) {
      if (threadIdx.x == 0) {
        int spins = 0;
        while (__hip_atomic_load(done + last, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <
               static_cast<uint32_t>(ntiles)) {
          if (++spins > (1 << 24)) {
            atomicOr(info, kInternalBit);
            break;
          }
          __builtin_amdgcn_s_sleep(1);
        }
      }
      __syncthreads();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    const uint32_t digit0 = block_exclusive_scan(hist[p * kRadix + threadIdx.x], s.wsum);
    const int taken = sort_pass<K, ITEMS, false>(s, cur ? k1 : k0, cur ? v1 : v0, cur ? k0 : k1, cur ? v0 : v1, n, p,
                                          plan && p == 0, digit0, tilectr + p, status, nullptr, 0, info);
    if (taken) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      __syncthreads();
      if (threadIdx.x == 0) atomicAdd(done + p, static_cast<uint32_t>(taken));
    }
    cur ^= 1;
    last = p;
  }
}

template <typename K, int ITEMS>
__global__ __launch_bounds__(kBlock) void k_sort_all(K* k0, K* k1, uint32_t* v0, uint32_t* v1, int64_t n, int passes,
                                                     const GridPlan* __restrict__ plan, const uint32_t* hist,
                                                     uint32_t* tilectr, uint32_t* done, uint64_t* status,
                                                     uint32_t* info) {
  __shared__ SortLds<K, ITEMS> s;
  if (plan && plan->key64 != (sizeof(K) == 8 ? 1 : 0)) return;  // the whole grid leaves
  sort_all<K, ITEMS>(s, k0, k1, v0, v1, n, passes, plan, hist, tilectr, done, status, info);
}

// Both key widths of a planned sort in one launch.
template <int ITEMS>
__global__ __launch_bounds__(kBlock) void k_sort_all_planned(void* k0, void* k1, uint32_t* v0, uint32_t* v1, int64_t n,
                                                             const GridPlan* __restrict__ plan, const uint32_t* hist,
                                                             uint32_t* tilectr, uint32_t* done, uint64_t* status,
                                                             uint32_t* info) {
  __shared__ alignas(16) unsigned char lds[sizeof(SortLds<uint64_t, ITEMS>)];
  if (plan->key64)
    sort_all<uint64_t, ITEMS>(*reinterpret_cast<SortLds<uint64_t, ITEMS>*>(lds), static_cast<uint64_t*>(k0),
                              static_cast<uint64_t*>(k1), v0, v1, n, 8, plan, hist, tilectr, done, status, info);
  else
    sort_all<uint32_t, ITEMS>(*reinterpret_cast<SortLds<uint32_t, ITEMS>*>(lds), static_cast<uint32_t*>(k0),
                              static_cast<uint32_t*>(k1), v0, v1, n, 4, plan, hist, tilectr, done, status, info);
}

// Workgroups of a look-back pass: at most what is resident at once on 256 CUs
// (two 64-bit or three 32-bit tiles per CU, bound by registers); they loop over
// the tiles.
template <typename K>
unsigned lookback_grid(int64_t tiles) {
  const int64_t cap = (sizeof(K) == 8 ? 2 : 3) * 256;
  return static_cast<unsigned>(tiles < cap ? tiles : cap);
}

// Which sort a number of keys takes: all passes in one launch, or passes of their own.
// One launch saves what a launch costs (4 to 5 us, three launches a pass with 32-bit
// keys, and as many again of the other width), but its passes are separated by
// release and acquire fences of every workgroup, which empty the XCD's L2 under those
// still running. From the end of the key kernel to the permute, one launch / passes of
// their own, us: planned, 32-bit keys, 131,072: 54 / 206; 524,288: 100 / 231; 1M: 161
// (kernel) / 144; planned, 64-bit keys, 524,288: 127 / 264; 1M: 393 / 290; 4M: 876 /
// 350. Eight 64-bit passes (Morton) 131,072: 172 / 178; 262,144: 195 / 200; 524,288:
// 285 / 226.
constexpr int64_t kSortAllMax = int64_t(1) << 19, kSortAllUnplanned = int64_t(1) << 18;
// Keys per thread of a tile: fewer while they put more CUs to work, until the look-back
// over more tiles costs more (one launch, 32-bit / 64-bit keys, us, with 4, 8 and 22 keys
// per thread: 16,384 keys 18/78, 22/90, 33/137; 32,768: 23/100, 23/98, 34/143; 65,536:
// 29/154, 27/115, 37/152; 131,072: 81/259, 56/170, 59/167).
constexpr int64_t kSort4Max = int64_t(1) << 15, kSort8Max = int64_t(1) << 17;
template <typename K>
int64_t sort_tile(int64_t n) {
  return 256 * (n <= kSort4Max ? 4 : n <= kSort8Max ? 8 : sort_items<K>());
}

template <typename K, int ITEMS>
void launch_sort_all(K* keys0, K* keys1, uint32_t* vals0, uint32_t* vals1, int64_t n, int passes, const GridPlan* plan,
                     const uint32_t* hist, uint32_t* tilectr, uint64_t* status, uint32_t* info, hipStream_t s) {
  hipLaunchKernelGGL((k_sort_all<K, ITEMS>), dim3(lookback_grid<K>(ceil_div(n, 256 * ITEMS))), dim3(kBlock), 0, s,
                     keys0, keys1, vals0, vals1, n, passes, plan, hist, tilectr, tilectr + 8, status, info);
}

template <int ITEMS>
void launch_sort_all_planned(void* keys0, void* keys1, uint32_t* vals0, uint32_t* vals1, int64_t n,
                             const GridPlan* plan, const uint32_t* hist, uint32_t* tilectr, uint64_t* status,
                             uint32_t* info, hipStream_t s) {
  hipLaunchKernelGGL(k_sort_all_planned<ITEMS>, dim3(lookback_grid<uint64_t>(ceil_div(n, 256 * ITEMS))), dim3(kBlock),
                     0, s, keys0, keys1, vals0, vals1, n, plan, hist, tilectr, tilectr + 8, status, info);
}

}  // namespace

int radix_sort(uint64_t* keys0, uint64_t* keys1, uint32_t* vals0, uint32_t* vals1, int64_t n, int bits,
               const uint32_t* hist, uint32_t* pass_plan, uint32_t* tilectr, uint64_t* status, uint32_t* info,
               hipStream_t s) {
  using K = uint64_t;
  const int passes = (bits + 7) / 8;
  if (n <= 1 || passes == 0) return 0;
  const int64_t tiles = ceil_div(n, 256 * sort_items<K>());
  fill_u32(tilectr, 0, 16, s);
  fill_u32(reinterpret_cast<uint32_t*>(status), 0, sort_status_words(n, true), s);
  if (n <= kSortAllUnplanned) {
    if (n <= kSort4Max)
      launch_sort_all<K, 4>(keys0, keys1, vals0, vals1, n, passes, nullptr, hist, tilectr, status, info, s);
    else if (n <= kSort8Max)
      launch_sort_all<K, 8>(keys0, keys1, vals0, vals1, n, passes, nullptr, hist, tilectr, status, info, s);
    else
      launch_sort_all<K, sort_items<K>()>(keys0, keys1, vals0, vals1, n, passes, nullptr, hist, tilectr, status, info,
                                          s);
    return passes & 1;
  }
  hipLaunchKernelGGL(k_pass_plan, dim3(1), dim3(kBlock), 0, s, hist, n, passes, pass_plan);
  // (look-back passes: for 64-bit keys, a count kernel's second read of the keys
  // and its extra launches cost more than the look-back; measured on the Morton
  // and batch sorts)
  int cur = 0;
  for (int p = 0; p < passes; ++p) {
    hipLaunchKernelGGL((k_onesweep<K, false>), dim3(lookback_grid<K>(tiles)), dim3(kBlock), 0, s, keys0, keys1,
                       vals0, vals1, n, p, static_cast<const GridPlan*>(nullptr), pass_plan, hist, tilectr, status,
                       static_cast<const uint32_t*>(nullptr), int64_t(0), info);
    cur ^= 1;
  }
  return cur;
}

int64_t sort_status_words(int64_t n, bool key64) {
  return ceil_div(n, key64 ? sort_tile<uint64_t>(n) : sort_tile<uint32_t>(n)) * kRadix * 2;
}
// Either width's (the separate 32-bit passes keep their tile counts in the same buffer;
// a call runs one width only).
int64_t planned_status_words(int64_t n) { return sort_status_words(n, false); }

void radix_sort_planned(void* keys0, void* keys1, uint32_t* vals0, uint32_t* vals1, int64_t n, const GridPlan* plan,
                        const uint32_t* hist, uint32_t* tilectr, uint64_t* status, uint32_t* info, hipStream_t s) {
  if (n <= 1) return;  // the key kernel's start buffer already is buffer 1 when there is nothing to sort
  if (n <= kSort4Max) {
    launch_sort_all_planned<4>(keys0, keys1, vals0, vals1, n, plan, hist, tilectr, status, info, s);
    return;
  }
  if (n <= kSort8Max) {
    launch_sort_all_planned<8>(keys0, keys1, vals0, vals1, n, plan, hist, tilectr, status, info, s);
    return;
  }
  uint32_t* k32[2] = {static_cast<uint32_t*>(keys0), static_cast<uint32_t*>(keys1)};
  uint64_t* k64[2] = {static_cast<uint64_t*>(keys0), static_cast<uint64_t*>(keys1)};
  if (n <= kSortAllMax) {
    launch_sort_all<uint32_t, sort_items<uint32_t>()>(k32[0], k32[1], vals0, vals1, n, 4, plan, hist, tilectr, status,
                                                      info, s);
    launch_sort_all<uint64_t, sort_items<uint64_t>()>(k64[0], k64[1], vals0, vals1, n, 8, plan, hist, tilectr, status,
                                                      info, s);
  } else {
    const int64_t tiles64 = ceil_div(n, 256 * sort_items<uint64_t>());
    // 32-bit keys (at most 4 passes): reduce, scan, then the pass, the tile counts
    // in the look-back buffer (tiles * 256 words of its tiles * 512)
    const int64_t tiles = ceil_div(n, 256 * sort_items<uint32_t>());
    uint32_t* counts = reinterpret_cast<uint32_t*>(status);
    for (int p = 0; p < 4; ++p) {
      hipLaunchKernelGGL(k_tile_counts<uint32_t>, dim3(static_cast<unsigned>(tiles)), dim3(kBlock), 0, s, k32[0],
                         k32[1], n, p, plan, counts, tiles);
      hipLaunchKernelGGL(k_tile_scan<uint32_t>, dim3(kRadix), dim3(kBlock), 0, s, counts, tiles, p, plan, hist);
      hipLaunchKernelGGL((k_onesweep<uint32_t, true>), dim3(static_cast<unsigned>(tiles)), dim3(kBlock), 0, s, k32[0],
                         k32[1], vals0, vals1, n, p, plan, static_cast<const uint32_t*>(nullptr), hist, tilectr,
                         status, static_cast<const uint32_t*>(counts), tiles, info);
    }
    for (int p = 0; p < 8; ++p)
      hipLaunchKernelGGL((k_onesweep<uint64_t, false>), dim3(lookback_grid<uint64_t>(tiles64)), dim3(kBlock), 0, s,
                         k64[0], k64[1], vals0, vals1, n, p, plan, static_cast<const uint32_t*>(nullptr), hist, tilectr,
                         status, static_cast<const uint32_t*>(nullptr), int64_t(0), info);
  }
}

}  // namespace fdb
