// The census by triangle listing: the Batagelj-Mrvar sums with the one-list
// third vertices counted from row totals instead of visited.
//
// For every edge {u, v} the sweep of Fig. 5 visits N(u) u N(v). A third vertex
// w adjacent to only one of u, v closes no triangle; over all edges these add
// up to the open wedges, which follow from each vertex's counts of out-, in-
// and mutual neighbours alone (an open wedge is a pair of neighbours of its
// centre, less the pairs that are adjacent, which are the triangles'). Only
// the third vertices adjacent to both are visited, each triangle once: edges
// are directed from the vertex of lower to the one of higher degree (rank 0 =
// highest degree), and for a vertex y the list N+(x) of every x below y is
// streamed against the set N+(y). The merge reads sum_x d(x)^2 list entries
// (3.57e12 at R-MAT scale 24), this reads sum_x d+(x)^2 / 2 (4.2e10). A whole
// call took 1,560 ms there by the merge and takes 42.2 ms; 37.0 and 2.07 ms at
// R-MAT scale 20, 469 and 10.1 ms on the Chung-Lu graph of 2^22 vertices, 566
// and 79 us at R-MAT scale 10, 24.1 and 7.4 ms on a grid of 2^25, 1,470 and 313 ms
// on 300,007 vertices of degree 3,000.
//
// Pipeline (one stream, no host synchronisation inside):
//   k_sw_rows    per row: offset checks, row starts, degree histogram
//   k_sw_rank    rank of each vertex by a counting sort on its degree
//   k_sw_orient  per tile of 2,048 entries: entry checks; each row split in
//                place into N+(x) (ranks and flags) and its in-list (the x
//                below it, ids and flags); per-row flag counts turned into
//                wedge and dyad sums
//   k_sw_cross   the rows that cross tile boundaries
//   k_sw_items   work items of k_sw_hubs and k_sw_mids
//   k_sw_pack    large graphs: places of the N+(x) in 16-bit ranks, the short ones
//   k_sw_sort_*  N+(x) sorted by rank where it is longer than one wavefront
//                (and packed)
//   k_sw_hubs    vertices with long in-lists: a workgroup holds N+(y) as a
//                byte table over the ranks and streams the N+(x)
//   k_sw_mids    in-lists of middling length: a smaller workgroup, 2-bit table
//   k_sw_dense   long N+ past the ranks of that table: one of 524,288 ranks
//   k_sw_rest    all others: up to 16 a wavefront, hash tables in LDS
//   k_sw_small   graphs of up to 16,384 vertices instead of the last three: lists
//                in ids, several rows a wavefront, a table field per id
//   k_sw_finish  classes from sums, 003 = C(n,3) less the rest
// A batch of graphs goes through k_sw_rows, k_sw_orient, k_sw_cross, k_sw_small
// (k_sw_items, k_sw_dense and k_sw_rest where a member is larger) as one disjoint
// union with ids local to each graph, its counters by graph
// (4,096 graphs of 64 to 8,192 vertices, 3e8 edges: 121 -> 16.7 ms a launch; 256
// graphs of up to 1,024, plan, launch and z-scores: 4.3 -> 0.37 ms). The labelled
// census adds k_lab_sums (54.7 -> 3.25 ms at R-MAT scale 20).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "lds_sort.h"
#include "sums.h"
#include "sweep.h"

namespace triad {
namespace {

constexpr int OT = 2048;  // entries of one orientation tile
constexpr int OTHREADS = 256, OPER = OT / OTHREADS, OWORDS = OT / 64;
constexpr int LONG_KEEP = 256;  // rows with long N+ kept in LDS before they are listed
constexpr int TILE_GRAPHS = 8;  // graphs of a batch whose sums a tile keeps in LDS
constexpr int ROWS_THREADS = 1024;  // of the ranking kernels, 4 or 16 rows a thread
constexpr int BUCKETS = 1024;          // degree buckets of the ranking
// Graphs up to here index their tables by vertex id, without ranks and sorts: R-MAT
// of 16,000 vertices 0.107 ms, ranked 0.223; of 9,001 0.095 and 0.205. The tables
// of two rows a wavefront then fill the LDS of four workgroups a CU. (Tables of
// 32,768 ids, two workgroups a CU, would take 30,000 vertices in 0.162 instead of 0.258
// ms, and, used for all, 16,000 in 0.119.)
constexpr int64_t DIRECT_N = 16384;
constexpr int64_t HUB_RANKS = 65536;   // ranks the workgroup tables cover (k_sw_pack: 16 bits)
// two workgroups a CU: six wavefronts a SIMD, four with the labels' counters
constexpr int hub_threads(bool lab) { return lab ? 512 : 768; }
// In-lists from here on: k_sw_hubs (ranks in its table). R-MAT scale 24, scale 20,
// labelled scale 20, ms: 128 42.3, 2.13, 3.42; 256 42.2, 2.12, 3.24; 512 42.3, 2.11, 3.24.
constexpr int64_t HUB_MIN_IN = 256;
constexpr int MID_THREADS = 256;
// In-lists from here on: k_sw_mids. Chung-Lu 2^22, R-MAT scale 20, R-MAT of 30,000
// vertices, ms: 32 10.86, 2.12, 0.257; 48 10.07, 2.06, 0.262; 64 9.73, 2.11, 0.266; 128
// 9.53, 2.13, 0.286. Labelled, scale 20: 24 3.25, 32 3.24, 48 3.31, 64 3.37.
template <bool LAB>
constexpr int64_t MID_MIN_IN = LAB ? 32 : 48;
// In-list entries of one of their work items. R-MAT scale 24, scale 20, ms: 1,024 43.6,
// 2.14; 2,048 42.2, 2.12; 4,096 42.2, 2.13.
constexpr int64_t CHUNK = 2048;
constexpr uint32_t TAB_MAX = 512;      // entries of one hash table
constexpr int TAB_WORDS = 1024;        // its slots
// threads and table of k_sw_dense's workgroups: one a CU, or four (batches of smaller members)
constexpr int DENSE_THREADS = 1024, DENSE_WORDS = 32768, DENSE_LOW = 8192;
constexpr int64_t DENSE_MIN_IN = 256;  // in-lists of a batch from here on, where it saves no pass
constexpr int REST_WAVES = 4;
constexpr int64_t PACK_MIN = 6 << 20;   // entries from which N+ lists are packed for k_sw_hubs
constexpr int64_t LIST_PAD = 4;        // list words read past a list's end
constexpr uint32_t SORT_MIN = 64, SORT_MID = 256, SORT_MAX = 4096;

// List words: id or rank in the low 30 bits, the direction flag in the top two.
// Labelled (LAB): the flag is seen from the lower id of the pair, bit 29 says
// which vertex that is, and ids take 29 bits.
template <bool LAB>
constexpr uint32_t IDM = LAB ? 0x1FFFFFFFu : 0x3FFFFFFFu;
constexpr uint32_t SLOT_FREE = 0xFFFFFFFFu;  // no id is 2^30 - 1
// Row words: first entry << 24 | length of N+; the top bit of the length marks
// a list that is not in rank order.
constexpr uint32_t LEN_MASK = 0x7FFFFFu, UNSORTED = 0x800000u;

__device__ __forceinline__ uint32_t rl(uint32_t x, int lane) {
  return (uint32_t)__builtin_amdgcn_readlane((int)x, lane);
}
__device__ __forceinline__ uint64_t rl64(uint64_t x, int lane) {
  return ((uint64_t)rl((uint32_t)(x >> 32), lane) << 32) | rl((uint32_t)x, lane);
}
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}
__device__ __forceinline__ uint64_t sum64(uint64_t x) {
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// Atomics on one cache line run one after another (88 ns each, measured with
// 9,216 of them): the counters are kept in SW_COPIES copies, summed at the end.
template <bool LAB>
__device__ __forceinline__ unsigned long long* copy_of(unsigned long long* acc) {
  return acc + (blockIdx.x % SW_COPIES) * (LAB ? SW_LAB_WORDS : SW_WORDS);
}

// Bucket of a degree, rising with it: exact below 32, then 32 steps an octave.
__device__ __forceinline__ uint32_t degree_bucket(uint32_t d) {
  if (d < 32) return d;
  const uint32_t e = 31 - (uint32_t)__builtin_clz(d);
  return ((e - 4) << 5) | ((d >> (e - 5)) & 31u);
}

// The start of a stage by the device's 100 MHz clock: an event per stage took
// 43 us of a 115 us call.
__device__ __forceinline__ void stamp(uint64_t* clk, int i) {
  if (clk && blockIdx.x == 0 && threadIdx.x == 0) clk[i] = __builtin_amdgcn_s_memrealtime();
}

// No kernel past k_sw_pack runs on a graph with an error; the symmetry check's
// and k_sw_pack's are in the third word.
__device__ __forceinline__ bool refused(const uint32_t* err) { return (err[0] | err[1] | err[2]) != 0; }

__global__ void k_sw_zero(uint32_t* __restrict__ p, int64_t m, uint64_t* __restrict__ clk) {
  stamp(clk, 0);
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) p[i] = 0;
}

// ------------------------------------------------------------ rows and ranks

struct RowArgs {
  int64_t n, nnz;
  const int64_t* off;
  uint32_t* deg;       // by id: the degree (tables indexed by id), or NULL
  uint32_t* hist;      // degree buckets, highest degree first, or NULL
  uint64_t* info;      // row words, N+ still empty
  uint32_t* list;      // the first word of each row that has one: its id
  uint32_t* mark;      // bit per entry: a row starts here
  uint32_t* tile_row;  // row that holds each tile's first entry
  uint32_t* err;
  // a batch: its graphs, their first rows, and the graph of each row (out)
  int32_t graphs;
  const int64_t* vbase;
  uint32_t* grow;
  // labelled: the entries below the row's own id, for rows that cross tiles
  const int32_t* nbr;
  struct Cross* cross;
};

// Counters of a row that crosses tile boundaries, at the first tile that it
// reaches into: entries placed so far, the neighbour counts (labelled: the
// entries below the row's own id).
struct Cross {
  uint32_t f, b, o, i, m, su, pad[2];
};

// PER rows a thread; PER > 1: with the degree histogram (workgroups of BUCKETS
// threads).
template <int PER>
__global__ void __launch_bounds__(PER > 1 ? ROWS_THREADS : 256) k_sw_rows(RowArgs a) {
  __shared__ uint32_t h[PER > 1 ? BUCKETS : 1];
  if (PER > 1) {
    h[threadIdx.x] = 0;
    __syncthreads();
  }
  const int64_t base = (int64_t)blockIdx.x * (blockDim.x * PER);
  for (int i = 0; i < PER; ++i) {
    const int64_t u = base + i * blockDim.x + threadIdx.x;
    if (u >= a.n) break;
    const int64_t b = a.off[u], e = a.off[u + 1];
    bool ok = true;
    if ((u == 0 && b != 0) || (u == a.n - 1 && e != a.nnz)) ok = false;
    if (e < b || b < 0 || e > a.nnz || e - b >= ((int64_t)1 << 31)) ok = false;
    const uint32_t d = ok ? (uint32_t)(e - b) : 0;
    if (!ok) atomicOr(a.err, ERR_RANGE);
    a.info[u] = ok ? (uint64_t)b << 24 : 0;
    if (a.vbase) {
      int32_t lo = 0, hi = a.graphs;  // the last graph with vbase[g] <= u
      while (hi - lo > 1) {
        const int32_t mid = (lo + hi) >> 1;
        if (a.vbase[mid] <= u) lo = mid; else hi = mid;
      }
      a.grow[u] = (uint32_t)lo;
    }
    if (a.deg) a.deg[u] = d;
    if (PER > 1) atomicAdd(&h[BUCKETS - 1 - degree_bucket(d)], 1u);
    if (d) {
      a.list[b] = (uint32_t)u;
      atomicOr(&a.mark[b >> 5], 1u << (b & 31));
      for (int64_t t = (b + OT - 1) / OT; t * OT < e; ++t) a.tile_row[t] = (uint32_t)u;
      if (a.cross && b / OT != (e - 1) / OT) {
        int64_t lo = b, hi = e;
        while (lo < hi) {
          const int64_t m = (lo + hi) >> 1;
          if (a.nbr[m] < (int32_t)u) lo = m + 1; else hi = m;
        }
        a.cross[b / OT + 1].su = (uint32_t)(lo - b);
      }
    }
  }
  if (PER == 1) return;
  __syncthreads();
  if (h[threadIdx.x]) atomicAdd(&a.hist[threadIdx.x], h[threadIdx.x]);
}

// Ranks by a counting sort on the degree bucket, highest first; the order
// within a bucket is free (any total order lists each triangle once).
template <int PER>
__global__ void __launch_bounds__(ROWS_THREADS) k_sw_rank(int64_t n, const int64_t* __restrict__ off,
                                                          const uint32_t* __restrict__ hist,
                                                          uint32_t* __restrict__ cursor, uint32_t* __restrict__ rank,
                                                          const uint32_t* __restrict__ err) {
  __shared__ uint32_t start[BUCKETS], cnt[BUCKETS], wsum[ROWS_THREADS / 64];
  if (err[0]) return;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  // exclusive prefix of the bucket counts
  const uint32_t v = hist[threadIdx.x];
  uint32_t x = v;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[w] = x;
  cnt[threadIdx.x] = 0;
  __syncthreads();
  uint32_t add = 0;
  for (int i = 0; i < w; ++i) add += wsum[i];
  start[threadIdx.x] = x - v + add;
  const int64_t base = (int64_t)blockIdx.x * (ROWS_THREADS * PER);
  uint32_t bk[PER];
  for (int i = 0; i < PER; ++i) {
    const int64_t u = base + i * ROWS_THREADS + threadIdx.x;
    bk[i] = BUCKETS;
    if (u < n) {
      bk[i] = BUCKETS - 1 - degree_bucket((uint32_t)(off[u + 1] - off[u]));
      atomicAdd(&cnt[bk[i]], 1u);
    }
  }
  __syncthreads();
  if (cnt[threadIdx.x]) start[threadIdx.x] += atomicAdd(&cursor[threadIdx.x], cnt[threadIdx.x]);
  __syncthreads();
  for (int i = 0; i < PER; ++i) {
    const int64_t u = base + i * ROWS_THREADS + threadIdx.x;
    if (u < n) {
      rank[u] = atomicAdd(&start[bk[i]], 1u);
    }
  }
}

// --------------------------------------------------------------- orientation

struct OrientArgs {
  int64_t n, nnz, ntiles;
  const int64_t* off;
  const int32_t* nbr;
  const uint8_t* flg;
  const uint32_t* key;  // rank (RANK) or degree, by row
  const uint32_t* mark;
  const uint32_t* tile_row;
  uint32_t* list;
  uint64_t* info;
  Cross* cross;
  uint32_t* mid;  // rows with N+ longer than SORT_MIN, than SORT_MID
  uint32_t* lng;
  uint32_t* counts;  // [0] of mid, [1] of lng
  unsigned long long* acc;
  uint32_t* err;
  // a batch: ids are local to their graph, the class sums go to gacc[graph][16]
  const int64_t* vbase;
  const uint32_t* grow;
  unsigned long long* gacc;
};

__device__ __forceinline__ uint64_t below(int k) { return (1ull << k) - 1; }  // k in [0, 63]

// One workgroup per tile of OT entries. The tile's row segments are compacted
// in LDS (a row start bit per entry marks them), so that every entry finds its
// row by two reads and a population count, and the counts of a segment are
// taken by one thread from bit planes without touching memory again: the only
// dependent reads of a tile are its entries, then the keys of their ends
// (tiles of 4,096 entries with a search and three row reads per segment in
// turn, at 2 wavefronts per SIMD: 11.4 ms at R-MAT scale 24 and 13.7 ms on the
// 4,096-graph batch, now 6.2 and 5.4; bound by the random reads of the keys).
// Five wavefronts per SIMD hide more of them than three without spills.
// RANK: lists hold ranks, else ids. BAT: a batch (ids). LAB: labelled words,
// the sums are k_lab_sums'.
template <bool RANK, bool BAT, bool LAB>
__global__ void __launch_bounds__(OTHREADS, 5) k_sw_orient(OrientArgs a) {
  __shared__ uint32_t srow[OT], skey[OT];  // per segment: its row (BAT: within its graph), its key; later N+ entries
  __shared__ uint16_t spos[OT + 1];        // its first entry
  __shared__ uint32_t sgr[BAT ? OT : 1];   // BAT: its graph, from the tile's first (any number without entries may lie between)
  __shared__ uint64_t heads[OWORDS], fwd[OWORDS + 1], b0[OWORDS], b1[OWORDS];
  __shared__ uint32_t hpre[OWORDS + 1];  // segments, N+ entries before each 64-entry word
  __shared__ uint32_t pre[OWORDS + 1];
  __shared__ int64_t cF[2], cB[2];       // crossing rows (first, last segment): where their entries go
  __shared__ int32_t edge[OWORDS + 1];   // the entry before each 64-entry word
  __shared__ int64_t ends[4];            // the first and the last segment's row: its entry range
  __shared__ uint32_t longs[2][RANK ? LONG_KEEP : 1], nlong[2], lbase[2];  // rows with long N+, over several tiles
  __shared__ unsigned long long gsum[BAT ? TILE_GRAPHS : 1][9];  // sums of the block, BAT: of the tile's first graphs
  if (a.err[0]) return;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t bad = 0, above = 0;
  // the rows with long N+ kept so far, to their list (one atomic; the whole block)
  auto put_longs = [&](int tid, int k) {
    if (tid == 0) lbase[k] = atomicAdd(&a.counts[k], nlong[k]);
    __syncthreads();
    for (int i = tid; i < (int)nlong[k]; i += OTHREADS) (k ? a.lng : a.mid)[lbase[k] + i] = longs[k][i];
    __syncthreads();
    if (tid == 0) nlong[k] = 0;
    __syncthreads();
  };
  if (!BAT && threadIdx.x < 9) gsum[0][threadIdx.x] = 0;
  if (threadIdx.x < 2) nlong[threadIdx.x] = 0;
  for (int64_t t = blockIdx.x; t < a.ntiles; t += gridDim.x) {
    // (made opaque: the values derived from it are recomputed per tile instead of
    // being hoisted out of the loop as live registers)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    const int64_t t0 = t * OT;
    const int len = (int)min((int64_t)OT, a.nnz - t0);
    const uint32_t xfirst = a.tile_row[t], xlast = t + 1 < a.ntiles ? a.tile_row[t + 1] : xfirst;
    const int32_t* nb = a.nbr + t0;
    int32_t y[OPER];
    uint32_t wd[OPER];
#pragma unroll
    for (int i = 0; i < OPER; ++i) {
      const int p = i * OTHREADS + tid;
      y[i] = p < len ? nb[p] : 0;
      wd[i] = p < len ? (uint32_t)(a.flg[(t0 + p) >> 2] >> (2 * (p & 3))) & 3u : 0u;
    }
    const int32_t left = tid == 0 && t > 0 ? nb[-1] : 0;
    __syncthreads();  // the tile before is done with LDS
#pragma unroll
    for (int i = 0; i < OPER; ++i)
      if (lane == 63) edge[i * (OTHREADS / 64) + w + 1] = y[i];
    if (tid == 0) edge[0] = left;
    if (w == 0) {
      uint64_t h = lane < OWORDS ? ((const uint64_t*)a.mark)[t * OWORDS + lane] | (lane == 0 ? 1ull : 0ull) : 0ull;
      const uint32_t c = (uint32_t)__popcll(h);
      uint32_t s = c;
      for (int o = 1; o < OWORDS; o <<= 1) {
        const uint32_t q = __shfl_up(s, o, 64);
        if (lane >= o) s += q;
      }
      if (lane < OWORDS) {
        heads[lane] = h;
        hpre[lane] = s - c;
        if (lane == OWORDS - 1) {
          hpre[OWORDS] = s;
          spos[s] = (uint16_t)len;
        }
      }
    } else if (w == 1) {
      // the rows that may cross a boundary: another tile may already have
      // placed entries over their start, so their ids come from the tile starts
      if (lane < 4) ends[lane] = a.off[(lane < 2 ? xfirst : xlast) + (lane & 1)];
    }
    if (BAT)
      for (int k = tid; k < TILE_GRAPHS * 9; k += OTHREADS) (&gsum[0][0])[k] = 0;
    __syncthreads();
    const int nseg = (int)hpre[OWORDS];
#pragma unroll
    for (int i = 0; i < OPER; ++i) {
      const int wi = i * (OTHREADS / 64) + w;
      if ((heads[wi] >> lane) & 1ull) spos[hpre[wi] + (uint32_t)__popcll(heads[wi] & below(lane))] = (uint16_t)(wi * 64 + lane);
    }
    const bool cross0 = ends[0] < t0 || ends[1] > t0 + len;                       // the first segment's row
    const bool cross1 = t + 1 < a.ntiles && ends[2] > t0 && ends[2] < t0 + len;  // the last one's, another row
    __syncthreads();
    const uint32_t g0 = BAT ? a.grow[xfirst] : 0u;
    for (int s = tid; s < nseg; s += OTHREADS) {
      const uint32_t x = s == 0 ? xfirst : s == nseg - 1 && cross1 ? xlast : a.list[t0 + spos[s]];
      skey[s] = a.key[x];
      if constexpr (BAT) {
        const uint32_t g = a.grow[x];
        sgr[s] = g - g0;
        srow[s] = (uint32_t)(x - a.vbase[g]);
      } else {
        srow[s] = x;
      }
    }
    __syncthreads();
    // entry checks, direction of each edge
    uint16_t sg[OPER];
    uint32_t ky[OPER];
#pragma unroll
    for (int i = 0; i < OPER; ++i) {
      const int p = i * OTHREADS + tid, wi = i * (OTHREADS / 64) + w;
      sg[i] = (uint16_t)(hpre[wi] + (uint32_t)__popcll(heads[wi] & (~0ull >> (63 - lane))) - 1);
      int64_t base = 0, ng = a.n;
      if (BAT) {
        const int64_t g = (int64_t)g0 + sgr[sg[i]];
        base = a.vbase[g];
        ng = a.vbase[g + 1] - base;
      }
      if (p < len && (y[i] < 0 || y[i] >= ng)) {
        bad |= ERR_RANGE;
        y[i] = 0;
      }
      ky[i] = a.key[base + y[i]];
    }
#pragma unroll
    for (int i = 0; i < OPER; ++i) {
      const int p = i * OTHREADS + tid, wi = i * (OTHREADS / 64) + w;
      const bool in = p < len;
      const int32_t x = (int32_t)srow[sg[i]];
      int32_t pv = __shfl_up(y[i], 1, 64);
      if (lane == 0) pv = edge[wi];
      // (the tile's first entry carries a start bit of its own: look at the row)
      const bool first = p == 0 ? ends[0] == t0 : (heads[wi] >> lane) & 1ull;
      if (in) {
        if (!first && pv >= y[i]) bad |= ERR_UNSORTED;
        if (y[i] == x) bad |= ERR_SELFLOOP;
        if (wd[i] == 0) bad |= ERR_RANGE;
      }
      const uint32_t kx = skey[sg[i]], g = wd[i];
      const bool f = in && (RANK ? ky[i] < kx : (ky[i] > kx || (ky[i] == kx && y[i] > x)));
      // N+ words carry f_xy and the rank (id) of y; in-list words of row x
      // the id of y and f_yx, the flag seen from y
      const uint32_t id = f && RANK ? ky[i] : (uint32_t)y[i], mirror = (g & 1u) << 1 | g >> 1;
      if (LAB)
        wd[i] = (y[i] > x ? g : mirror) << 30 | (uint32_t)(f == (y[i] < x)) << 29 | id;
      else
        wd[i] = (f ? g : mirror) << 30 | id;
      const uint64_t mf = __ballot(f), m0 = __ballot(g & 1u), m1 = __ballot(g >> 1);
      above += (uint32_t)__popcll(__ballot(in && y[i] > x));
      if (lane == 0) {
        fwd[wi] = mf;
        b0[wi] = m0;
        b1[wi] = m1;
      }
    }
    __syncthreads();
    if (w == 0) {
      const uint32_t c = lane < OWORDS ? (uint32_t)__popcll(fwd[lane]) : 0u;
      uint32_t s = c;
      for (int o = 1; o < OWORDS; o <<= 1) {
        const uint32_t q = __shfl_up(s, o, 64);
        if (lane >= o) s += q;
      }
      if (lane < OWORDS) pre[lane] = s - c;
      if (lane == OWORDS - 1) {
        pre[OWORDS] = s;
        fwd[OWORDS] = 0;
      }
    }
    __syncthreads();
    // the counts of each segment (its sums go to LDS at once: kept in registers
    // over the tiles they cost a wavefront per SIMD and spills)
    for (int s = tid; s < nseg; s += OTHREADS) {
      const int p = spos[s], e = spos[s + 1];
      const uint32_t nf = pre[e >> 6] + (uint32_t)__popcll(fwd[e >> 6] & below(e & 63)) - pre[p >> 6] -
                          (uint32_t)__popcll(fwd[p >> 6] & below(p & 63));
      uint32_t o = 0, in = 0, mu = 0;
      for (int wi = p >> 6; wi <= (e - 1) >> 6; ++wi) {
        uint64_t m = ~0ull;
        if (wi == p >> 6) m &= ~below(p & 63);
        if (wi == e >> 6) m &= below(e & 63);
        const uint64_t q0 = b0[wi] & m, q1 = b1[wi] & m;
        o += (uint32_t)__popcll(q0 & ~q1);
        in += (uint32_t)__popcll(q1 & ~q0);
        mu += (uint32_t)__popcll(q0 & q1);
      }
      const uint32_t g = BAT ? g0 + sgr[s] : 0u;
      const uint32_t x = srow[s] + (BAT ? (uint32_t)a.vbase[g] : 0u);
      skey[s] = nf;
      if (!((s == 0 && cross0) || (s == nseg - 1 && cross1))) {
        const uint32_t fl = nf > SORT_MAX ? UNSORTED : 0u;
        a.info[x] = (uint64_t)(t0 + p) << 24 | (min(nf, LEN_MASK) | (RANK ? fl : 0u));
        if constexpr (!LAB) {
          RowSums one;
          one.row(BAT ? (uint64_t)(a.vbase[g + 1] - a.vbase[g]) : (uint64_t)a.n, o, in, mu);
          for (int k = 0; k < 9; ++k) {
            if (!one.c[k]) continue;
            if (!BAT || g - g0 < TILE_GRAPHS) atomicAdd(&gsum[g - g0][k], (unsigned long long)one.c[k]);
            else atomicAdd(&a.gacc[(uint64_t)g * 16 + RowSums::batch_slot(k)], (unsigned long long)one.c[k]);
          }
        }
        if (RANK && nf > SORT_MIN && nf <= SORT_MAX) {
          const uint32_t k = nf > SORT_MID;
          longs[k][atomicAdd(&nlong[k], 1u)] = x;
        }
      } else {
        const int k = s == 0 ? 0 : 1;
        const int64_t ox = ends[2 * k], ex = ends[2 * k + 1];
        Cross* c = &a.cross[ox / OT + 1];
        cF[k] = ox + atomicAdd(&c->f, nf);
        cB[k] = ex - 1 - (int64_t)atomicAdd(&c->b, (uint32_t)(e - p) - nf);
        atomicAdd(&c->o, o);
        atomicAdd(&c->i, in);
        atomicAdd(&c->m, mu);
      }
    }
    __syncthreads();
    // place the entries
#pragma unroll
    for (int i = 0; i < OPER; ++i) {
      const int p = i * OTHREADS + tid, wi = i * (OTHREADS / 64) + w;
      if (p >= len) continue;
      const int s = sg[i], h = spos[s];
      const uint64_t fm = fwd[wi];
      const uint32_t c = pre[wi] + (uint32_t)__popcll(fm & below(lane)) - pre[h >> 6] -
                         (uint32_t)__popcll(fwd[h >> 6] & below(h & 63));
      const bool f = (fm >> lane) & 1ull;
      const uint32_t q = (uint32_t)(p - h) - c;  // in-list entries of the segment before this one
      int64_t to;
      if ((s == 0 && cross0) || (s == nseg - 1 && cross1)) {
        const int k = s == 0 ? 0 : 1;
        to = f ? cF[k] + c : cB[k] - q;
      } else {
        to = t0 + h + (f ? c : skey[s] + q);
      }
      a.list[to] = wd[i];
    }
    if (RANK && nlong[0] + OT / SORT_MIN > LONG_KEEP) put_longs(tid, 0);
    if (RANK && nlong[1] + OT / SORT_MIN > LONG_KEEP) put_longs(tid, 1);
    if (BAT)
      for (int k = tid; k < TILE_GRAPHS * 9; k += OTHREADS) {
        const unsigned long long v = gsum[k / 9][k % 9];
        if (v) atomicAdd(&a.gacc[(uint64_t)(g0 + k / 9) * 16 + RowSums::batch_slot(k % 9)], v);
      }
  }
  const int tid = threadIdx.x, lane = tid & 63;
  __syncthreads();
  if (RANK) {
    put_longs(tid, 0);
    put_longs(tid, 1);
  }
  for (int o = 32; o > 0; o >>= 1) bad |= __shfl_xor(bad, o, 64);
  if (lane == 0 && bad) atomicOr(&a.err[1], bad);
  if (lane == 0 && above) atomicAdd(&copy_of<LAB>(a.acc)[LAB ? SW_LAB_ABOVE : SW_ABOVE], (unsigned long long)above);
  __syncthreads();
  if (!BAT && !LAB && tid < 9 && gsum[0][tid]) atomicAdd(&copy_of<LAB>(a.acc)[RowSums::slot(tid)], gsum[0][tid]);
}

// Rows that cross tile boundaries, at the first boundary inside each.
template <bool RANK, bool BAT, bool LAB>
__global__ void __launch_bounds__(256) k_sw_cross(OrientArgs a) {
  if (a.err[0] | a.err[1]) return;
  const int lane = threadIdx.x & 63;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  RowSums sums;
  for (int64_t t0 = 1 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x - lane; t0 < a.ntiles; t0 += stride) {
    const int64_t t = t0 + lane;
    int kind = -1;  // list of long N+
    uint32_t x = 0;
    if (t < a.ntiles) {
      x = a.tile_row[t];
      const int64_t ox = a.off[x];
      if (ox < t * OT && ox / OT + 1 == t) {
        const Cross c = a.cross[t];
        const uint32_t fl = RANK && c.f > SORT_MAX ? UNSORTED : 0u;
        a.info[x] = (uint64_t)ox << 24 | (min(c.f, LEN_MASK) | fl);
        if constexpr (BAT) {
          const uint32_t g = a.grow[x];
          RowSums one;
          one.row((uint64_t)(a.vbase[g + 1] - a.vbase[g]), c.o, c.i, c.m);
          for (int k = 0; k < 9; ++k)
            if (one.c[k]) atomicAdd(&a.gacc[(uint64_t)g * 16 + RowSums::batch_slot(k)], (unsigned long long)one.c[k]);
        } else if constexpr (!LAB) {
          sums.row((uint64_t)a.n, c.o, c.i, c.m);
        }
        if (RANK && c.f > SORT_MIN && c.f <= SORT_MAX) kind = c.f > SORT_MID ? 1 : 0;
      }
    }
    if (RANK)
      for (int k = 0; k < 2; ++k) {  // one atomic a wavefront
        const uint64_t m = __ballot(kind == k);
        if (!m) continue;
        uint32_t base = 0;
        if (lane == 0) base = atomicAdd(&a.counts[k], (uint32_t)__popcll(m));
        base = rl(base, 0);
        if (kind == k) (k ? a.lng : a.mid)[base + __popcll(m & below(lane))] = x;
      }
  }
  if (BAT || LAB) return;
  for (int k = 0; k < 9; ++k) {
    const uint64_t v = sum64(sums.c[k]);
    if (lane == 0 && v) atomicAdd(&copy_of<LAB>(a.acc)[RowSums::slot(k)], (unsigned long long)v);
  }
}

// ------------------------------------------------------------- labelled sums
// The open wedges and dyads of the 64-state census in closed form (states of a
// triple a < b < c: f_ab | f_ac << 2 | f_bc << 4; h below is a pair's flag seen
// from its lower id). A wedge at centre x is two of its entries: both below x
// (states h << 2 | h' << 4, in id order), one on each side (h | h' << 4), both
// above (h | h' << 2); the counts of ordered flag pairs on one side come from
// running counts of the flags 1 and 2 along the row. An edge u < v of flag h has
// third vertices adjacent to neither below u (state h << 4),
// between (h << 2) and above (h), less the common neighbours there:
//   below  u - s_u - s_v, between (v - u - 1) - (k - s_u) - (d'_v - s_v - 1),
//   above  (n - 1 - v) - (d_u - k - 1) - (d_v - d'_v)
// with k the index of v in row u, s_u, d'_v the entries of rows u, v below
// their own ids and s_v the index of u in row v, so each entry adds its own
// row's part. (The common neighbours are added with the triangles.)
struct SegCounts {
  uint32_t lo[3], hi[3];  // entries below and above the row's id, by h - 1
};

struct LabArgs {
  int64_t n, nnz, ntiles;
  const int64_t* off;
  const int32_t* nbr;
  const uint8_t* flg;
  const uint32_t* mark;
  const uint32_t* tile_row;
  const uint32_t* list;  // a row's id at its first entry
  const Cross* cross;    // entries below the own id of rows that cross tiles
  SegCounts* segs;       // [tile][2]: the counts of a crossing first, last segment
  unsigned long long* acc;
  const uint32_t* err;
};

// Row totals into the wedge states (hist: 64 words): pairs of unlike flags on
// one side all in the order (higher flag, lower flag); the running counts move
// those that come the other way round.
template <class Add>
__device__ __forceinline__ void lab_row(const uint64_t (&lo)[3], const uint64_t (&hi)[3], Add add) {
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) {
      if (lo[i] && hi[j]) add((i + 1) | (j + 1) << 4, lo[i] * hi[j]);
      if (i == j) {
        if (lo[i] > 1) add((i + 1) << 2 | (j + 1) << 4, lo[i] * (lo[i] - 1) / 2);
        if (hi[i] > 1) add((i + 1) | (j + 1) << 2, hi[i] * (hi[i] - 1) / 2);
      } else if (i > j) {
        if (lo[i] && lo[j]) add((i + 1) << 2 | (j + 1) << 4, lo[i] * lo[j]);
        if (hi[i] && hi[j]) add((i + 1) | (j + 1) << 2, hi[i] * hi[j]);
      }
    }
}

// Pairs (earlier flag i, later flag j), i < j, k = 0..2 for (1,2) (1,3) (2,3):
// moved from the state of (j, i) to that of (i, j).
__device__ __forceinline__ void lab_move(unsigned long long* acc, int side, int k, uint64_t v) {
  if (!v) return;
  const int i = k == 2 ? 2 : 1, j = k == 0 ? 2 : 3;
  const int s0 = side ? (i | j << 2) : (i << 2 | j << 4), s1 = side ? (j | i << 2) : (j << 2 | i << 4);
  atomicAdd(&acc[s0], (unsigned long long)v);
  atomicAdd(&acc[s1], (unsigned long long)(0 - v));
}

__global__ void __launch_bounds__(OTHREADS, 4) k_lab_sums(LabArgs a) {
  __shared__ uint32_t srow[OT], ssu[OT];
  __shared__ uint16_t spos[OT + 1];
  __shared__ uint64_t heads[OWORDS];
  __shared__ uint32_t hpre[OWORDS + 1];
  __shared__ uint64_t pl[6][OWORDS + 1];  // planes: below 1, 2, 3; above 1, 2, 3
  __shared__ uint32_t pp[6][OWORDS + 1];  // their counts before each word
  __shared__ int64_t ends[4];
  __shared__ unsigned long long hist[64];
  if (a.err[0]) return;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (threadIdx.x < 64) hist[threadIdx.x] = 0;
  uint64_t dy[3][3] = {}, pr[2][3] = {};  // dyads [below, between, above][h - 1], ordered pairs [side][k]
  for (int64_t t = blockIdx.x; t < a.ntiles; t += gridDim.x) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    const int64_t t0 = t * OT;
    const int len = (int)min((int64_t)OT, a.nnz - t0);
    const uint32_t xfirst = a.tile_row[t], xlast = t + 1 < a.ntiles ? a.tile_row[t + 1] : xfirst;
    int32_t y[OPER];
    uint32_t h[OPER];
#pragma unroll
    for (int i = 0; i < OPER; ++i) {
      const int p = i * OTHREADS + tid;
      y[i] = p < len ? a.nbr[t0 + p] : 0;
      h[i] = p < len ? (uint32_t)(a.flg[(t0 + p) >> 2] >> (2 * (p & 3))) & 3u : 0u;
    }
    __syncthreads();
    if (w == 0) {
      uint64_t m = lane < OWORDS ? ((const uint64_t*)a.mark)[t * OWORDS + lane] | (lane == 0 ? 1ull : 0ull) : 0ull;
      const uint32_t c = (uint32_t)__popcll(m);
      uint32_t s = c;
      for (int o = 1; o < OWORDS; o <<= 1) {
        const uint32_t q = __shfl_up(s, o, 64);
        if (lane >= o) s += q;
      }
      if (lane < OWORDS) {
        heads[lane] = m;
        hpre[lane] = s - c;
        if (lane == OWORDS - 1) {
          hpre[OWORDS] = s;
          spos[s] = (uint16_t)len;
        }
      }
    } else if (w == 1 && lane < 4) {
      ends[lane] = a.off[(lane < 2 ? xfirst : xlast) + (lane & 1)];
    }
    __syncthreads();
    const int nseg = (int)hpre[OWORDS];
#pragma unroll
    for (int i = 0; i < OPER; ++i) {
      const int wi = i * (OTHREADS / 64) + w;
      if ((heads[wi] >> lane) & 1ull) spos[hpre[wi] + (uint32_t)__popcll(heads[wi] & below(lane))] = (uint16_t)(wi * 64 + lane);
    }
    const bool cross0 = ends[0] < t0 || ends[1] > t0 + len;
    const bool cross1 = t + 1 < a.ntiles && ends[2] > t0 && ends[2] < t0 + len;
    __syncthreads();
    for (int s = tid; s < nseg; s += OTHREADS)
      srow[s] = s == 0 ? xfirst : s == nseg - 1 && cross1 ? xlast : a.list[t0 + spos[s]];
    __syncthreads();
    uint16_t sg[OPER];
#pragma unroll
    for (int i = 0; i < OPER; ++i) {
      const int wi = i * (OTHREADS / 64) + w;
      sg[i] = (uint16_t)(hpre[wi] + (uint32_t)__popcll(heads[wi] & (~0ull >> (63 - lane))) - 1);
      const bool up = y[i] > (int32_t)srow[sg[i]];
      if (!up) h[i] = (h[i] & 1u) << 1 | h[i] >> 1;
#pragma unroll
      for (uint32_t f = 1; f <= 3; ++f) {
        const uint64_t ml = __ballot(h[i] == f && !up), mh = __ballot(h[i] == f && up);
        if (lane == 0) {
          pl[f - 1][wi] = ml;
          pl[f + 2][wi] = mh;
        }
      }
    }
    __syncthreads();
    for (int k = w; k < 6; k += OTHREADS / 64) {
      const uint32_t c = lane < OWORDS ? (uint32_t)__popcll(pl[k][lane]) : 0u;
      uint32_t s = c;
      for (int o = 1; o < OWORDS; o <<= 1) {
        const uint32_t q = __shfl_up(s, o, 64);
        if (lane >= o) s += q;
      }
      if (lane < OWORDS) pp[k][lane] = s - c;
      if (lane == OWORDS - 1) {
        pp[k][OWORDS] = s;
        pl[k][OWORDS] = 0;
      }
    }
    __syncthreads();
    // entries of plane k before position p of the tile
    auto before = [&](int k, int p) { return pp[k][p >> 6] + (uint32_t)__popcll(pl[k][p >> 6] & below(p & 63)); };
    for (int s = tid; s < nseg; s += OTHREADS) {
      const int p = spos[s], e = spos[s + 1];
      uint64_t lo[3], hi[3];
      for (int f = 0; f < 3; ++f) {
        lo[f] = before(f, e) - before(f, p);
        hi[f] = before(f + 3, e) - before(f + 3, p);
      }
      if ((s == 0 && cross0) || (s == nseg - 1 && cross1)) {
        const int k = s == 0 ? 0 : 1;
        SegCounts c;
        for (int f = 0; f < 3; ++f) {
          c.lo[f] = (uint32_t)lo[f];
          c.hi[f] = (uint32_t)hi[f];
        }
        a.segs[2 * t + k] = c;
        ssu[s] = a.cross[ends[2 * k] / OT + 1].su;
      } else {
        ssu[s] = (uint32_t)(lo[0] + lo[1] + lo[2]);
        lab_row(lo, hi, [&](int st, uint64_t v) { atomicAdd(&hist[st], (unsigned long long)v); });
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < OPER; ++i) {
      const int p = i * OTHREADS + tid, s = sg[i], p0 = spos[s];
      if (p >= len) continue;
      const int64_t x = srow[s], su = ssu[s];
      int64_t k = p - p0, d = spos[s + 1] - p0;
      if ((s == 0 && cross0) || (s == nseg - 1 && cross1)) {
        const int q = s == 0 ? 0 : 1;
        k = t0 + p - ends[2 * q];
        d = ends[2 * q + 1] - ends[2 * q];
      }
      const bool up = y[i] > (int32_t)x;
      const int64_t d0 = up ? x - su : -k, d1 = up ? (y[i] - x - 1) - (k - su) : -(su - k - 1),
                    d2 = up ? (a.n - 1 - y[i]) - (d - 1 - k) : -(d - su);
      const int side = up ? 3 : 0;
      const uint32_t c1 = before(side, p) - before(side, p0), c2 = before(side + 1, p) - before(side + 1, p0);
#pragma unroll
      for (uint32_t f = 1; f <= 3; ++f) {
        const bool me = h[i] == f;
        dy[0][f - 1] += me ? (uint64_t)d0 : 0;
        dy[1][f - 1] += me ? (uint64_t)d1 : 0;
        dy[2][f - 1] += me ? (uint64_t)d2 : 0;
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const bool me = (q != 0) == up;
        pr[q][0] += me && h[i] == 2 ? c1 : 0u;
        pr[q][1] += me && h[i] == 3 ? c1 : 0u;
        pr[q][2] += me && h[i] == 3 ? c2 : 0u;
      }
    }
  }
  unsigned long long* acc = copy_of<true>(a.acc);
  const int lane = threadIdx.x & 63;
  for (int f = 1; f <= 3; ++f)
    for (int k = 0; k < 3; ++k) {
      const uint64_t v = sum64(dy[k][f - 1]);
      if (lane == 0 && v) atomicAdd(&acc[f << (4 - 2 * k)], (unsigned long long)v);
    }
  for (int q = 0; q < 2; ++q)
    for (int k = 0; k < 3; ++k) {
      const uint64_t v = sum64(pr[q][k]);
      if (lane == 0) lab_move(acc, q, k, v);
    }
  __syncthreads();
  if (threadIdx.x < 64 && hist[threadIdx.x]) atomicAdd(&acc[threadIdx.x], hist[threadIdx.x]);
}

// Rows that cross tiles, one wavefront each: their totals, and the ordered pairs
// whose entries lie in different tiles.
__global__ void __launch_bounds__(256) k_lab_cross(LabArgs a) {
  if (a.err[0]) return;
  const int lane = threadIdx.x & 63;
  unsigned long long* acc = copy_of<true>(a.acc);
  const int64_t nw = (int64_t)gridDim.x * 4;
  for (int64_t t = 1 + (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); t < a.ntiles; t += nw) {
    const uint32_t x = a.tile_row[t];
    const int64_t ox = a.off[x], ex = a.off[x + 1];
    if (ox >= t * OT || ox / OT + 1 != t) continue;
    const int64_t ta = t - 1, te = (ex - 1) / OT;  // first and last tile of the row
    uint64_t tot[6] = {}, pr[2][3] = {};
    for (int64_t b = ta; b <= te; b += 64) {
      uint64_t c[6] = {}, run[6];
      const int64_t q = b + lane;
      if (q <= te) {
        const SegCounts g = a.segs[2 * q + (q == ta && ox > ta * OT ? 1 : 0)];
        for (int f = 0; f < 3; ++f) {
          c[f] = g.lo[f];
          c[f + 3] = g.hi[f];
        }
      }
      for (int k = 0; k < 6; ++k) {
        uint64_t v = c[k];
        for (int o = 1; o < 64; o <<= 1) {
          const uint64_t u = __shfl_up(v, o, 64);
          if (lane >= o) v += u;
        }
        run[k] = tot[k] + v - c[k];  // in the row's tiles before this one
        tot[k] += __shfl(v, 63, 64);
      }
      for (int s = 0; s < 2; ++s) {
        pr[s][0] += run[3 * s] * c[3 * s + 1];
        pr[s][1] += run[3 * s] * c[3 * s + 2];
        pr[s][2] += run[3 * s + 1] * c[3 * s + 2];
      }
    }
    for (int s = 0; s < 2; ++s)
      for (int k = 0; k < 3; ++k) {
        const uint64_t v = sum64(pr[s][k]);
        if (lane == 0) lab_move(acc, s, k, v);
      }
    if (lane == 0) {
      const uint64_t lo[3] = {tot[0], tot[1], tot[2]}, hi[3] = {tot[3], tot[4], tot[5]};
      lab_row(lo, hi, [&](int st, uint64_t v) { atomicAdd(&acc[st], (unsigned long long)v); });
    }
  }
}

// ------------------------------------------------------------------- sorting

// Sort keys: the rank in the high bits (a list word rotated left by its flag
// bits, 2, or 3 with labels).
__device__ __forceinline__ uint32_t to_key(uint32_t w, int r) { return __builtin_amdgcn_alignbit(w, w, 32 - r); }
__device__ __forceinline__ uint32_t of_key(uint32_t k, int r) { return __builtin_amdgcn_alignbit(k, k, r); }

// Half a packed block from four sort keys (flags of 2 bits): 16-bit ranks, and
// flags, those of the even entries in the low byte (the order in which k_sw_hubs
// assembles what it reads from its table); the second half's flags go 4 bits up.
// Ranks past the table and places past a list's end (key ~0) get the flag 0,
// which counts for nothing.
__device__ __forceinline__ uint2 pack_ranks(const uint32_t* k) {
  uint32_t h[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) h[i] = min(k[i] >> 2, 0xFFFFu);
  return make_uint2(h[0] | h[1] << 16, h[2] | h[3] << 16);
}
__device__ __forceinline__ uint32_t pack_flags(const uint32_t* k) {
  uint32_t f[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) f[i] = k[i] >> 2 < (uint32_t)HUB_RANKS ? k[i] & 3u : 0u;
  return f[0] | f[2] << 2 | f[1] << 8 | f[3] << 10;
}

// Where the lists go packed (see k_sw_pack); prow NULL: nowhere.
struct Packed {
  const uint64_t* prow;
  uint4* pack;
  const uint32_t* hubs;  // number of items of k_sw_hubs: without any, prow is not written
};
// Block k of a packed list that starts at unit u: its ranks' unit, its flags'
// 16-bit word.
__device__ __forceinline__ uint32_t rank_unit(uint32_t u, uint32_t k) { return u + (k >> 3) * 9 + 1 + (k & 7); }
__device__ __forceinline__ uint64_t flag_word(uint32_t u, uint32_t k) {
  return (uint64_t)(u + (k >> 3) * 9) * 8 + (k & 7);
}

// N+ lists of 65 to 256 entries, one wavefront each: a bitonic network over
// four registers a lane.
__global__ void __launch_bounds__(256) k_sw_sort_mid(const uint32_t* __restrict__ rows,
                                                     const uint32_t* __restrict__ count,
                                                     const uint64_t* __restrict__ info, uint32_t* __restrict__ list,
                                                     const uint32_t* __restrict__ err, int rot, Packed pk) {
  if (refused(err)) return;
  const bool pack = pk.prow && *pk.hubs;
  const int lane = threadIdx.x & 63;
  const uint32_t nw = gridDim.x * 4, cnt = *count;
  for (uint32_t r = blockIdx.x * 4 + (threadIdx.x >> 6); r < cnt; r += nw) {
    const uint64_t in = info[rows[r]];
    const uint32_t len = (uint32_t)in & LEN_MASK;
    uint32_t* p = list + (in >> 24);
    uint32_t k[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) k[e] = (uint32_t)(e * 64 + lane) < len ? to_key(p[e * 64 + lane], rot) : 0xFFFFFFFFu;
    // element lane * 4 + e
#pragma unroll
    for (int sz = 2; sz <= 256; sz <<= 1) {
#pragma unroll
      for (int j = sz >> 1; j > 0; j >>= 1) {
        if (j >= 4) {
          const int lm = j >> 2;
          const bool up = ((lane * 4) & sz) == 0, lo = (lane & lm) == 0;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t o = __shfl_xor(k[e], lm, 64);
            k[e] = (lo == up) ? min(k[e], o) : max(k[e], o);
          }
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (e & j) continue;
            const bool up = ((lane * 4 + e) & sz) == 0;
            const uint32_t x = k[e], y = k[e | j];
            k[e] = up ? min(x, y) : max(x, y);
            k[e | j] = up ? max(x, y) : min(x, y);
          }
        }
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if ((uint32_t)(lane * 4 + e) < len) p[lane * 4 + e] = of_key(k[e], rot);
    if (pack) {
      const uint32_t u = (uint32_t)(pk.prow[rows[r]] >> 32), b = lane >> 1;
      const uint32_t f = pack_flags(k), f1 = __shfl_xor(f, 1, 64);
      if (8 * b < len) {
        reinterpret_cast<uint2*>(pk.pack)[2 * (uint64_t)rank_unit(u, b) + (lane & 1)] = pack_ranks(k);
        if (!(lane & 1)) reinterpret_cast<uint16_t*>(pk.pack)[flag_word(u, b)] = (uint16_t)(f | f1 << 4);
      }
    }
  }
}

// N+ lists of 257 to 4,096 entries, one workgroup each: a radix sort in LDS on
// the bits of a rank (no z of an N+ has the last rank, which fills the places
// past a list's end): 1.24 ms at R-MAT scale 24, 2.09 by a bitonic network in LDS;
// 146 and 213 us on the Chung-Lu graph of 2^22 vertices. Bound by the passes'
// vector instructions and waits.
__global__ void __launch_bounds__(256, 5) k_sw_sort_long(const uint32_t* __restrict__ rows,
                                                         const uint32_t* __restrict__ count,
                                                         const uint64_t* __restrict__ info, uint32_t* list,
                                                         const uint32_t* __restrict__ err, int bits, Packed pk) {
  __shared__ uint32_t s[SORT_MAX];
  __shared__ alignas(16) uint32_t cnt[4][256];
  __shared__ uint32_t sh[4];
  if (refused(err)) return;
  const bool pack = pk.prow && *pk.hubs;
  const uint32_t rows_listed = *count;
  for (uint32_t r = blockIdx.x; r < rows_listed; r += gridDim.x) {
    const uint64_t in = info[rows[r]];
    const uint32_t len = min((uint32_t)in & LEN_MASK, SORT_MAX);
    uint32_t* p = list + (in >> 24);
    __syncthreads();
    lds_sort<256, SORT_MAX / 256>(s, cnt, sh, p, len, bits);
    for (uint32_t i = threadIdx.x; i < len; i += 256) p[i] = s[i];
    if (pack) {
      const uint32_t u = (uint32_t)(pk.prow[rows[r]] >> 32);
      for (uint32_t b = threadIdx.x; 8 * b < len; b += 256) {
        uint32_t k[8];
#pragma unroll
        for (uint32_t i = 0; i < 8; ++i) k[i] = 8 * b + i < len ? to_key(s[8 * b + i], 2) : 0xFFFFFFFFu;
        const uint2 r0 = pack_ranks(k), r1 = pack_ranks(k + 4);
        pk.pack[rank_unit(u, b)] = make_uint4(r0.x, r0.y, r1.x, r1.y);
        reinterpret_cast<uint16_t*>(pk.pack)[flag_word(u, b)] = (uint16_t)(pack_flags(k) | pack_flags(k + 4) << 4);
      }
    }
  }
}

// ------------------------------------------------------------------ triangles

// Flags of 16 candidate triangles a lane, two bits each: X = f_xz, Y = f_yz
// (0: z is not in N+(y)), G = f_xy; counted by class 16 at a time.
struct Tri {
  static constexpr bool LAB = false;
  uint32_t X = 0, Y = 0, G = 0;
  uint32_t c[7] = {};  // all, 030C, 120D, 120U, 120C, 210, 300

  __device__ __forceinline__ void count() {
    constexpr uint32_t L = 0x55555555u;
    const uint32_t xl = X & L, xh = (X >> 1) & L, yl = Y & L, yh = (Y >> 1) & L, gl = G & L, gh = (G >> 1) & L;
    const uint32_t x1 = xl & ~xh, x2 = xh & ~xl, x3 = xl & xh;
    const uint32_t y1 = yl & ~yh, y2 = yh & ~yl, y3 = yl & yh;
    const uint32_t g1 = gl & ~gh, g2 = gh & ~gl, g3 = gl & gh;
    const uint32_t hit = (xl | xh) & (yl | yh);
    // the vertex outside the mutual pair (z, y or x) sends both, receives both
    const uint32_t d = (g3 & x2 & y2) | (x3 & g2 & y1) | (y3 & g1 & x1);
    const uint32_t u = (g3 & x1 & y1) | (x3 & g1 & y2) | (y3 & g2 & x2);
    const uint32_t p = (g3 & ((x1 & y2) | (x2 & y1))) | (x3 & ((g1 & y1) | (g2 & y2))) | (y3 & ((g1 & x2) | (g2 & x1)));
    const uint32_t two = (g3 & x3 & (y1 | y2)) | (g3 & (x1 | x2) & y3) | ((g1 | g2) & x3 & y3);
    c[0] += __popc(hit);
    c[1] += __popc((g1 & x2 & y1) | (g2 & x1 & y2));
    c[2] += __popc(d);
    c[3] += __popc(u);
    c[4] += __popc(p);
    c[5] += __popc(two);
    c[6] += __popc(g3 & x3 & y3);
  }
  // Four candidates of one x: x holds f_xz in the top two bits, y f_yz in the
  // top (TOP) or the low ones; as many of the last as r, taken to 0 .. 8, has
  // pairs of bits are dropped. g8: f_xy in each field of a byte.
  template <bool TOP>
  __device__ __forceinline__ void add4(const uint32_t (&x)[4], const uint32_t (&y)[4], int r, uint32_t g8) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      X = __builtin_amdgcn_alignbit(X, x[e], 30);
      Y = TOP ? __builtin_amdgcn_alignbit(Y, y[e], 30) : (Y << 2 | y[e]);
    }
    X &= ~((1u << min(max(r, 0), 8)) - 1u);
    G = G << 8 | g8;
  }
  // May a counter pass 32 bits with the next item? (A wavefront adds at most 2^30
  // a lane per item; on a whole chip a lane does not get that far, but the launch
  // shape of a batch is the caller's.)
  __device__ __forceinline__ bool full() const { return __ballot(c[0] >> 30) != 0; }
  __device__ __forceinline__ void flush(unsigned long long* acc, int lane) {
    uint64_t s[7];
    for (int k = 0; k < 7; ++k) {
      s[k] = sum64(c[k]);
      c[k] = 0;
    }
    if (lane == 0 && s[0]) {
      s[0] -= s[1] + s[2] + s[3] + s[4] + s[5] + s[6];
      const int slot[7] = {8, 9, 11, 12, 13, 14, 15};
      for (int k = 0; k < 7; ++k)
        if (s[k]) atomicAdd(&acc[slot[k]], (unsigned long long)s[k]);
    }
  }
};

// The labelled counterpart: X, Y, G hold the flags seen from the lower id of
// each pair, LX, LY, LG (the high bit of each field) whether z < x, z < y, y <
// x by id. The three pairs are told apart by id order (ab, ac, bc of a < b < c)
// with masks, then each of the 27 states has its counter.
struct TriLab {
  static constexpr bool LAB = true;
  uint32_t X = 0, Y = 0, G = 0, LX = 0, LY = 0, LG = 0;
  uint32_t c[27] = {};

  __device__ __forceinline__ void count() {
    constexpr uint32_t L = 0x55555555u;
    const uint32_t xl = X & L, xh = (X >> 1) & L, yl = Y & L, yh = (Y >> 1) & L, gl = G & L, gh = (G >> 1) & L;
    const uint32_t lx = LX >> 1, ly = LY >> 1, lg = LG >> 1;  // (fields masked below)
    const uint32_t hit = (xl | xh) & (yl | yh);
    // the pair without the largest vertex is ab, the one without the smallest bc
    const uint32_t big_x = lg & lx, big_y = ~lg & ly, big_z = ~lx & ~ly;
    const uint32_t low_x = ~lg & ~lx, low_y = lg & ~ly, low_z = lx & ly;
    const uint32_t abl = (big_x & yl) | (big_y & xl) | (big_z & gl), abh = (big_x & yh) | (big_y & xh) | (big_z & gh);
    const uint32_t bcl = (low_x & yl) | (low_y & xl) | (low_z & gl), bch = (low_x & yh) | (low_y & xh) | (low_z & gh);
    const uint32_t acl = gl ^ xl ^ yl ^ abl ^ bcl, ach = gh ^ xh ^ yh ^ abh ^ bch;
    const uint32_t ab[3] = {abl & ~abh & hit, abh & ~abl & hit, abl & abh & hit};
    const uint32_t ac[3] = {acl & ~ach, ach & ~acl, acl & ach};
    const uint32_t bc[3] = {bcl & ~bch, bch & ~bcl, bcl & bch};
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const uint32_t q = ab[i] & ac[j];
#pragma unroll
        for (int k = 0; k < 3; ++k) c[i * 9 + j * 3 + k] += __popc(q & bc[k]);
      }
  }
  // g8: the flag in each field of the low byte, y < x in those of the next
  template <bool TOP>
  __device__ __forceinline__ void add4(const uint32_t (&x)[4], const uint32_t (&y)[4], int r, uint32_t g8) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      X = __builtin_amdgcn_alignbit(X, x[e], 30);
      LX = __builtin_amdgcn_alignbit(LX, x[e] << 2, 30);
      Y = TOP ? __builtin_amdgcn_alignbit(Y, y[e], 30) : (Y << 2 | y[e] >> 1);
      LY = TOP ? __builtin_amdgcn_alignbit(LY, y[e] << 2, 30) : (LY << 2 | (y[e] << 1 & 2u));
    }
    X &= ~((1u << min(max(r, 0), 8)) - 1u);
    G = G << 8 | (g8 & 0xFFu);
    LG = LG << 8 | g8 >> 8;
  }
  __device__ __forceinline__ bool full() const {
    uint32_t o = 0;
#pragma unroll
    for (int k = 0; k < 27; ++k) o |= c[k];
    return __ballot(o >> 30) != 0;
  }
  __device__ __forceinline__ void flush(unsigned long long* acc, int lane) {
#pragma unroll
    for (int k = 0; k < 27; ++k) {
      const uint64_t v = sum64(c[k]);
      const int state = (k / 9 + 1) | (k / 3 % 3 + 1) << 2 | (k % 3 + 1) << 4;
      if (lane == 0 && v) atomicAdd(&acc[state], (unsigned long long)v);
      c[k] = 0;
    }
  }
};

// Table of two-bit (LAB: four-bit) fields: id z in word z / 16 (z / 8), the
// fields from the top down. Ids past the last of W words read that word, which
// the caller keeps zero if it can meet such ids.
template <bool LAB>
constexpr int FB = LAB ? 3 : 4;  // log2 of the fields of a word
template <int W, bool LAB>
__device__ __forceinline__ uint32_t probe_bits(const uint32_t* tab, uint32_t w) {
  return tab[min((w & IDM<LAB>) >> FB<LAB>, (uint32_t)W - 1)] << ((w << (LAB ? 2 : 1)) & 31u);
}
template <bool LAB>
__device__ __forceinline__ void set_bits(uint32_t* tab, uint32_t w) {
  const uint32_t f = LAB ? (w >> 28 & 0xEu) << (28 - 4 * (w & 7u)) : (w >> 30) << (30 - 2 * (w & 15u));
  atomicOr(&tab[(w & IDM<LAB>) >> FB<LAB>], f);
}

// Hash table of list words, open addressing on the low bits of the id; at most
// half of its mask + 1 slots are taken, so every search ends.
template <bool LAB>
__device__ __forceinline__ uint32_t probe_hash(const uint32_t* tab, uint32_t w, uint32_t mask = TAB_WORDS - 1) {
  const uint32_t key = w & IDM<LAB>;
  uint32_t h = key & mask, v = tab[h];
  while (v != SLOT_FREE && (v & IDM<LAB>) != key) {
    h = (h + 1) & mask;
    v = tab[h];
  }
  return (v & IDM<LAB>) == key ? v : 0u;
}
__device__ __forceinline__ void set_hash(uint32_t* tab, uint32_t w, uint32_t mask = TAB_WORDS - 1) {
  uint32_t h = w & mask;
  while (atomicCAS(&tab[h], SLOT_FREE, w) != SLOT_FREE) h = (h + 1) & mask;
}

// The in-list vertices x of one batch: byte offset of N+(x); its length, the
// unsorted mark, and f_xy on top. Offsets take 32 bits where those of the whole
// list do (a load then adds them to a scalar base).
template <bool WIDE>
struct XList {
  typename std::conditional<WIDE, uint64_t, uint32_t>::type p[64];
  uint32_t m[64];
};

// Lists the vertices of up to `cnt` in-list words g (one a lane) whose N+ has
// at least two entries (y is one of them). PACK: their blocks instead (from
// prow, in place of info).
template <bool LAB, bool WIDE, bool PACK = false>
__device__ __forceinline__ int list_x(XList<WIDE>& L, const uint32_t* __restrict__ in, int cnt,
                                      const uint64_t* __restrict__ info, int lane) {
  uint64_t xi = 0;
  uint32_t g = 0;
  if (lane < cnt) {
    g = in[lane];
    xi = info[g & IDM<LAB>];
  }
  const bool has = ((uint32_t)xi & LEN_MASK) >= (PACK ? 1 : 2);
  const uint64_t m = __ballot(has);
  if (has) {
    const int k = __popcll(m & below(lane));
    L.p[k] = PACK ? xi >> 32 : xi >> 24 << 2;
    L.m[k] = (g & ~IDM<LAB>) | ((uint32_t)xi & (LEN_MASK | UNSORTED));
  }
  return __popcll(m);
}

// Streams the cnt listed N+(x) against the table of y: one list per GL lanes
// and four entries a lane, in two such sets in turn, so that one set's loads
// are in flight while the other is counted (loads are never skipped, an idle
// lane rereads the list's first words: the wait for a set is then for its own
// loads only). A list in rank order ends with the step that reaches y's rank.
// MULTI: of several y, each list with the number of its y's table, and yranks
// their ranks if SORTED.
template <int GL, bool SORTED, bool TOP, bool WIDE, bool MULTI, class T, class Probe>
__device__ __forceinline__ void stream(const uint32_t* __restrict__ list, const XList<WIDE>& L, int cnt,
                                       uint32_t yrank, int lane, T& tri, Probe probe,
                                       const uint32_t* yranks = nullptr) {
  constexpr uint64_t G0 = GL == 16 ? 0x0001000100010001ull : 0x0101010101010101ull;  // first lane of each group
  constexpr int STEP = 4 * GL, SETS = 64 / GL;
  const int l4 = (lane & (GL - 1)) * 4;
  const uint64_t before = below(lane & (64 - GL));
  struct Slot {
    typename std::conditional<WIDE, uint64_t, uint32_t>::type o;  // byte offset of the lane's next entries
    int r;         // 8 - 2 * entries of the list from there on (8 or more: none)
    uint32_t g8;
    uint32_t lim;  // SORTED: the rank that ends the list
    uint32_t tab;  // MULTI: the list's table
    uint32_t w[4];
  } sl[2];
  auto load = [&](Slot& s) {
    const auto o = s.r < 8 ? s.o : 0;
    __builtin_memcpy(s.w, (const char*)list + o, 16);
  };
  auto take = [&](Slot& s, int k) {
    s.r = 8;
    if (k < cnt) {
      const uint32_t m = L.m[k];
      s.o = L.p[k] + 4 * l4;
      s.r = 8 + 2 * (l4 - (int)(m & LEN_MASK));
      s.g8 = (m >> 30) * 0x55u | (T::LAB ? (m >> 29 & 1u) * 0xAA00u : 0u);
      // (lists of up to SORT_MIN entries are not sorted)
      if (MULTI) s.tab = m >> 24 & 15u;
      if (SORTED)
        s.lim = (m & UNSORTED) || (STEP < (int)SORT_MIN && (m & LEN_MASK) <= SORT_MIN) ? ~0u : MULTI ? yranks[s.tab] : yrank;
    }
  };
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    sl[i].o = 0;
    sl[i].g8 = sl[i].lim = sl[i].tab = 0;
    take(sl[i], i * SETS + lane / GL);
    load(sl[i]);
  }
  int next = 2 * SETS;
  auto step = [&](Slot& s) {
    uint32_t y[4];
    probe(s.w, y, s.tab);
    tri.template add4<TOP>(s.w, y, s.r, s.g8);
    // lists that end here: their first lane has at most one step left, or the
    // last entry read has reached y
    uint64_t d = __ballot(s.r >= 8 - 2 * STEP) & G0;
    if (SORTED) d |= (__ballot((s.w[3] & IDM<T::LAB>) >= s.lim) >> (GL - 1)) & G0;
    s.o += 4 * STEP;
    s.r += 2 * STEP;
    if (d) {
      const uint64_t all = (d << GL) - d;
      if (__builtin_amdgcn_inverse_ballot_w64(all)) take(s, next + __popcll(d & before));
      next += __popcll(d);
    }
    load(s);
  };
  auto any = [&]() { return __ballot(min(sl[0].r, sl[1].r) < 8) != 0; };
  if (!any()) return;
  do {
    step(sl[0]);
    step(sl[1]);
    step(sl[0]);
    step(sl[1]);
    // (the last loads stay before the count: merged with those above the loop
    // they would move to its head, right before their use)
    __builtin_amdgcn_sched_barrier(0);
    tri.count();
  } while (any());
}

struct CountArgs {
  int64_t n, nnz, ntiles;
  const int64_t* off;
  const uint32_t* list;
  const uint64_t* info;
  const uint32_t* rank;
  const uint32_t* tile_row;
  uint64_t* items[3];  // of k_sw_hubs, k_sw_mids, k_sw_dense: y << 32 | chunk
  uint64_t* clk;       // stage starts, or NULL
  uint32_t* counts;    // [2 .. 4] items listed, [5 .. 7] items taken, [8] units packed
  int64_t range;       // k_sw_rest: entries of one wavefront
  uint32_t window;     // a batch: ids of k_sw_dense's table
  unsigned long long* acc;
  uint32_t* err;
  // a batch (see OrientArgs)
  const int64_t* vbase;
  const uint32_t* grow;
  unsigned long long* gacc;
  // N+ lists packed (k_sw_pack) in so many units, or NULL
  uint64_t* prow;
  uint4* pack;
  uint32_t units;
};

// Ranks of k_sw_dense's table.
template <bool LAB, int WORDS = DENSE_WORDS>
constexpr uint32_t DENSE_RANKS = (uint32_t)WORDS << FB<LAB>;

// Which kernel counts the triangles of y: 0 k_sw_hubs, 1 k_sw_mids, 2
// k_sw_dense, 3 k_sw_rest, 4 none. k_sw_mids reads the lists again for every
// TAB_MAX entries of N+(y) past its bits, k_sw_dense for every window of its
// table: the one with fewer passes (at most, by the number of such ranks).
template <bool LAB>
__device__ __forceinline__ uint32_t route(uint32_t rank, uint32_t plus, int64_t minus) {
  if (plus == 0 || minus == 0) return 4;
  if (rank < HUB_RANKS && minus >= HUB_MIN_IN) return 0;
  if (plus <= TAB_MAX) return minus >= MID_MIN_IN<LAB> ? 1 : 3;
  if (rank <= HUB_RANKS) return 1;
  const uint32_t high = min(plus, rank - (uint32_t)HUB_RANKS);
  return (high + TAB_MAX - 1) / TAB_MAX > (rank - 1) / DENSE_RANKS<LAB> + 1 ? 2 : 1;
}

// A batch (members above DIRECT_N): does k_sw_dense take y, of a graph of n
// vertices, rather than k_sw_rest? Where it needs fewer passes, or no more and
// the in-list feeds a workgroup. ms before / now: 8 members of 20,011 vertices of
// degree 1,000 202 / 39, 16 of 50,021 of degree 600 191 / 136, of degree 300 (few
// in-lists so long) 38 / 38; with workgroups of 1,024 alone 110, 200, 53.
__device__ __forceinline__ bool dense_member(uint32_t window, uint32_t plus, int64_t minus, uint32_t n) {
  const uint32_t there = (plus + TAB_MAX - 1) / TAB_MAX, here = (n - 1) / window + 1;
  return there > here || (there == here && minus >= DENSE_MIN_IN);
}

template <bool BAT, bool LAB>
__global__ void __launch_bounds__(256) k_sw_items(CountArgs a) {
  __shared__ uint32_t cnt[3], base[3];
  stamp(a.clk, 1);
  if (a.err[0] | a.err[1]) return;
  for (int64_t x0 = (int64_t)blockIdx.x * 4096; x0 < a.n; x0 += (int64_t)gridDim.x * 4096) {
    __syncthreads();
    if (threadIdx.x < 3) cnt[threadIdx.x] = 0;
    __syncthreads();
    uint32_t at[16], num[16], kind = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int64_t x = x0 + i * 256 + threadIdx.x;
      num[i] = 0;
      if (x < a.n) {
        const uint64_t in = a.info[x];
        const uint32_t plus = (uint32_t)in & LEN_MASK;
        const int64_t minus = a.off[x + 1] - (int64_t)(in >> 24) - plus;
        bool listed = plus && minus && (minus >= (BAT ? DENSE_MIN_IN : MID_MIN_IN<LAB>) || plus > TAB_MAX);
        if (BAT && listed) {
          const uint32_t g = a.grow[x];
          listed = dense_member(a.window, plus, minus, (uint32_t)(a.vbase[g + 1] - a.vbase[g]));
        }
        if (listed) {
          const uint32_t r = BAT ? 2 : route<LAB>(a.rank[x], plus, minus);
          kind |= r << (2 * i);
          num[i] = (uint32_t)((minus + CHUNK - 1) / CHUNK);
          at[i] = atomicAdd(&cnt[r], num[i]);
        }
      }
    }
    __syncthreads();
    if (threadIdx.x < 3 && cnt[threadIdx.x]) base[threadIdx.x] = atomicAdd(&a.counts[2 + threadIdx.x], cnt[threadIdx.x]);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const uint32_t r = (kind >> (2 * i)) & 3u;
      for (uint32_t c = 0; c < num[i]; ++c)
        a.items[r][base[r] + at[i] + c] = (uint64_t)(x0 + i * 256 + threadIdx.x) << 32 | c;
    }
  }
}

// N+ of two entries or more in blocks of eight for k_sw_hubs: 16 bytes of 16-bit
// ranks and two bytes of flags, in groups of up to eight blocks: one unit of 16
// bytes with the flags, then a unit of ranks a block, so that a step of k_sw_hubs
// reads 144 bytes in a row. prow[x]: first unit << 32, the unsorted mark and the
// blocks (0: none). Lists of 65 to SORT_MAX entries are written by the
// kernels that sort them. Half the entries are in N+ only if the graph is
// symmetric, which nothing has shown yet (the symmetry check is an option and the
// entries above the diagonal are compared at the end): a workgroup whose units do
// not fit refuses the graph and leaves its lists out. One atomic takes the units of 256 * PER vertices (one
// for 256 took 2.6 ms at 2^24 vertices: atomics on one word queue).
template <int PER>
__global__ void __launch_bounds__(256) k_sw_pack(CountArgs a) {
  constexpr int V = 256 * PER;
  __shared__ uint32_t pre[V], dst[V], ws[8], base;
  __shared__ uint64_t row[V];
  if (a.err[0] | a.err[1] || a.counts[2] == 0) return;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  for (int64_t x0 = (int64_t)blockIdx.x * V; x0 < a.n; x0 += (int64_t)gridDim.x * V) {
    uint64_t xi[PER];
    uint32_t nb[PER], fill[PER], all = 0, mine = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int64_t x = x0 + t * PER + i;
      xi[i] = x < a.n ? a.info[x] : 0;
      const uint32_t l = (uint32_t)xi[i] & LEN_MASK;
      nb[i] = l >= 2 ? (l + 7) / 8 : 0;
      fill[i] = l <= SORT_MIN || l > SORT_MAX ? nb[i] : 0;
      all += nb[i] + (nb[i] + 7) / 8;
      mine += fill[i];
    }
    uint32_t ea = all, em = mine;
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t va = __shfl_up(ea, o, 64), vm = __shfl_up(em, o, 64);
      if (lane >= o) {
        ea += va;
        em += vm;
      }
    }
    __syncthreads();
    if (lane == 63) {
      ws[w] = ea;
      ws[4 + w] = em;
    }
    __syncthreads();
    ea -= all;
    em -= mine;
    for (int q = 0; q < w; ++q) {
      ea += ws[q];
      em += ws[4 + q];
    }
    const uint32_t total = ws[0] + ws[1] + ws[2] + ws[3], todo = ws[4] + ws[5] + ws[6] + ws[7];
    if (t == 0 && total) base = atomicAdd(&a.counts[8], total);
    __syncthreads();
    const bool fits = total == 0 || (uint64_t)base + total <= a.units;
    if (!fits && t == 0) atomicOr(&a.err[2], ERR_ASYM);
    ea += base;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int64_t x = x0 + t * PER + i;
      if (!fits) nb[i] = 0;
      pre[t * PER + i] = em;
      dst[t * PER + i] = ea;
      row[t * PER + i] = xi[i];
      if (x < a.n) a.prow[x] = nb[i] ? (uint64_t)ea << 32 | ((uint32_t)xi[i] & UNSORTED) | nb[i] : 0ull;
      em += fill[i];
      ea += nb[i] + (nb[i] + 7) / 8;
    }
    __syncthreads();
    for (uint32_t b = t; fits && b < todo; b += 256) {
      uint32_t v = 0;  // the last list that starts at or before b
#pragma unroll
      for (int o = V / 2; o; o >>= 1)
        if (pre[v + o] <= b) v += o;
      const uint32_t k = b - pre[v], left = ((uint32_t)row[v] & LEN_MASK) - 8 * k;
      const uint32_t* p = a.list + (row[v] >> 24) + 8 * k;
      uint32_t q[8] = {0, 0, 0, 0, 0, 0, 0, 0};
      __builtin_memcpy(q, p, 16);
      if (left > 4) __builtin_memcpy(q + 4, p + 4, 16);
#pragma unroll
      for (int i = 0; i < 8; ++i) q[i] = (uint32_t)i < left ? to_key(q[i], 2) : 0xFFFFFFFFu;
      const uint2 r0 = pack_ranks(q), r1 = pack_ranks(q + 4);
      a.pack[rank_unit(dst[v], k)] = make_uint4(r0.x, r0.y, r1.x, r1.y);
      reinterpret_cast<uint16_t*>(a.pack)[flag_word(dst[v], k)] = (uint16_t)(pack_flags(q) | pack_flags(q + 4) << 4);
    }
  }
}

// Streams the cnt listed packed N+(x) against the table of y, one list per
// eight lanes and a block of eight entries a lane, in two sets in turn as in
// stream(). A step assembles 8 fields of f_yz, two bits each in the order of the
// packed flags, without a shift a field: the table's bytes arrive in pairs.
template <class T, class Table>
__device__ __forceinline__ void stream_packed(const CountArgs& a, const XList<false>& L, int cnt, uint32_t yrank,
                                              int lane, T& tri, const Table& tab) {
  constexpr uint64_t G0 = 0x0101010101010101ull;
  const int l8 = lane & 7;
  const uint32_t lane_ranks = 16 + 16 * l8, to_flags = 16 + 14 * l8;
  const uint64_t before = below(lane & 56);
  struct Slot {
    uint32_t o, g, lim;  // byte offset of the lane's next ranks; f_xy in each field; the rank that ends the list
    int r;               // blocks of the list from there on (0 or less: none)
    uint32_t w[4], f;
  } sl[2];
  auto load = [&](Slot& s) {
    const uint32_t o = s.r > 0 ? s.o : lane_ranks;
    __builtin_memcpy(s.w, (const char*)a.pack + o, 16);
    s.f = *(const uint16_t*)((const char*)a.pack + (o - to_flags));
  };
  auto take = [&](Slot& s, int k) {
    s.r = 0;
    if (k < cnt) {
      const uint32_t m = L.m[k];
      s.o = (L.p[k] << 4) + lane_ranks;
      s.r = (int)(m & LEN_MASK) - l8;
      s.g = (m >> 30) * 0x00550055u;
      // (lists of up to SORT_MIN entries, one step, are not sorted)
      s.lim = (m & UNSORTED) || (m & LEN_MASK) <= SORT_MIN / 8 ? ~0u : yrank;
    }
  };
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    sl[i].o = sl[i].g = sl[i].lim = 0;
    take(sl[i], i * 8 + lane / 8);
    load(sl[i]);
  }
  int next = 16;
  auto step = [&](Slot& s, uint32_t& X, uint32_t& Y, uint32_t& G) {
    Y = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      Y |= (uint32_t)tab[s.w[i] & 0xFFFFu] << (2 * i);
      Y |= (uint32_t)tab[s.w[i] >> 16] << (16 + 2 * i);
    }
    X = s.r > 0 ? s.f : 0u;
    G = s.g;
    uint64_t d = __ballot(s.r <= 8) & G0;
    d |= (__ballot((s.w[3] >> 16) >= s.lim) >> 7) & G0;
    s.o += 144;
    s.r -= 8;
    if (d) {
      const uint64_t all = (d << 8) - d;
      if (__builtin_amdgcn_inverse_ballot_w64(all)) take(s, next + __popcll(d & before));
      next += __popcll(d);
    }
    load(s);
    // (the loads stay here, before the count: merged with those above the loop
    // they would move to its head, half a round before their use)
    __builtin_amdgcn_sched_barrier(0);
  };
  auto any = [&]() { return __ballot(max(sl[0].r, sl[1].r) > 0) != 0; };
  if (!any()) return;
  do {
    uint32_t X0, Y0, G0_, X1, Y1, G1;
    step(sl[0], X0, Y0, G0_);
    step(sl[1], X1, Y1, G1);
    tri.X = __builtin_amdgcn_perm(X1, X0, 0x05010400);  // bytes X0[0], X1[0], X0[1], X1[1]
    tri.Y = Y0 | Y1 << 8;
    tri.G = G0_ | G1 << 8;
    tri.count();
  } while (any());
}

// Vertices with long in-lists: a workgroup takes up to CHUNK of one's in-list
// and holds N+(y) as a byte per rank (z of N+(y) has a lower rank than y). Bound
// by the bytes read past L2, 7.4 TB/s at R-MAT scale 24: 28.2 ms with lists of
// 32-bit words; packed (PACK) 18.1, where ranks and flags in arrays of their own
// took 21.9 (a line of flags for every line or two of ranks). Counting the classes
// 32 candidates at a time instead of 16 saves a tenth of the vector instructions
// but no time (35 ms: registers spill).
template <bool LAB, bool WIDE, bool PACK>
__global__ void __launch_bounds__(hub_threads(LAB), LAB ? 4 : 6) k_sw_hubs(CountArgs a) {
  constexpr int HUB_THREADS = hub_threads(LAB);
  __shared__ __align__(16) uint8_t tab[HUB_RANKS + 16];  // f_yz by rank of z; past the ranks: 0
  __shared__ XList<WIDE> xl[HUB_THREADS / 64];
  __shared__ uint32_t item, next;
  stamp(a.clk, 2);
  if (refused(a.err)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  for (int i = tid; i < (int)sizeof(tab) / 4; i += HUB_THREADS) ((uint32_t*)tab)[i] = 0;
  const uint32_t nitems = a.counts[2];
  XList<WIDE>& L = xl[tid >> 6];
  typename std::conditional<LAB, TriLab, Tri>::type tri;
  for (;;) {
    if (tid == 0) {
      item = atomicAdd(&a.counts[5], 1u);
      next = 0;
    }
    __syncthreads();
    const uint32_t it = item;
    if (it >= nitems) break;
    const uint64_t q = a.items[0][it];
    const uint32_t y = (uint32_t)(q >> 32);
    const uint64_t in = a.info[y];
    const uint32_t plus = (uint32_t)in & LEN_MASK, yr = a.rank[y];
    const int64_t s = (int64_t)(in >> 24), b = s + plus + (int64_t)(uint32_t)q * CHUNK;
    const int cnt = (int)min(CHUNK, a.off[y + 1] - b);
    for (uint32_t i = tid; i < plus; i += HUB_THREADS) {
      const uint32_t z = a.list[s + i];
      tab[z & IDM<LAB>] = (uint8_t)(z >> (LAB ? 29 : 30));
    }
    // wavefronts claim up to 64 in-list entries at a time
    const int claim = cnt >= 1024 ? 64 : cnt >= 512 ? 32 : 16;
    __syncthreads();
    for (;;) {
      int k = 0;
      if (lane == 0) k = (int)atomicAdd(&next, (uint32_t)claim);
      k = __builtin_amdgcn_readfirstlane(k);
      if (k >= cnt) break;
      const int nx = list_x<LAB, WIDE, PACK>(L, a.list + b + k, min(claim, cnt - k), PACK ? a.prow : a.info, lane);
      wave_sync();
      if constexpr (PACK)
        stream_packed(a, L, nx, yr, lane, tri, tab);
      else
        stream<16, true, false, WIDE, false>(a.list, L, nx, yr, lane, tri, [&](const uint32_t (&w)[4], uint32_t (&f)[4], uint32_t) {
#pragma unroll
          for (int e = 0; e < 4; ++e) f[e] = tab[min(w[e] & IDM<LAB>, (uint32_t)HUB_RANKS)];
        });
      wave_sync();
    }
    __syncthreads();
    for (uint32_t i = tid; i < plus; i += HUB_THREADS) tab[a.list[s + i] & IDM<LAB>] = 0;
    if (tri.full()) tri.flush(copy_of<LAB>(a.acc), lane);
  }
  tri.flush(copy_of<LAB>(a.acc), lane);
}

// Vertices with in-lists of middling length, of any rank: a smaller workgroup,
// N+(y) as two bits per rank up to HUB_RANKS and a hash table beyond, which takes
// TAB_MAX entries of the list at a time whatever their ranks.
template <bool LAB, bool WIDE>
__global__ void __launch_bounds__(MID_THREADS, LAB ? 4 : 5) k_sw_mids(CountArgs a) {
  constexpr int W = (HUB_RANKS >> FB<LAB>) + 1;
  __shared__ uint32_t tab[W], high[TAB_WORDS];
  __shared__ XList<WIDE> xl[MID_THREADS / 64];
  __shared__ uint32_t item, next;
  if (refused(a.err)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  for (int i = tid; i < W; i += MID_THREADS) tab[i] = 0;
  for (int i = tid; i < TAB_WORDS; i += MID_THREADS) high[i] = SLOT_FREE;
  const uint32_t nitems = a.counts[3];
  XList<WIDE>& L = xl[tid >> 6];
  typename std::conditional<LAB, TriLab, Tri>::type tri;
  for (;;) {
    if (tid == 0) item = atomicAdd(&a.counts[6], 1u);
    __syncthreads();
    const uint32_t it = item;
    if (it >= nitems) break;
    const uint64_t q = a.items[1][it];
    const uint32_t y = (uint32_t)(q >> 32);
    const uint64_t in = a.info[y];
    const uint32_t plus = (uint32_t)in & LEN_MASK, yr = a.rank[y];
    const int64_t s = (int64_t)(in >> 24), b = s + plus + (int64_t)(uint32_t)q * CHUNK;
    const int cnt = (int)min(CHUNK, a.off[y + 1] - b);
    const int claim = cnt >= 256 ? 64 : cnt >= 128 ? 32 : 16;
    const bool far = yr > HUB_RANKS;  // N+(y) may reach past the bits
    for (uint32_t f = 0; f < plus && (f == 0 || far); f += TAB_MAX) {
      const uint32_t fe = min(f + TAB_MAX, plus);
      // the first pass has all the bits
      bool any = f == 0;
      for (uint32_t i = f + tid; i < (f ? fe : plus); i += MID_THREADS) {
        const uint32_t z = a.list[s + i];
        if ((z & IDM<LAB>) < HUB_RANKS) {
          if (f == 0) set_bits<LAB>(tab, z);
        } else if (i < fe) {
          set_hash(high, z);
          any = true;
        }
      }
      if (tid == 0) next = 0;
      if (f == 0) __syncthreads();
      else if (!__syncthreads_or(any)) continue;
      for (;;) {
        int k = 0;
        if (lane == 0) k = (int)atomicAdd(&next, (uint32_t)claim);
        k = __builtin_amdgcn_readfirstlane(k);
        if (k >= cnt) break;
        const int nx = list_x<LAB, WIDE>(L, a.list + b + k, min(claim, cnt - k), a.info, lane);
        wave_sync();
        stream<16, true, true, WIDE, false>(a.list, L, nx, yr, lane, tri, [&](const uint32_t (&w)[4], uint32_t (&g)[4], uint32_t) {
          uint32_t top = 0;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            g[e] = probe_bits<W, LAB>(tab, w[e]);
            top = max(top, w[e] & IDM<LAB>);
          }
          if (far && __ballot(top >= HUB_RANKS)) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if ((w[e] & IDM<LAB>) >= HUB_RANKS) g[e] = probe_hash<LAB>(high, w[e]);
          }
        });
        wave_sync();
      }
      __syncthreads();
      if (f == 0)
        for (uint32_t i = tid; i < plus; i += MID_THREADS) {
          const uint32_t z = a.list[s + i] & IDM<LAB>;
          if (z < HUB_RANKS) tab[z >> FB<LAB>] = 0;
        }
      if (far)
        for (int i = tid; i < TAB_WORDS; i += MID_THREADS) high[i] = SLOT_FREE;
      if (fe < plus) __syncthreads();
    }
    if (tri.full()) tri.flush(copy_of<LAB>(a.acc), lane);
  }
  tri.flush(copy_of<LAB>(a.acc), lane);
}

// Vertices with N+ longer than k_sw_mids takes in few passes, past its bits: bits
// for a window of ranks at a time, 128 KB of them and one workgroup a CU. (Dense
// graphs of more than 65,536 vertices: with hash tables of 512 entries only,
// every list was read plus / 512 times, 2,041 ms where this takes 313 on 300,007
// vertices of degree 3,000.) BAT: the same for members of a batch, by ids, in a
// quarter of the size where the largest member fits (see dense_member).
template <bool BAT, bool LAB, bool WIDE, int WORDS>
__global__ void __launch_bounds__(DENSE_THREADS / (DENSE_WORDS / WORDS), 4) k_sw_dense(CountArgs a) {
  constexpr int THREADS = DENSE_THREADS / (DENSE_WORDS / WORDS), W = WORDS + 1;
  constexpr uint32_t RANKS = DENSE_RANKS<LAB, WORDS>;
  __shared__ uint32_t tab[W];  // past the window: 0
  __shared__ XList<WIDE> xl[THREADS / 64];
  __shared__ uint32_t item, next;
  if (refused(a.err)) return;
  const uint32_t nitems = a.counts[4];
  if (blockIdx.x >= nitems) return;
  const int tid = threadIdx.x, lane = tid & 63;
  for (int i = tid; i < W; i += THREADS) tab[i] = 0;
  XList<WIDE>& L = xl[tid >> 6];
  typename std::conditional<LAB, TriLab, Tri>::type tri;
  for (;;) {
    if (tid == 0) item = atomicAdd(&a.counts[7], 1u);
    __syncthreads();
    const uint32_t it = item;
    if (it >= nitems) break;
    const uint64_t q = a.items[2][it];
    const uint32_t y = (uint32_t)(q >> 32);
    const uint64_t in = a.info[y];
    const uint32_t plus = (uint32_t)in & LEN_MASK;
    const uint32_t graph = BAT ? a.grow[y] : 0u;
    const int64_t base = BAT ? a.vbase[graph] : 0;
    const uint32_t yr = BAT ? (uint32_t)(a.vbase[graph + 1] - base) : a.rank[y];  // above every z
    const int64_t s = (int64_t)(in >> 24), b = s + plus + (int64_t)(uint32_t)q * CHUNK;
    const int cnt = (int)min(CHUNK, a.off[y + 1] - b);
    const int claim = cnt >= 1024 ? 64 : cnt >= 512 ? 32 : 16;
    for (uint32_t from = 0; from < yr; from += RANKS) {
      bool any = false;
      for (uint32_t i = tid; i < plus; i += THREADS) {
        const uint32_t z = a.list[s + i];
        if ((z & IDM<LAB>) - from < RANKS) {
          set_bits<LAB>(tab, z - from);
          any = true;
        }
      }
      if (tid == 0) next = 0;
      if (!__syncthreads_or(any)) continue;
      for (;;) {
        int k = 0;
        if (lane == 0) k = (int)atomicAdd(&next, (uint32_t)claim);
        k = __builtin_amdgcn_readfirstlane(k);
        if (k >= cnt) break;
        const int nx = list_x<LAB, WIDE>(L, a.list + b + k, min(claim, cnt - k), a.info + base, lane);
        wave_sync();
        stream<16, !BAT, true, WIDE, false>(a.list, L, nx, yr, lane, tri, [&](const uint32_t (&w)[4], uint32_t (&g)[4], uint32_t) {
#pragma unroll
          for (int e = 0; e < 4; ++e) g[e] = probe_bits<W, LAB>(tab, (w[e] & IDM<LAB>) - from);
        });
        wave_sync();
      }
      __syncthreads();
      for (uint32_t i = tid; i < plus; i += THREADS) {
        const uint32_t z = (a.list[s + i] & IDM<LAB>) - from;
        if (z < RANKS) tab[z >> FB<LAB>] = 0;
      }
      __syncthreads();
    }
    if (BAT) tri.flush(a.gacc + (uint64_t)graph * 16, lane);
    else if (tri.full()) tri.flush(copy_of<LAB>(a.acc), lane);
  }
  if (!BAT) tri.flush(copy_of<LAB>(a.acc), lane);
}

// The row that holds entry j, by a 64-way search between tile starts.
__device__ __forceinline__ int64_t row_of(const CountArgs& a, int64_t j, int lane) {
  const int64_t t = j / OT;
  int64_t r = a.tile_row[t];
  int64_t span = (t + 1 < a.ntiles ? (int64_t)a.tile_row[t + 1] : a.n - 1) - r + 1;
  while (span > 1) {
    const int64_t step = (span + 63) / 64;
    const bool le = lane * step < span && a.off[r + lane * step] <= j;
    const int k = __popcll(__ballot(le)) - 1;
    r += k * step;
    span = min(step, span - k * step);
  }
  return r;
}

// Workgroups are dealt to the 8 XCDs in turn; this numbering gives each XCD
// consecutive ones, whose ranges share lists in its L2.
__device__ __forceinline__ uint32_t xcd_block() {
  const uint32_t g = gridDim.x, q = g / 8, r = g % 8, x = blockIdx.x % 8;
  return x * q + min(x, r) + blockIdx.x / 8;
}

// inclusive maximum over the lanes of a wavefront
__device__ __forceinline__ uint32_t wave_max(uint32_t x) {
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false));  // row_shr:1, 2, 4, 8
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false));  // row_bcast:15, 31
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false));
  return x;
}

// The other vertices of a ranked graph (RANK), and all vertices of a batch with
// members above DIRECT_N that k_sw_dense does not take: a wavefront takes a range
// of entries and the rows whose in-lists lie in it, up to 16 at once, each with
// its share of the hash table (at most a quarter full), their in-lists of up to 64
// entries in all as one list whose x carry their row's table. Longer ones go alone,
// the table filled TAB_MAX entries at a time (at most half full). Bound by the
// dependent reads of short lists: one row at a time took 33 of 37.4 ms on a grid of
// 2^25 vertices (24.1 in all by the merge), now 3.1 of 7.4; 3.8 and 3.0 ms at R-MAT
// scale 24. Four wavefronts a SIMD (three: Chung-Lu 2^22 10.85 -> 11.09 ms); with
// labels three, where four spill 30 registers. BAT: a batch, counted by graph.
template <bool RANK, bool BAT, bool LAB, bool WIDE>
__global__ void __launch_bounds__(REST_WAVES * 64, LAB ? 3 : 4) k_sw_rest(CountArgs a) {
  __shared__ alignas(16) uint32_t tabs[REST_WAVES][TAB_WORDS];
  __shared__ uint32_t marks[REST_WAVES][64], rows[REST_WAVES][16], ranks[RANK ? REST_WAVES : 1][16];
  __shared__ XList<WIDE> xl[REST_WAVES];
  using Pos = typename std::conditional<WIDE, uint64_t, uint32_t>::type;  // in the list
  struct Row {
    Pos start, lo;  // of N+, of the part of the in-list
    uint32_t plus, num, key;  // their lengths; the rank or the graph
  };
  __shared__ Row kept[REST_WAVES][64];  // (in registers, they spill in every step over the rows)
  if (refused(a.err)) return;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t *tab = tabs[w], *mark = marks[w], *row = rows[w], *yranks = ranks[RANK ? w : 0];
  XList<WIDE>& L = xl[w];
  Row* keep = kept[w];
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < TAB_WORDS / 256; ++i)
      reinterpret_cast<uint4*>(tab)[i * 64 + lane] = make_uint4(SLOT_FREE, SLOT_FREE, SLOT_FREE, SLOT_FREE);
  };
  clear();
  typename std::conditional<LAB, TriLab, Tri>::type tri;
  uint32_t graph = 0;
  const int64_t nw = (int64_t)gridDim.x * (blockDim.x >> 6);
  for (int64_t j0 = ((int64_t)xcd_block() * (blockDim.x >> 6) + w) * a.range; j0 < a.nnz; j0 += nw * a.range) {
    const int64_t j1 = min(j0 + a.range, a.nnz);
    for (int64_t r = row_of(a, j0, lane);; r += 64) {
      // 64 rows, one a lane: N+ and the part of the in-list in the range
      uint32_t num = 0;
      int64_t e = a.nnz;
      if (r + lane < a.n) {
        const uint64_t in = a.info[r + lane];
        e = a.off[r + lane + 1];
        const uint32_t plus = (uint32_t)in & LEN_MASK;
        const int64_t bs = (int64_t)(in >> 24) + plus, b = max(bs, j0);
        const int64_t hi = min(e, j1);
        if (plus && hi > b) {
          num = (uint32_t)(hi - b);
          uint32_t key = 0;
          if (RANK) {
            key = a.rank[r + lane];
            if (route<LAB>(key, plus, e - bs) != 3) num = 0;
          }
          if (BAT) {
            key = a.grow[r + lane];
            if ((plus > TAB_MAX || e - bs >= DENSE_MIN_IN) &&
                dense_member(a.window, plus, e - bs, (uint32_t)(a.vbase[key + 1] - a.vbase[key])))
              num = 0;
          }
          keep[lane] = Row{(Pos)(in >> 24), (Pos)b, plus, num, key};
        }
      }
      const bool done = rl64((uint64_t)e, 63) >= (uint64_t)j1 || r + 64 >= a.n;
      uint64_t todo = __ballot(num > 0);
      while (todo) {
        const int s = __builtin_ctzll(todo);
        const uint64_t* info = a.info;
        const Row me = keep[lane];  // (rows not listed: of an earlier step, out of `todo`)
        if (BAT) {
          const uint32_t g = rl(me.key, s);
          if (g != graph) {
            tri.flush(a.gacc + (uint64_t)graph * 16, lane);
            graph = g;
          }
          info += a.vbase[graph];
        }
        // the next rows that take a table of this size: 2^bits slots, 2^lanes lanes
        const uint32_t first = rl(me.plus, s);
        int bits = first <= 16 ? 6 : min(34 - (int)__builtin_clz(first - 1), 10);  // at most a quarter of them taken
        uint64_t sel = todo & __ballot(me.plus <= 1u << (bits - 2) && (!BAT || me.key == graph));
        if (bits == 10) sel = 1ull << s;
        const uint32_t v = sel >> lane & 1 ? me.num : 0u, upto = wave_scan(v);
        const uint32_t q = (uint32_t)__popcll(sel & below(lane));
        sel = __ballot(v && (q == 0 || (upto <= 64 && q < 1u << (10 - bits))));
        todo &= ~sel;
        const int n0 = (int)__popcll(sel);
        const bool alone = n0 == 1;  // (also a row whose in-list fills more than a step)
        bits = alone ? 10 : 10 - (32 - (int)__builtin_clz(n0 - 1));  // as large as so few rows leave it
        const int lanes = bits - 4;
        const bool mine = sel >> lane & 1;
        mark[lane] = 0;
        wave_sync();
        if (mine) {
          mark[upto - v] = (uint32_t)lane + 1;
          row[q] = (uint32_t)lane;
          if (RANK) yranks[q] = me.key;
        }
        wave_sync();
        // entry p of the in-lists is of row `own`; lanes 2^lanes k .. fill the table of row k
        const int own = (int)wave_max(mark[lane]) - 1, k0 = lane >> lanes;
        const uint32_t total = rl(upto, 63 - __builtin_clzll(sel)), tag = __shfl(q, own, 64) << 24;
        const Pos from = keep[own].lo - (Pos)__shfl(upto - v, own, 64);
        const int of = k0 < n0 ? (int)row[k0] : -1;
        const Pos mylist = keep[max(of, 0)].start;
        const uint32_t mylen = of < 0 ? 0u : keep[of].plus, mask = (1u << bits) - 1;
        uint32_t* mytab = tab + (k0 << bits);
        const uint32_t longest = alone ? first : 1u;  // (the others take one filling)
        for (uint32_t f = 0; f < longest; f += TAB_MAX) {
          for (uint32_t i = f + (lane & ((1 << lanes) - 1)); i < min(f + TAB_MAX, mylen); i += 1u << lanes)
            set_hash(mytab, a.list[mylist + i], mask);
          wave_sync();
          for (uint32_t k = 0; k < total; k += 64) {
            uint32_t g = 0;
            uint64_t xi = 0;
            if (k + lane < total) {
              g = a.list[from + (k + lane)];
              xi = info[g & IDM<LAB>];
            }
            const bool has = ((uint32_t)xi & LEN_MASK) >= 2;
            const uint64_t m = __ballot(has);
            if (has) {
              const int i = __popcll(m & below(lane));
              L.p[i] = xi >> 24 << 2;
              L.m[i] = (g & ~IDM<LAB>) | tag | ((uint32_t)xi & (LEN_MASK | UNSORTED));
            }
            wave_sync();
            stream<8, RANK, true, WIDE, true>(a.list, L, __popcll(m), 0, lane, tri,
                                              [&](const uint32_t (&z)[4], uint32_t (&y)[4], uint32_t t) {
              const uint32_t* mt = tab + (t << bits);
#pragma unroll
              for (int i = 0; i < 4; ++i) y[i] = probe_hash<LAB>(mt, z[i], mask);
            }, yranks);
            wave_sync();
          }
          clear();
          wave_sync();
        }
        if (BAT && tri.full()) tri.flush(a.gacc + (uint64_t)graph * 16, lane);
      }
      if (done) break;
    }
  }
  if (BAT) tri.flush(a.gacc + (uint64_t)graph * 16, lane);
  else tri.flush(copy_of<LAB>(a.acc), lane);
}

// One walk of k_sw_small over a wavefront's ranges. LARGE: the members of a batch
// past the tables, their ids N at a time; else the others (true if it met such).
template <int N, int R, bool BAT, bool LAB, bool WIDE, bool LARGE, class T>
__device__ __forceinline__ bool small_walk(const CountArgs& a, uint32_t* tab, XList<WIDE>& L, T& tri, uint32_t& graph,
                                           int lane, int w) {
  constexpr int TW = N >> FB<LAB>, LR = 64 / R;  // words of one table, lanes of one row
  uint32_t* mine = tab + lane / LR * TW;
  bool large = false;
  const int64_t nw = (int64_t)gridDim.x * (blockDim.x >> 6);
  for (int64_t j0 = ((int64_t)xcd_block() * (blockDim.x >> 6) + w) * a.range; j0 < a.nnz; j0 += nw * a.range) {
    const int64_t j1 = min(j0 + a.range, a.nnz);
    for (int64_t r = row_of(a, j0, lane);; r += 64) {
      // 64 rows, one a lane: N+ and the part of the in-list in the range
      int64_t lo = 0, e = a.nnz;
      uint64_t in = 0;
      uint32_t num = 0, gr = 0;
      if (r + lane < a.n) {
        in = a.info[r + lane];
        e = a.off[r + lane + 1];
        const uint32_t plus = (uint32_t)in & LEN_MASK;
        lo = max((int64_t)(in >> 24) + plus, j0);
        const int64_t hi = min(e, j1);
        if (plus && hi > lo) {
          num = (uint32_t)(hi - lo);
          if (BAT) gr = a.grow[r + lane];
        }
      }
      uint64_t todo = __ballot(num > 0);
      while (todo) {
        const uint64_t* info = a.info;
        uint32_t ids = 0;
        if (BAT) {
          const uint32_t g = rl(gr, __builtin_ctzll(todo));
          if (g != graph) {
            tri.flush(a.gacc + (uint64_t)graph * 16, lane);
            graph = g;
          }
          const int64_t base = a.vbase[graph], ng = a.vbase[graph + 1] - base;
          if ((ng > N) != LARGE) {
            large = true;
            todo &= ~__ballot(gr == graph);
            continue;
          }
          ids = (uint32_t)ng;
          info += base;
        }
        // the next R rows (of one graph): lanes LR q .. take the q-th
        int src = -1;
        uint32_t end[R];  // in-list entries of rows 0 .. q
        uint64_t at[R];   // list position of row q's in-list, less the entries before
        uint32_t total = 0;
#pragma unroll
        for (int q = 0; q < R; ++q) {
          at[q] = 0;
          if (todo && (!BAT || q == 0 || rl(gr, __builtin_ctzll(todo)) == graph)) {
            const int s = __builtin_ctzll(todo);
            todo &= todo - 1;
            if (lane / LR == q) src = s;
            at[q] = rl64((uint64_t)lo, s) - total;
            total += rl(num, s);
          }
          end[q] = total;
        }
        const uint64_t yi = __shfl(in, max(src, 0), 64);
        const uint32_t plus = src < 0 ? 0u : (uint32_t)yi & LEN_MASK;
        const uint32_t* mylist = a.list + (yi >> 24);
        uint32_t first = 0;  // of the ids in the table
        do {
          for (uint32_t i = lane % LR; i < plus; i += LR)
            if (!LARGE || (mylist[i] & IDM<LAB>) - first < (uint32_t)N) set_bits<LAB>(mine, mylist[i] - first);
          wave_sync();
          for (uint32_t k = 0; k < total; k += 64) {
            const uint32_t p = k + lane;
            uint32_t q = 0, g = 0;
            uint64_t xi = 0, from = at[0];
#pragma unroll
            for (int i = 1; i < R; ++i)
              if (p >= end[i - 1]) {
                q = i;
                from = at[i];
              }
            if (p < total) {
              g = a.list[from + p];
              xi = info[g & IDM<LAB>];
            }
            const bool has = ((uint32_t)xi & LEN_MASK) >= 2;
            const uint64_t m = __ballot(has);
            if (has) {
              const int i = __popcll(m & below(lane));
              L.p[i] = xi >> 24 << 2;
              L.m[i] = (g & ~IDM<LAB>) | q << 24 | ((uint32_t)xi & LEN_MASK);
            }
            wave_sync();
            stream<8, false, true, WIDE, true>(a.list, L, __popcll(m), 0, lane, tri,
                                               [&](const uint32_t (&q)[4], uint32_t (&f)[4], uint32_t t) {
              const uint32_t* mt = tab + t * TW;
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                if constexpr (LARGE) {
                  const uint32_t z = (q[i] & IDM<LAB>) - first;
                  f[i] = z < (uint32_t)N ? probe_bits<TW, LAB>(mt, z) : 0u;
                } else {
                  f[i] = probe_bits<TW, LAB>(mt, q[i]);
                }
              }
            });
            wave_sync();
          }
          for (uint32_t i = lane % LR; i < plus; i += LR) {
            const uint32_t z = (mylist[i] & IDM<LAB>) - first;
            if (!LARGE || z < (uint32_t)N) mine[z >> FB<LAB>] = 0;
          }
          wave_sync();
        } while (LARGE && (first += N) < ids);
        if (BAT && tri.full()) tri.flush(a.gacc + (uint64_t)graph * 16, lane);
      }
      if (rl64((uint64_t)e, 63) >= (uint64_t)j1 || r + 64 >= a.n) break;
    }
  }
  return large;
}

// Graphs and batch members of up to N vertices, lists in ids: a wavefront takes
// a range of entries and R rows at a time, 64 / R lanes each filling that row's
// table of N+(y) (a field per id), then the R in-lists as one list whose x carry
// their row's table: short rows fill the steps of one stream together, and
// their dependent reads overlap. (One row at a time: 17.3 ms on the 4,096-graph
// batch, 0.19 ms on 256 graphs of up to 1,024 vertices; R rows: 12.3 and 0.10,
// and 10.3 with longer turns and the loads of stream() ahead of its count.
// Bound by vector issue on the large batch, by the reads' latency on small ones.)
// WAVES: a batch plan's launch shape; tables for as many as the workgroup has
// (with tables for four, workgroups of two took 26 ms on the large batch).
template <int N, int R, bool BAT, bool LAB, bool WIDE, int WAVES>
__global__ void __launch_bounds__(WAVES * 64, LAB && N > 4096 ? 2 : 4) k_sw_small(CountArgs a) {
  constexpr int TW = N >> FB<LAB>;
  __shared__ uint32_t tabs[WAVES][R * TW];
  __shared__ XList<WIDE> xl[WAVES];
  stamp(a.clk, 1);
  stamp(a.clk, 2);
  if (refused(a.err)) return;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t* tab = tabs[w];
  XList<WIDE>& L = xl[w];
  for (int i = lane; i < R * TW; i += 64) tab[i] = 0;
  typename std::conditional<LAB, TriLab, Tri>::type tri;
  uint32_t graph = 0;
  const bool large = small_walk<N, R, BAT, LAB, WIDE, false>(a, tab, L, tri, graph, lane, w);
  // A plan's launches read the graph bases as they are then: they may have been
  // rewritten with a member past the tables.
  if constexpr (BAT) {
    if (large) small_walk<N, R, BAT, LAB, WIDE, true>(a, tab, L, tri, graph, lane, w);
  }
  if (BAT) tri.flush(a.gacc + (uint64_t)graph * 16, lane);
  else tri.flush(copy_of<LAB>(a.acc), lane);
}

// k_sw_small by the largest member: tables of 8 KB a wavefront in all (labelled
// 16 KB), so that four workgroups fit a CU's LDS.
template <bool BAT, bool LAB, bool WIDE, int WAVES>
void launch_small_of(int64_t nmax, unsigned grid, const CountArgs& ca, hipStream_t s) {
  if (nmax <= 4096) k_sw_small<4096, 4, BAT, LAB, WIDE, WAVES><<<grid, WAVES * 64, 0, s>>>(ca);
  else if (nmax <= 8192) k_sw_small<8192, 4, BAT, LAB, WIDE, WAVES><<<grid, WAVES * 64, 0, s>>>(ca);
  else k_sw_small<DIRECT_N, 2, BAT, LAB, WIDE, WAVES><<<grid, WAVES * 64, 0, s>>>(ca);
}
template <bool BAT, bool LAB, bool WIDE>
void launch_small(int64_t nmax, unsigned grid, int waves, const CountArgs& ca, hipStream_t s) {
  if constexpr (BAT) {
    if (waves == 1) return launch_small_of<BAT, LAB, WIDE, 1>(nmax, grid, ca, s);
    if (waves == 2) return launch_small_of<BAT, LAB, WIDE, 2>(nmax, grid, ca, s);
  }
  launch_small_of<BAT, LAB, WIDE, REST_WAVES>(nmax, grid, ca, s);
}

// ------------------------------------------------------------------- results

__global__ void k_sw_finish(const unsigned long long* __restrict__ acc, uint32_t* __restrict__ err, int64_t nnz,
                            uint64_t n, uint64_t clo, uint64_t chi, uint64_t* __restrict__ out,
                            uint64_t* __restrict__ status) {
  stamp(status + SW_CLK, 3);
  __shared__ uint64_t sum[SW_WORDS];
  if (threadIdx.x < SW_WORDS) {
    uint64_t t = 0;
    for (int k = 0; k < SW_COPIES; ++k) t += acc[k * SW_WORDS + threadIdx.x];
    sum[threadIdx.x] = t;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  uint32_t e = err[0] | err[1] | err[2];
  if (!e && (int64_t)sum[SW_ABOVE] * 2 != nnz) e = ERR_ASYM;
  status[17] = e;
  if (e) return;  // an error writes no output
  uint64_t c[16];
  for (int k = 0; k < 16; ++k) c[k] = sum[k];
  c[2] += n * (sum[SUMS_MUT] / 2);
  open_wedges(c);
  uint64_t s = 0;
  for (int k = 1; k < 16; ++k) {
    status[k] = out[k] = c[k];
    s += c[k];
  }
  status[0] = out[0] = clo - s;
  status[16] = out[16] = chi - (clo < s ? 1u : 0u);
  stamp(status + SW_CLK, 4);
}

// Labelled: a triangle a < b < c takes its three pairs of neighbours out of the
// wedge states and gives the common neighbour back to the dyads of its edges
// (bc with the third vertex below, ac between, ab above).
__global__ void k_sw_finish_lab(const unsigned long long* __restrict__ acc, uint32_t* __restrict__ err, int64_t nnz,
                                uint64_t clo, uint64_t chi, uint64_t* __restrict__ out,
                                uint64_t* __restrict__ status) {
  stamp(status + SW_CLK, 3);
  __shared__ uint64_t c[SW_LAB_WORDS];
  for (int i = threadIdx.x; i < SW_LAB_WORDS; i += blockDim.x) {
    uint64_t t = 0;
    for (int k = 0; k < SW_COPIES; ++k) t += acc[k * SW_LAB_WORDS + i];
    c[i] = t;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  uint32_t e = err[0] | err[1] | err[2];
  if (!e && (int64_t)c[SW_LAB_ABOVE] * 2 != nnz) e = ERR_ASYM;
  status[65] = e;
  if (e) return;  // an error writes no output
  for (uint32_t st = 21; st < 64; ++st) {
    const uint32_t ab = st & 3u, ac = st >> 2 & 3u, bc = st >> 4;
    if (!ab || !ac || !bc) continue;
    const uint64_t t = c[st];
    c[ab | ac << 2] -= t;
    c[ab | bc << 4] -= t;
    c[ac << 2 | bc << 4] -= t;
    c[ab] += t;
    c[ac << 2] += t;
    c[bc << 4] += t;
  }
  uint64_t s = 0;
  for (int k = 1; k < 64; ++k) {
    status[k] = out[k] = c[k];
    s += c[k];
  }
  status[0] = out[0] = clo - s;
  status[64] = out[64] = chi - (clo < s ? 1u : 0u);
  stamp(status + SW_CLK, 4);
}

// Per graph: the classes from its sums; 003 = C(n_g, 3) less the rest (n_g <
// 4,801,281 keeps C(n_g, 3) below 2^64). err[3] keeps the batch's error bits.
__global__ void k_sw_finish_batch(int32_t graphs, int64_t nnz, const int64_t* __restrict__ vbase,
                                  const unsigned long long* __restrict__ gacc,
                                  const unsigned long long* __restrict__ acc, uint32_t* __restrict__ err,
                                  uint64_t* __restrict__ out) {
  uint64_t above = threadIdx.x < SW_COPIES ? acc[threadIdx.x * SW_WORDS + SW_ABOVE] : 0;
  __shared__ uint64_t part[4];
  above = sum64(above);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = above;
  __syncthreads();
  uint32_t e = err[0] | err[1];
  if (!e && (int64_t)(part[0] + part[1] + part[2] + part[3]) * 2 != nnz) e = ERR_ASYM;
  if (blockIdx.x == 0 && threadIdx.x == 0) err[3] = e;
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= graphs || e) return;  // an error writes no output
  const uint64_t n = (uint64_t)(vbase[g + 1] - vbase[g]);
  uint64_t c3 = 0;
  if (n >= 3) {
    // n(n-1)(n-2)/6 without overflow: divide the factors first
    uint64_t x = n, y = n - 1, z = n - 2;
    if (x % 2 == 0) x /= 2; else y /= 2;
    if (x % 3 == 0) x /= 3; else if (y % 3 == 0) y /= 3; else z /= 3;
    c3 = x * y * z;
  }
  uint64_t c[16];
  for (int k = 1; k < 16; ++k) c[k] = gacc[16 * (uint64_t)g + k];
  c[2] += n * (gacc[16 * (uint64_t)g] / 2);
  open_wedges(c);
  uint64_t s = 0;
  for (int k = 1; k < 16; ++k) {
    out[16 * (uint64_t)g + k] = c[k];
    s += c[k];
  }
  out[16 * (uint64_t)g] = c3 - s;
}

// Symmetry check: every entry's mirror with swapped direction bits.
__global__ void k_sw_symmetry(int64_t n, int64_t nnz, const int64_t* __restrict__ off, const int32_t* __restrict__ nbr,
                              const uint8_t* __restrict__ flg, uint32_t* __restrict__ err) {
  if (err[0]) return;
  const int64_t nw = (int64_t)gridDim.x * (blockDim.x >> 6);
  const int lane = threadIdx.x & 63;
  bool bad = false;
  for (int64_t x = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); x < n; x += nw) {
    const int64_t b = off[x], e = off[x + 1];
    for (int64_t j = b + lane; j < e; j += 64) {
      const int32_t y = nbr[j];
      if (y < 0 || y >= n) continue;  // an entry check reports it
      const uint32_t f = (flg[j >> 2] >> (2 * (j & 3))) & 3u;
      int64_t lo = off[y], hi = off[y + 1];
      const int64_t end = hi;
      while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (nbr[mid] < (int32_t)x) lo = mid + 1; else hi = mid;
      }
      if (lo >= end || nbr[lo] != (int32_t)x ||
          ((flg[lo >> 2] >> (2 * (lo & 3))) & 3u) != (((f & 1u) << 1) | (f >> 1)))
        bad = true;
    }
  }
  if (bad) atomicOr(&err[2], ERR_ASYM);
}

unsigned grid_of_work(int64_t work, int per, int64_t cap) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>((work + per - 1) / per, cap));
}

}  // namespace

int sweep_census(const SweepIn& in, bool validate, bool labelled, unsigned long long** acc_out, uint32_t** err_out, Scratch& scratch,
                 uint64_t* status, hipStream_t s) {
  uint64_t* clk = status + SW_CLK;
  const int64_t n = in.n, nnz = in.nnz;
  DeviceInfo di;
  if (int st = device_info(&di)) return st;
  const bool rank = n > DIRECT_N;
  const int64_t ntiles = (nnz + OT - 1) / OT;
  // everything that starts at zero, in one block
  int64_t words = 0;
  auto place = [&](int64_t w) {
    const int64_t at = words;
    words += (w + 1) & ~(int64_t)1;
    return at;
  };
  const int64_t w_acc = place(2 * (labelled ? SW_LAB_WORDS : SW_WORDS) * SW_COPIES), w_err = place(SW_ERRS), w_cnt = place(10);
  const int64_t w_hist = place(rank ? 2 * BUCKETS : 0);
  const int64_t w_cross = place((ntiles + 1) * (int64_t)(sizeof(Cross) / 4));
  const int64_t w_mark = place(ntiles * (OT / 32));
  uint32_t* zero = nullptr;
  ALLOC(zero, words);
  unsigned long long* acc = (unsigned long long*)(zero + w_acc);
  uint32_t* err = zero + w_err;
  *acc_out = acc;
  *err_out = err;
  k_sw_zero<<<grid_of_work(words, 1024, 2048), 256, 0, s>>>(zero, words, clk);
  if (n == 0) return TRIAD_OK;
  uint32_t *key = nullptr, *list = nullptr, *tile_row = nullptr, *mid = nullptr, *lng = nullptr;
  uint64_t *info = nullptr, *hub_items = nullptr, *mid_items = nullptr, *dense_items = nullptr;
  SegCounts* segs = nullptr;
  if (labelled) ALLOC(segs, 2 * ntiles);
  ALLOC(key, n);
  ALLOC(info, n);
  ALLOC(list, nnz + LIST_PAD);
  ALLOC(tile_row, ntiles);
  if (rank) {
    ALLOC(mid, nnz / SORT_MIN + 1);
    ALLOC(lng, nnz / SORT_MID + 1);
    // an in-list of `minus` entries makes at most minus / CHUNK + 1 items, and
    // only in-lists of MID_MIN_IN entries (hubs: HUB_MIN_IN) or N+ of more than
    // TAB_MAX make any
    ALLOC(hub_items, std::min(std::min(n, HUB_RANKS), nnz / HUB_MIN_IN) + nnz / CHUNK + 1);
    ALLOC(mid_items, std::min(n, nnz / MID_MIN_IN<true> + nnz / TAB_MAX) + nnz / CHUNK + 1);
    ALLOC(dense_items, nnz / TAB_MAX + nnz / CHUNK + 1);
  }
  const RowArgs ra{n, nnz, in.off, rank ? nullptr : key, rank ? zero + w_hist : nullptr, info, list, zero + w_mark,
                   tile_row, err, 0, nullptr, nullptr, in.nbr, labelled ? (Cross*)(zero + w_cross) : nullptr};
  // (16 rows a thread: fewer atomics on the bucket counters; 4 while that
  // leaves fewer workgroups than four a CU. 2^26 vertices in 2^25 pairs: 6.02 ms
  // with 16, 6.60 with 4; 2^24, R-MAT: 42.3 and 42.2)
  const bool many = n > (int64_t)di.cus * 4 * ROWS_THREADS * 16;
  const unsigned rgrid = grid_of_work(n, ROWS_THREADS * (many ? 16 : 4), INT32_MAX);
  if (!rank) k_sw_rows<1><<<grid_of_work(n, 256, INT32_MAX), 256, 0, s>>>(ra);
  else if (many) k_sw_rows<16><<<rgrid, ROWS_THREADS, 0, s>>>(ra);
  else k_sw_rows<4><<<rgrid, ROWS_THREADS, 0, s>>>(ra);
  if (nnz == 0) return TRIAD_OK;
  if (rank) {
    uint32_t* hist = zero + w_hist;
    if (many) k_sw_rank<16><<<rgrid, ROWS_THREADS, 0, s>>>(n, in.off, hist, hist + BUCKETS, key, err);
    else k_sw_rank<4><<<rgrid, ROWS_THREADS, 0, s>>>(n, in.off, hist, hist + BUCKETS, key, err);
  }
  if (validate)
    k_sw_symmetry<<<grid_of_work(n, 4, 65536), 256, 0, s>>>(n, nnz, in.off, in.nbr, in.flg, err);
  const OrientArgs oa{n,        nnz,  ntiles, in.off, in.nbr, in.flg, key, zero + w_mark, tile_row, list, info,
                      (Cross*)(zero + w_cross), mid, lng, zero + w_cnt, acc, err, nullptr, nullptr, nullptr};
  const unsigned ogrid = grid_of_work(ntiles, 1, (int64_t)di.cus * 8);
  const unsigned cgrid = grid_of_work(ntiles, 256, 256);
  CountArgs ca{n, nnz, ntiles, in.off, list, info, key, tile_row, {hub_items, mid_items, dense_items}, clk, zero + w_cnt, 0, 0, acc, err,
               nullptr, nullptr, nullptr, nullptr, nullptr, 0};
  // N+ packed for the hubs: at most as many units as entries (two for two; half
  // of all of them in a symmetric graph), whose byte offsets take 32 bits. R-MAT, by
  // entries, not packed / packed, us: 1.7 M 304 / 316, 3.4 M 434 / 441, 5.4 M 541 /
  // 543, 7.6 M 690 / 672, 14.8 M 1,154 / 1,077, 31 M 2,338 / 2,053; 521 M 51.2 / 42.2
  // ms. With fewer than two entries a vertex its scratch could pass the documented bound.
  const bool pack = rank && !labelled && nnz >= 2 * n && nnz >= PACK_MIN && nnz < (int64_t)1 << 29;
  if (pack) {
    ALLOC(ca.prow, n);
    ca.units = (uint32_t)(nnz / 2 + 16);
    ALLOC(ca.pack, ca.units);
  }
  // a wavefront's range: small graphs spread over the chip, large ones in
  // ranges that spread the row search over more entries
  const int64_t waves = (int64_t)di.cus * (rank ? 32 : 16);
  ca.range = std::max<int64_t>(64, std::min<int64_t>(rank ? 1024 : 512, (nnz / waves + 63) & ~(int64_t)63));
  const unsigned wgrid = grid_of_work((nnz + ca.range - 1) / ca.range, REST_WAVES, (int64_t)di.cus * 8);
  if (labelled) {
    const LabArgs la{n, nnz, ntiles, in.off, in.nbr, in.flg, zero + w_mark, tile_row, list, (Cross*)(zero + w_cross),
                     segs, acc, err};
    k_lab_sums<<<ogrid, OTHREADS, 0, s>>>(la);
    k_lab_cross<<<grid_of_work(ntiles, 4, 2048), 256, 0, s>>>(la);
  }
  const int rank_bits = n > 1 ? 64 - __builtin_clzll((unsigned long long)(n - 1)) : 1;
  auto run = [&](auto lab) {
    constexpr bool LAB = decltype(lab)::value;
    if (rank) {
      k_sw_orient<true, false, LAB><<<ogrid, OTHREADS, 0, s>>>(oa);
      k_sw_cross<true, false, LAB><<<cgrid, 256, 0, s>>>(oa);
      k_sw_items<false, LAB><<<grid_of_work(n, 4096, 4096), 256, 0, s>>>(ca);
      // (2^24 vertices 42.2 ms with 8 a thread, 42.6 with one; 600,011 1.11 and 1.12;
      // 300,007 0.876 and 0.848)
      if (pack && n > 1 << 19) k_sw_pack<8><<<grid_of_work(n, 2048, INT32_MAX), 256, 0, s>>>(ca);
      else if (pack) k_sw_pack<1><<<grid_of_work(n, 256, INT32_MAX), 256, 0, s>>>(ca);
      const Packed pk{pack ? ca.prow : nullptr, ca.pack, ca.counts + 2};
      k_sw_sort_mid<<<grid_of_work(nnz / SORT_MIN, 4, (int64_t)di.cus * 8), 256, 0, s>>>(mid, zero + w_cnt, info, list, err, LAB ? 3 : 2, pk);
      k_sw_sort_long<<<grid_of_work(nnz / SORT_MID, 1, (int64_t)di.cus * 8), 256, 0, s>>>(lng, zero + w_cnt + 1, info, list, err, rank_bits, pk);
      auto count = [&](auto wide) {
        constexpr bool W = decltype(wide)::value;
        if constexpr (!LAB && !W) {
          if (pack) {
            k_sw_hubs<false, false, true><<<(unsigned)(di.cus * 2), hub_threads(false), 0, s>>>(ca);
          } else {
            k_sw_hubs<false, false, false><<<(unsigned)(di.cus * 2), hub_threads(false), 0, s>>>(ca);
          }
        } else {
          k_sw_hubs<LAB, W, false><<<(unsigned)(di.cus * 2), hub_threads(LAB), 0, s>>>(ca);
        }
        k_sw_mids<LAB, W><<<(unsigned)(di.cus * (LAB ? 4 : 6)), MID_THREADS, 0, s>>>(ca);
        // (an N+ of more than TAB_MAX entries takes as many rows of about its degree)
        if (n > HUB_RANKS && nnz >= (int64_t)TAB_MAX * TAB_MAX / 2) k_sw_dense<false, LAB, W, DENSE_WORDS><<<(unsigned)di.cus, DENSE_THREADS, 0, s>>>(ca);
        k_sw_rest<true, false, LAB, W><<<wgrid, REST_WAVES * 64, 0, s>>>(ca);
      };
      if (nnz + LIST_PAD < ((int64_t)1 << 30)) count(std::false_type{}); else count(std::true_type{});
    } else {
      // (n <= DIRECT_N: fewer than 2^28 entries)
      k_sw_orient<false, false, LAB><<<ogrid, OTHREADS, 0, s>>>(oa);
      k_sw_cross<false, false, LAB><<<cgrid, 256, 0, s>>>(oa);
      launch_small<false, LAB, false>(n, wgrid, REST_WAVES, ca, s);
    }
  };
  if (labelled) run(std::true_type{}); else run(std::false_type{});
  HIPCHK(hipGetLastError());
  return TRIAD_OK;
}

// A batch: the pieces of its scratch block in order (sizes in bytes, rounded
// up as Scratch hands them out).
struct BatchSizes {
  int64_t ntiles, dense_items, zero_words, w_err, w_cnt, w_gacc, w_cross, w_mark;
  BatchSizes(int32_t graphs, int64_t nnz) {
    ntiles = (nnz + OT - 1) / OT;
    dense_items = nnz / DENSE_MIN_IN + nnz / TAB_MAX + nnz / CHUNK + 1;
    zero_words = 0;
    auto place = [&](int64_t w) {
      const int64_t at = zero_words;
      zero_words += (w + 1) & ~(int64_t)1;
      return at;
    };
    place(2 * SW_WORDS * SW_COPIES);  // acc first
    w_err = place(SW_ERRS);
    // Atomics on 64 bytes queue: a graph's triangle counters (8, 9, 11 .. 15) fall
    // three and four into two such pieces when the first counter is 32 bytes into
    // one (85 graphs of up to 455 vertices 92 us; at 48 bytes, two and five, 97; at 56
    // 105; at 0, all seven, 112; 64 of up to 4,000: 190, 212, 219, 237).
    w_cnt = place(20);
    w_gacc = place(32 * (int64_t)graphs);
    static_assert((2 * SW_WORDS * SW_COPIES + SW_ERRS + 20) % 16 == 8, "see above");
    w_cross = place((ntiles + 1) * (int64_t)(sizeof(Cross) / 4));
    w_mark = place(ntiles * (OT / 32));
  }
};

size_t sweep_batch_bytes(int32_t graphs, int64_t nv, int64_t nnz) {
  const BatchSizes z(graphs, nnz);
  auto r = [](int64_t b) { return (size_t)((std::max<int64_t>(b, 1) + 255) & ~(int64_t)255); };
  return r(4 * z.zero_words) + 2 * r(4 * nv) + r(8 * nv) + r(4 * (nnz + LIST_PAD)) + r(4 * z.ntiles) +
         r(8 * z.dense_items);
}

int sweep_batch_groups(int waves) {
  DeviceInfo di;
  if (device_info(&di) != TRIAD_OK) return 1024;
  return di.cus * 64 / waves;
}

int sweep_batch(int32_t graphs, int64_t nv, const SweepIn& in, const int64_t* vbase, int64_t nmax, int waves,
                int groups, int64_t range, uint64_t* d_out, uint32_t** err_out, Scratch& scratch, hipStream_t s) {
  const int64_t nnz = in.nnz;
  const BatchSizes z(graphs, nnz);
  uint32_t *zero = nullptr, *key = nullptr, *grow = nullptr, *list = nullptr, *tile_row = nullptr;
  uint64_t *info = nullptr, *dense_items = nullptr;
  ALLOC(zero, z.zero_words);
  ALLOC(key, nv);
  ALLOC(grow, nv);
  ALLOC(info, nv);
  ALLOC(list, nnz + LIST_PAD);
  ALLOC(tile_row, z.ntiles);
  ALLOC(dense_items, z.dense_items);
  unsigned long long* acc = (unsigned long long*)zero;
  unsigned long long* gacc = (unsigned long long*)(zero + z.w_gacc);
  uint32_t* err = zero + z.w_err;
  *err_out = err + 3;
  k_sw_zero<<<grid_of_work(z.zero_words, 1024, 2048), 256, 0, s>>>(zero, z.zero_words, nullptr);
  if (nv > 0) {
    const RowArgs ra{nv, nnz, in.off, key, nullptr, info, list, zero + z.w_mark, tile_row, err, graphs, vbase, grow,
                     nullptr, nullptr};
    k_sw_rows<1><<<grid_of_work(nv, 256, INT32_MAX), 256, 0, s>>>(ra);
  }
  if (nv > 0 && nnz > 0) {
    DeviceInfo di;
    if (int st = device_info(&di)) return st;
    const OrientArgs oa{nv, nnz, z.ntiles, in.off, in.nbr, in.flg, key, zero + z.w_mark, tile_row, list, info,
                        (Cross*)(zero + z.w_cross), nullptr, nullptr, zero + z.w_cnt, acc, err, vbase, grow, gacc};
    k_sw_orient<false, true, false><<<grid_of_work(z.ntiles, 1, (int64_t)di.cus * 8), OTHREADS, 0, s>>>(oa);
    k_sw_cross<false, true, false><<<grid_of_work(z.ntiles, 256, 256), 256, 0, s>>>(oa);
    CountArgs ca{nv, nnz, z.ntiles, in.off, list, info, key, tile_row, {nullptr, nullptr, dense_items}, nullptr, zero + z.w_cnt, range, 0, acc,
                 err, vbase, grow, gacc};
    // (by default 2,048 entries a turn, fewer where that leaves less than four
    // turns a wavefront; 4,096 graphs, 3e8 edges: 19.5 ms with 512, 17.5 with
    // these and twice the workgroups; 256 graphs of up to 1,024 vertices: 0.24
    // with 2,048, 0.21 with fewer)
    if (range <= 0) range = std::max<int64_t>(64, std::min<int64_t>(2048, (nnz / (di.cus * 64) + 63) & ~(int64_t)63));
    ca.range = range;
    const bool low = nmax <= DENSE_RANKS<false, DENSE_LOW>;
    ca.window = low ? DENSE_RANKS<false, DENSE_LOW> : DENSE_RANKS<false>;
    const unsigned grid = grid_of_work((nnz + range - 1) / range, waves, groups);
    auto count = [&](auto wide) {
      constexpr bool W = decltype(wide)::value;
      if (nmax <= DIRECT_N) {
        launch_small<true, false, W>(nmax, grid, waves, ca, s);
      } else {
        k_sw_items<true, false><<<grid_of_work(nv, 4096, 4096), 256, 0, s>>>(ca);
        if (low) k_sw_dense<true, false, W, DENSE_LOW><<<(unsigned)di.cus * 4, DENSE_THREADS / 4, 0, s>>>(ca);
        else k_sw_dense<true, false, W, DENSE_WORDS><<<(unsigned)di.cus, DENSE_THREADS, 0, s>>>(ca);
        k_sw_rest<false, true, false, W><<<grid, waves * 64, 0, s>>>(ca);
      }
    };
    if (nnz + LIST_PAD < ((int64_t)1 << 30)) count(std::false_type{}); else count(std::true_type{});
  }
  k_sw_finish_batch<<<grid_of_work(graphs, 256, INT32_MAX), 256, 0, s>>>(graphs, nnz, vbase, gacc, acc, err, d_out);
  return TRIAD_OK;
}

void sweep_finish(const unsigned long long* acc, uint32_t* err, bool labelled, int64_t nnz, int64_t n,
                  uint64_t* d_out, uint64_t* status, hipStream_t s) {
  uint64_t clo, chi;
  choose3(n, &clo, &chi);
  if (labelled) k_sw_finish_lab<<<1, 128, 0, s>>>(acc, err, nnz, clo, chi, d_out, status);
  else k_sw_finish<<<1, 64, 0, s>>>(acc, err, nnz, (uint64_t)n, clo, chi, d_out, status);
}

}  // namespace triad
