// Directed triad census on CDNA4 (gfx950): kernels and the single-graph
// pipeline behind triad_census_device().
//
// Pipeline (one HIP stream; the host reads two sizes on the way):
//   k_rows      per row u: offset checks, first entry > u (binary search on the
//               sorted row), self-loop check, tasks(u) = entries above u
//   k_entries   per entry: neighbour/flag checks, sortedness, and the packed
//               word id << 2 | flag (the compact id+direction encoding of
//               Sec. 6 / Fig. 7, built once on the device)
//   scan        exclusive prefix of tasks(u): the collapsed (u,v) task space
//               of Fig. 5 steps 2 and 2.1
//   k_emit_entries  task list in CSR order, one thread per entry; tasks whose
//               merge length d(u)+d(v) exceeds the hub threshold are flagged.
//               The entries below their row's id are listed as (id, index)
//               pairs, which a stable radix sort by id puts in task order:
//               their indices are the tasks' counts of N(v) ids below u
//               (k_low_words; the no-allocation census searches u in N(v)
//               per task instead). k_hub_list lists the flagged tasks.
//   k_census    persistent wavefronts: hub chunks first, then tasks; each
//               item merges a range of N(u) with a range of N(v)
//   k_finalize  the common-neighbour part of 012 and 102 from the triangle
//               classes; 003 = C(n,3) - sum of the rest, in two 64-bit words
// The batched census (many graphs in one captured launch) and the labelled
// (64-state) census can use the same kernels; by default graphs and batches
// take the triangle listing of sweep.hip instead.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <type_traits>
#include <vector>

#include "device_sort.h"
#include "sweep.h"
#include "tile_rows.h"
#include "triad_internal.h"

namespace triad {

constexpr uint32_t KEY_INF = 0xFFFFFFFFu;  // larger than any key (ids < 2^30 - 1)

__device__ __forceinline__ uint32_t key_of(uint32_t p) { return p | 3u; }

__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

__device__ __forceinline__ uint32_t bcast32(uint32_t x, int lane) {
  return (uint32_t)__builtin_amdgcn_readlane((int)x, lane);
}
__device__ __forceinline__ uint64_t bcast64(uint64_t x, int lane) {
  uint32_t lo = bcast32((uint32_t)x, lane), hi = bcast32((uint32_t)(x >> 32), lane);
  return ((uint64_t)hi << 32) | lo;
}
// Marks a wave-uniform value as such for the compiler, which otherwise keeps
// loop state that passes through divergent code in vector registers.
__device__ __forceinline__ uint32_t uni(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }

__device__ __forceinline__ uint64_t wave_sum64(uint64_t x) {
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// ------------------------------------------------------------------ checks

// Per row: offsets monotone, first entry above u, self-loop, task count.
__global__ void k_rows(int64_t n, int64_t nnz, const int64_t* __restrict__ off, const int32_t* __restrict__ nbr,
                       uint32_t* __restrict__ ustart, int64_t* __restrict__ ntask, uint32_t* __restrict__ rowmark,
                       uint32_t* __restrict__ err) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < n; u += stride) {
    int64_t b = off[u], e = off[u + 1];
    if (u == 0 && b != 0) atomicOr(err, ERR_RANGE);
    if (u == n - 1 && e != nnz) atomicOr(err, ERR_RANGE);
    if (e < b || b < 0 || e > nnz || e - b >= ((int64_t)1 << 31)) {
      atomicOr(err, ERR_RANGE);
      ustart[u] = 0;
      ntask[u] = 0;
      continue;
    }
    // first position with nbr > u (rows are sorted; checked by k_entries)
    int64_t lo = b, hi = e;
    while (lo < hi) {
      int64_t mid = (lo + hi) >> 1;
      if (nbr[mid] <= (int32_t)u) lo = mid + 1; else hi = mid;
    }
    if (lo > b && nbr[lo - 1] == (int32_t)u) atomicOr(err, ERR_SELFLOOP);
    ustart[u] = (uint32_t)(lo - b);
    ntask[u] = e - lo;
    if (e > b) atomicOr(&rowmark[b >> 5], 1u << (b & 31));
  }
}

// Per entry: id range, non-zero flag, strictly increasing rows; packed words.
__global__ void k_entries(int64_t n, int64_t nnz, const int32_t* __restrict__ nbr, const uint8_t* __restrict__ flg,
                          const uint32_t* __restrict__ rowmark, uint32_t* __restrict__ packed,
                          uint32_t* __restrict__ err) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  uint32_t bits = 0;
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < nnz; j += stride) {
    int32_t y = nbr[j];
    uint32_t f = (flg[j >> 2] >> (2 * (j & 3))) & 3u;
    if (y < 0 || y >= n || f == 0) bits |= ERR_RANGE;
    if (j + 1 < nnz) {
      bool row_start = (rowmark[(j + 1) >> 5] >> ((j + 1) & 31)) & 1u;
      if (!row_start && nbr[j + 1] <= y) bits |= ERR_UNSORTED;
    }
    packed[j] = ((uint32_t)y << 2) | f;
  }
  if (bits) atomicOr(err, bits);
}

// Full validation: every entry has its mirror with swapped direction bits.
__global__ void k_symmetry(int64_t n, const int64_t* __restrict__ off, const uint32_t* __restrict__ packed,
                           const uint32_t* __restrict__ err_in, uint32_t* __restrict__ err) {
  if (*err_in) return;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n; x += stride) {
    for (int64_t j = off[x]; j < off[x + 1]; ++j) {
      uint32_t p = packed[j];
      uint32_t y = p >> 2, f = p & 3u;
      int64_t lo = off[y], hi = off[y + 1];
      uint32_t want = ((uint32_t)x << 2) | 3u;
      while (lo < hi) {
        int64_t mid = (lo + hi) >> 1;
        if (key_of(packed[mid]) < want) lo = mid + 1; else hi = mid;
      }
      uint32_t g = ((f & 1u) << 1) | (f >> 1);
      if (lo >= off[y + 1] || packed[lo] != (((uint32_t)x << 2) | g)) {
        atomicOr(err, ERR_ASYM);
        return;
      }
    }
  }
}

// ---------------------------------------------------------- exclusive scan
// out[0..m] = exclusive prefix of in[0..m) (out[m] = total). Three passes:
// block sums, a single-block scan of the block sums, block-local scans.
constexpr int SCAN_T = 256, SCAN_I = 16, SCAN_B = SCAN_T * SCAN_I;

__device__ int64_t block_excl_scan(int64_t v, int64_t* sh, int64_t* total) {
  // sh: SCAN_T/64 + 1 slots
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int64_t x = v;
  for (int o = 1; o < 64; o <<= 1) {
    int64_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) sh[w] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t run = 0;
    for (int k = 0; k < SCAN_T / 64; ++k) {
      int64_t t = sh[k];
      sh[k] = run;
      run += t;
    }
    sh[SCAN_T / 64] = run;
  }
  __syncthreads();
  int64_t r = x - v + sh[w];
  *total = sh[SCAN_T / 64];
  __syncthreads();
  return r;
}

__global__ void k_scan_sums(const int64_t* __restrict__ in, int64_t m, int64_t* __restrict__ bsum) {
  __shared__ int64_t sh[SCAN_T / 64 + 1];
  const int64_t base = (int64_t)blockIdx.x * SCAN_B + threadIdx.x;
  int64_t s = 0;
  for (int k = 0; k < SCAN_I; ++k)
    if (base + k * SCAN_T < m) s += in[base + k * SCAN_T];
  int64_t tot;
  block_excl_scan(s, sh, &tot);
  if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

__global__ void k_scan_top(int64_t* __restrict__ bsum, int64_t nb) {
  __shared__ int64_t sh[SCAN_T / 64 + 1];
  int64_t carry = 0;
  for (int64_t c = 0; c < nb; c += SCAN_B) {
    int64_t base = c + (int64_t)threadIdx.x * SCAN_I, loc[SCAN_I], s = 0;
    for (int k = 0; k < SCAN_I; ++k) {
      loc[k] = (base + k < nb) ? bsum[base + k] : 0;
      s += loc[k];
    }
    int64_t tot, ex = block_excl_scan(s, sh, &tot);
    int64_t run = carry + ex;
    for (int k = 0; k < SCAN_I; ++k)
      if (base + k < nb) { bsum[base + k] = run; run += loc[k]; }
    carry += tot;
  }
}

// in may be out: a thread reads its values before it writes them.
__global__ void k_scan_apply(const int64_t* in, int64_t m, const int64_t* __restrict__ bsum, int64_t* out) {
  __shared__ int64_t sh[SCAN_T / 64 + 1];
  int64_t base = (int64_t)blockIdx.x * SCAN_B + (int64_t)threadIdx.x * SCAN_I, loc[SCAN_I], s = 0;
  for (int k = 0; k < SCAN_I; ++k) {
    loc[k] = (base + k < m) ? in[base + k] : 0;
    s += loc[k];
  }
  int64_t tot, run = block_excl_scan(s, sh, &tot) + bsum[blockIdx.x];
  for (int k = 0; k < SCAN_I; ++k)
    if (base + k < m) { out[base + k] = run; run += loc[k]; }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == SCAN_T - 1) out[m] = run;
}

// --------------------------------------------------------------- task list

// Task list in CSR order: the tasks of row u are its entries above u, written
// as (u << 32 | local index), each with its count of N(v) ids below u; tasks
// longer than the hub threshold are flagged and listed afterwards
// (k_hub_list, one atomic per tile of tasks).
struct EmitArgs {
  int64_t n;
  const int64_t* off;
  const uint32_t* packed;
  const uint32_t* ustart;
  const int64_t* tpre;
  uint64_t* tasks;
  uint32_t* tskip;        // per task: entries of N(v) below u
  // 1: tskip by a search of u in N(v); 0: no search, tskip gets 0 (the merge
  // then takes all of N(v)), or nothing when `lower` is given (its sort does)
  int32_t count_below;
  int64_t hub_threshold;  // < 0: no hub tasks
  const uint32_t* err;
  // optional: every entry below its row's own id, as (id << 32 | index in the
  // row), at lpre[row] + index (lpre: exclusive prefix of those counts)
  uint64_t* lower;
  const int64_t* lpre;
};

// One task per active lane: row u (entries from b, degree du), k = index of v
// in the row, t = task index. Also records how many ids of N(v) lie below u
// (binary search in N(v)): a whole task's merge starts N(v) at u. With the
// lower entries listed (e.lower), those counts come from their sort instead.
__device__ __forceinline__ void emit_task(const EmitArgs& e, bool act, int64_t u, int64_t b, int64_t du, uint32_t k,
                                          int64_t t) {
  if (!act) return;
  uint64_t tk = ((uint64_t)u << 32) | k;
  const uint32_t v = e.packed[b + k] >> 2;
  const int64_t bv = e.off[v];
  const uint32_t dv = (uint32_t)(e.off[v + 1] - bv);
  if (e.hub_threshold >= 0 && du + dv > e.hub_threshold) tk |= HUB_BIT;
  e.tasks[t] = tk;
  // ids of N(v) below u
  const uint32_t key = (uint32_t)u << 2;
  uint32_t lo = 0, len = e.count_below ? dv : 0u;
  while (len > 0) {
    const uint32_t half = len >> 1;
    if (e.packed[bv + lo + half] < key) {
      lo += half + 1;
      len -= half + 1;
    } else {
      len = half;
    }
  }
  if (!e.lower) e.tskip[t] = lo;
}

// Hub list: the flagged tasks, compacted with one atomic per tile of HUB_TILE
// tasks (list order is free), with the chunk count of each.
constexpr int HUB_TILE = 256 * 16;
__global__ void __launch_bounds__(256) k_hub_list(const uint64_t* __restrict__ tasks, int64_t ntasks,
                                                  const int64_t* __restrict__ off, const uint32_t* __restrict__ packed,
                                                  const uint32_t* __restrict__ ustart, const uint32_t* __restrict__ tskip,
                                                  int64_t chunk, uint64_t* __restrict__ hub_task,
                                                  int64_t* __restrict__ hub_nch, unsigned long long* __restrict__ hub_count,
                                                  const uint32_t* __restrict__ err) {
  if (*err) return;
  __shared__ unsigned int wsum[4];
  __shared__ unsigned long long base;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int64_t t0 = (int64_t)blockIdx.x * HUB_TILE; t0 < ntasks; t0 += (int64_t)gridDim.x * HUB_TILE) {
    // each wavefront counts its quarter of the tile, 64 tasks per step
    const int64_t q0 = t0 + (int64_t)w * (HUB_TILE / 4), q1 = min(q0 + HUB_TILE / 4, ntasks);
    unsigned int c = 0;
    for (int64_t t = q0 + lane; t - lane < q1; t += 64)
      c += (unsigned int)__popcll(__ballot(t < q1 && (tasks[t] & HUB_BIT)));
    if (lane == 0) wsum[w] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
      const unsigned int tot = wsum[0] + wsum[1] + wsum[2] + wsum[3];
      base = tot ? atomicAdd(hub_count, (unsigned long long)tot) : 0ull;
    }
    __syncthreads();
    uint64_t slot = base;
    for (int i = 0; i < w; ++i) slot += wsum[i];
    for (int64_t t = q0 + lane; t - lane < q1; t += 64) {
      const uint64_t tk = t < q1 ? tasks[t] : 0;
      const bool hub = (tk & HUB_BIT) != 0;
      const uint64_t m = __ballot(hub);
      if (hub) {
        const uint64_t h = slot + (uint64_t)__popcll(m & ((1ull << lane) - 1));
        const uint32_t u = (uint32_t)(tk >> 32) & 0x3FFFFFFFu, k = (uint32_t)tk;
        const int64_t au = off[u], du = off[u + 1] - au;
        const uint32_t v = packed[au + k] >> 2;
        // the merged length: N(u) above u and N(v) from u on
        const int64_t dv = off[v + 1] - off[v];
        const int64_t len = (du - ustart[u]) + dv - min((int64_t)tskip[t], dv);
        hub_task[h] = (uint64_t)t;
        hub_nch[h] = (len + chunk - 1) / chunk;
      }
      slot += (uint64_t)__popcll(m);
    }
    __syncthreads();
  }
}

// Task list from the CSR entries, one thread per entry: entry j of row u with
// an id above u is task tpre[u] + (j - off[u] - ustart[u]) (CSR order), with
// its hub flag and, searched or left to the sort of the lower entries, its
// count of N(v) ids below u (emit_task); an entry below u goes to the lower
// entry list when there is one. Every task is as cheap as the next, whatever
// the lengths of the rows.
// STAGED: the tile's row starts come from LDS (the sort path, whose entries do
// no global search of their own).
template <bool STAGED>
__global__ void __launch_bounds__(256) k_emit_entries(EmitArgs e, int64_t nnz) {
  __shared__ typename std::conditional<STAGED, TileRows, int64_t[2]>::type T;
  if (*e.err) return;
  for (int64_t t0 = (int64_t)blockIdx.x * ETILE; t0 < nnz; t0 += (int64_t)gridDim.x * ETILE) {
    const int64_t t1 = min(t0 + (int64_t)ETILE, nnz);
    int64_t r0 = 0, r1 = 0;
    if constexpr (STAGED) {
      tile_stage(e.off, e.n, t0, t1, T);
    } else {
      tile_rows(e.off, e.n, t0, t1, T);
      r0 = T[0];
      r1 = T[1];
    }
    for (int64_t j = t0 + threadIdx.x; j < t1; j += blockDim.x) {
      int64_t u;
      if constexpr (STAGED) u = tile_row(e.off, T, t0, j);
      else u = row_search(e.off, r0, r1 + 1, j);
      const int64_t b = e.off[u];
      const uint32_t k = (uint32_t)(j - b), su = e.ustart[u];
      if (k >= su)
        emit_task(e, true, u, b, e.off[u + 1] - b, k, e.tpre[u] + (k - su));
      else if (e.lower)
        e.lower[e.lpre[u] + k] = ((uint64_t)(e.packed[j] >> 2) << 32) | k;
    }
  }
}

// Per row: the number of its entries below its own id (as 64-bit counts for the scan).
__global__ void k_lower_counts(int64_t n, const uint32_t* __restrict__ ustart, int64_t* __restrict__ cnt) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n; x += stride) cnt[x] = ustart[x];
}

// tskip[t] = the low word of the t-th sorted lower entry.
__global__ void k_low_words(const uint64_t* __restrict__ items, int64_t m, uint32_t* __restrict__ tskip) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < m; t += stride) tskip[t] = (uint32_t)items[t];
}

static void launch_emit_entries(const EmitArgs& e, int64_t nnz, hipStream_t s) {
  const int64_t tiles = (nnz + ETILE - 1) / ETILE;
  const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>(tiles, 65536));
  if (e.lower) k_emit_entries<true><<<grid, 256, 0, s>>>(e, nnz);
  else k_emit_entries<false><<<grid, 256, 0, s>>>(e, nnz);
}

// ------------------------------------------------------------ the census

struct CensusArgs {
  int64_t n;
  const int64_t* off;
  const uint32_t* packed;
  const uint32_t* ustart;  // per row: entries below the row's own id
  const uint32_t* tskip;   // per task (indexed like tasks): entries of N(v) below u
  const uint64_t* tasks;   // the task queue
  const uint64_t* htasks;  // the task words the hub list indexes
  const int64_t* order;    // optional: queue position -> index into tasks
  int64_t ntasks;
  const uint64_t* hub_task;
  const int64_t* hub_pre;  // [nhub+1] exclusive prefix of chunk counts
  int64_t nhub;
  int64_t chunk;
  unsigned long long* qctr;  // [2]: hub items, tasks
  unsigned long long* acc;   // [16]
  uint32_t* cycles;          // optional per-task cycles
  uint64_t* wave_span;       // optional [waves][2]: realtime at wave start, end
  const uint32_t* grow;      // batched census: graph of each row
  const int64_t* vbase;      // batched census: first row of each graph
  unsigned long long* gout;  // batched census: [graphs][16] accumulators
  const uint32_t* err;
  ClassSlices cls;           // nibble idx = fa | fb << 2 -> class; idx 0 -> 0 (not counted)
  LabTables lab;             // labelled census: states of ids found in one list only
};

constexpr int PAD = 1024;   // readable entries past the end of the packed array
// rounds with at most LOP_S ids in one window and at least LOP_G in the other
// take the entry-by-entry path (lopsided_round) instead of the merged walk
constexpr uint32_t LOP_S = 64, LOP_G = 128;

// Per-wavefront LDS: two sorted windows (plus a sentinel slot each) and the
// class counters, one per (class, lane). HH = true shares each counter between
// lanes l and l+32, which the LDS serves in different halves of a wave64
// access, halving the array.
template <int W, bool HH, int NC = 16>
struct WaveLds {
  static constexpr int COLS = HH ? 32 : 64;
  static constexpr int NCLS = NC;
  // the labelled census keeps two 16-bit counters per word (states 2r and
  // 2r + 1 in row r), halving its counter array
  static constexpr int ROWS = NC == 64 ? NC / 2 : NC;
  uint32_t a[W + 1];
  uint32_t b[W + 1];
  uint32_t hist[ROWS * COLS];  // [class or state row][column]
};

// Adds d (which may be negative, as two's complement) to counter k of a
// lane's column hcol: one word per class, or half a word per labelled state.
template <int W, bool HH, int NC>
__device__ __forceinline__ void hist_add(uint32_t* hcol, uint32_t k, uint32_t d) {
  constexpr uint32_t C = WaveLds<W, HH, NC>::COLS;
  if constexpr (NC == 64)
    atomicAdd(hcol + (k >> 1) * C, d << ((k & 1u) << 4));
  else
    atomicAdd(hcol + k * C, d);
}

// Labelled counters are flushed before any 16-bit field can leave +-32767:
// a round changes a field by less than its share of `steps`, and the check
// runs every round.
constexpr uint32_t LAB_FLUSH_STEPS = 1u << 14;

// Labelled census (64 states of a triple a < b < c by id order, Sec. 3): the
// state of the triple of task (u, v) and a counted third vertex w, from the
// flags fa = f_uw (0 if w is not in N(u)) and fb = f_vw: above v the triple
// is (u, v, w) and its state f | fa << 2 | fb << 4 (f = f_uv); between u and
// v it is (u, w, v), w not adjacent to u, and its state f << 2 | f_wv << 4,
// f_wv the mirror of fb.
__device__ __forceinline__ uint32_t mirror_flag(uint32_t f) { return ((f & 1u) << 1) | (f >> 1); }
__device__ __forceinline__ uint32_t lab_state(bool above_v, uint32_t f, uint32_t fa, uint32_t fb) {
  return above_v ? (f | fa << 2 | fb << 4) : (f << 2 | mirror_flag(fb) << 4);
}

// Merge-path split of the diagonal d of A (la) and B (lb) in global memory:
// the number of A elements among the first d merged (A first on equal ids).
__device__ uint32_t global_split(const uint32_t* A, uint32_t la, const uint32_t* B, uint32_t lb, uint32_t d) {
  uint32_t lo = d > lb ? d - lb : 0, hi = d < la ? d : la;
  while (lo < hi) {
    uint32_t mid = (lo + hi) >> 1;
    if (key_of(A[mid]) <= key_of(B[d - mid - 1])) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// One batch of work items, one item per lane (lane < cnt). An item merges
// A = packed[aoff .. aoff+la) (a range of N(u)) with B = packed[boff ..
// boff+lb) (a range of N(v)). A starts at the first id of N(u) above u and,
// B at u: an id w < u is never counted (Fig. 5 step 2.1.4), and the
// intersection sizes that complete the dyadic counts follow from the triangle
// classes (k_finalize), so the ids below u are not needed. A split task's
// chunks divide that same trimmed merge.
// uf = u | kind << 30 with kind 0 = a later chunk of a split task, 1 = its
// first chunk, 2 = a whole task; the first two kinds also add their task's
// dyadic term dyad = n - d(u) - d(v) (Fig. 5 step 2.1.3). vf = v << 2 | f_uv.
struct Batch {
  int cnt;
  int64_t aoff, boff, tid;
  uint32_t la, lb, uf, vf, gid;
  int32_t dyad;
  // labelled census: the dyadic triads of the task with the third vertex
  // below u, between u and v, above v, less the common neighbours there
  int32_t dlo, dmid, dhi;
};

// Adds the batch's dyadic terms n - d(u) - d(v) (Fig. 5 step 2.1.3; the
// common-neighbour part is added by k_finalize) to counter 012 or 102 by the
// u-v dyad: one wave reduction and one atomic per counter when the whole batch
// belongs to one graph, per-lane atomics otherwise (batched census only).
template <bool BAT, bool LAB>
__device__ void add_dyads(const CensusArgs& g, int lane, const Batch& bt) {
  if constexpr (LAB) {
    // per range and u-v flag f: states f << 4 (w < u), f << 2 (u < w < v), f
    const uint32_t f = bt.vf & 3u;
#pragma unroll
    for (uint32_t ff = 1; ff <= 3; ++ff) {
      const bool mine = f == ff;  // lanes without a task, and later chunks, hold zeros
      const uint64_t lo = wave_sum64(mine ? (uint64_t)(int64_t)bt.dlo : 0);
      const uint64_t mid = wave_sum64(mine ? (uint64_t)(int64_t)bt.dmid : 0);
      const uint64_t hi = wave_sum64(mine ? (uint64_t)(int64_t)bt.dhi : 0);
      if (lane == 0) {
        if (lo) atomicAdd(&g.acc[ff << 4], (unsigned long long)lo);
        if (mid) atomicAdd(&g.acc[ff << 2], (unsigned long long)mid);
        if (hi) atomicAdd(&g.acc[ff], (unsigned long long)hi);
      }
    }
    return;
  }
  const uint64_t dv = (uint64_t)(int64_t)bt.dyad;
  const bool mut = (bt.vf & 3u) == 3u;
  const uint32_t g0 = bcast32(bt.gid, 0);
  if (!BAT || __ballot(bt.dyad != 0 && bt.gid != g0) == 0) {
    const uint64_t sa = wave_sum64(mut ? 0 : dv), sm = wave_sum64(mut ? dv : 0);
    unsigned long long* tgt = BAT ? g.gout + 16 * (uint64_t)g0 : g.acc;
    if (lane == 0) {
      if (sa) atomicAdd(&tgt[1], (unsigned long long)sa);
      if (sm) atomicAdd(&tgt[2], (unsigned long long)sm);
    }
  } else if (bt.dyad != 0) {
    atomicAdd(&g.gout[16 * (uint64_t)bt.gid + (mut ? 2 : 1)], (unsigned long long)dv);
  }
}

// Claims the next batch: hub chunks first (phase 0), then whole tasks
// (phase 1). Returns false when both queues are drained.
// Labelled census: the dyadic terms of task (u, v) by range of w, less the
// common neighbours in each range (added back from the triangle states at the
// end): k = index of v in row u, su = ids of N(u) below u, sv = ids of N(v)
// below u, dvm = ids of N(v) below v.
__device__ __forceinline__ void lab_dyads(Batch& bt, int64_t n, int64_t u, int64_t v, int64_t du, int64_t k, int64_t su,
                                          int64_t sv, int64_t dv, int64_t dvm) {
  bt.dlo = (int32_t)(u - su - sv);
  bt.dmid = (int32_t)((v - u - 1) - (k - su) - (dvm - sv - 1));
  bt.dhi = (int32_t)((n - 1 - v) - (du - k - 1) - (dv - dvm));
}

template <bool BAT, bool LAB>
__device__ bool fetch_batch(const CensusArgs& g, int lane, int& phase, Batch& bt) {
  const int64_t hub_items = g.nhub ? g.hub_pre[g.nhub] : 0;
  for (;;) {
    const int q = phase == 0 ? 0 : 1;
    const int64_t limit = phase == 0 ? hub_items : g.ntasks;
    uint64_t base = 0;
    if (lane == 0) base = atomicAdd(&g.qctr[q], (unsigned long long)BATCH);
    base = bcast64(base, 0);
    if ((int64_t)base >= limit) {
      if (phase == 0) { phase = 1; continue; }
      return false;
    }
    bt.cnt = (int)uni((uint32_t)min((int64_t)BATCH, limit - (int64_t)base));
    bt.la = bt.lb = bt.uf = bt.vf = bt.gid = 0;
    bt.dyad = 0;
    bt.dlo = bt.dmid = bt.dhi = 0;
    bt.aoff = bt.boff = bt.tid = 0;
    if (lane < bt.cnt) {
      if (phase == 0) {
        const int64_t item = (int64_t)base + lane;
        int64_t lo = 0, hi = g.nhub;  // last h with hub_pre[h] <= item
        while (hi - lo > 1) {
          const int64_t mid = (lo + hi) >> 1;
          if (g.hub_pre[mid] <= item) lo = mid; else hi = mid;
        }
        const int64_t c = item - g.hub_pre[lo];
        bt.tid = (int64_t)g.hub_task[lo];
        const uint64_t tk = g.htasks[bt.tid] & ~HUB_BIT;
        const uint32_t u = (uint32_t)(tk >> 32);
        const int64_t au0 = g.off[u];
        const uint32_t du = (uint32_t)(g.off[u + 1] - au0);
        const uint32_t pv = g.packed[au0 + (uint32_t)tk];
        const int64_t bv0 = g.off[pv >> 2];
        const uint32_t dv = (uint32_t)(g.off[(pv >> 2) + 1] - bv0);
        // the ids of N(u) above u and of N(v) from u on
        const uint32_t su = g.ustart[u], sv = min(g.tskip[bt.tid], dv);
        const int64_t au = au0 + su, bv = bv0 + sv;
        const uint32_t dla = du - su, dlb = dv - sv;
        const uint32_t* Ag = g.packed + au;
        const uint32_t* Bg = g.packed + bv;
        const uint64_t Ltot = (uint64_t)dla + dlb;
        // the chunks split the merged length (a trailing chunk may be empty)
        const uint64_t d0 = min((uint64_t)c * g.chunk, Ltot), d1 = min(d0 + (uint64_t)g.chunk, Ltot);
        const uint32_t i0 = global_split(Ag, dla, Bg, dlb, (uint32_t)d0);
        const uint32_t i1 = global_split(Ag, dla, Bg, dlb, (uint32_t)d1);
        uint32_t k0 = (uint32_t)d0 - i0, k1 = (uint32_t)d1 - i1;
        // an id shared by A and B stays with the chunk holding its A copy
        if (i0 > 0 && k0 < dlb && key_of(Ag[i0 - 1]) == key_of(Bg[k0])) ++k0;
        if (i1 > 0 && k1 < dlb && key_of(Ag[i1 - 1]) == key_of(Bg[k1])) ++k1;
        if (k1 < k0) k1 = k0;
        bt.aoff = au + i0;
        bt.la = i1 - i0;
        bt.boff = bv + k0;
        bt.lb = k1 - k0;
        bt.uf = u | ((c == 0 ? 1u : 0u) << 30);
        bt.vf = pv;
        int64_t nn = g.n;
        if (BAT) {
          bt.gid = g.grow[u];
          nn = g.vbase[bt.gid + 1] - g.vbase[bt.gid];
        }
        bt.dyad = c == 0 ? (int32_t)(nn - (int64_t)du - (int64_t)dv) : 0;
        if constexpr (LAB) {
          if (c == 0) {
            const uint32_t vv = pv >> 2;
            lab_dyads(bt, g.n, u, vv, du, (int64_t)(uint32_t)tk, su, sv, dv, g.ustart[vv]);
          }
        }
      } else {
        bt.tid = g.order ? g.order[base + lane] : (int64_t)base + lane;
        const uint64_t tk = g.tasks[bt.tid];
        if (!(tk & HUB_BIT)) {  // hub tasks were merged in phase 0: empty item here
          const uint32_t u = (uint32_t)(tk >> 32) & 0x3FFFFFFFu;
          const int64_t au0 = g.off[u], au1 = g.off[u + 1];
          const uint32_t pv = g.packed[au0 + (uint32_t)tk];
          const int64_t bv0 = g.off[pv >> 2], bv1 = g.off[(pv >> 2) + 1];
          // never past the list's end, whatever the count says
          const uint32_t sv = min(g.tskip[bt.tid], (uint32_t)(bv1 - bv0));
          bt.boff = bv0 + sv;
          bt.lb = (uint32_t)(bv1 - bt.boff);
          // the ids of N(u) above u
          bt.aoff = au0 + g.ustart[u];
          bt.la = (uint32_t)(au1 - bt.aoff);
          const uint32_t du = (uint32_t)(au1 - au0), dv = bt.lb + sv;
          bt.uf = u | (2u << 30);
          bt.vf = pv;
          int64_t nn = g.n;
          if (BAT) {
            bt.gid = g.grow[u];
            nn = g.vbase[bt.gid + 1] - g.vbase[bt.gid];
          }
          bt.dyad = (int32_t)(nn - (int64_t)du - (int64_t)dv);
          if constexpr (LAB) {
            const uint32_t vv = pv >> 2;
            lab_dyads(bt, g.n, u, vv, du, (int64_t)(uint32_t)tk, g.ustart[u], sv, dv, g.ustart[vv]);
          }
        }
      }
    }
    add_dyads<BAT, LAB>(g, lane, bt);
    return true;
  }
}

// Uniform view of the item a wavefront is working on.
struct Item {
  const uint32_t* A;
  const uint32_t* B;
  uint32_t la, lb, uq, vq, f, kind, gid;
  uint64_t slice;  // class table slice of f = f_uv
  int64_t tid;
};

__device__ __forceinline__ void item_of(const Batch& bt, int it, const CensusArgs& g, Item& x) {
  x.A = g.packed + (int64_t)bcast64((uint64_t)bt.aoff, it);
  x.B = g.packed + (int64_t)bcast64((uint64_t)bt.boff, it);
  x.la = bcast32(bt.la, it);
  x.lb = bcast32(bt.lb, it);
  const uint32_t uf = bcast32(bt.uf, it), vf = bcast32(bt.vf, it);
  x.uq = (uf << 2) | 3u;  // the kind bits shift out
  x.vq = vf | 3u;
  x.f = vf & 3u;
  x.kind = uf >> 30;
  // a select between kernel arguments: no load is queued behind the window
  // prefetch, whose completion the merge must not wait for
  x.slice = x.f == 3u ? g.cls.s[3] : (x.f == 2u ? g.cls.s[2] : g.cls.s[1]);
  x.gid = bcast32(bt.gid, it);
  x.tid = (int64_t)bcast64((uint64_t)bt.tid, it);
}

// Buffer resource over n 32-bit words at p: a load past the n-th word returns
// 0 and does not access memory.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t words_rsrc(const uint32_t* p, uint32_t n) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(p), (short)0, (int)(n * 4u), 0x00020000);
}

// Issue the loads of one round's windows into registers (no wait). Every
// chunk is loaded without a branch; lanes past the window end read 0.
template <int W>
__device__ __forceinline__ void load_round(const uint32_t* A, uint32_t na_ld, const uint32_t* B, uint32_t nb_ld,
                                           int lane, uint32_t (&ra)[W / 64], uint32_t (&rb)[W / 64]) {
  // the lane's byte offset is made opaque here, in the loop, so that the
  // chunk offsets j * 256 go into the loads' immediate fields instead of
  // being hoisted out of the round loop as seven live registers
  uint32_t l4 = (uint32_t)lane * 4u;
  asm volatile("" : "+v"(l4));
  if (na_ld) {
    const __amdgpu_buffer_rsrc_t r = words_rsrc(A, na_ld);
#pragma unroll
    for (int j = 0; j < W / 64; ++j) ra[j] = __builtin_amdgcn_raw_buffer_load_b32(r, l4 + j * 256, 0, 0);
  }
  if (nb_ld) {
    const __amdgpu_buffer_rsrc_t r = words_rsrc(B, nb_ld);
#pragma unroll
    for (int j = 0; j < W / 64; ++j) rb[j] = __builtin_amdgcn_raw_buffer_load_b32(r, l4 + j * 256, 0, 0);
  }
}

// Number of entries of the sorted window x[0, n) with key <= bound, 0 < n <= W:
// a 64-ary search, one LDS read per lane for the last key of each of 64
// blocks of W/64 entries, then one per lane in the block holding the boundary.
template <int W>
__device__ __forceinline__ uint32_t count_le(const uint32_t* x, uint32_t n, uint32_t bound, int lane) {
  constexpr uint32_t S = W / 64;
  // recomputed from the lane id in every round: a loop-invariant index kept
  // live across the round loop would be spilled
  uint32_t l = (uint32_t)lane;
  asm volatile("" : "+v"(l));
  if (n <= 64) {
    // a window of at most 64 ids (the short list of most lopsided rounds):
    // one read and one compare per lane
    const uint32_t v = key_of(x[min(l, n - 1)]);
    return (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(l < n) & __builtin_amdgcn_ballot_w64(v <= bound));
  }
  const uint32_t last = key_of(x[min(l * S + S - 1, n - 1)]);
  // (each ballot of one compare is that compare's lane mask as it stands;
  // masks are combined on the scalar unit)
  const uint32_t c1 = (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(l * S < n) &
                                         __builtin_amdgcn_ballot_w64(last <= bound));  // whole blocks <= bound
  if (c1 * S >= n) return n;
  const uint32_t e = c1 * S + l;
  const bool in2 = l < S && e < n;
  const uint32_t v = key_of(x[in2 ? e : 0]);
  return c1 * S + (uint32_t)__popcll(((1ull << S) - 1) & __builtin_amdgcn_ballot_w64(e < n) &
                                     __builtin_amdgcn_ballot_w64(v <= bound));
}

// Per-lane two-pointer walk of the lane's merge-path range of one round:
// one distinct w per step, classified in situ from its direction bits
// (Fig. 5 steps 2.1.4-2.1.4.2, Sec. 6).
template <int W, bool HH, int NC>
__device__ __forceinline__ void merge_round(WaveLds<W, HH, NC>& L, uint32_t na, uint32_t nb, uint32_t uq,
                                                uint32_t vq, uint64_t slice, uint32_t fuv, uint32_t col, int lane) {
  constexpr bool LAB = NC == 64;
  const uint32_t D = na + nb;
  const uint32_t d0 = (uint32_t)(((uint64_t)lane * D) >> 6), d1 = (uint32_t)(((uint64_t)(lane + 1) * D) >> 6);
  uint32_t lo = d0 > nb ? d0 - nb : 0, hi = d0 < na ? d0 : na;
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if (key_of(L.a[mid]) <= key_of(L.b[d0 - mid - 1])) lo = mid + 1; else hi = mid;
  }
  uint32_t i = lo, k = d0 - lo;
  // an id shared by A[i-1] and B[k] was consumed with A[i-1] by a lane before
  if (i > 0 && k < nb && key_of(L.a[i - 1]) == key_of(L.b[k])) ++k;
  const uint32_t start = i + k;
  uint32_t pos = start;
  uint32_t* const hcol = L.hist + col;
  // The lane predicates are kept as wavefront masks so that their logic runs
  // on the scalar unit; the vector unit only compares, selects and adds.
  while (pos < d1) {
    const uint32_t a = L.a[i], b = L.b[k];
    const uint32_t ea = a | 3u, eb = b | 3u;
    const bool ta = ea <= eb, tb = eb <= ea;  // w is in N(u), in N(v)
    const uint64_t tA = __builtin_amdgcn_ballot_w64(ta), tB = __builtin_amdgcn_ballot_w64(tb);
    // canonical selection (Fig. 5 step 2.1.4): a w taken from N(u), alone or
    // shared, is counted iff v < w; a w found in N(v) only iff u < w
    const uint64_t mA = tA & __builtin_amdgcn_ballot_w64(ea > vq);
    const uint64_t mB = (tB & mA) | (__builtin_amdgcn_ballot_w64(eb > uq) & ~tA);
    // nibble shift 4 * (fa | fb << 2) of the class table, with the flag of a
    // list that does not hold w, or of an uncounted w, taken as 0
    const uint32_t fa = __builtin_amdgcn_inverse_ballot_w64(mA) ? a & 3u : 0u;
    const uint32_t sb = __builtin_amdgcn_inverse_ballot_w64(mB) ? b : 0u;
    uint32_t cls;
    if constexpr (LAB) {
      // a counted w from N(u) lies above v; one from N(v) only may lie below it
      const bool cnt = __builtin_amdgcn_inverse_ballot_w64(mA | mB);
      const uint32_t st = lab_state(__builtin_amdgcn_inverse_ballot_w64(mA) | (eb > vq), fuv, fa, sb & 3u);
      cls = cnt ? st : 0u;
    } else {
      const uint32_t sh = (((sb << 2) | fa) << 2) & 63u;  // the id bits of b shift out
      cls = (uint32_t)(slice >> sh) & 15u;
    }
    hist_add<W, HH, NC>(hcol, cls, 1u);
    i += (uint32_t)ta;
    k += (uint32_t)tb;
    pos = i + k;
  }
}

// Deferred counts of the long window of lopsided rounds whose ids are all
// counted as found in one list only: such an id's class depends only on its
// flag and on the round's class row (uniform), so each lane counts flags 1..3
// in bytes 1..3 of one register (1 << 8f: a shift and a shift-add per id, no
// LDS atomic), and the counts go to the LDS counters when the class row
// changes, after pack_rounds<W>() rounds (a byte then holds at most that many
// times W / 64 ids, below 256), and before every flush.
struct FlagPack {
  uint32_t acc;     // per lane: byte f = ids of flag f counted since the drain
  uint32_t tbl;     // the class row those counts belong to (uniform)
  uint32_t rounds;  // rounds counted since the drain (uniform)
  // labelled census: ids above v in acc, the rest in acc0 (byte 0 of both
  // collects the uncounted ids); tbl and tbl0 are the state tables of the two
  uint32_t acc0, tbl0;
};
template <int W>
constexpr uint32_t pack_rounds() {
  return 255u / (uint32_t)(W / 64);
}

template <int W, bool HH, int NC>
__device__ __forceinline__ void pack_drain(WaveLds<W, HH, NC>& L, FlagPack& p, uint32_t col) {
  static_assert(pack_rounds<W>() * (W / 64) < 256, "a byte counter would overflow");
  constexpr uint32_t C = WaveLds<W, HH, NC>::COLS;
  if (p.rounds == 0) return;
  uint32_t* const hcol = L.hist + col;
  if constexpr (NC == 64) {
    // state of flag f: 6-bit field f of the table (8-bit fields; field 0 unused)
#pragma unroll
    for (uint32_t f = 1; f < 4; ++f) {
      hist_add<W, HH, NC>(hcol, (p.tbl >> (8 * f)) & 63u, (p.acc >> (8 * f)) & 255u);
      hist_add<W, HH, NC>(hcol, (p.tbl0 >> (8 * f)) & 63u, (p.acc0 >> (8 * f)) & 255u);
    }
    p.acc0 = 0;
  } else {
#pragma unroll
    for (uint32_t f = 1; f < 4; ++f) atomicAdd(hcol + ((p.tbl >> (4 * f)) & 15u) * C, (p.acc >> (8 * f)) & 255u);
  }
  p.acc = 0;
  p.rounds = 0;
}

// A round in which one window holds few ids (S, ns of them) and the other many
// (G, ng): the same classification as the walk, entry by entry instead of in
// merged order. Each id of S finds its match in G by a branchless lower-bound
// search and is classified with both flags; every id of G is classified as
// found in its own list only, in 64-wide chunks, and the match of an S id
// takes that one-list count back. Counter columns can therefore dip below
// zero between flushes; flush_wave sums them as signed values.
template <int W, bool HH, int NC>
__device__ __forceinline__ void lopsided_round(WaveLds<W, HH, NC>& L, uint32_t na, uint32_t nb, uint32_t uq,
                                                   uint32_t vq, uint64_t slice, uint32_t ga, uint32_t gb, uint32_t fuv,
                                                   const LabTables& lt, uint32_t col, int lane, FlagPack& pk) {
  constexpr uint32_t C = WaveLds<W, HH, NC>::COLS;
  constexpr bool LAB = NC == 64;
  const bool sA = na <= nb;  // the short window is N(u)'s
  const uint32_t* S = sA ? L.a : L.b;
  const uint32_t* G = sA ? L.b : L.a;
  const uint32_t ns = sA ? na : nb, ng = sA ? nb : na;
  // class of an id found in G only, by its flag f: N(v) only (sA) is counted
  // iff u < w, N(u) only iff v < w. Nibble f of rowtbl holds that class
  // (nibble 0: not counted), and the four nibbles are repeated at bit 16 so
  // that a bit-field extract at offset (y << 2) mod 32 finds them whatever the
  // lowest id bit of y.
  const uint32_t thrG = sA ? uq : vq;
  const uint32_t rowtbl = sA ? gb : ga;
  uint32_t* const hcol = L.hist + col;
  for (uint32_t t0 = 0; t0 < ns; t0 += 64) {
    const uint32_t t = t0 + (uint32_t)lane;
    const bool act = t < ns;
    const uint32_t x = S[act ? t : 0];
    const uint32_t kx = x | 3u, x0 = x & ~3u;
    // lower bound of x's id in G[0, ng), ng >= 1: a packed word is below x0
    // iff its id is below x's; the cursor is an LDS address, so each probe is
    // a read at an immediate offset. A full window (the usual case) takes a
    // fixed, unrolled sequence of halvings.
    const uint32_t* p = G;
    if (ng == (uint32_t)W) {
#pragma unroll
      for (uint32_t len = W; len > 1;) {
        const uint32_t half = len >> 1;
        p = p[half] < x0 ? p + half : p;
        len -= half;
      }
    } else {
      for (uint32_t len = ng; len > 1;) {
        const uint32_t half = len >> 1;
        p = p[half] < x0 ? p + half : p;
        len -= half;
      }
    }
    // both candidates in one read (G[ng] is the sentinel)
    const uint32_t g0 = p[0], g1 = p[1];
    const uint32_t gr = g0 < x0 ? g1 : g0;
    const bool common = act & (key_of(gr) == kx);
    const uint32_t fs = x & 3u, fg = common ? gr & 3u : 0u;
    // canonical selection (Fig. 5 step 2.1.4) for the S id
    const bool counted = act & ((sA | common) ? kx > vq : kx > uq);
    uint32_t cls, gcls;
    if constexpr (LAB) {
      const uint32_t fa = sA ? fs : fg, fb = sA ? fg : fs;
      cls = counted ? lab_state(kx > vq, fuv, fa, fb) : 0u;
      // the G-only state the matched G id gets below
      gcls = (common & (kx > thrG)) ? (sA ? lab_state(kx > vq, fuv, 0u, fg) : lab_state(true, fuv, fg, 0u)) : 0u;
    } else {
      const uint32_t idx = sA ? fs | fg << 2 : fg | fs << 2;
      cls = counted ? (uint32_t)(slice >> (idx << 2)) & 15u : 0u;
      gcls = (common & (kx > thrG)) ? (rowtbl >> (4u * fg)) & 15u : 0u;
    }
    hist_add<W, HH, NC>(hcol, cls, 1u);
    // the matched G id is counted below as found in G only: take that back
    if (common) hist_add<W, HH, NC>(hcol, gcls, ~0u);
  }
  if constexpr (LAB) {
    // ids of G as found in G only: N(v) only (sA) counts above u, its state
    // depending on the side of v; N(u) only counts above v. Tables hold the
    // state per flag in 8-bit fields (field 0 = uncounted).
    const uint32_t thi = sA ? lt.gb_hi[fuv] : lt.ga_hi[fuv], tlo = sA ? lt.gb_lo[fuv] : 0u;
    if (ng == (uint32_t)W) {
      // a full window: all reads first, then per-lane byte counts by flag and
      // side of v (an uncounted id into byte 0), drained when the tables change
      uint32_t y[W / 64];
#pragma unroll
      for (int j = 0; j < W / 64; ++j) y[j] = G[j * 64 + lane];
      if (pk.tbl != thi || pk.tbl0 != tlo || pk.rounds >= pack_rounds<W>()) {
        pack_drain(L, pk, col);
        pk.tbl = thi;
        pk.tbl0 = tlo;
      }
      uint32_t a1 = pk.acc, a0 = pk.acc0;
#pragma unroll
      for (int j = 0; j < W / 64; ++j) {
        const uint32_t inc = 1u << (((y[j] > thrG ? y[j] : 0u) << 3) & 31u);
        if (y[j] > vq) a1 += inc; else a0 += inc;
      }
      pk.acc = a1;
      pk.acc0 = a0;
      pk.rounds += 1;
      return;
    }
    for (uint32_t e = (uint32_t)lane; e - (uint32_t)lane < ng; e += 64) {
      const uint32_t y = G[e < ng ? e : 0];
      const uint32_t off = ((e < ng) & (y > thrG)) ? y << 3 : 0u;
      hist_add<W, HH, NC>(hcol, __builtin_amdgcn_ubfe(y > vq ? thi : tlo, off, 6), 1u);
    }
    return;
  }
  // ids of G, classified as found in G only, 64 per step. G is sorted: if
  // its last id is not above the threshold none is counted, if its first is
  // every one is.
  const uint32_t gfirst = uni(G[0]), glast = uni(G[ng - 1]);
  if (glast <= thrG) return;
  const uint32_t nfull = ng & ~63u;
  uint32_t e = (uint32_t)lane;
  if (nfull == (uint32_t)W) {
    // all reads first: one wait instead of one per chunk
    uint32_t y[W / 64];
#pragma unroll
    for (int j = 0; j < W / 64; ++j) y[j] = G[j * 64 + lane];
    if (gfirst > thrG) {
      if (pk.tbl != rowtbl || pk.rounds >= pack_rounds<W>()) {
        pack_drain(L, pk, col);
        pk.tbl = rowtbl;
      }
      uint32_t acc = pk.acc;
#pragma unroll
      for (int j = 0; j < W / 64; ++j) acc += 1u << ((y[j] << 3) & 31u);  // byte f of the id's flag f
      pk.acc = acc;
      pk.rounds += 1;
    } else {
#pragma unroll
      for (int j = 0; j < W / 64; ++j) {
        const uint32_t off = y[j] > thrG ? y[j] << 2 : 0u;
        atomicAdd(hcol + __builtin_amdgcn_ubfe(rowtbl, off, 4) * C, 1u);
      }
    }
    return;
  }
  for (; e < nfull; e += 64) {
    const uint32_t y = G[e];
    const uint32_t off = y > thrG ? y << 2 : 0u;
    atomicAdd(hcol + __builtin_amdgcn_ubfe(rowtbl, off, 4) * C, 1u);
  }
  if (nfull < ng) {
    const uint32_t y = G[e];
    const uint32_t off = ((e < ng) & (y > thrG)) ? y << 2 : 0u;
    atomicAdd(hcol + __builtin_amdgcn_ubfe(rowtbl, off, 4) * C, 1u);
  }
}

template <int W, bool HH, int NC>
__device__ void flush_wave(WaveLds<W, HH, NC>& L, int lane, unsigned long long* acc) {
  constexpr int C = WaveLds<W, HH, NC>::COLS;
  wave_lds_sync();
  // counters are signed: a lopsided round may take a count back from a column
  // other than the one that received it
  if constexpr (NC == 64) {
    for (int r = 0; r < NC / 2; ++r) {
      // two signed 16-bit fields, each within +-32767 (LAB_FLUSH_STEPS)
      const int32_t w = lane < C ? (int32_t)L.hist[r * C + lane] : 0;
      const int32_t lo = (int32_t)(int16_t)(uint16_t)(w & 0xFFFF), hi = (w - lo) >> 16;
      const uint64_t slo = wave_sum64((uint64_t)(int64_t)lo), shi = wave_sum64((uint64_t)(int64_t)hi);
      if (lane == 0) {
        if (r > 0 && slo) atomicAdd(&acc[2 * r], (unsigned long long)slo);
        if (shi) atomicAdd(&acc[2 * r + 1], (unsigned long long)shi);
      }
    }
  } else {
    for (int c = 1; c < NC; ++c) {
      const uint64_t x = lane < C ? (uint64_t)(int64_t)(int32_t)L.hist[c * C + lane] : 0u;
      const uint64_t sum = wave_sum64(x);
      if (lane == 0 && sum) atomicAdd(&acc[c], (unsigned long long)sum);
    }
  }
  for (int c = 0; c < WaveLds<W, HH, NC>::ROWS; ++c)
    if (lane < C) L.hist[c * C + lane] = 0;
  wave_lds_sync();
}

// Persistent census kernel. Each wavefront claims batches of items and runs a
// two-stage pipeline over "rounds": while round r is merged from LDS, the
// global loads of round r+1 (same item, or the next item of the batch) are in
// flight in registers. MODE 1 adds per-task cycle recording; MODE 2 is the
// batched census: every graph of the batch accumulates into its own counters
// (a wavefront flushes its LDS counters when it moves to another graph).
template <int WAVES, int W, bool HH, int MODE, int MINW>
__global__ void __launch_bounds__(WAVES * 64, MINW) k_census(CensusArgs g) {
  constexpr bool CYC = MODE == 1, BAT = MODE == 2, LAB = MODE == 3;
  constexpr int NC = LAB ? 64 : 16;
  __shared__ WaveLds<W, HH, NC> lds[WAVES];
  constexpr int C = WaveLds<W, HH, NC>::COLS;
  if (*g.err) return;
  const int lane = threadIdx.x & 63;
  WaveLds<W, HH, NC>& L = lds[threadIdx.x >> 6];
  const int64_t wave_id = (int64_t)blockIdx.x * WAVES + (threadIdx.x >> 6);
  if (g.wave_span && lane == 0) g.wave_span[2 * wave_id] = __builtin_amdgcn_s_memrealtime();
  for (int c = 0; c < WaveLds<W, HH, NC>::ROWS; ++c)
    if (lane < C) L.hist[c * C + lane] = 0;
  wave_lds_sync();
  const uint32_t col = (uint32_t)(lane & (C - 1));
  // counters 1 (012) and 2 (102) receive n - d(u) - d(v) per task when the
  // batch is claimed; the common-neighbour part is added at the end
  uint32_t steps = 0;  // bound on any counter's increments since the last flush

  // The pipeline starts on an empty item: its round is a no-op that is
  // immediately "done", so the first real item is claimed by the same code
  // path as every later one.
  int phase = 0;
  Batch bt;
  bt.cnt = 0;
  int it = 0;
  Item cur;
  cur.A = cur.B = g.packed;
  cur.la = cur.lb = 0;
  cur.uq = cur.vq = 0;
  cur.f = 1;
  cur.kind = 0;
  cur.gid = 0;
  cur.slice = 0;
  cur.tid = 0;
  uint32_t wg = 0xFFFFFFFFu;  // graph whose counters the wavefront holds (batched)
  uint32_t ia = 0, ib = 0;  // position of the current round in the item
  uint64_t t_start = CYC ? __builtin_amdgcn_s_memtime() : 0;
  uint32_t ra[W / 64], rb[W / 64];
  uint32_t na_ld = 0, nb_ld = 0;
  FlagPack pk{0u, 0u, 0u, 0u, 0u};

  for (;;) {
    // ---- stage the loaded round in LDS (slots past the window get zeros or
    // stale values; every reader stops at the window end or its sentinel)
#pragma unroll
    for (int j = 0; j < W / 64; ++j) {
      const uint32_t k = (uint32_t)(j * 64 + lane);
      L.a[k] = ra[j];
      L.b[k] = rb[j];
    }
    wave_lds_sync();
    // every element up to the smaller of the two window maxima is merged now:
    // all of the window that ends lower, and the other one up to that key
    const uint32_t ra_rem = cur.la - ia, rb_rem = cur.lb - ib;
    const uint32_t lastA = na_ld < ra_rem ? uni(key_of(L.a[na_ld - 1])) : KEY_INF;
    const uint32_t lastB = nb_ld < rb_rem ? uni(key_of(L.b[nb_ld - 1])) : KEY_INF;
    uint32_t na = na_ld, nb = nb_ld;
    if (lastA < lastB) {
      if (nb_ld) nb = count_le<W>(L.b, nb_ld, lastA, lane);
    } else if (lastB < lastA) {
      if (na_ld) na = count_le<W>(L.a, na_ld, lastB, lane);
    }
    if (lane == 0) {
      L.a[na] = KEY_INF;  // sentinels: the walk never reads past them
      L.b[nb] = KEY_INF;
    }
    // ---- choose and issue the next round
    const bool item_done = (ia + na >= cur.la) && (ib + nb >= cur.lb);
    Item nxt;  // the next item; read only when item_done
    uint32_t nia = ia + na, nib = ib + nb;
    bool more = true;
    if (item_done) {
      nia = nib = 0;
      int nit = it + 1;
      // skip empty items (hub tasks in the task queue)
      while (nit < bt.cnt && bcast32(bt.la, nit) + bcast32(bt.lb, nit) == 0) ++nit;
      if (nit < bt.cnt) {
        item_of(bt, nit, g, nxt);
        it = nit;
      } else {
        // batch exhausted: claim the next one (the current item is already in
        // scalars, so bt can be overwritten; this latency is not hidden)
        for (;;) {
          more = uni(fetch_batch<BAT, LAB>(g, lane, phase, bt));
          if (!more) break;
          int k0 = 0;
          while (k0 < bt.cnt && bcast32(bt.la, k0) + bcast32(bt.lb, k0) == 0) ++k0;
          if (k0 < bt.cnt) {
            it = k0;
            item_of(bt, k0, g, nxt);
            break;
          }
        }
      }
    }
    // the next round's windows: more of this item, or the start of the next
    const uint32_t* const nA = item_done ? nxt.A : cur.A;
    const uint32_t* const nB = item_done ? nxt.B : cur.B;
    const uint32_t nla = item_done ? nxt.la : cur.la, nlb = item_done ? nxt.lb : cur.lb;
    const uint32_t nna_ld = more ? min(nla - nia, (uint32_t)W) : 0u;
    const uint32_t nnb_ld = more ? min(nlb - nib, (uint32_t)W) : 0u;
    wave_lds_sync();
    // ra/rb are consumed (counts done, LDS staged): refill them for the next round
    if (more) load_round<W>(nA + nia, nna_ld, nB + nib, nnb_ld, lane, ra, rb);
    // ---- merge this round from LDS
    if (BAT && cur.gid != wg && cur.la + cur.lb > 0) {
      if (wg != 0xFFFFFFFFu) {
        pack_drain(L, pk, col);
        flush_wave(L, lane, g.gout + 16 * (uint64_t)wg);
        steps = 0;
      }
      wg = cur.gid;
    }
    if (min(na, nb) <= LOP_S && max(na, nb) >= LOP_G)
      lopsided_round<W, HH, NC>(L, na, nb, cur.uq, cur.vq, cur.slice, g.cls.ga[cur.f], g.cls.gb[cur.f], cur.f, g.lab,
                                col, lane, pk);
    else
      merge_round<W, HH, NC>(L, na, nb, cur.uq, cur.vq, cur.slice, cur.f, col, lane);
    steps += (na + nb) / (HH ? 16 : 32) + 4;
    if (item_done) {
      if constexpr (CYC) {
        const uint64_t t_end = __builtin_amdgcn_s_memtime();
        if (lane == 0 && cur.kind == 2) g.cycles[cur.tid] = (uint32_t)min(t_end - t_start, (uint64_t)0xFFFFFFFFu);
        t_start = t_end;
      }
      if (!LAB && steps > (1u << 30)) {
        pack_drain(L, pk, col);
        flush_wave(L, lane, BAT ? g.gout + 16 * (uint64_t)wg : g.acc);
        steps = 0;
      }
    }
    if (LAB && steps > LAB_FLUSH_STEPS) {
      pack_drain(L, pk, col);  // counts still packed belong to the rounds steps covers
      flush_wave(L, lane, g.acc);
      steps = 0;
    }
    wave_lds_sync();
    if (!more) break;
    if (item_done) cur = nxt;
    ia = nia;
    ib = nib;
    na_ld = nna_ld;
    nb_ld = nnb_ld;
  }
  unsigned long long* tgt = g.acc;
  if (BAT) tgt = wg != 0xFFFFFFFFu ? g.gout + 16 * (uint64_t)wg : nullptr;
  pack_drain(L, pk, col);
  if (tgt) flush_wave(L, lane, tgt);
  if (lane == 0 && g.wave_span) g.wave_span[2 * wave_id + 1] = __builtin_amdgcn_s_memrealtime();
}

// The dyadic counts (Fig. 5 step 2.1.3) need each task's number of common
// neighbours of u and v, added to 012 or 102 by the task's dyad. Summed over
// the tasks of each dyad kind these follow from the triangle classes: a
// triangle is a common neighbour of each of its three edges, and its class
// fixes how many of them are mutual (030T, 030C: none; 120D, 120U, 120C: one;
// 210: two; 300: three).
__device__ __forceinline__ void add_common_neighbours(uint64_t* c) {
  const uint64_t t1 = c[11] + c[12] + c[13];
  c[1] += 3 * (c[8] + c[9]) + 2 * t1 + c[14];
  c[2] += t1 + 2 * c[14] + 3 * c[15];
}

__global__ void k_finalize(const unsigned long long* __restrict__ acc, uint64_t clo, uint64_t chi,
                           const uint32_t* __restrict__ err, uint64_t* __restrict__ out) {
  if (threadIdx.x != 0 || blockIdx.x != 0 || *err) return;  // an error writes no output
  uint64_t c[16];
  for (int k = 0; k < 16; ++k) c[k] = acc[k];
  add_common_neighbours(c);
  uint64_t s = 0;
  for (int k = 1; k < 16; ++k) {
    out[k] = c[k];
    s += c[k];
  }
  out[0] = clo - s;
  out[16] = chi - (clo < s ? 1u : 0u);
}

// Labelled census: each triangle {a < b < c} is a common neighbour of three
// of its edges' tasks, so the dyadic terms of those tasks (which subtracted
// it) get it back: the task (b, c) below u (state f_bc << 4), the task (a, c)
// between u and v (state f_ac << 2), the task (a, b) above v (state f_ab).
// State 0 (no arc) = C(n,3) minus the rest, in two 64-bit words (out[64] is
// the high word).
__global__ void k_finalize_lab(const unsigned long long* __restrict__ acc, uint64_t clo, uint64_t chi,
                               const uint32_t* __restrict__ err, uint64_t* __restrict__ out) {
  if (threadIdx.x != 0 || blockIdx.x != 0 || *err) return;  // an error writes no output
  uint64_t c[64];
  for (int k = 0; k < 64; ++k) c[k] = acc[k];
  for (uint32_t st = 1; st < 64; ++st) {
    const uint32_t fab = st & 3u, fac = (st >> 2) & 3u, fbc = st >> 4;
    if (fab && fac && fbc) {
      c[fbc << 4] += acc[st];
      c[fac << 2] += acc[st];
      c[fab] += acc[st];
    }
  }
  uint64_t s = 0;
  for (int k = 1; k < 64; ++k) {
    out[k] = c[k];
    s += c[k];
  }
  out[0] = clo - s;
  out[64] = chi - (clo < s ? 1u : 0u);
}

__global__ void k_fill_u64(uint64_t* p, int64_t m, uint64_t v) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) p[i] = v;
}
__global__ void k_fill_u32(uint32_t* p, int64_t m, uint32_t v) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) p[i] = v;
}

// ------------------------------------------------------------------- host

static int grid_for(int64_t work, int threads, int cap = 65536) {
  int64_t g = (work + threads - 1) / threads;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (int)g;
}

int64_t scan_sums(int64_t m) { return (m + SCAN_B - 1) / SCAN_B + 1; }

int scan_i64_with(const int64_t* in, int64_t m, int64_t* out, int64_t* sums, hipStream_t s) {
  const int64_t nb = (m + SCAN_B - 1) / SCAN_B;
  if (m > 0) {
    k_scan_sums<<<(unsigned)nb, SCAN_T, 0, s>>>(in, m, sums);
    k_scan_top<<<1, SCAN_T, 0, s>>>(sums, nb);
    k_scan_apply<<<(unsigned)nb, SCAN_T, 0, s>>>(in, m, sums, out);
  } else {
    k_fill_u64<<<1, 64, 0, s>>>((uint64_t*)out, 1, 0);
  }
  HIPCHK(hipGetLastError());
  return TRIAD_OK;
}

int scan_i64(const int64_t* in, int64_t m, int64_t* out, Scratch& scratch, hipStream_t s) {
  int64_t* sums = nullptr;
  ALLOC(sums, scan_sums(m));
  return scan_i64_with(in, m, out, sums, s);
}

// Kernel variants: LDS window per list x counter array layout x occupancy hint.
enum Variant { V_W512 = 0, V_W1024 = 1, V_W512_HH = 2, V_W256_HH = 3, V_W512_HH6 = 4, V_W448_HH7 = 5,
               V_W384_HH7 = 6, V_W320_HH8 = 7, NUM_VARIANTS };

template <int WAVES, int W, bool HH, int MINW>
static hipError_t launch_t(const CensusArgs& a, int mode, int groups, hipStream_t s) {
  if (mode == 1) k_census<WAVES, W, HH, 1, MINW><<<groups, WAVES * 64, 0, s>>>(a);
  else if (mode == 2) k_census<WAVES, W, HH, 2, MINW><<<groups, WAVES * 64, 0, s>>>(a);
  else k_census<WAVES, W, HH, 0, MINW><<<groups, WAVES * 64, 0, s>>>(a);
  return hipGetLastError();
}
template <int WAVES, int W, bool HH, int MINW>
static int occ_t(int mode) {
  // a property of the code object (gfx950), asked for once: every timed call
  // reports the launch size
  static std::atomic<int> known[3];
  if (const int k = known[mode].load(std::memory_order_relaxed)) return k;
  int per_cu = 0;
  hipError_t e;
  if (mode == 1) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_census<WAVES, W, HH, 1, MINW>, WAVES * 64, 0);
  else if (mode == 2) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_census<WAVES, W, HH, 2, MINW>, WAVES * 64, 0);
  else e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_census<WAVES, W, HH, 0, MINW>, WAVES * 64, 0);
  if (e != hipSuccess) return 1;
  known[mode].store(std::max(per_cu, 1), std::memory_order_relaxed);
  return std::max(per_cu, 1);
}
template <int WAVES>
static hipError_t launch_v(int variant, const CensusArgs& a, int cyc, int groups, hipStream_t s) {
  switch (variant) {
    case V_W1024: return launch_t<WAVES, 1024, false, 1>(a, cyc, groups, s);
    case V_W512_HH: return launch_t<WAVES, 512, true, 1>(a, cyc, groups, s);
    case V_W256_HH: return launch_t<WAVES, 256, true, 1>(a, cyc, groups, s);
    case V_W512_HH6: return launch_t<WAVES, 512, true, 6>(a, cyc, groups, s);
    case V_W448_HH7: return launch_t<WAVES, 448, true, 7>(a, cyc, groups, s);
    case V_W384_HH7: return launch_t<WAVES, 384, true, 7>(a, cyc, groups, s);
    case V_W320_HH8: return launch_t<WAVES, 320, true, 8>(a, cyc, groups, s);
    default: return launch_t<WAVES, 512, false, 1>(a, cyc, groups, s);
  }
}
template <int WAVES>
static int occ_v(int variant, int cyc) {
  switch (variant) {
    case V_W1024: return occ_t<WAVES, 1024, false, 1>(cyc);
    case V_W512_HH: return occ_t<WAVES, 512, true, 1>(cyc);
    case V_W256_HH: return occ_t<WAVES, 256, true, 1>(cyc);
    case V_W512_HH6: return occ_t<WAVES, 512, true, 6>(cyc);
    case V_W448_HH7: return occ_t<WAVES, 448, true, 7>(cyc);
    case V_W384_HH7: return occ_t<WAVES, 384, true, 7>(cyc);
    case V_W320_HH8: return occ_t<WAVES, 320, true, 8>(cyc);
    default: return occ_t<WAVES, 512, false, 1>(cyc);
  }
}

static hipError_t launch_census(int waves, int variant, const CensusArgs& a, int groups, hipStream_t s) {
  const int cyc = a.gout ? 2 : a.cycles ? 1 : 0;
  switch (waves) {
    case 1: return launch_v<1>(variant, a, cyc, groups, s);
    case 2: return launch_v<2>(variant, a, cyc, groups, s);
    default: return launch_v<4>(variant, a, cyc, groups, s);
  }
}

// The labelled census (64 state counters per column, two 16-bit counters per
// LDS word: 4 KB per wavefront) runs one launch shape: 448-entry windows, two
// wavefronts per workgroup, up to 5 per SIMD.
constexpr int LAB_WAVES = 2;
static hipError_t launch_lab(const CensusArgs& a, int groups, hipStream_t s) {
  k_census<LAB_WAVES, 448, true, 3, 5><<<groups, LAB_WAVES * 64, 0, s>>>(a);
  return hipGetLastError();
}
static int lab_groups(int requested) {
  if (requested > 0) return requested;
  DeviceInfo di;
  if (device_info(&di) != TRIAD_OK) return 1024;
  static std::atomic<int> known;
  int per_cu = known.load(std::memory_order_relaxed);
  if (!per_cu) {
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_census<LAB_WAVES, 448, true, 3, 5>, LAB_WAVES * 64, 0) !=
            hipSuccess || per_cu < 1)
      return di.cus;
    known.store(per_cu, std::memory_order_relaxed);
  }
  return di.cus * per_cu;
}

static int census_groups(int waves, int variant, int cyc, int requested) {
  if (requested > 0) return requested;
  DeviceInfo di;
  if (device_info(&di) != TRIAD_OK) return 1024;
  const int per_cu = waves == 1 ? occ_v<1>(variant, cyc) : waves == 2 ? occ_v<2>(variant, cyc) : occ_v<4>(variant, cyc);
  return di.cus * per_cu;
}

static int default_variant() {
  const char* e = getenv("TRIAD_VARIANT");
  if (e && *e >= '0' && *e < '0' + NUM_VARIANTS) return *e - '0';
  return V_W448_HH7;
}

// The kernel variant of a call and its wavefronts per workgroup: 448-entry
// windows at 7 wavefronts per SIMD run best with two wavefronts per workgroup.
static int pick_variant(const triad_opts& o) {
  return o.kernel_variant > 0 && o.kernel_variant <= NUM_VARIANTS ? o.kernel_variant - 1 : default_variant();
}
static int pick_waves(const triad_opts& o, int variant) {
  if (o.waves_per_group) return o.waves_per_group;
  return variant == V_W448_HH7 ? 2 : 1;
}

struct Events {
  hipEvent_t e[5] = {nullptr, nullptr, nullptr, nullptr, nullptr};
  bool on = false;
  ~Events() {
    for (auto& x : e)
      if (x) (void)hipEventDestroy(x);
  }
  hipError_t init() {
    on = true;
    for (auto& x : e) {
      hipError_t r = hipEventCreate(&x);
      if (r != hipSuccess) return r;
    }
    return hipSuccess;
  }
  void rec(int i, hipStream_t s) {
    if (on) (void)hipEventRecord(e[i], s);
  }
  float ms(int a, int b) {
    float t = 0;
    if (on) (void)hipEventElapsedTime(&t, e[a], e[b]);
    return t;
  }
};

// Upper bound of the scratch bytes census_device takes from an arena for a
// plain-schedule call (each request rounded up to 256 bytes): per row the
// first-task index, task count and its scan, per entry the packed word and a
// row-start bit, per task its word, N(v) count and hub-list slots, plus the
// emission segment list and the scans' block sums.
static size_t census_scratch_bound(int64_t n, int64_t nnz) {
  const int64_t m = nnz / 2;
  auto r = [](int64_t bytes) { return (size_t)((std::max<int64_t>(bytes, 1) + 255) & ~(int64_t)255); };
  size_t b = r(4) + r((16 + 5) * 8);  // errors; counters, queues
  if (n > 0) {
    b += r(4 * n) + r(8 * n) + r(8 * (n + 1)) + r(4 * ((nnz >> 5) + 1)) + r(4 * (nnz + PAD));
    b += r(8 * ((n + SCAN_B - 1) / SCAN_B + 1));
  }
  if (m > 0) {
    b += r(8 * m) + r(4 * m) + r(8 * m) + r(8 * m) + r(8 * (m + 1));
    b += r(8 * ((m + SCAN_B - 1) / SCAN_B + 1));
  }
  return b;
}

// The census of one device-resident graph. labelled: the 64-state census
// (65 output words) instead of the 16 classes (17 words). allocated_before:
// device bytes the caller allocated for this call (counted against the
// memory cap). Outputs are written only on success.
int census_device(int64_t n, int64_t nnz, const int64_t* off, const int32_t* nbr, const uint8_t* flg,
                  const triad_opts* opts, hipStream_t s, uint64_t* d_out, uint64_t* h_out, void* arena = nullptr,
                  size_t arena_bytes = 0, bool labelled = false, size_t allocated_before = 0) {
  triad_opts o{};
  if (opts) o = *opts;
  const int NC = labelled ? 64 : 16;  // census counters
  if (labelled && (o.task_cycles || o.kernel_variant || o.waves_per_group))
    return fail(TRIAD_EINVAL, "the labelled census takes no cycle recording and no kernel variant");
  if (n < 0 || n >= ((int64_t)1 << 30)) return fail(TRIAD_EINVAL, "n must be in [0, 2^30)");
  if (nnz < 0 || nnz >= ((int64_t)1 << 40)) return fail(TRIAD_EINVAL, "nnz must be in [0, 2^40)");
  if (!off || !d_out || (nnz > 0 && (!nbr || !flg))) return fail(TRIAD_EINVAL, "NULL pointer argument");
  if (o.validate < 0 || o.validate > 1) return fail(TRIAD_EINVAL, "validate must be 0 or 1");
  if (o.schedule < 0 || o.schedule > 2) return fail(TRIAD_EINVAL, "unknown schedule");
  const int variant = pick_variant(o);
  const int waves = pick_waves(o, variant);
  if (waves != 1 && waves != 2 && waves != 4) return fail(TRIAD_EINVAL, "waves_per_group must be 1, 2 or 4");
  const int64_t chunk = o.chunk > 0 ? o.chunk : 32768;
  const int64_t hub_thr = o.hub_threshold == 0 ? 65536 : o.hub_threshold;
  // schedule key: 0 none (CSR order), 1 d(u)+d(v), 2 the learned cost model
  const int sched = o.schedule == TRIAD_SCHED_PLAIN ? 0 : (o.schedule == TRIAD_SCHED_LEARNED && o.model) ? 2 : 1;
  if (chunk < 256 || chunk > ((int64_t)1 << 30)) return fail(TRIAD_EINVAL, "chunk must be in [256, 2^30]");
  DeviceInfo di;
  if (int st = device_info(&di)) return st;

  if (arena) {
    if (o.schedule != TRIAD_SCHED_PLAIN || o.task_cycles || o.timing)
      return fail(TRIAD_EINVAL, "the no-allocation census takes the plain schedule, no cycle recording and no timing");
    const size_t need = census_scratch_bound(n, nnz);
    if (need > arena_bytes)
      return fail(TRIAD_EINVAL, "graph too large for the no-allocation census: it needs " + std::to_string(need) +
                                    " bytes of scratch, the static scratch holds " + std::to_string(arena_bytes));
  }
  Scratch scratch = arena ? Scratch(s, arena, arena_bytes) : Scratch(s, allocated_before, true);
  // The default call lists triangles (sweep.hip). The merge below remains for
  // calls that ask for what only it has: a work queue of tasks to order
  // (schedules), to time (per-task cycles, wave spans) or to shape.
  if ((!labelled || n < SW_LAB_MAX_N) && o.schedule == TRIAD_SCHED_PLAIN && !o.task_cycles && !o.wave_span &&
      !o.hub_threshold && !o.chunk && !o.waves_per_group && !o.grid_groups && !o.kernel_variant) {
    unsigned long long* acc = nullptr;
    uint32_t* err = nullptr;
    uint64_t* status = nullptr;
    ALLOC(status, SW_STATUS);
    const SweepIn in{n, nnz, off, nbr, flg};
    if (int st = sweep_census(in, o.validate == 1, labelled, &acc, &err, scratch, status, s)) return st;
    // test hook: a call that passes validation reports a device fault
    if (injected_fault_pending()) {
      uint32_t eh[SW_ERRS];
      const size_t words = labelled ? SW_LAB_WORDS : SW_WORDS;
      std::vector<unsigned long long> sums(SW_COPIES * words);
      HIPCHK(hipMemcpyAsync(eh, err, sizeof eh, hipMemcpyDeviceToHost, s));
      HIPCHK(hipMemcpyAsync(sums.data(), acc, sums.size() * sizeof sums[0], hipMemcpyDeviceToHost, s));
      HIPCHK(hipStreamSynchronize(s));
      unsigned long long above = 0;
      for (int k = 0; k < SW_COPIES; ++k) above += sums[k * words + (labelled ? SW_LAB_ABOVE : SW_ABOVE)];
      if (!(eh[0] | eh[1] | eh[2]) && (int64_t)above * 2 == nnz && take_injected_fault()) k_fill_u32<<<1, 64, 0, s>>>(err + 2, 1, ERR_DEVICE);
    }
    sweep_finish(acc, err, labelled, nnz, n, d_out, status, s);
    HIPCHK(hipGetLastError());
    uint64_t hres[SW_STATUS];
    HIPCHK(hipMemcpyAsync(hres, status, sizeof hres, hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    if (int st = status_from_bits((uint32_t)hres[NC + 1]))
      return fail(st, st == TRIAD_ERANGE      ? "neighbour id out of range, zero flag, or bad offsets"
                      : st == TRIAD_ESELFLOOP ? "self-loop in the CSR"
                      : st == TRIAD_EUNSORTED ? "row not strictly increasing"
                      : st == TRIAD_EASYM     ? "CSR not symmetric or flags not mirrored"
                                              : "the device reported a fault during the census");
    if (h_out) std::memcpy(h_out, hres, (NC + 1) * sizeof(uint64_t));
    if (o.timing) {
      const uint64_t* clk = hres + SW_CLK;
      auto ms = [&](int i, int j) { return (float)((double)(int64_t)(clk[j] - clk[i]) / 1e5); };
      const bool ran = nnz > 0;  // else the counting stages were not launched
      o.timing->prep_ms = ms(0, ran ? 1 : 3);
      o.timing->tasks_ms = ran ? ms(1, 2) : 0.0f;
      o.timing->census_ms = ran ? ms(2, 3) : 0.0f;
      o.timing->finalize_ms = ms(3, 4);
      o.timing->tasks = nnz / 2;
      o.timing->hub_tasks = 0;
      o.timing->items = nnz / 2;
      o.timing->waves = labelled ? (int64_t)lab_groups(0) * LAB_WAVES
                                 : (int64_t)census_groups(waves, variant, 0, 0) * waves;
    }
    return hres[NC] ? TRIAD_OK_003_WRAPPED : TRIAD_OK;
  }
  Events ev;
  if (o.timing) HIPCHK(ev.init());
  uint32_t* err = nullptr;
  // NC census counters, 2 queue counters, hub tasks
  unsigned long long* acc = nullptr;
  ALLOC(err, 1);
  ALLOC(acc, NC + 5);
  k_fill_u32<<<1, 64, 0, s>>>(err, 1, 0);
  k_fill_u64<<<1, 64, 0, s>>>((uint64_t*)acc, NC + 5, 0);
  uint64_t clo, chi;
  choose3(n, &clo, &chi);
  ev.rec(0, s);
  uint32_t *ustart = nullptr, *rowmark = nullptr, *packed = nullptr;
  int64_t *ntask = nullptr, *tpre = nullptr;
  if (n > 0) {
    ALLOC(ustart, n);
    ALLOC(ntask, n);
    ALLOC(tpre, n + 1);
    ALLOC(rowmark, (nnz >> 5) + 1);
    ALLOC(packed, nnz + PAD);
    k_fill_u32<<<grid_for((nnz >> 5) + 1, 256, 4096), 256, 0, s>>>(rowmark, (nnz >> 5) + 1, 0);
    k_rows<<<grid_for(n, 256), 256, 0, s>>>(n, nnz, off, nbr, ustart, ntask, rowmark, err);
    if (nnz > 0) {
      k_entries<<<grid_for(nnz, 256, 16384), 256, 0, s>>>(n, nnz, nbr, flg, rowmark, packed, err);
      if (o.validate == 1) k_symmetry<<<grid_for(n, 256), 256, 0, s>>>(n, off, packed, err, err);
    }
    HIPCHK(hipGetLastError());
  }
  ev.rec(1, s);
  // the task space and hub list need sizes on the host: read the task total
  int64_t ntasks = 0, nhub = 0;
  uint32_t errh = 0;
  uint64_t* tasks = nullptr;
  uint32_t* tskip = nullptr;
  int64_t* order = nullptr;
  uint64_t* hub_task = nullptr;
  int64_t *hub_nch = nullptr, *hub_pre = nullptr;
  if (n > 0) {
    if (int st = scan_i64(ntask, n, tpre, scratch, s)) return st;
    HIPCHK(hipMemcpyAsync(&ntasks, tpre + n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    HIPCHK(hipMemcpyAsync(&errh, err, sizeof(uint32_t), hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    if (errh) {
      int st = status_from_bits(errh);
      return fail(st, st == TRIAD_ERANGE ? "neighbour id out of range, zero flag, or bad offsets"
                      : st == TRIAD_ESELFLOOP ? "self-loop in the CSR"
                      : st == TRIAD_EUNSORTED ? "row not strictly increasing"
                                              : "CSR not symmetric or flags not mirrored");
    }
    if (ntasks * 2 != nnz) return fail(TRIAD_EASYM, "CSR is not symmetric (entries above and below the diagonal differ)");
  }
  if (ntasks > 0) {
    ALLOC(tasks, ntasks);
    ALLOC(tskip, ntasks);
    const int64_t hub_cap = hub_thr >= 0 ? ntasks : 0;
    ALLOC(hub_task, hub_cap);
    ALLOC(hub_nch, hub_cap);
    ALLOC(hub_pre, hub_cap + 1);
    // Each task's count of N(v) ids below u. The entries of row v below v,
    // listed in CSR order, are the tasks (w, v) with that count as their index
    // in the row; sorted by w (stably, so v stays in order within each w) they
    // come out in task order, and their indices are the counts. The
    // no-allocation census, whose scratch is bounded, searches u in N(v) per
    // task instead.
    const bool by_sort = !arena && ntasks < ((int64_t)1 << 32);
    uint64_t *items = nullptr, *itmp = nullptr;
    int64_t* lpre = nullptr;
    if (by_sort) {
      ALLOC(items, ntasks);
      ALLOC(itmp, ntasks);
      ALLOC(lpre, n + 1);
      k_lower_counts<<<grid_for(n, 256), 256, 0, s>>>(n, ustart, ntask);
      if (int st = scan_i64(ntask, n, lpre, scratch, s)) return st;
    }
    const EmitArgs e{n, off, packed, ustart, tpre, tasks, tskip, by_sort ? 0 : 1, hub_thr, err, items, lpre};
    launch_emit_entries(e, nnz, s);
    if (by_sort) {
      const int rbu = n > 1 ? 64 - __builtin_clzll((unsigned long long)(n - 1)) : 1;  // ids below 2^rbu
      if (int st = radix_sort_u64(&items, &itmp, ntasks, 32, 32 + rbu, scratch, s)) return st;
      k_low_words<<<grid_for(ntasks, 256, 65536), 256, 0, s>>>(items, ntasks, tskip);
    }
    // A schedule reorders the last batches of the queue: in place, or, with
    // per-task cycle recording, through a queue-position -> task index map
    // that keeps the tasks (and so the cycles) in CSR order.
    if (sched) {
      if (o.task_cycles) ALLOC(order, ntasks);
      const int64_t nwaves = (int64_t)census_groups(waves, variant, o.task_cycles ? 1 : 0, o.grid_groups) * waves;
      if (int st = schedule_tail(sched, o.model, n, off, ustart, packed, tasks, tskip, ntasks, order, o.tail_share,
                                 nwaves, scratch, s))
        return st;
    }
    if (hub_thr >= 0)
      k_hub_list<<<grid_for(ntasks, HUB_TILE, 32768), 256, 0, s>>>(tasks, ntasks, off, packed, ustart, tskip, chunk,
                                                                   hub_task, hub_nch, acc + NC + 2, err);
    HIPCHK(hipGetLastError());
    if (hub_thr >= 0) {
      unsigned long long hc = 0;
      HIPCHK(hipMemcpyAsync(&hc, acc + NC + 2, sizeof(hc), hipMemcpyDeviceToHost, s));
      HIPCHK(hipStreamSynchronize(s));
      nhub = (int64_t)hc;
      if (nhub > 0) {
        if (int st = scan_i64(hub_nch, nhub, hub_pre, scratch, s)) return st;
      }
    }
  }
  ev.rec(2, s);
  int groups = 0;
  if (ntasks > 0) {
    CensusArgs a{};
    a.n = n;
    a.off = off;
    a.packed = packed;
    a.ustart = ustart;
    a.tskip = tskip;
    a.tasks = tasks;
    a.htasks = tasks;
    a.order = order;
    a.ntasks = ntasks;
    a.hub_task = hub_task;
    a.hub_pre = hub_pre;
    a.nhub = nhub;
    a.chunk = chunk;
    a.qctr = acc + NC;
    a.acc = acc;
    a.cycles = o.task_cycles;
    a.wave_span = o.wave_span;
    a.err = err;
    a.cls = class_slices();
    a.lab = lab_tables();
    if (labelled) {
      groups = lab_groups(o.grid_groups);
      HIPCHK(launch_lab(a, groups, s));
    } else {
      groups = census_groups(waves, variant, a.cycles != nullptr ? 1 : 0, o.grid_groups);
      HIPCHK(launch_census(waves, variant, a, groups, s));
    }
    HIPCHK(hipGetLastError());
  }
  // test hook: the census reports a device fault through the error flag
  if (take_injected_fault()) k_fill_u32<<<1, 64, 0, s>>>(err, 1, ERR_DEVICE);
  ev.rec(3, s);
  if (labelled)
    k_finalize_lab<<<1, 64, 0, s>>>(acc, clo, chi, err, d_out);
  else
    k_finalize<<<1, 64, 0, s>>>(acc, clo, chi, err, d_out);
  HIPCHK(hipGetLastError());
  ev.rec(4, s);
  // staged on the host: h_out is written only once the error flag is clear
  uint64_t hres[65];
  HIPCHK(hipMemcpyAsync(hres, d_out, (NC + 1) * sizeof(uint64_t), hipMemcpyDeviceToHost, s));
  HIPCHK(hipMemcpyAsync(&errh, err, sizeof(uint32_t), hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  if (errh)
    return fail(status_from_bits(errh), errh & ERR_DEVICE ? "the device reported a fault during the census"
                                                          : "input validation failed on the device");
  if (h_out) std::memcpy(h_out, hres, (NC + 1) * sizeof(uint64_t));
  const uint64_t hi0 = hres[NC];  // high word of the null count
  if (o.timing) {
    o.timing->prep_ms = ev.ms(0, 1);
    o.timing->tasks_ms = ev.ms(1, 2);
    o.timing->census_ms = ev.ms(2, 3);
    o.timing->finalize_ms = ev.ms(3, 4);
    o.timing->tasks = ntasks;
    o.timing->hub_tasks = nhub;
    o.timing->items = ntasks;
    o.timing->waves = (int64_t)groups * (labelled ? LAB_WAVES : waves);
  }
  return hi0 ? TRIAD_OK_003_WRAPPED : TRIAD_OK;
}


// ---------------------------------------------------------------- batches
// G graphs in one concatenated CSR (rows of graph g: [vbase[g], vbase[g+1]),
// graph-local neighbour ids). Rebasing every id by vbase[g] turns the batch
// into one disjoint union; a task never leaves its graph, so the single-graph
// kernels apply unchanged except that each graph keeps its own counters.

// Per row of a batch: its graph, offset checks, the first entry above the
// row (binary search over its graph-local ids), the self-loop check, the task
// count and the row-start mark.
__global__ void k_rows_batch(int32_t G, int64_t nv, int64_t nnz, const int64_t* __restrict__ vbase,
                             const int64_t* __restrict__ off, const int32_t* __restrict__ nbr,
                             uint32_t* __restrict__ grow, uint32_t* __restrict__ ustart, int64_t* __restrict__ ntask,
                             uint32_t* __restrict__ rowmark, uint32_t* __restrict__ err) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < nv; u += stride) {
    int32_t lo = 0, hi = G;  // last graph with vbase[g] <= u
    while (hi - lo > 1) {
      const int32_t mid = (lo + hi) >> 1;
      if (vbase[mid] <= u) lo = mid; else hi = mid;
    }
    grow[u] = (uint32_t)lo;
    const int64_t g0 = vbase[lo];
    const int64_t b = off[u], e = off[u + 1];
    ustart[u] = 0;
    ntask[u] = 0;
    if ((u == 0 && b != 0) || (u == nv - 1 && e != nnz) || e < b || b < 0 || e > nnz) {
      atomicOr(err, ERR_RANGE);
      continue;
    }
    const int32_t ul = (int32_t)(u - g0);
    int64_t p = b, q = e;  // first entry with a local id above ul
    while (p < q) {
      const int64_t m = (p + q) >> 1;
      if (nbr[m] <= ul) p = m + 1; else q = m;
    }
    if (p > b && nbr[p - 1] == ul) atomicOr(err, ERR_SELFLOOP);
    ustart[u] = (uint32_t)(p - b);
    ntask[u] = e - p;
    if (e > b) atomicOr(&rowmark[b >> 5], 1u << (b & 31));
  }
}

// Per entry of a batch: graph-local id in range, flag not 0, rows strictly
// increasing, and the packed word with the id moved to the disjoint union
// (graph base added). An entry's graph is the last one whose first entry
// (off[vbase[g]]) is not after it; a tile of ETILE entries usually lies in one
// graph (found once per tile), else its entries search the tile's few graphs.
__device__ __forceinline__ int32_t graph_of_entry(const int64_t* __restrict__ off, const int64_t* __restrict__ vbase,
                                                  int32_t lo, int32_t hi, int64_t j) {
  // off[vbase[lo]] <= j; the answer lies in [lo, hi)
  while (hi - lo > 1) {
    const int32_t mid = (lo + hi) >> 1;
    if (off[vbase[mid]] <= j) lo = mid; else hi = mid;
  }
  return lo;
}
__global__ void __launch_bounds__(256) k_entries_batch(int32_t G, int64_t nnz, const int64_t* __restrict__ vbase,
                                                       const int64_t* __restrict__ off, const int32_t* __restrict__ nbr,
                                                       const uint8_t* __restrict__ flg,
                                                       const uint32_t* __restrict__ rowmark,
                                                       uint32_t* __restrict__ packed, uint32_t* __restrict__ err) {
  __shared__ int32_t gr[2];
  uint32_t bits = 0;
  for (int64_t t0 = (int64_t)blockIdx.x * ETILE; t0 < nnz; t0 += (int64_t)gridDim.x * ETILE) {
    const int64_t t1 = min(t0 + (int64_t)ETILE, nnz);
    if (threadIdx.x < 2) gr[threadIdx.x] = graph_of_entry(off, vbase, 0, G, threadIdx.x ? t1 - 1 : t0);
    __syncthreads();
    const int32_t ga = gr[0], gb = gr[1];
    for (int64_t j = t0 + threadIdx.x; j < t1; j += blockDim.x) {
      const int32_t gx = ga == gb ? ga : graph_of_entry(off, vbase, ga, gb + 1, j);
      const int64_t g0 = vbase[gx], ng = vbase[gx + 1] - g0;
      const int32_t y = nbr[j];
      const uint32_t f = (flg[j >> 2] >> (2 * (j & 3))) & 3u;
      if (y < 0 || y >= ng || f == 0) bits |= ERR_RANGE;
      if (j + 1 < nnz) {
        const bool row_start = (rowmark[(j + 1) >> 5] >> ((j + 1) & 31)) & 1u;
        if (!row_start && nbr[j + 1] <= y) bits |= ERR_UNSORTED;
      }
      packed[j] = ((uint32_t)(y + g0) << 2) | f;
    }
    __syncthreads();
  }
  if (bits) atomicOr(err, bits);
}

__global__ void k_check_tasks(const int64_t* __restrict__ tpre, int64_t nv, int64_t nnz, uint32_t* __restrict__ err) {
  if (threadIdx.x == 0 && blockIdx.x == 0 && tpre[nv] * 2 != nnz) atomicOr(err, ERR_ASYM);
}

// Per graph: 003 = C(n_g, 3) minus the rest (n_g < 4,801,281 keeps C(n_g,3) < 2^64).
__global__ void k_finalize_batch(int32_t G, const int64_t* __restrict__ vbase,
                                 const unsigned long long* __restrict__ gout, const uint32_t* __restrict__ err,
                                 uint64_t* __restrict__ out) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= G || *err) return;
  const uint64_t n = (uint64_t)(vbase[g + 1] - vbase[g]);
  uint64_t c3 = 0;
  if (n >= 3) {
    // n(n-1)(n-2)/6 without overflow: divide the factors first
    uint64_t a = n, b = n - 1, c = n - 2;
    if (a % 2 == 0) a /= 2; else b /= 2;
    if (a % 3 == 0) a /= 3; else if (b % 3 == 0) b /= 3; else c /= 3;
    c3 = a * b * c;
  }
  uint64_t c[16];
  for (int k = 0; k < 16; ++k) c[k] = gout[16 * (uint64_t)g + k];
  add_common_neighbours(c);
  uint64_t s = 0;
  for (int k = 1; k < 16; ++k) {
    out[16 * (uint64_t)g + k] = c[k];
    s += c[k];
  }
  out[16 * (uint64_t)g] = c3 - s;
}

// Content signature of a batch for the autotuner's cache: a sum of hashes of
// (row, offset) pairs and of the graph bases, and the sum of squared degrees.
__device__ __forceinline__ uint64_t sig_mix(uint64_t z) {
  z ^= z >> 30;
  z *= 0xbf58476d1ce4e5b9ull;
  z ^= z >> 27;
  z *= 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}
__global__ void k_batch_signature(int32_t G, int64_t nv, const int64_t* __restrict__ vbase,
                                  const int64_t* __restrict__ off, unsigned long long* __restrict__ sig) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  uint64_t h = 0, s2 = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i <= nv; i += stride) {
    h += sig_mix((uint64_t)off[i] * 0x9e3779b97f4a7c15ull + (uint64_t)i);
    if (i < nv) {
      const uint64_t d = (uint64_t)(off[i + 1] - off[i]);
      s2 += d * d;
    }
    if (i <= G) h += sig_mix(~((uint64_t)vbase[i] * 0xd1b54a32d192ed03ull + (uint64_t)i));
  }
  h = wave_sum64(h);
  s2 = wave_sum64(s2);
  if ((threadIdx.x & 63) == 0) {
    atomicAdd(&sig[0], (unsigned long long)h);
    atomicAdd(&sig[1], (unsigned long long)s2);
  }
}

}  // namespace triad

struct triad_batch_plan {
  int32_t G = 0;
  int64_t nv = 0, nnz = 0;
  const int64_t* vbase = nullptr;
  uint64_t* out = nullptr;
  std::vector<void*> bufs;
  uint32_t* err = nullptr;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  hipStream_t last = nullptr;
  int launched = 0;
  bool drained = true;  // nothing launched since the last wait
  bool several = false;  // launches on several streams that no wait has covered
  size_t bytes = 0;  // device memory the plan holds (counted against the memory cap)
  void* block = nullptr;  // its one scratch block, from the held blocks of `device`
  size_t block_bytes = 0;
  int device = -1;
};

namespace triad {

static void plan_free(triad_batch_plan* p) {
  if (!p) return;
  if (p->exec) (void)hipGraphExecDestroy(p->exec);
  if (p->graph) (void)hipGraphDestroy(p->graph);
  for (void* b : p->bufs) (void)hipFree(b);
  if (p->block) {
    // hipFree would wait for the device; a kept block has to wait as well
    // before another call may take it
    int dev = -1;
    (void)hipGetDevice(&dev);
    if (dev != p->device) (void)hipSetDevice(p->device);
    const bool idle = p->drained || hipDeviceSynchronize() == hipSuccess;
    if (dev != p->device) (void)hipSetDevice(dev);
    if (idle) held_give(p->block, p->block_bytes, p->device);
    else (void)hipFree(p->block);
  }
  delete p;
}

template <class T>
static hipError_t plan_alloc(triad_batch_plan* p, T** ptr, int64_t count) {
  const size_t bytes = (size_t)std::max<int64_t>(count, 1) * sizeof(T);
  if (!within_cap(p->bytes + bytes)) return hipErrorOutOfMemory;
  hipError_t e = hipMalloc((void**)ptr, bytes);
  if (e == hipSuccess) {
    p->bufs.push_back(*ptr);
    p->bytes += bytes;
  }
  return e;
}

// Graph bases of a batch: vbase[0] = 0, non-decreasing, vbase[G] = nv, and
// every member below BATCH_MAX_N vertices (C(n_g, 3) < 2^64).
constexpr int64_t BATCH_MAX_N = 4801281;
static int check_vbase(int32_t G, int64_t nv, const int64_t* hv, int64_t* nmax = nullptr) {
  if (nmax) *nmax = 0;
  if (hv[0] != 0) return fail(TRIAD_EINVAL, "vbase[0] must be 0");
  if (hv[G] != nv) return fail(TRIAD_EINVAL, "vbase[G] must equal the number of rows nv");
  for (int32_t g = 0; g < G; ++g) {
    if (hv[g + 1] < hv[g]) return fail(TRIAD_EINVAL, "vbase is not non-decreasing at graph " + std::to_string(g));
    if (hv[g + 1] - hv[g] >= BATCH_MAX_N)
      return fail(TRIAD_EINVAL, "graph " + std::to_string(g) + " has 4,801,281 or more vertices (its 003 count "
                                "would not fit in 64 bits); census it on its own");
    if (nmax) *nmax = std::max(*nmax, hv[g + 1] - hv[g]);
  }
  return TRIAD_OK;
}

// Entries that a wavefront of the batched triangle listing takes per turn, by
// kernel variant (0: left to sweep_batch): 512, 1,024, 2,048 and 256 for 1 .. 4, the
// autotuner's candidates (5 .. 8 the same). Workgroups of two wavefronts on 4,096
// graphs of up to 8,192 vertices: 17.7, 16.8, 16.7, 19.8 ms; on 64 of up to 900: 0.106,
// 0.131, 0.174, 0.099.
static int64_t batch_range(int32_t variant) {
  return variant <= 0 || variant > NUM_VARIANTS ? 0 : (int64_t)128 << (variant % 4 + 1);
}

static int plan_build(int32_t G, int64_t nv, int64_t nnz, const int64_t* vbase, const int64_t* off, const int32_t* nbr,
                      const uint8_t* flg, uint64_t* d_out, const triad_opts* opts, hipStream_t s,
                      triad_batch_plan** out_plan) {
  triad_opts o{};
  if (opts) o = *opts;
  if (G < 1 || nv < 0 || nv >= ((int64_t)1 << 30) || nnz < 0 || nnz >= ((int64_t)1 << 40))
    return fail(TRIAD_EINVAL, "bad batch sizes");
  if (!vbase || !off || !d_out || (nnz > 0 && (!nbr || !flg)) || !out_plan) return fail(TRIAD_EINVAL, "NULL pointer");
  const int variant = pick_variant(o);
  const int waves = pick_waves(o, variant);
  if (waves != 1 && waves != 2 && waves != 4) return fail(TRIAD_EINVAL, "waves_per_group must be 1, 2 or 4");
  DeviceInfo di;
  if (int st = device_info(&di)) return st;
  int64_t nmax = 0;
  // The graph bases are checked on the host before anything is captured or
  // launched: every kernel indexes rows through them, and each member's null
  // count C(n_g, 3) is formed in 64 bits.
  {
    std::vector<int64_t> hv((size_t)G + 1);
    HIPCHK(hipMemcpyAsync(hv.data(), vbase, sizeof(int64_t) * ((size_t)G + 1), hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    if (int st = check_vbase(G, nv, hv.data(), &nmax)) return st;
  }
  triad_batch_plan* p = new triad_batch_plan;
  p->G = G;
  p->nv = nv;
  p->nnz = nnz;
  p->vbase = vbase;
  p->out = d_out;
  // Triangles are listed unless the caller asks for the per-task merge
  const bool merge = o.short_tasks < 0;
  uint32_t *grow = nullptr, *ustart = nullptr, *packed = nullptr, *tskip = nullptr, *rowmark = nullptr;
  int64_t *ntask = nullptr, *tpre = nullptr, *bsum = nullptr;
  uint64_t* tasks = nullptr;
  unsigned long long* q = nullptr;  // census queue [2]
  const int64_t ntasks = nnz / 2;
  unsigned long long* gacc = nullptr;  // per-graph counters; d_out is written only by a clean finalize
  bool failed = false;
  if (merge) {
    failed = plan_alloc(p, &p->err, 1) || plan_alloc(p, &q, 2) || plan_alloc(p, &gacc, (int64_t)G * 16) ||
             plan_alloc(p, &grow, nv) || plan_alloc(p, &ustart, nv) || plan_alloc(p, &ntask, nv) ||
             plan_alloc(p, &tpre, nv + 1) || plan_alloc(p, &bsum, nv / SCAN_B + 2) ||
             plan_alloc(p, &packed, nnz + PAD) || plan_alloc(p, &tasks, ntasks) || plan_alloc(p, &tskip, ntasks) ||
             plan_alloc(p, &rowmark, (nnz >> 5) + 1);
  } else {
    p->device = di.device;
    const size_t bytes = sweep_batch_bytes(G, nv, nnz);
    failed = !within_cap(bytes) || held_take(&p->block, bytes, &p->block_bytes) != hipSuccess;
    p->bytes = bytes;
  }
  if (failed) {
    p->block_bytes = 0;
    plan_free(p);
    (void)hipGetLastError();
    return fail(TRIAD_ENOMEM, "device allocation for the batch plan failed");
  }
  // capture the whole batched census as one graph (fills instead of memsets)
  // on a private stream: the caller's stream may be the legacy null stream,
  // which cannot be captured; launches replay it on the caller's stream
  hipStream_t cs = nullptr;
  hipError_t e = hipStreamCreateWithFlags(&cs, hipStreamNonBlocking);
  if (e == hipSuccess) e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
  if (e != hipSuccess) {
    if (cs) (void)hipStreamDestroy(cs);
    plan_free(p);
    return fail(TRIAD_EDEVICE, std::string("hipStreamBeginCapture: ") + hipGetErrorString(e));
  }
  s = cs;
  int st = TRIAD_OK;
  if (merge) {
    k_fill_u32<<<1, 64, 0, s>>>(p->err, 1, 0);
    k_fill_u64<<<1, 64, 0, s>>>((uint64_t*)q, 2, 0);  // queue counters
    k_fill_u64<<<grid_for((int64_t)G * 16, 256, 4096), 256, 0, s>>>((uint64_t*)gacc, (int64_t)G * 16, 0);
    if (nv > 0) {
      k_fill_u32<<<grid_for((nnz >> 5) + 1, 256, 4096), 256, 0, s>>>(rowmark, (nnz >> 5) + 1, 0);
      k_rows_batch<<<grid_for(nv, 256, 65535), 256, 0, s>>>(G, nv, nnz, vbase, off, nbr, grow, ustart, ntask, rowmark,
                                                            p->err);
      if (nnz > 0)
        k_entries_batch<<<grid_for(nnz, ETILE, 65536), 256, 0, s>>>(G, nnz, vbase, off, nbr, flg, rowmark, packed,
                                                                   p->err);
      st = scan_i64_with(ntask, nv, tpre, bsum, s);  // (a failure: the capture is ended and the plan freed below)
      k_check_tasks<<<1, 64, 0, s>>>(tpre, nv, nnz, p->err);
      if (ntasks > 0) {
        const EmitArgs ea{nv, off, packed, ustart, tpre, tasks, tskip, 0, -1, p->err, nullptr, nullptr};
        launch_emit_entries(ea, nnz, s);
        CensusArgs a{};
        a.off = off;
        a.packed = packed;
        a.ustart = ustart;
        a.tskip = tskip;
        a.tasks = tasks;
        a.htasks = tasks;
        a.ntasks = ntasks;
        a.chunk = 1;
        a.qctr = q;
        a.acc = gacc;
        a.grow = grow;
        a.vbase = vbase;
        a.gout = gacc;
        a.err = p->err;
        a.cls = class_slices();
        (void)launch_census(waves, variant, a, census_groups(waves, variant, 2, o.grid_groups), s);
      }
    }
    k_finalize_batch<<<(G + 255) / 256, 256, 0, s>>>(G, vbase, gacc, p->err, d_out);
  } else {
    Scratch arena(s, p->block, p->block_bytes);
    const SweepIn in{nv, nnz, off, nbr, flg};
    const int wpg = o.waves_per_group ? o.waves_per_group : 4;
    const int groups = o.grid_groups > 0 ? o.grid_groups : 2 * sweep_batch_groups(wpg);
    st = sweep_batch(G, nv, in, vbase, nmax, wpg, groups, batch_range(o.kernel_variant), d_out, &p->err, arena, s);
  }
  e = hipStreamEndCapture(s, &p->graph);
  if (e == hipSuccess) e = hipGraphInstantiate(&p->exec, p->graph, nullptr, nullptr, 0);
  (void)hipStreamDestroy(cs);
  if (st != TRIAD_OK || e != hipSuccess) {
    plan_free(p);
    return st != TRIAD_OK ? st
                          : fail(TRIAD_EDEVICE, std::string("batch graph capture failed: ") + hipGetErrorString(e));
  }
  *out_plan = p;
  return TRIAD_OK;
}

}  // namespace triad

using namespace triad;

// Scratch of the no-allocation census: one copy per GPU, held until the
// process ends. Host code never passes this name to a kernel (on the host it
// is a stand-in, not a device address); it takes each device's address once
// with hipGetSymbolAddress and uses that.
static __device__ __align__(256) unsigned char scratch[TRIAD_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
std::mutex g_noalloc_mu;
void* g_noalloc_ptr[MAX_DEVICES] = {};

// The calling thread's current device's copy of `scratch` (address taken on
// the first call for that device, with it current).
int noalloc_scratch(void** out) {
  int dev = -1;
  HIPCHK(hipGetDevice(&dev));
  if (dev < 0 || dev >= MAX_DEVICES) return fail(TRIAD_EDEVICE, "device index out of range for the static scratch");
  std::lock_guard<std::mutex> lk(g_noalloc_mu);
  if (!g_noalloc_ptr[dev]) {
    void* p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      return fail(TRIAD_EDEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
    g_noalloc_ptr[dev] = p;
  }
  *out = g_noalloc_ptr[dev];
  return TRIAD_OK;
}
}  // namespace

extern "C" {

int triad_census_device_noalloc(int64_t n, int64_t nnz, const int64_t* off, const int32_t* nbr, const uint8_t* flg,
                                const triad_opts* opts, void* stream, uint64_t* d_out, uint64_t* h_out) {
  void* base = nullptr;
  if (int st = noalloc_scratch(&base)) return st;
  return census_device(n, nnz, off, nbr, flg, opts, (hipStream_t)stream, d_out, h_out, base,
                       (size_t)TRIAD_NOALLOC_SCRATCH_BYTES);
}

int triad_census_device(int64_t n, int64_t nnz, const int64_t* off, const int32_t* nbr, const uint8_t* flg,
                        const triad_opts* opts, void* stream, uint64_t* d_out, uint64_t* h_out) {
  return census_device(n, nnz, off, nbr, flg, opts, (hipStream_t)stream, d_out, h_out);
}

int triad_labelled_census_device(int64_t n, int64_t nnz, const int64_t* off, const int32_t* nbr, const uint8_t* flg,
                                 const triad_opts* opts, void* stream, uint64_t* d_out, uint64_t* h_out) {
  return census_device(n, nnz, off, nbr, flg, opts, (hipStream_t)stream, d_out, h_out, nullptr, 0, true);
}

int triad_census_ex(int64_t n, const int64_t* off, const int32_t* nbr, const uint8_t* flg, const triad_opts* opts,
                    uint64_t out_u64[16], uint64_t* out_003_hi) {
  if (!out_u64) return fail(TRIAD_EINVAL, "out_u64 is NULL");
  const int level = opts ? opts->validate : 0;
  // The offsets are checked here (the copies are sized by them), the entries on
  // the device, which finds the same faults in the same order of importance: one
  // host thread took 5.3 of 6.9 ms for 5.4 M entries. A call that fails before
  // the device has looked reports what the host check finds, if anything.
  if (int st = validate_offsets(n, off, nbr, flg)) return st;
  auto failed = [&](int status, const char* msg) {
    const int st = triad_validate_host(n, off, nbr, flg, level);
    return st ? st : fail(status, msg);
  };
  const int64_t nnz = off[n];
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return failed(TRIAD_EDEVICE, "no HIP device available");
  const size_t in_bytes = sizeof(int64_t) * (n + 1) + sizeof(int32_t) * std::max<int64_t>(nnz, 1) +
                          std::max<int64_t>((nnz + 3) / 4, 1) + 17 * sizeof(uint64_t);
  if (!within_cap(in_bytes)) return failed(TRIAD_ENOMEM, "the input copy alone exceeds the memory cap");
  hipStream_t s;
  if (hipStreamCreate(&s) != hipSuccess) return failed(TRIAD_EDEVICE, "hipStreamCreate failed");
  uint64_t h[17];
  int st = TRIAD_OK;
  {
    Scratch copies(s, 0, true);  // gives its blocks back once the stream has drained
    int64_t* d_off = nullptr;
    int32_t* d_nbr = nullptr;
    uint8_t* d_flg = nullptr;
    uint64_t* d_out = nullptr;
    if (copies.get(&d_off, n + 1) != hipSuccess || copies.get(&d_nbr, nnz) != hipSuccess ||
        copies.get(&d_flg, (nnz + 3) / 4) != hipSuccess || copies.get(&d_out, 17) != hipSuccess) {
      (void)hipGetLastError();
      st = failed(TRIAD_ENOMEM, "device allocation for the input copy failed");
    } else if (hipMemcpyAsync(d_off, off, sizeof(int64_t) * (n + 1), hipMemcpyHostToDevice, s) != hipSuccess ||
               (nnz > 0 && hipMemcpyAsync(d_nbr, nbr, sizeof(int32_t) * nnz, hipMemcpyHostToDevice, s) != hipSuccess) ||
               (nnz > 0 && hipMemcpyAsync(d_flg, flg, (nnz + 3) / 4, hipMemcpyHostToDevice, s) != hipSuccess)) {
      st = failed(TRIAD_EDEVICE, "host to device copy failed");
    } else {
      st = census_device(n, nnz, d_off, d_nbr, d_flg, opts, s, d_out, h, nullptr, 0, false, in_bytes);
      // (the status a host check would have given before memory was asked for)
      if (st == TRIAD_ENOMEM || st == TRIAD_EINVAL) {
        const std::string msg = triad_last_error();
        st = failed(st, msg.c_str());
      }
    }
  }
  (void)hipStreamDestroy(s);
  if (st >= 0) {
    std::memcpy(out_u64, h, 16 * sizeof(uint64_t));
    if (out_003_hi) *out_003_hi = h[16];
  }
  return st;
}

int triad_census(int64_t n, const int64_t* off, const int32_t* nbr, const uint8_t* flg, uint64_t out_u64[16]) {
  return triad_census_ex(n, off, nbr, flg, nullptr, out_u64, nullptr);
}


int triad_batch_plan_create(int32_t G, int64_t nv, int64_t nnz, const int64_t* d_vbase, const int64_t* d_offsets,
                            const int32_t* d_nbrs, const uint8_t* d_flags, uint64_t* d_out, const triad_opts* opts,
                            void* hip_stream, triad_batch_plan** plan) {
  return plan_build(G, nv, nnz, d_vbase, d_offsets, d_nbrs, d_flags, d_out, opts, (hipStream_t)hip_stream, plan);
}

int triad_batch_plan_launch(triad_batch_plan* plan, void* hip_stream) {
  if (!plan || !plan->exec) return fail(TRIAD_EINVAL, "invalid plan");
  hipStream_t s = (hipStream_t)hip_stream;
  HIPCHK(hipGraphLaunch(plan->exec, s));
  if (!plan->drained && plan->last != s) plan->several = true;
  plan->last = s;
  plan->launched = 1;
  plan->drained = false;
  return TRIAD_OK;
}

int triad_batch_plan_status(triad_batch_plan* plan) {
  if (!plan) return fail(TRIAD_EINVAL, "invalid plan");
  if (!plan->launched) return fail(TRIAD_EINVAL, "plan not launched");
  uint32_t e = 0;
  HIPCHK(hipMemcpyAsync(&e, plan->err, sizeof(e), hipMemcpyDeviceToHost, plan->last));
  HIPCHK(hipStreamSynchronize(plan->last));
  plan->drained = !plan->several;  // (only the last launch's stream was waited for)
  if (e) return fail(status_from_bits(e), "batch input validation failed on the device");
  return TRIAD_OK;
}

void triad_batch_plan_destroy(triad_batch_plan* plan) { plan_free(plan); }

int triad_census_batch(int32_t G, int64_t nv, int64_t nnz, const int64_t* d_vbase, const int64_t* d_offsets,
                       const int32_t* d_nbrs, const uint8_t* d_flags, const triad_opts* opts, void* hip_stream,
                       uint64_t* d_out) {
  triad_batch_plan* p = nullptr;
  if (int st = triad_batch_plan_create(G, nv, nnz, d_vbase, d_offsets, d_nbrs, d_flags, d_out, opts, hip_stream, &p))
    return st;
  int st = triad_batch_plan_launch(p, hip_stream);
  if (st == TRIAD_OK) st = triad_batch_plan_status(p);
  triad_batch_plan_destroy(p);
  return st;
}

int triad_batch_autotune(int32_t G, int64_t nv, int64_t nnz, const int64_t* d_vbase, const int64_t* d_offsets,
                         const int32_t* d_nbrs, const uint8_t* d_flags, void* hip_stream, const char* cache_path,
                         triad_opts* best) {
  if (!best) return fail(TRIAD_EINVAL, "best is NULL");
  if (G < 1 || nv < 0 || nv >= ((int64_t)1 << 30) || nnz < 0 || !d_vbase || !d_offsets)
    return fail(TRIAD_EINVAL, "bad batch sizes or NULL pointer");
  DeviceInfo di;
  if (int st = device_info(&di)) return st;
  hipStream_t s = (hipStream_t)hip_stream;
  {
    std::vector<int64_t> hv((size_t)G + 1);
    HIPCHK(hipMemcpyAsync(hv.data(), d_vbase, sizeof(int64_t) * ((size_t)G + 1), hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    if (int st = check_vbase(G, nv, hv.data())) return st;
  }
  // the batch's content signature: equal sizes alone do not make equal batches
  unsigned long long hsig[2] = {0, 0};
  {
    unsigned long long* dsig = nullptr;
    HIPCHK(hipMallocAsync((void**)&dsig, 2 * sizeof(unsigned long long), s));
    k_fill_u64<<<1, 64, 0, s>>>((uint64_t*)dsig, 2, 0);
    k_batch_signature<<<grid_for(nv + 1, 256, 4096), 256, 0, s>>>(G, nv, d_vbase, d_offsets, dsig);
    hipError_t e = hipMemcpyAsync(hsig, dsig, sizeof hsig, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipFreeAsync(dsig, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail(TRIAD_EDEVICE, std::string("batch signature: ") + hipGetErrorString(e));
  }
  char sig[256];
  snprintf(sig, sizeof sig, "%s|G=%d|nv=%lld|nnz=%lld|h=%016llx|d2=%llu", di.name.c_str(), (int)G, (long long)nv,
           (long long)nnz, hsig[0], hsig[1]);
  // the candidate launch shapes; a cached line naming any other is ignored. (The
  // default's four wavefronts are not among them: one and two are as fast or faster,
  // 16.55 against 16.78 ms on 4,096 graphs of up to 8,192 vertices, 0.099 against 0.153
  // on 64 of up to 900.)
  const int variants[4] = {1, 2, 3, 4};
  const int wavess[2] = {1, 2};
  auto candidate = [&](int kv, int wv, int gg) {
    for (int vi = 0; vi < 4; ++vi)
      for (int wi = 0; wi < 2; ++wi)
        for (int gm = 1; gm <= 2; ++gm)
          if (kv == variants[vi] && wv == wavess[wi] && gg == sweep_batch_groups(wv) * gm) return true;
    return false;
  };
  // cache: one JSON object per line: {"sig": "...", "kernel_variant": k, "waves_per_group": w, "grid_groups": g, "ms": t}
  if (cache_path) {
    if (FILE* f = fopen(cache_path, "r")) {
      char line[512];
      while (fgets(line, sizeof line, f)) {
        char want[300];
        snprintf(want, sizeof want, "\"sig\": \"%s\"", sig);
        if (!strstr(line, want)) continue;
        int kv = 0, wv = 0, gg = 0;
        const char* p1 = strstr(line, "\"kernel_variant\": ");
        const char* p2 = strstr(line, "\"waves_per_group\": ");
        const char* p3 = strstr(line, "\"grid_groups\": ");
        if (p1 && p2 && p3 && sscanf(p1 + 18, "%d", &kv) == 1 && sscanf(p2 + 19, "%d", &wv) == 1 &&
            sscanf(p3 + 15, "%d", &gg) == 1 && candidate(kv, wv, gg)) {
          *best = triad_opts{};
          best->kernel_variant = kv;
          best->waves_per_group = wv;
          best->grid_groups = gg;
          fclose(f);
          return TRIAD_OK;
        }
      }
      fclose(f);
    }
  }
  uint64_t* out = nullptr;
  HIPCHK(hipMalloc(&out, sizeof(uint64_t) * 16 * (size_t)G));
  hipEvent_t e0, e1;
  HIPCHK(hipEventCreate(&e0));
  HIPCHK(hipEventCreate(&e1));
  float best_ms = 1e30f;
  triad_opts bo{};
  int status = TRIAD_OK;
  for (int vi = 0; vi < 4 && status == TRIAD_OK; ++vi)
    for (int wi = 0; wi < 2 && status == TRIAD_OK; ++wi)
      for (int gm = 1; gm <= 2; ++gm) {
        triad_opts o{};
        o.kernel_variant = variants[vi];
        o.waves_per_group = wavess[wi];
        o.grid_groups = sweep_batch_groups(o.waves_per_group) * gm;
        triad_batch_plan* p = nullptr;
        status = triad_batch_plan_create(G, nv, nnz, d_vbase, d_offsets, d_nbrs, d_flags, out, &o, hip_stream, &p);
        if (status != TRIAD_OK) break;
        float t = 1e30f;
        for (int rep = 0; rep < 3 && status == TRIAD_OK; ++rep) {
          (void)hipEventRecord(e0, s);
          status = triad_batch_plan_launch(p, hip_stream);
          (void)hipEventRecord(e1, s);
          if (status == TRIAD_OK) status = triad_batch_plan_status(p);
          float ms = 0;
          (void)hipEventElapsedTime(&ms, e0, e1);
          if (rep > 0 && ms < t) t = ms;  // first launch is a warm-up
        }
        triad_batch_plan_destroy(p);
        if (status == TRIAD_OK && t < best_ms) {
          best_ms = t;
          bo = o;
        }
      }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  (void)hipFree(out);
  if (status != TRIAD_OK) return status;
  *best = bo;
  if (cache_path) {
    if (FILE* f = fopen(cache_path, "a")) {
      fprintf(f, "{\"sig\": \"%s\", \"kernel_variant\": %d, \"waves_per_group\": %d, \"grid_groups\": %d, \"ms\": %.3f}\n",
              sig, bo.kernel_variant, bo.waves_per_group, bo.grid_groups, best_ms);
      fclose(f);
    }
  }
  return TRIAD_OK;
}

}  // extern "C"
