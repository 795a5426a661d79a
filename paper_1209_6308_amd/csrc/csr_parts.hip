// CSR construction by parts: the arcs' entries are split into buckets of whole
// rows that one workgroup sorts in LDS.
//
// A radix sort of 64-bit (row, column) keys moves every key once per 8 bits of
// row and column: six passes at 2^24 vertices, each a read for the digit
// counts, a read and a write. Here an entry moves twice before its bucket fits
// into LDS, and it shrinks on the way. The bucket of an entry is given by the
// top B bits of mix(row), a bijection of the row ids that spreads the heavy
// rows evenly, and the 32-bit key of an entry in its bucket is
//     low bits of mix(row) | column | direction
// with direction 0 for the arc row -> column. The order of the buckets does not
// matter, only that each holds whole rows: rows go to their places in id order
// at the end.
//
//   k_bp_count1   range check, self-loops dropped, counts of the first digit
//                 of the bucket (per block of a fixed range of arcs)
//   k_bp_split1   arcs -> keys by the first digit, with the second digit
//                 (16 bits) beside them
//   k_bp_parts    the first digit's buckets cut into parts of equal size
//   k_bp_count2, k_bp_split2   keys by the second digit
//   k_bp_sizes    bucket starts, lists of the buckets too long for k_bp_sort
//   k_bp_sort     a bucket: sorted in LDS, runs of equal (row, column) merged to
//                 one entry (column << 2 | flags), places of the rows
//   k_bp_mid      the same for up to 32,768 keys (listed)
//   k_bp_long_*   longer buckets (listed): sorted through memory by all workgroups
//   k_bp_row_*    places of the rows -> offsets
//   k_bp_out      ids and packed flags in row order
//
// R-MAT scale 24, 268 M arcs of which 2.1 GB are read and 2.1
// GB written at least: 25.4 ms by the general sort, 9.8 so; the splits move 11.6
// GB in 3.9 ms with their counts (1.95 + 1.95), the LDS sorts of 537 M keys take
// 4.0 (bound by vector instructions), long buckets 0.6, rows and ids 1.3.
// Within a split, order does not matter (the buckets are sorted after it), so
// a key's place comes from an LDS counter; a block keeps its places in each
// digit's run for its whole range, so that consecutive tiles of a block
// continue the same lines.
#include <hip/hip_runtime.h>

#include <string>

#include "csr_parts.h"
#include "device_sort.h"
#include "lds_sort.h"

namespace triad {
namespace {

constexpr int ST = 1024;                // threads of the split kernels
constexpr int S1_ARCS = 8192;           // arcs of one tile of k_bp_split1 (two entries each)
constexpr int S1_PER = S1_ARCS / ST;
constexpr int S1_GROUPS = 1024;         // blocks of k_bp_count1 and k_bp_split1 at most
constexpr int S2_TILE = 16384, S2_PER = S2_TILE / ST;
constexpr int64_t PART = 1 << 16;       // entries of one block of k_bp_count2 and k_bp_split2
constexpr int DIGITS = 1024;            // of one split at most (10 bits)
constexpr int AVG_BITS = 11;            // a bucket holds about 2^11 keys at most
constexpr int CAP = 4096, MID_CAP = 16384, TOP_CAP = 32768;  // keys of a bucket: k_bp_sort, k_bp_mid
constexpr int LT = 512, L_PER = 16, L_PART = LT * L_PER;  // keys of one block of the long buckets' kernels
constexpr int RT = 256, RI = 8;          // rows: threads of a block, rows of a thread
constexpr int OT = 4096;                // entries of one tile of k_bp_out

// W_LPARTS, W_NLONG: one 64-bit word, so that the parts' numbers grow with the list
enum { W_ERR = 0, W_NMID = 1, W_NTOP = 2, W_LPARTS = 4, W_NLONG = 5, W_WORDS = 8 };

struct Bp {
  int64_t n, narcs;
  const int32_t *src, *dst;
  int rb;               // ids below 2^rb
  int b1, b2, low;      // bits of the two digits, row bits left in the key: rb = b1 + b2 + low
  uint32_t mul, inv, mask;
  uint32_t* w;          // W_ words
};

__device__ __forceinline__ uint32_t mix(const Bp& a, uint32_t x) { return (x * a.mul) & a.mask; }
__device__ __forceinline__ uint32_t digit1(const Bp& a, uint32_t m) { return a.b1 ? m >> (a.rb - a.b1) : 0u; }
__device__ __forceinline__ uint32_t digit2(const Bp& a, uint32_t m) { return (m >> a.low) & ((1u << a.b2) - 1u); }
__device__ __forceinline__ uint32_t key_of(const Bp& a, uint32_t m, uint32_t col, uint32_t dir) {
  // low + rb + 1 <= 32; a shift by 32 when nothing of the row is left is avoided
  const uint32_t r = m & ((1u << a.low) - 1u);
  return (a.low ? r << (a.rb + 1) : 0u) | col << 1 | dir;
}

// exclusive sum over the threads of a block; sh has a word per wavefront
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t* sh) {
  const int w = threadIdx.x >> 6;
  const uint32_t x = wave_scan(v);
  if ((threadIdx.x & 63) == 63) sh[w] = x;
  __syncthreads();
  uint32_t base = x - v;
  for (int q = 0; q < w; ++q) base += sh[q];
  return base;
}

// The last split also clears the rows' ends (outputs: not before the host has
// looked).
__device__ __forceinline__ void no_rows(int64_t n, int64_t* end) {
  for (int64_t x = (int64_t)blockIdx.x * ST + threadIdx.x; x < n; x += (int64_t)gridDim.x * ST) end[x] = 0;
}

__global__ void __launch_bounds__(ST) k_bp_count1(Bp a, int64_t per, uint32_t* __restrict__ counts) {
  __shared__ uint32_t cnt[DIGITS];
  const int D = 1 << a.b1;
  for (int d = threadIdx.x; d < D; d += ST) cnt[d] = 0;
  __syncthreads();
  const int64_t i1 = min((int64_t)(blockIdx.x + 1) * per, a.narcs);
  uint32_t bad = 0;
  for (int64_t i = (int64_t)blockIdx.x * per + threadIdx.x; i < i1; i += ST) {
    const int32_t x = a.src[i], y = a.dst[i];
    if (x < 0 || y < 0 || x >= a.n || y >= a.n) bad = 1;
    else if (x != y) {
      atomicAdd(&cnt[digit1(a, mix(a, (uint32_t)x))], 1u);
      atomicAdd(&cnt[digit1(a, mix(a, (uint32_t)y))], 1u);
    }
  }
  if (bad) atomicOr(&a.w[W_ERR], ERR_RANGE);
  __syncthreads();
  for (int d = threadIdx.x; d < D; d += ST) counts[(int64_t)d * gridDim.x + blockIdx.x] = cnt[d];
}

// Bound by its scattered writes: 1.6 ms for 268 M arcs, 3.4 TB/s. The longer the
// runs the better: with tiles of 16,384 entries and 256 digits a run is 64 keys
// (256 B; 128 B of second digits); tiles of 8,192 took 1.92 ms, and 512 digits
// 1.96 with the larger tile and 2.30 with the smaller. One workgroup fills the
// CU's LDS.
__global__ void __launch_bounds__(ST) k_bp_split1(Bp a, int64_t per, const uint32_t* __restrict__ offs,
                                                     uint32_t* __restrict__ keys, uint16_t* __restrict__ digs,
                                                     int64_t* __restrict__ end) {
  __shared__ uint64_t buf[2 * S1_ARCS];
  __shared__ uint32_t cnt[DIGITS], start[DIGITS], cur[DIGITS], sh[ST / 64];
  if (a.w[W_ERR]) return;
  if (end) no_rows(a.n, end);
  const int D = 1 << a.b1, t = threadIdx.x;
  for (int d = t; d < DIGITS; d += ST) {
    cnt[d] = 0;
    cur[d] = d < D ? offs[(int64_t)d * gridDim.x + blockIdx.x] : 0u;
  }
  const int64_t i0 = (int64_t)blockIdx.x * per, i1 = min(i0 + per, a.narcs);
  uint32_t x[S1_PER], y[S1_PER];
  auto load = [&](int64_t b) {
#pragma unroll
    for (int k = 0; k < S1_PER; ++k) {
      const int64_t i = b + k * ST + t;
      x[k] = i < i1 ? (uint32_t)a.src[i] : 0u;
      y[k] = i < i1 ? (uint32_t)a.dst[i] : 0u;
    }
  };
  if (i0 < i1) load(i0);
  for (int64_t b = i0; b < i1; b += S1_ARCS) {
    __syncthreads();
    uint32_t rank[S1_PER];
#pragma unroll
    for (int k = 0; k < S1_PER; ++k) {
      rank[k] = 0;
      if (x[k] != y[k]) {
        const uint32_t r0 = atomicAdd(&cnt[digit1(a, mix(a, x[k]))], 1u);
        const uint32_t r1 = atomicAdd(&cnt[digit1(a, mix(a, y[k]))], 1u);
        rank[k] = r0 | r1 << 16;  // below 16,384 (both ends of an arc may share a digit)
      }
    }
    __syncthreads();
    start[t] = block_scan(cnt[t], sh);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < S1_PER; ++k)
      if (x[k] != y[k]) {
        const uint32_t mx = mix(a, x[k]), my = mix(a, y[k]);
        const uint32_t dx = digit1(a, mx), dy = digit1(a, my);
        buf[start[dx] + (rank[k] & 0xFFFFu)] = (uint64_t)(dx << 16 | digit2(a, mx)) << 32 | key_of(a, mx, y[k], 0u);
        buf[start[dy] + (rank[k] >> 16)] = (uint64_t)(dy << 16 | digit2(a, my)) << 32 | key_of(a, my, x[k], 1u);
      }
    if (b + S1_ARCS < i1) load(b + S1_ARCS);
    const uint32_t total = start[DIGITS - 1] + cnt[DIGITS - 1];
    __syncthreads();
    for (uint32_t i = t; i < total; i += ST) {
      const uint64_t v = buf[i];
      const uint32_t d = (uint32_t)(v >> 48);
      const uint32_t at = cur[d] + (i - start[d]);
      keys[at] = (uint32_t)v;
      if (digs) digs[at] = (uint16_t)(v >> 32);
    }
    __syncthreads();
    for (int d = t; d < DIGITS; d += ST) {
      cur[d] += cnt[d];
      cnt[d] = 0;
    }
  }
}

// pbase[d] = first part of bucket d of the first digit, pbase[D] = their number
// (at most gridDim of the kernels that take parts); start1: the buckets' starts.
__global__ void __launch_bounds__(DIGITS) k_bp_parts(Bp a, const uint32_t* __restrict__ offs, int64_t groups,
                                                     const uint32_t* __restrict__ total, uint32_t* __restrict__ pbase,
                                                     uint32_t* __restrict__ start1) {
  __shared__ uint32_t sh[DIGITS / 64];
  const int D = 1 << a.b1, d = threadIdx.x;
  const uint32_t s0 = d < D ? offs[(int64_t)d * groups] : *total;
  const uint32_t s1 = d + 1 < D ? offs[(int64_t)(d + 1) * groups] : *total;
  const uint32_t np = (uint32_t)(((int64_t)s1 - s0 + PART - 1) / PART);
  const uint32_t base = block_scan(np, sh);
  if (d < D) {
    pbase[d] = base;
    start1[d] = s0;
    if (d == D - 1) {
      pbase[D] = base + np;
      start1[D] = s1;
    }
  }
}

struct Part {
  uint32_t base, np, p;  // first part of the bucket, their number, this one
  int64_t i0, i1;
};
// Called by every thread of the block (one looks at one bucket).
__device__ __forceinline__ bool part_of(const Bp& a, const uint32_t* pbase, const uint32_t* start1, Part& r) {
  static_assert(ST >= DIGITS, "a thread for every digit");
  __shared__ uint32_t mine;
  const uint32_t D = 1u << a.b1, t = threadIdx.x;
  if (blockIdx.x >= pbase[D]) return false;
  if (t < D && pbase[t] <= blockIdx.x && blockIdx.x < pbase[t + 1]) mine = t;
  __syncthreads();
  const uint32_t d = mine;
  r.base = pbase[d];
  r.np = pbase[d + 1] - r.base;
  r.p = blockIdx.x - r.base;
  r.i0 = start1[d] + (int64_t)r.p * PART;
  r.i1 = min(r.i0 + PART, (int64_t)start1[d + 1]);
  return true;
}

__global__ void __launch_bounds__(ST) k_bp_count2(Bp a, const uint32_t* __restrict__ pbase,
                                                  const uint32_t* __restrict__ start1,
                                                  const uint16_t* __restrict__ digs, uint32_t* __restrict__ counts) {
  __shared__ uint32_t cnt[DIGITS];
  if (a.w[W_ERR]) return;
  Part r;
  const int D = 1 << a.b2;
  if (!part_of(a, pbase, start1, r)) {
    // the scan runs over every part's counts
    for (int d = threadIdx.x; d < D; d += ST) counts[(int64_t)blockIdx.x * D + d] = 0;
    return;
  }
  for (int d = threadIdx.x; d < D; d += ST) cnt[d] = 0;
  __syncthreads();
  // pairs of digits from the first even place on
  const int64_t e0 = r.i0 + (r.i0 & 1), np = (r.i1 - e0) >> 1;
  const uint32_t* pair = reinterpret_cast<const uint32_t*>(digs + e0);
  for (int64_t i = threadIdx.x; i < np; i += ST) {
    const uint32_t v = pair[i];
    atomicAdd(&cnt[v & 0xFFFFu], 1u);
    atomicAdd(&cnt[v >> 16], 1u);
  }
  if (threadIdx.x == 0) {
    if (e0 > r.i0) atomicAdd(&cnt[digs[r.i0]], 1u);
    if (e0 + 2 * np < r.i1) atomicAdd(&cnt[digs[r.i1 - 1]], 1u);
  }
  __syncthreads();
  for (int d = threadIdx.x; d < D; d += ST) counts[(int64_t)r.base * D + (int64_t)d * r.np + r.p] = cnt[d];
}

// As the first split, with 4 bytes out: 1.5 ms for 537 M keys at 1,024 digits
// (runs of 64 B; tiles of 8,192: 1.8).
__global__ void __launch_bounds__(ST) k_bp_split2(Bp a, const uint32_t* __restrict__ pbase,
                                                     const uint32_t* __restrict__ start1,
                                                     const uint32_t* __restrict__ offs,
                                                     const uint32_t* __restrict__ keys,
                                                     const uint16_t* __restrict__ digs, uint32_t* __restrict__ out,
                                                     int64_t* __restrict__ end) {
  __shared__ uint32_t bk[S2_TILE];
  __shared__ uint16_t bd[S2_TILE];
  __shared__ uint32_t cnt[DIGITS], start[DIGITS], cur[DIGITS], sh[ST / 64];
  Part p;
  no_rows(a.n, end);
  if (!part_of(a, pbase, start1, p)) return;
  const int D = 1 << a.b2, t = threadIdx.x;
  for (int d = t; d < DIGITS; d += ST) {
    cnt[d] = 0;
    cur[d] = d < D ? offs[(int64_t)p.base * D + (int64_t)d * p.np + p.p] : 0u;
  }
  uint32_t k[S2_PER], d[S2_PER];
  auto load = [&](int64_t b) {
#pragma unroll
    for (int j = 0; j < S2_PER; ++j) {
      const int64_t i = b + j * ST + t;
      k[j] = i < p.i1 ? keys[i] : 0u;
      d[j] = i < p.i1 ? (uint32_t)digs[i] : ~0u;
    }
  };
  load(p.i0);
  for (int64_t b = p.i0; b < p.i1; b += S2_TILE) {
    __syncthreads();
    uint32_t rank[S2_PER];
#pragma unroll
    for (int j = 0; j < S2_PER; ++j) rank[j] = d[j] != ~0u ? atomicAdd(&cnt[d[j]], 1u) : 0u;
    __syncthreads();
    start[t] = block_scan(cnt[t], sh);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < S2_PER; ++j)
      if (d[j] != ~0u) {
        const uint32_t at = start[d[j]] + rank[j];
        bk[at] = k[j];
        bd[at] = (uint16_t)d[j];
      }
    if (b + S2_TILE < p.i1) load(b + S2_TILE);
    const uint32_t total = start[DIGITS - 1] + cnt[DIGITS - 1];
    __syncthreads();
    for (uint32_t i = t; i < total; i += ST) {
      const uint32_t q = bd[i];
      out[cur[q] + (i - start[q])] = bk[i];
    }
    __syncthreads();
    for (int q = t; q < DIGITS; q += ST) {
      cur[q] += cnt[q];
      cnt[q] = 0;
    }
  }
}

// Buckets of more than CAP and of more than MID_CAP keys (their numbers), and
// those of more than TOP_CAP: (bucket, start, keys, first part).
struct Lists {
  uint32_t *mid, *top;
  uint4* longs;
  uint32_t mid_cap, top_cap, long_cap, nlong;
};

// Bucket starts from the scanned counts (of k_bp_count2, or of k_bp_count1 when
// there is one digit: pbase NULL).
__global__ void k_bp_sizes(Bp a, const uint32_t* __restrict__ offs, int64_t noffs, int64_t groups,
                           const uint32_t* __restrict__ pbase, const uint32_t* __restrict__ total,
                           uint32_t* __restrict__ bstart, Lists l) {
  if (a.w[W_ERR]) return;
  const int64_t nb = 1ll << (a.b1 + a.b2);
  auto at = [&](int64_t q) -> uint32_t {
    if (q >= nb) return *total;
    int64_t i;
    if (pbase) {
      const uint32_t d = (uint32_t)(q >> a.b2), e = (uint32_t)q & ((1u << a.b2) - 1u), p0 = pbase[d];
      // a bucket of the first digit without entries starts where the next one does
      const uint32_t np = pbase[d + 1] - p0;
      i = ((int64_t)p0 << a.b2) + (int64_t)e * np;
    } else {
      i = q * groups;
    }
    return i < noffs ? offs[i] : *total;
  };
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  uint32_t len = 0;
  if (q < nb) {
    const uint32_t s0 = at(q);
    len = at(q + 1) - s0;
    bstart[q] = s0;
    if (q == nb - 1) bstart[nb] = *total;
    if (len > TOP_CAP) {
      const uint64_t np = ((uint64_t)len + L_PART - 1) / L_PART;
      const uint64_t at = atomicAdd(reinterpret_cast<unsigned long long*>(&a.w[W_LPARTS]), 1ull << 32 | np);
      // always: each holds more than TOP_CAP of the entries
      if ((uint32_t)(at >> 32) < l.long_cap) l.longs[at >> 32] = make_uint4((uint32_t)q, s0, len, (uint32_t)at);
    } else if (len > MID_CAP) {
      const uint32_t k = atomicAdd(&a.w[W_NTOP], 1u);
      if (k < l.top_cap) l.top[k] = (uint32_t)q;  // always, likewise
    }
  }
  const bool mid = len > CAP && len <= MID_CAP;
  const uint64_t mm = __ballot(mid);
  if (mm) {
    uint32_t k = 0;
    if ((threadIdx.x & 63) == 0) k = atomicAdd(&a.w[W_NMID], (uint32_t)__popcll(mm));
    k = __shfl(k, 0, 64) + (uint32_t)__popcll(mm & ((1ull << (threadIdx.x & 63)) - 1));
    if (mid && k < l.mid_cap) l.mid[k] = (uint32_t)q;  // always, likewise
  }
}

// ------------------------------------------------------------ bucket sort
struct Rows {
  uint32_t* ent;   // merged entries, column << 2 | flags, at their bucket's start
  uint32_t* pos;   // first entry of a row in ent
  int64_t* end;    // the place after its last one (0 for a row without entries)
};

// Has the run of equal (row, column) that k belongs to, which is sorted by
// direction and goes on at lo, a key of direction 1? Its last key is found by
// doubling steps.
__device__ __forceinline__ uint32_t run_back(const uint32_t* s, uint32_t lo, uint32_t len, uint32_t k) {
  uint32_t step = 1;  // s[lo] is in the run
  while (lo + step < len && (s[lo + step] ^ k) <= 1u) {
    lo += step;
    step <<= 1;
  }
  for (; step; step >>= 1)
    if (lo + step < len && (s[lo + step] ^ k) <= 1u) lo += step;
  return s[lo] & 1u;
}

// Is the key at i < len the first of its (row, column)?
__device__ __forceinline__ bool run_head(const uint32_t* s, uint32_t i) { return i == 0 || (s[i] ^ s[i - 1]) > 1u; }

// Runs of sorted keys -> entries: keys [i0, i1) of a bucket of len keys, at most
// R rounds of T, with `run` entries before them.
template <int T, int R>
__device__ __forceinline__ void emit_runs(const Bp& a, const Rows& o, const uint32_t* s, uint32_t i0, uint32_t i1,
                                          uint32_t len, uint32_t bucket, uint32_t b0, uint32_t run, uint32_t* sh) {
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int nr = (int)((i1 - i0 + T - 1) / T);
  const uint32_t first = i0 + (uint32_t)(w * nr * 64 + lane), cm = (1u << a.rb) - 1u;
  uint64_t hm[R];
  uint32_t c = 0;
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (r < nr) {
      const uint32_t i = first + r * 64;
      hm[r] = __ballot(i < i1 && run_head(s, i));
      c += (uint32_t)__popcll(hm[r]);
    }
  if (lane == 0) sh[w] = c;
  __syncthreads();
  for (int q = 0; q < w; ++q) run += sh[q];
  run += b0;
  const uint64_t above = lane == 63 ? 0ull : ~0ull << (lane + 1);
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (r < nr) {
      const uint32_t i = first + r * 64;
      const uint32_t k = i < i1 ? s[i] : 0u;
      const uint32_t pv = i && i < i1 ? s[i - 1] : ~k, nx = i + 1 < len ? s[i + 1] : ~k;
      const uint64_t back = __ballot(i < i1 && (k & 1u));
      const uint32_t j = i - lane + 64, kj = (uint32_t)__builtin_amdgcn_readlane((int)nx, 63);  // after these 64
      if (i < i1) {
        const uint32_t e = __builtin_amdgcn_mbcnt_hi((uint32_t)(hm[r] >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)hm[r], run));
        const bool head = (k ^ pv) > 1u;
        if (head) {
          // directions in the run: this key's, and direction 1 if a later key has it
          const uint64_t rest = hm[r] & above;
          uint32_t f = 1u + (k & 1u);
          if (f == 1u) {
            if (back & above & (rest - 1) & ~rest) f = 3u;
            else if (rest == 0 && j < len && (kj ^ k) <= 1u) f |= run_back(s, j, len, k) << 1;
          }
          o.ent[e] = (k >> 1 & cm) << 2 | f;
        }
        // the first and last key of a row
        const bool rf = ((k ^ pv) >> 1) > cm || i == 0, rl = ((k ^ nx) >> 1) > cm || i + 1 == len;
        if (rf || rl) {
          const uint32_t q = a.low ? k >> (a.rb + 1) : 0u;
          const uint32_t x = ((bucket << a.low | q) * a.inv) & a.mask;
          if (rf) o.pos[x] = e;
          if (rl) o.end[x] = e + (head ? 1u : 0u);
        }
      }
      run += (uint32_t)__popcll(hm[r]);
    }
}

// Bound by vector instructions: 2.7 ms for 345 M keys in 244,000 buckets (R-MAT
// scale 24), about 250 a wavefront and 64 keys, half of them the three passes'
// matching. The scans of the digit counts run by DPP and places are kept as 16
// bits, two a register (3.3 ms with shuffles and spills).
__global__ void __launch_bounds__(256, 6) k_bp_sort(Bp a, const uint32_t* __restrict__ bstart,
                                                    const uint32_t* __restrict__ keys, Rows o) {
  __shared__ uint32_t s[CAP];
  __shared__ alignas(16) uint32_t cnt[4][256];
  __shared__ uint32_t sh[4];
  const uint32_t b0 = bstart[blockIdx.x], len = bstart[blockIdx.x + 1] - b0;
  if (len == 0 || len > CAP) return;
  lds_sort<256, CAP / 256>(s, cnt, sh, keys + b0, len, a.low + a.rb + 1);
  emit_runs<256, CAP / 256>(a, o, s, 0, len, len, blockIdx.x, b0, 0, sh);
}

// Listed buckets of up to T * R keys, those of the list `top` first. With 512
// threads two workgroups fit on a CU; with 1,024 one bucket ends sooner, which
// counts where there are fewer buckets than CUs (45 against 58 us): then one
// launch takes both lists.
template <int T, int R>
__global__ void __launch_bounds__(T, 4) k_bp_mid(Bp a, const uint32_t* __restrict__ bstart,
                                                 const uint32_t* __restrict__ top, uint32_t ntop,
                                                 const uint32_t* __restrict__ mid, const uint32_t* __restrict__ keys,
                                                 Rows o) {
  __shared__ uint32_t s[T * R];
  __shared__ alignas(16) uint32_t cnt[T / 64][256];
  __shared__ uint32_t sh[T / 64];
  const uint32_t q = blockIdx.x < ntop ? top[blockIdx.x] : mid[blockIdx.x - ntop], b0 = bstart[q], len = bstart[q + 1] - b0;
  if (len > T * R) return;
  lds_sort<T, R>(s, cnt, sh, keys + b0, len, a.low + a.rb + 1);
  emit_runs<T, R>(a, o, s, 0, len, len, q, b0, 0, sh);
}

// The longest buckets (few, but one may hold all entries) are sorted by all
// workgroups together, least significant digit first through memory:
// counts of a part, a scan over (bucket, digit, part), a stable scatter. (In the
// last part of a bucket, the places past its end take the highest digit: they come
// after every key and are not written.)
struct LPart {
  uint32_t bucket, start, len, first;  // its keys, its first part
  uint32_t np, p;                      // its parts, this one
  uint64_t base;                       // its counts start here
  int64_t i0, i1;
};
__device__ __forceinline__ LPart long_part(const Lists& l) {
  uint32_t lo = 0, hi = l.nlong;  // the last one whose first part is not past this block
  while (hi - lo > 1) {
    const uint32_t m = (lo + hi) >> 1;
    if (l.longs[m].w <= blockIdx.x) lo = m; else hi = m;
  }
  const uint4 b = l.longs[lo];
  LPart r;
  r.bucket = b.x;
  r.start = b.y;
  r.len = b.z;
  r.first = b.w;
  r.np = (uint32_t)(((uint64_t)b.z + L_PART - 1) / L_PART);
  r.p = blockIdx.x - b.w;
  r.base = (uint64_t)b.w * 256;
  r.i0 = (int64_t)b.y + (int64_t)r.p * L_PART;
  r.i1 = min(r.i0 + L_PART, (int64_t)b.y + b.z);
  return r;
}

__global__ void __launch_bounds__(LT) k_bp_long_count(Lists l, const uint32_t* __restrict__ keys, int lo, int wd,
                                                      uint32_t* __restrict__ counts) {
  __shared__ uint32_t cnt[256];
  const LPart p = long_part(l);
  const int t = threadIdx.x;
  if (t < 256) cnt[t] = 0;
  __syncthreads();
  uint32_t key[L_PER];
#pragma unroll
  for (int r = 0; r < L_PER; ++r) key[r] = p.i0 + r * LT + t < p.i1 ? keys[p.i0 + r * LT + t] : 0u;
#pragma unroll
  for (int r = 0; r < L_PER; ++r)
    if (p.i0 + r * LT + t < p.i1) atomicAdd(&cnt[__builtin_amdgcn_ubfe(key[r], lo, wd)], 1u);
  __syncthreads();
  if (t < 256) counts[p.base + (uint64_t)t * p.np + p.p] = cnt[t];
}

__global__ void __launch_bounds__(LT, 4) k_bp_long_scatter(Lists l, const uint32_t* __restrict__ in,
                                                           uint32_t* __restrict__ out, int lo, int wd,
                                                           const uint32_t* __restrict__ offs) {
  constexpr int W = LT / 64;
  __shared__ uint32_t cnt[W][256], sh[W], cur[256];
  const LPart p = long_part(l);
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const uint64_t below = (1ull << lane) - 1, above = ~below << 1;
  if (t < 256) cur[t] = p.start + (offs[p.base + (uint64_t)t * p.np + p.p] - offs[p.base]);
  for (int k = t; k < W * 256; k += LT) (&cnt[0][0])[k] = 0;
  uint32_t key[L_PER], pos[L_PER];
  const int64_t i0 = p.i0 + w * (L_PER * 64) + lane;
#pragma unroll
  for (int r = 0; r < L_PER; ++r) key[r] = i0 + r * 64 < p.i1 ? in[i0 + r * 64] : ~0u;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < L_PER; ++r) pos[r] = match_rank(__builtin_amdgcn_ubfe(key[r], lo, wd), cnt[w], below, above);
  __syncthreads();
  digit_starts<W>(cnt, sh, cur);
#pragma unroll
  for (int r = 0; r < L_PER; ++r)
    if (i0 + r * 64 < p.i1) out[cnt[w][__builtin_amdgcn_ubfe(key[r], lo, wd)] + pos[r]] = key[r];
}

// The runs of a part's keys: their number, then (scanned) their entries.
__global__ void __launch_bounds__(LT) k_bp_long_heads(Lists l, const uint32_t* __restrict__ keys,
                                                      uint32_t* __restrict__ heads) {
  __shared__ uint32_t sh[LT / 64];
  const LPart p = long_part(l);
  const uint32_t* s = keys + p.start;
  const uint32_t i0 = (uint32_t)(p.i0 - p.start) + threadIdx.x, i1 = (uint32_t)(p.i1 - p.start);
  uint32_t c = 0;
#pragma unroll
  for (int r = 0; r < L_PER; ++r)
    c += (uint32_t)__popcll(__ballot(i0 + r * LT < i1 && run_head(s, i0 + r * LT)));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int q = 1; q < LT / 64; ++q) c += sh[q];
    heads[blockIdx.x] = c;
  }
}

__global__ void __launch_bounds__(LT, 4) k_bp_long_emit(Bp a, Lists l, const uint32_t* __restrict__ keys,
                                                        const uint32_t* __restrict__ heads, Rows o) {
  __shared__ uint32_t sh[LT / 64];
  const LPart p = long_part(l);
  emit_runs<LT, L_PER>(a, o, keys + p.start, (uint32_t)(p.i0 - p.start), (uint32_t)(p.i1 - p.start), p.len, p.bucket,
                       p.start, heads[blockIdx.x] - heads[p.first], sh);
}

// Ends of rows (in off) -> offsets, and the first row of every tile of k_bp_out
// (after them the last row that is not empty): block sums, their scan, the rows.
__device__ __forceinline__ int64_t degree(const int64_t* off, const uint32_t* pos, int64_t x, int64_t n) {
  if (x >= n) return 0;
  const int64_t e = off[x];
  return e ? e - pos[x] : 0;
}
__device__ __forceinline__ int64_t wave_sum(int64_t x) {
#pragma unroll
  for (int o = 32; o; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

__global__ void __launch_bounds__(RT) k_bp_row_sums(int64_t n, const int64_t* __restrict__ off,
                                                    const uint32_t* __restrict__ pos, int64_t* __restrict__ sums) {
  __shared__ int64_t sh[RT / 64];
  const int64_t x = (int64_t)blockIdx.x * (RT * RI) + threadIdx.x;
  int64_t c = 0;
#pragma unroll
  for (int k = 0; k < RI; ++k) c += degree(off, pos, x + k * RT, n);
  c = wave_sum(c);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int q = 1; q < RT / 64; ++q) c += sh[q];
    sums[blockIdx.x] = c;
  }
}

// sums[0, m) -> their exclusive scan, sums[m] = the total
__global__ void __launch_bounds__(1024) k_bp_row_top(int64_t* __restrict__ sums, int64_t m) {
  __shared__ int64_t sh[16];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  int64_t carry = 0;
  for (int64_t c = 0; c < m; c += 4096) {
    const int64_t b = c + 4 * t;
    int64_t v[4], x = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[k] = b + k < m ? sums[b + k] : 0;
      x += v[k];
    }
    const int64_t own = x;
    for (int o = 1; o < 64; o <<= 1) {
      const int64_t y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    __syncthreads();
    if (lane == 63) sh[w] = x;
    __syncthreads();
    int64_t run = carry + x - own;
    for (int q = 0; q < 16; ++q) {
      if (q < w) run += sh[q];
      carry += sh[q];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (b + k < m) {
        sums[b + k] = run;
        run += v[k];
      }
  }
  if (t == 0) sums[m] = carry;
}

__global__ void __launch_bounds__(RT) k_bp_rows(int64_t n, int64_t* __restrict__ off, const uint32_t* __restrict__ pos,
                                                const int64_t* __restrict__ sums, uint32_t* __restrict__ trow) {
  __shared__ int64_t sh[RT / 64];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int64_t x0 = (int64_t)blockIdx.x * (RT * RI) + t * RI, nnz = sums[gridDim.x];
  int64_t d[RI], x = 0;
#pragma unroll
  for (int k = 0; k < RI; ++k) {
    d[k] = degree(off, pos, x0 + k, n);
    x += d[k];
  }
  const int64_t own = x;
  for (int o = 1; o < 64; o <<= 1) {
    const int64_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) sh[w] = x;
  __syncthreads();
  int64_t b = sums[blockIdx.x] + x - own;
  for (int q = 0; q < w; ++q) b += sh[q];
#pragma unroll
  for (int k = 0; k < RI; ++k)
    if (x0 + k < n) {
      const int64_t e = b + d[k];
      off[x0 + k] = b;
      for (int64_t q = (b + OT - 1) / OT; q * OT < e; ++q) trow[q] = (uint32_t)(x0 + k);
      if (b < e && e == nnz) trow[(nnz + OT - 1) / OT] = (uint32_t)(x0 + k);
      if (x0 + k == n - 1) off[n] = e;
      b = e;
    }
}

// Entries in row order, four a thread and round. The tile's rows mark their
// starts in a bitmap in LDS, with their places in ent beside it; an entry's row
// is the last mark at or before it: 1.07 ms for R-MAT scale 24, bound by memory
// (rows lie scattered in ent: lines are read in part). A binary search over
// staged row starts took 1.65 ms, and a tile of many empty rows searched in
// memory; handing the places to consecutive lanes through LDS, so that the reads
// coalesce, 1.85.
__global__ void __launch_bounds__(256) k_bp_out(int64_t n, const int64_t* __restrict__ off,
                                                const uint32_t* __restrict__ trow, const uint32_t* __restrict__ pos,
                                                const uint32_t* __restrict__ ent, int32_t* __restrict__ nbr,
                                                uint8_t* __restrict__ flg) {
  constexpr int R = OT / (4 * 256), WORDS = OT / 32;
  static_assert(WORDS == 128, "two words a lane of one wavefront");
  __shared__ uint32_t from[OT];      // at a row's start: place in ent less the place in the tile
  __shared__ uint32_t mark[WORDS];
  __shared__ uint16_t last[WORDS];   // last mark in this word or before
  const int64_t nnz = off[n], t0 = (int64_t)blockIdx.x * OT, t1 = min(t0 + (int64_t)OT, nnz);
  if (t0 >= nnz) return;
  const int t = threadIdx.x;
  const int64_t r0 = trow[blockIdx.x], r1 = trow[blockIdx.x + 1];  // r1 may start at t1
  if (t < WORDS) mark[t] = 0;
  __syncthreads();
  for (int64_t x = r0 + t; x <= r1; x += 256) {
    const int64_t b = off[x], e = off[x + 1];
    if (b < e && b < t1) {
      const uint32_t at = (uint32_t)max(b - t0, (int64_t)0);
      from[at] = pos[x] - (uint32_t)(b - t0);
      atomicOr(&mark[at >> 5], 1u << (at & 31));
    }
  }
  __syncthreads();
  if (t < 64) {
    const uint32_t a = mark[2 * t], b = mark[2 * t + 1];
    const int la = a ? 64 * t + 31 - __clz((int)a) : 0, lb = b ? 64 * t + 63 - __clz((int)b) : la;
    int x = lb;  // marks grow with the lane: a running maximum
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(x, o, 64);
      if (t >= o) x = max(x, y);
    }
    int before = __shfl_up(x, 1, 64);
    if (t == 0) before = 0;
    last[2 * t] = (uint16_t)max(before, la);
    last[2 * t + 1] = (uint16_t)x;
  }
  __syncthreads();
  const int m = (int)(t1 - t0);
  uint32_t v[R][4];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int j = 4 * (r * 256 + t);
#pragma unroll
    for (int k = 0; k < 4; ++k) v[r][k] = 0;
    if (j >= m) continue;
    const uint32_t wd = mark[j >> 5], b4 = wd >> (j & 31), upto = wd & (2u << (j & 31)) - 1u;
    uint32_t at = upto ? (uint32_t)((j & ~31) + 31 - __clz((int)upto)) : last[(j >> 5) - 1];
    uint32_t f = from[at];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (k && (b4 >> k & 1u)) f = from[j + k];
      if (j + k < m) v[r][k] = ent[f + j + k];
    }
  }
  const bool wide = ((uintptr_t)nbr & 15) == 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int j = 4 * (r * 256 + t);
    if (j >= m) continue;
    if (wide && j + 4 <= m) {
      *reinterpret_cast<int4*>(nbr + t0 + j) =
          make_int4((int)(v[r][0] >> 2), (int)(v[r][1] >> 2), (int)(v[r][2] >> 2), (int)(v[r][3] >> 2));
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (j + k < m) nbr[t0 + j + k] = (int32_t)(v[r][k] >> 2);
    }
    flg[(t0 + j) >> 2] = (uint8_t)((v[r][0] & 3u) | (v[r][1] & 3u) << 2 | (v[r][2] & 3u) << 4 | (v[r][3] & 3u) << 6);
  }
}

__global__ void k_bp_zero(uint32_t* w) {
  if (threadIdx.x < W_WORDS) w[threadIdx.x] = 0;
}

}  // namespace

// Bits of the bucket for N entries of ids below 2^rb, or -1 where the general
// sort is taken: where the key does not fit into 32 bits even in buckets of a
// quarter of the usual size (at 2^24 ids from 67 M entries on it does, at 2^20
// always), and with more ids than entries, where passes over the ids would cost
// more than the sort. Below that the parts are never slower: 94 against 200 us
// for 3,500 arcs, 464 against 473 for 4 M on 200,003 vertices (the longest
// bucket's passes), 0.9 against 2.3 ms for 16.8 M at random, 1.6 against 2.2 ms
// for a star of 16.8 M.
static int bucket_bits(int64_t n, int64_t N, int rb) {
  if (n > N) return -1;
  int b = 0;
  while ((N - 1) >> AVG_BITS >> b > 0) ++b;  // N <= 2^(b + AVG_BITS)
  b = std::min(b, rb);
  const int need = 2 * rb + 1 - 32;
  if (need > b + 2) return -1;
  b = std::max(b, need);
  return b > 20 ? -1 : b;
}

int csr_by_parts(int64_t n, int64_t narcs, int rb, const int32_t* src, const int32_t* dst, hipStream_t s, int64_t* off,
                 int32_t* nbr, uint8_t* flg, int64_t* nnz_out, bool* done) {
  *done = false;
  const int64_t N = 2 * narcs;
  const int bits = bucket_bits(n, N, rb);
  if (bits < 0) return TRIAD_OK;
  Scratch scratch(s, 0, true);
  Bp a{};
  a.n = n;
  a.narcs = narcs;
  a.src = src;
  a.dst = dst;
  a.rb = rb;
  a.b1 = bits <= 10 ? bits : std::max(bits - 10, bits / 2 - 1);  // the first split writes two arrays: longer runs
  a.b2 = bits - a.b1;
  a.low = rb - bits;
  // the golden ratio's fraction in rb bits, odd, and its inverse modulo 2^32
  a.mul = (uint32_t)(0x9E3779B97F4A7C15ull >> (64 - rb)) | 1u;
  a.inv = 1;
  for (int k = 0; k < 5; ++k) a.inv *= 2u - a.mul * a.inv;
  a.mask = (uint32_t)((1ull << rb) - 1);
  const int64_t nb = 1ll << bits, D1 = 1ll << a.b1, D2 = 1ll << a.b2;
  const int64_t tiles = (narcs + S1_ARCS - 1) / S1_ARCS;
  const int64_t per = (tiles + S1_GROUPS - 1) / S1_GROUPS * S1_ARCS, groups = (narcs + per - 1) / per;
  const int64_t parts = a.b2 ? N / PART + D1 : 0;
  const int64_t row_blocks = (n + RT * RI - 1) / (RT * RI);
  Lists l{};
  l.mid_cap = (uint32_t)(N / CAP + 1);
  l.top_cap = (uint32_t)(N / MID_CAP + 1);
  l.long_cap = (uint32_t)(N / TOP_CAP + 1);
  uint32_t *ka = nullptr, *kb = nullptr, *pos = nullptr, *bstart = nullptr, *trow = nullptr, *c1 = nullptr,
           *o1 = nullptr, *c2 = nullptr, *o2 = nullptr, *pbase = nullptr, *start1 = nullptr, *tot = nullptr;
  uint16_t* digs = nullptr;
  int64_t* sums = nullptr;
  ALLOC(a.w, W_WORDS);
  ALLOC(tot, 2);
  ALLOC(ka, N);
  ALLOC(kb, N);
  ALLOC(pos, n);
  ALLOC(sums, row_blocks + 1);
  ALLOC(bstart, nb + 1);
  ALLOC(trow, N / OT + 2);
  ALLOC(l.mid, l.mid_cap);
  ALLOC(l.top, l.top_cap);
  ALLOC(l.longs, l.long_cap);
  ALLOC(c1, D1 * groups);
  ALLOC(o1, D1 * groups);
  if (a.b2) {
    ALLOC(digs, N);
    ALLOC(c2, D2 * parts);
    ALLOC(o2, D2 * parts);
    ALLOC(pbase, D1 + 1);
    ALLOC(start1, D1 + 1);
  }
  k_bp_zero<<<1, 64, 0, s>>>(a.w);
  k_bp_count1<<<(unsigned)groups, ST, 0, s>>>(a, per, c1);
  if (int st = scan_u32(c1, D1 * groups, o1, tot, scratch, s)) return st;
  const uint32_t* in = ka;
  if (a.b2) {
    k_bp_parts<<<1, DIGITS, 0, s>>>(a, o1, groups, tot, pbase, start1);
    k_bp_split1<<<(unsigned)groups, ST, 0, s>>>(a, per, o1, ka, digs, nullptr);
    k_bp_count2<<<(unsigned)parts, ST, 0, s>>>(a, pbase, start1, digs, c2);
    if (int st = scan_u32(c2, D2 * parts, o2, nullptr, scratch, s)) return st;
    k_bp_sizes<<<grid_of(nb, 256, 1 << 20), 256, 0, s>>>(a, o2, D2 * parts, 0, pbase, tot, bstart, l);
  } else {
    k_bp_sizes<<<grid_of(nb, 256, 1 << 20), 256, 0, s>>>(a, o1, D1 * groups, groups, nullptr, tot, bstart, l);
  }
  HIPCHK(hipGetLastError());
  uint32_t h[W_WORDS];
  HIPCHK(hipMemcpyAsync(h, a.w, sizeof h, hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  if (h[W_ERR]) return fail(TRIAD_ERANGE, "arc endpoint outside [0, n)");
  l.nlong = h[W_NLONG];
  // everything that may fail for want of memory comes before the first output
  uint32_t *lc = nullptr, *loffs = nullptr, *heads = nullptr;
  const int64_t lcounts = (int64_t)h[W_LPARTS] * 256;
  if (l.nlong) {
    ALLOC(lc, lcounts);
    ALLOC(loffs, lcounts);
    ALLOC(heads, h[W_LPARTS]);
  }
  uint32_t* lsums = nullptr;
  ALLOC(lsums, scan_u32_sums(lcounts));
  if (a.b2) {
    k_bp_split2<<<(unsigned)parts, ST, 0, s>>>(a, pbase, start1, o2, ka, digs, kb, off);
    in = kb;
  } else {
    k_bp_split1<<<(unsigned)groups, ST, 0, s>>>(a, per, o1, ka, nullptr, off);
  }
  const Rows o{in == ka ? kb : ka, pos, off};
  const int kbits = a.low + a.rb + 1;
  if (l.nlong) {
    uint32_t *from = in == ka ? ka : kb, *to = o.ent;
    const int P = ((kbits + 7) / 8 + 1) & ~1;  // even: the sorted keys are where they were
    for (int p = 0, lo = 0; p < P; ++p) {
      const int hi = kbits * (p + 1) / P, wd = hi - lo;
      k_bp_long_count<<<h[W_LPARTS], LT, 0, s>>>(l, from, lo, wd, lc);
      if (int st = scan_u32_with(lc, lcounts, loffs, nullptr, lsums, s)) return st;
      k_bp_long_scatter<<<h[W_LPARTS], LT, 0, s>>>(l, from, to, lo, wd, loffs);
      std::swap(from, to);
      lo = hi;
    }
    k_bp_long_heads<<<h[W_LPARTS], LT, 0, s>>>(l, in, lc);
    if (int st = scan_u32_with(lc, h[W_LPARTS], heads, nullptr, lsums, s)) return st;
  }
  if (l.nlong) k_bp_long_emit<<<h[W_LPARTS], LT, 0, s>>>(a, l, in, heads, o);
  const uint32_t ntop = h[W_NTOP], nmid = h[W_NMID];
  const bool few = ntop + nmid <= 256;
  if (const uint32_t g = few ? ntop + nmid : ntop)
    k_bp_mid<1024, TOP_CAP / 1024><<<g, 1024, 0, s>>>(a, bstart, l.top, ntop, l.mid, in, o);
  if (!few && nmid) k_bp_mid<512, MID_CAP / 512><<<nmid, 512, 0, s>>>(a, bstart, nullptr, 0, l.mid, in, o);
  k_bp_sort<<<(unsigned)nb, 256, 0, s>>>(a, bstart, in, o);
  HIPCHK(hipGetLastError());
  k_bp_row_sums<<<(unsigned)row_blocks, RT, 0, s>>>(n, off, pos, sums);
  k_bp_row_top<<<1, 1024, 0, s>>>(sums, row_blocks);
  k_bp_rows<<<(unsigned)row_blocks, RT, 0, s>>>(n, off, pos, sums, trow);
  k_bp_out<<<grid_of(N, OT, INT32_MAX), 256, 0, s>>>(n, off, trow, pos, o.ent, nbr, flg);
  HIPCHK(hipGetLastError());
  int64_t nnz = 0;
  HIPCHK(hipMemcpyAsync(&nnz, off + n, sizeof nnz, hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  *nnz_out = nnz;
  *done = true;
  return TRIAD_OK;
}

}  // namespace triad
