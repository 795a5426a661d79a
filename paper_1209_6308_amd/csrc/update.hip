// Incremental census of a graph that changes by arc insertions and deletions:
// the census of the graph after a batch of updates, from the census before it
// and the changed pairs only (the census at fixed time intervals of Sec. 3,
// Figs. 3-4, without a full sweep per interval).
//
// A batch is a sequence of arc operations applied in order (insert x->y, or
// delete it). Only its net effect on each unordered pair {a, b} matters: the
// pair's flag goes from f0 to f1, each bit being set by the last operation on
// its arc (or kept). The census is a sum of row terms and triangles (see
// sweep.hip), so its change is
//   - for every row with a changed entry, the row's sums after less before, from
//     its counts of out-, in- and mutual neighbours (a pass over its 2-bit flags),
//   - for every changed pair {a, b}, a < b, the triangles {a, b, w} after less
//     before, each counted by the smallest of its changed pairs (pair order a <<
//     RB | b). The w adjacent to both a and b before come from the shorter of the
//     two rows searched in the longer; the others are among the changes of a or
//     b. (Merging both rows of every changed pair took 6.5 of 8.2 ms per 100,000
//     updates on 90 M entries, R-MAT; row sums, pairs and parts now 1.3 ms. Bound
//     by the latency of the searches' dependent reads.)
// The classes come from the 64-state table of the census (Fig. 5 step
// 2.1.4.1). The null count stays C(n,3) minus the rest.
//
//   k_upd_small     up to UPD_SMALL operations: the next four in one workgroup
//   k_upd_keys      two keys per operation (one a row): row, column, direction, kind
//   radix sort      by (row, column, direction), stable: operations keep their order
//   k_upd_state     f0 from the CSR, f1 from the last operation on each arc
//   k_upd_emit      the changed entries E in order, their places in the old rows
//   k_upd_rows      changed rows: their sums
//   k_upd_pairs     changed pairs: their triangles
//   k_new_offsets, k_upd_copy   the CSR after the batch
// Nothing waits for the host until the end: counts stay on the device and grids
// are sized for their bounds.
#include <hip/hip_runtime.h>

#include <cstring>
#include <string>

#include "device_sort.h"
#include "sums.h"
#include "triad_internal.h"

namespace triad {
namespace {

constexpr int UT = 256;
constexpr int UPD_SMALL = 2048;      // operations that one workgroup sorts in LDS
constexpr int SMALL_T = 1024;
constexpr int64_t UPD_PART = 1024;   // entries of the shorter row that one wavefront searches
constexpr int64_t UPD_PARTS = 64;    // parts of one pair at most
constexpr int64_t UPD_QUEUE = 1 << 18;  // parts put off at most

__device__ __forceinline__ uint32_t entry_flag(const uint8_t* flg, int64_t j) {
  return (flg[j >> 2] >> (2 * (j & 3))) & 3u;
}

// first position in nbr[b, e) with an id >= y
__device__ __forceinline__ int64_t lower_id(const int32_t* nbr, int64_t b, int64_t e, int32_t y) {
  while (b < e) {
    const int64_t m = (b + e) >> 1;
    if (nbr[m] < y) b = m + 1; else e = m;
  }
  return b;
}

// first position in keys[b, e) whose key is >= k
__device__ __forceinline__ int64_t lower_key(const uint64_t* keys, int64_t b, int64_t e, uint64_t k) {
  while (b < e) {
    const int64_t m = (b + e) >> 1;
    if (keys[m] < k) b = m + 1; else e = m;
  }
  return b;
}

struct UpdGraph {
  int64_t n, nnz;
  const int64_t* off;
  const int32_t* nbr;
  const uint8_t* flg;
  int rb;  // ids below 2^rb
};

// Words the kernels share (zeroed first).
// U_PARTS is one of 64 bits: every long pair draws a ticket, full queue or not.
enum { U_ERR = 0, U_NE = 1, U_PARTS = 2, U_WORDS = 4 };
__device__ __forceinline__ unsigned long long* parts_of(uint32_t* u) {
  return reinterpret_cast<unsigned long long*>(u + U_PARTS);
}

// Operation i as two keys (row << rb | column) << 2 | direction << 1 | insert,
// direction 0 for the arc row -> column.
__device__ __forceinline__ uint32_t op_keys(const UpdGraph& g, int32_t s, int32_t d, uint32_t op, uint64_t* k0,
                                            uint64_t* k1) {
  *k0 = *k1 = ~0ull;
  if (s < 0 || d < 0 || s >= g.n || d >= g.n || op > 1u) return ERR_RANGE;
  *k0 = ((((uint64_t)s << g.rb) | (uint64_t)d) << 2) | op;
  *k1 = ((((uint64_t)d << g.rb) | (uint64_t)s) << 2) | 2u | op;
  return s == d ? (uint32_t)ERR_SELFLOOP : 0u;
}

__global__ void k_upd_keys(UpdGraph g, int64_t k, const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                           const uint8_t* __restrict__ ins, uint64_t* __restrict__ keys, uint32_t* __restrict__ u) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  uint32_t bits = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < k; i += stride)
    bits |= op_keys(g, src[i], dst[i], ins[i], &keys[2 * i], &keys[2 * i + 1]);
  if (bits) atomicOr(&u[U_ERR], bits);
}

// The entry of key's (row, column): where it stands (or would stand) in the old
// row, and f0 << 2 | f1, f1 = f0 with each arc's bit set by the last operation
// on it (the run's operations are sorted by direction, in order within it).
// key(q) is the sorted key at q < N.
template <class Key>
__device__ __forceinline__ uint32_t entry_state(const UpdGraph& g, int64_t i, int64_t N, Key key, int64_t* pos) {
  const uint64_t pr = key(i) >> 2;
  const int64_t x = (int64_t)(pr >> g.rb);
  const int32_t y = (int32_t)(pr & ((1ull << g.rb) - 1));
  const int64_t e = g.off[x + 1], j = lower_id(g.nbr, g.off[x], e, y);
  const uint32_t f0 = j < e && g.nbr[j] == y ? entry_flag(g.flg, j) : 0u;
  uint32_t f1 = f0;
  for (int64_t q = i; q < N && (key(q) >> 2) == pr; ++q) {
    const uint64_t kq = key(q);
    const uint32_t bit = 1u << ((kq >> 1) & 1u);
    f1 = (kq & 1u) ? (f1 | bit) : (f1 & ~bit);
  }
  *pos = j;
  return f0 << 2 | f1;
}

__global__ void k_upd_state(UpdGraph g, const uint64_t* __restrict__ keys, int64_t N, uint32_t* __restrict__ chg,
                            uint8_t* __restrict__ st, uint32_t* __restrict__ pos, const uint32_t* __restrict__ u) {
  if (u[U_ERR]) return;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += stride) {
    chg[i] = 0;
    if (i > 0 && (keys[i] >> 2) == (keys[i - 1] >> 2)) continue;
    int64_t p;
    const uint32_t f = entry_state(g, i, N, [&](int64_t q) { return keys[q]; }, &p);
    st[i] = (uint8_t)f;
    pos[i] = (uint32_t)p;
    chg[i] = (f >> 2) != (f & 3u) ? 1u : 0u;
  }
}

// Changed entries: E = (row << rb | column) << 4 | f0 << 2 | f1 in order, P their
// places, net = +1 for an inserted entry, -1 for a deleted one.
__device__ __forceinline__ int64_t net_of(uint32_t f) { return (f >> 2) == 0 ? 1 : (f & 3u) == 0 ? -1 : 0; }

__global__ void k_upd_emit(const uint64_t* __restrict__ keys, int64_t N, const uint32_t* __restrict__ chg,
                           const uint32_t* __restrict__ cpos, const uint8_t* __restrict__ st,
                           const uint32_t* __restrict__ pos, uint64_t* __restrict__ E, uint32_t* __restrict__ P,
                           int64_t* __restrict__ net, const uint32_t* __restrict__ u) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const bool bad = u[U_ERR] != 0;
  const int64_t nE = bad ? 0 : u[U_NE];
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += stride) {
    if (!bad && chg[i]) {
      const uint32_t c = cpos[i], f = st[i];
      E[c] = (keys[i] >> 2) << 4 | f;
      P[c] = pos[i];
      net[c] = net_of(f);
    }
    if (i >= nE) net[i] = 0;  // the scan runs over all N
  }
}

// All of the above for at most UPD_SMALL operations, in one workgroup: keys and
// their order of arrival sorted by a bitonic network in LDS, the changed entries
// compacted and their shifts S (sum of net before each; S[nE] = the total)
// scanned (36 us for 601 updates, bound by the network's barriers and the row
// searches; as sort passes of five launches each, scans and waits for the host
// it was most of a call of 534 us, now 143).
__global__ void __launch_bounds__(SMALL_T) k_upd_small(UpdGraph g, int k, const int32_t* __restrict__ src,
                                                       const int32_t* __restrict__ dst, const uint8_t* __restrict__ ins,
                                                       uint64_t* __restrict__ E, uint32_t* __restrict__ P,
                                                       int64_t* __restrict__ S, uint32_t* __restrict__ u) {
  constexpr int M = 2 * UPD_SMALL, PER = M / SMALL_T;
  __shared__ uint64_t key[M];
  __shared__ uint16_t ord[M];
  __shared__ uint32_t err, wsum[SMALL_T / 64][2];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int N = 2 * k;
  int L = 64;
  while (L < N) L <<= 1;
  if (tid == 0) err = 0;
  __syncthreads();
  uint32_t bits = 0;
  for (int i = tid; i < L / 2; i += SMALL_T) {
    uint64_t k0 = ~0ull, k1 = ~0ull;
    if (i < k) bits |= op_keys(g, src[i], dst[i], ins[i], &k0, &k1);
    key[2 * i] = k0;
    key[2 * i + 1] = k1;
    ord[2 * i] = (uint16_t)(2 * i);
    ord[2 * i + 1] = (uint16_t)(2 * i + 1);
  }
  if (bits) atomicOr(&err, bits);
  __syncthreads();
  if (err) {
    if (tid == 0) u[U_ERR] = err;
    return;
  }
  for (int sz = 2; sz <= L; sz <<= 1)
    for (int j = sz >> 1; j > 0; j >>= 1) {
      for (int q = tid; q < L / 2; q += SMALL_T) {
        const int a = ((q & ~(j - 1)) << 1) | (q & (j - 1)), b = a | j;
        const uint64_t ka = key[a], kb = key[b];
        const uint16_t oa = ord[a], ob = ord[b];
        const bool gt = (ka >> 1) != (kb >> 1) ? (ka >> 1) > (kb >> 1) : oa > ob;
        if (gt == ((a & sz) == 0)) {
          key[a] = kb;
          key[b] = ka;
          ord[a] = ob;
          ord[b] = oa;
        }
      }
      __syncthreads();
    }
  // each thread: PER consecutive keys
  uint32_t f[PER], c = 0;
  int64_t pos[PER], d = 0;
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const int i = tid * PER + r;
    f[r] = 0;
    pos[r] = 0;
    if (i < N && (i == 0 || (key[i] >> 2) != (key[i - 1] >> 2))) {
      f[r] = entry_state(g, i, N, [&](int64_t q) { return key[q]; }, &pos[r]);
      if ((f[r] >> 2) == (f[r] & 3u)) f[r] = 0;
    }
    if (f[r]) {
      ++c;
      d += net_of(f[r]);
    }
  }
  // exclusive prefix of (changed entries, net) over the threads
  uint32_t sc = c;
  int32_t sd = (int32_t)d;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t qc = __shfl_up(sc, o, 64);
    const int32_t qd = __shfl_up(sd, o, 64);
    if (lane >= o) {
      sc += qc;
      sd += qd;
    }
  }
  if (lane == 63) {
    wsum[w][0] = sc;
    wsum[w][1] = (uint32_t)sd;
  }
  __syncthreads();
  uint32_t at = sc - c;
  int64_t sh = sd - d;
  for (int q = 0; q < w; ++q) {
    at += wsum[q][0];
    sh += (int32_t)wsum[q][1];
  }
#pragma unroll
  for (int r = 0; r < PER; ++r)
    if (f[r]) {
      E[at] = (key[tid * PER + r] >> 2) << 4 | f[r];
      P[at] = (uint32_t)pos[r];
      S[at] = sh;
      ++at;
      sh += net_of(f[r]);
    }
  if (tid == SMALL_T - 1) {
    S[at] = sh;
    u[U_NE] = at;
  }
}

// ----------------------------------------------------------------- row sums

struct DeltaArgs {
  UpdGraph g;
  const uint64_t* E;  // sorted changed entries
  uint64_t lut[4];    // class of code c: nibble c & 15 of lut[c >> 4]
  unsigned long long* acc;  // UPD_COPIES x UPD_ACC words, two's complement
  uint32_t* u;
  uint64_t* queue;    // parts put off: entry << 8 | part
  uint32_t room;      // their number at most
};
constexpr int UPD_COPIES = 32, UPD_ACC = 32;
__device__ __forceinline__ unsigned long long* acc_of(const DeltaArgs& a) {
  return a.acc + (blockIdx.x % UPD_COPIES) * UPD_ACC;
}
__device__ __forceinline__ uint64_t wave_sum(uint64_t x) {
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}
__device__ __forceinline__ uint64_t lane64(uint64_t x, int l) {
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(x >> 32), l) << 32) |
         (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, l);
}

// Neighbour counts by flag of the entries [b, e), by one wavefront: 16 entries a
// lane and read.
__device__ __forceinline__ void flag_counts(const UpdGraph& g, int64_t b, int64_t e, int lane, uint32_t (&c)[3]) {
  const int64_t nbytes = (g.nnz + 3) / 4;
  uint32_t o = 0, i = 0, m = 0;
#pragma unroll 4
  for (int64_t p = (b >> 2) + 4 * lane; p * 4 < e; p += 256) {
    uint32_t w = 0;
    if (p + 4 <= nbytes) __builtin_memcpy(&w, g.flg + p, 4);
    else
      for (int q = 0; q < 4 && p + q < nbytes; ++q) w |= (uint32_t)g.flg[p + q] << (8 * q);
    const int64_t at = p * 4;  // the word's first entry
    if (at < b) w &= ~0u << (2 * (b - at));
    if (at + 16 > e) w &= ~(~0u << (2 * (e - at)));
    const uint32_t lo = w & 0x55555555u, hi = (w >> 1) & 0x55555555u;
    o += __popc(lo & ~hi);
    i += __popc(hi & ~lo);
    m += __popc(lo & hi);
  }
  for (int s = 32; s > 0; s >>= 1) {
    o += __shfl_xor(o, s, 64);
    i += __shfl_xor(i, s, 64);
    m += __shfl_xor(m, s, 64);
  }
  c[0] = o;
  c[1] = i;
  c[2] = m;
}

// One wavefront per changed row (at the first of its changed entries).
__global__ void __launch_bounds__(UT) k_upd_rows(DeltaArgs a) {
  if (a.u[U_ERR]) return;
  const UpdGraph& g = a.g;
  const int lane = threadIdx.x & 63;
  const int64_t nw = ((int64_t)gridDim.x * UT) >> 6, nE = a.u[U_NE];
  RowSums sums;
  for (int64_t i = ((int64_t)blockIdx.x * UT + threadIdx.x) >> 6; i < nE; i += nw) {
    const uint64_t x = a.E[i] >> (4 + g.rb);
    if (i > 0 && (a.E[i - 1] >> (4 + g.rb)) == x) continue;
    uint32_t c0[3];
    flag_counts(g, g.off[x], g.off[x + 1], lane, c0);
    int64_t c1[3] = {c0[0], c0[1], c0[2]};
    for (int64_t j = i;; j += 64) {
      const uint64_t ent = j + lane < nE ? a.E[j + lane] : ~0ull;
      const bool mine = j + lane < nE && (ent >> (4 + g.rb)) == x;
      for (uint32_t f = 1; f <= 3; ++f)
        c1[f - 1] += (int64_t)__popcll(__ballot(mine && (ent & 3u) == f)) -
                     (int64_t)__popcll(__ballot(mine && (ent >> 2 & 3u) == f));
      if (!__builtin_amdgcn_readlane(mine, 63)) break;
    }
    if (lane == 0) {
      RowSums p, q;
      p.row((uint64_t)g.n, c0[0], c0[1], c0[2]);
      q.row((uint64_t)g.n, (uint64_t)c1[0], (uint64_t)c1[1], (uint64_t)c1[2]);
      for (int k = 0; k < 9; ++k) sums.c[k] += q.c[k] - p.c[k];
    }
  }
  // (lane 0 holds each wavefront's sums)
  if (lane == 0)
    for (int k = 0; k < 9; ++k)
      if (sums.c[k]) atomicAdd(&acc_of(a)[RowSums::slot(k)], (unsigned long long)sums.c[k]);
}

// ---------------------------------------------------------------- triangles

__device__ __forceinline__ uint32_t class_of(const DeltaArgs& g, uint32_t code) {
  const uint64_t w = code < 16 ? g.lut[0] : code < 32 ? g.lut[1] : code < 48 ? g.lut[2] : g.lut[3];
  return (uint32_t)(w >> (4 * (code & 15u))) & 15u;
}

// Change entry of (x, y) in E[b, e) (the row x range): index or -1.
__device__ __forceinline__ int64_t find_change(const DeltaArgs& a, int64_t b, int64_t e, int64_t x, int32_t y) {
  const uint64_t k = (((uint64_t)x << a.g.rb) | (uint64_t)y) << 4;
  const int64_t p = lower_key(a.E, b, e, k);
  return (p < e && (a.E[p] >> 4) == (k >> 4)) ? p : -1;
}

struct Pair {
  int64_t a;
  int32_t b;
  uint32_t f0, f1;
  int64_t oa, ea, ob, eb;      // rows a and b
  int64_t da0, da1, db0, db1;  // their changed entries
};

// The pair is the smallest changed one of the triad {a, b, w} (the changed ones
// among its other two: cha, chb).
__device__ __forceinline__ bool owns(int rb, const Pair& p, int32_t w, bool cha, bool chb) {
  const uint64_t pk = ((uint64_t)p.a << rb) | (uint64_t)p.b;
  const int64_t a = p.a, b = p.b;
  return !(cha && ((((uint64_t)min((int64_t)w, a)) << rb) | (uint64_t)max((int64_t)w, a)) < pk) &&
         !(chb && ((((uint64_t)min((int64_t)w, b)) << rb) | (uint64_t)max((int64_t)w, b)) < pk);
}

// Entries [s0, s1) of the shorter of rows a and b searched in the longer: the w
// adjacent to both before.
__device__ void pair_part(const DeltaArgs& A, const Pair& p, int64_t s0, int64_t s1, int lane, int32_t* h) {
  const UpdGraph& g = A.g;
  const bool aside = p.ea - p.oa <= p.eb - p.ob;  // row a is the shorter
  const int64_t base = aside ? p.oa : p.ob, lb = aside ? p.ob : p.oa, le = aside ? p.eb : p.ea;
  for (int64_t j = s0 + lane; j < s1; j += 64) {
    const int32_t w = g.nbr[base + j];
    const int64_t q = lower_id(g.nbr, lb, le, w);
    if (q >= le || g.nbr[q] != w) continue;
    const uint32_t fs = entry_flag(g.flg, base + j), fl = entry_flag(g.flg, q);
    const uint32_t g0a = aside ? fs : fl, g0b = aside ? fl : fs;
    const int64_t ca = p.da1 - p.da0 > 1 ? find_change(A, p.da0, p.da1, p.a, w) : -1;
    const int64_t cb = p.db1 - p.db0 > 1 ? find_change(A, p.db0, p.db1, p.b, w) : -1;
    if (!owns(g.rb, p, w, ca >= 0, cb >= 0)) continue;
    const uint32_t g1a = ca >= 0 ? (uint32_t)A.E[ca] & 3u : g0a, g1b = cb >= 0 ? (uint32_t)A.E[cb] & 3u : g0b;
    if (p.f0) h[class_of(A, p.f0 | g0a << 2 | g0b << 4) * 64 + lane] -= 1;
    if (p.f1 && g1a && g1b) h[class_of(A, p.f1 | g1a << 2 | g1b << 4) * 64 + lane] += 1;
  }
}

// The triangles after that need an inserted entry of a or of b.
__device__ void pair_changes(const DeltaArgs& A, const Pair& p, int lane, int32_t* h) {
  if (!p.f1) return;
  const UpdGraph& g = A.g;
  const uint64_t cmask = (1ull << g.rb) - 1;
  auto old_flag = [&](int64_t b, int64_t e, int32_t w) {
    const int64_t j = lower_id(g.nbr, b, e, w);
    return j < e && g.nbr[j] == w ? entry_flag(g.flg, j) : 0u;
  };
  for (int side = 0; side < 2; ++side) {
    const int64_t L0 = side ? p.db0 : p.da0, L1 = side ? p.db1 : p.da1;
    for (int64_t j = L0 + lane; j < L1; j += 64) {
      const uint64_t ent = A.E[j];
      const int32_t w = (int32_t)((ent >> 4) & cmask);
      const uint32_t g0 = (uint32_t)(ent >> 2) & 3u, g1 = (uint32_t)ent & 3u;  // with this side
      if (w == p.a || w == p.b || !g1) continue;
      const int64_t q = side ? find_change(A, p.da0, p.da1, p.a, w) : find_change(A, p.db0, p.db1, p.b, w);
      if (side && q >= 0) continue;  // taken by the changes of a
      uint32_t h0, h1;               // with the other side
      if (q >= 0) {
        h0 = (uint32_t)(A.E[q] >> 2) & 3u;
        h1 = (uint32_t)A.E[q] & 3u;
      } else {
        h0 = h1 = side ? old_flag(p.oa, p.ea, w) : old_flag(p.ob, p.eb, w);
      }
      if (!h1 || (g0 && h0) || !owns(g.rb, p, w, side == 0 || q >= 0, side == 1 || q >= 0)) continue;
      h[class_of(A, p.f1 | (side ? h1 : g1) << 2 | (side ? g1 : h1) << 4) * 64 + lane] += 1;
    }
  }
}

__device__ __forceinline__ Pair pair_of(const DeltaArgs& A, int64_t q) {
  const UpdGraph& g = A.g;
  const uint64_t ent = A.E[q];
  Pair p;
  p.a = (int64_t)(ent >> (4 + g.rb));
  p.b = (int32_t)((ent >> 4) & ((1ull << g.rb) - 1));
  p.f0 = (uint32_t)(ent >> 2) & 3u;
  p.f1 = (uint32_t)ent & 3u;
  p.oa = g.off[p.a];
  p.ea = g.off[p.a + 1];
  p.ob = g.off[p.b];
  p.eb = g.off[p.b + 1];
  return p;
}
// The rows' changed entries: four searches, one a lane.
__device__ __forceinline__ void pair_ranges(const DeltaArgs& A, Pair& p, int64_t nE, int lane) {
  const int64_t x = (lane & 2 ? (int64_t)p.b : p.a) + (lane & 1);
  const int64_t r = lane < 4 ? lower_key(A.E, 0, nE, (uint64_t)x << (A.g.rb + 4)) : 0;
  p.da0 = (int64_t)lane64((uint64_t)r, 0);
  p.da1 = (int64_t)lane64((uint64_t)r, 1);
  p.db0 = (int64_t)lane64((uint64_t)r, 2);
  p.db1 = (int64_t)lane64((uint64_t)r, 3);
}
__device__ __forceinline__ int64_t part_size(int64_t len) {
  return len > UPD_PART * UPD_PARTS ? (len + UPD_PARTS - 1) / UPD_PARTS : UPD_PART;
}

__device__ void flush_classes(int32_t* h, int lane, unsigned long long* acc) {
  __builtin_amdgcn_wave_barrier();
  for (int c = 8; c < 16; ++c) {
    const uint64_t x = wave_sum((uint64_t)(int64_t)h[c * 64 + lane]);
    if (lane == 0 && x) atomicAdd(&acc[c], (unsigned long long)x);
    h[c * 64 + lane] = 0;
  }
  __builtin_amdgcn_wave_barrier();
}

// One wavefront per changed pair (the entries with row < column): the first
// UPD_PART entries of its shorter row, and its changes. Further parts go to
// other wavefronts (MORE, a second launch) through a queue, or are taken here if
// it is full.
template <bool MORE>
__global__ void __launch_bounds__(UT) k_upd_pairs(DeltaArgs A) {
  __shared__ int32_t hist[UT / 64][16 * 64];
  if (A.u[U_ERR]) return;
  const uint64_t listed = MORE ? *parts_of(A.u) : 0;
  if (MORE && listed == 0) return;
  const int lane = threadIdx.x & 63;
  int32_t* h = hist[threadIdx.x >> 6];
  for (int c = 0; c < 16; ++c) h[c * 64 + lane] = 0;
  const int64_t nw = ((int64_t)gridDim.x * UT) >> 6, nE = A.u[U_NE];
  const int64_t items = MORE ? (int64_t)min(listed, (uint64_t)A.room) : nE;
  uint64_t steps = 0;
  for (int64_t it = ((int64_t)blockIdx.x * UT + threadIdx.x) >> 6; it < items; it += nw) {
    const int64_t q = MORE ? (int64_t)(A.queue[it] >> 8) : it;
    Pair p = pair_of(A, q);
    if (!MORE && p.b < p.a) continue;
    pair_ranges(A, p, nE, lane);
    const int64_t len = min(p.ea - p.oa, p.eb - p.ob), sz = part_size(len);
    int64_t s0 = 0, s1 = min(len, sz);
    if (MORE) {
      s0 = min(len, (int64_t)(A.queue[it] & 255u) * sz);
      s1 = min(len, s0 + sz);
    } else {
      pair_changes(A, p, lane, h);
      const int parts = (int)((len + sz - 1) / sz);
      if (parts > 1) {
        uint32_t at = 0;
        if (lane == 0) at = (uint32_t)min((uint64_t)atomicAdd(parts_of(A.u), (unsigned long long)(parts - 1)), (uint64_t)A.room);
        at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
        for (int c = 1 + lane; c < parts; c += 64)
          if ((int64_t)at + c - 1 < A.room) A.queue[at + c - 1] = (uint64_t)q << 8 | (uint64_t)c;
        // the parts that found no room
        const int64_t room = max((int64_t)0, min((int64_t)parts - 1, (int64_t)A.room - (int64_t)at));
        if (room < parts - 1) pair_part(A, p, (1 + room) * sz, len, lane, h);
      }
    }
    pair_part(A, p, s0, s1, lane, h);
    steps += (uint64_t)(len + p.da1 - p.da0 + p.db1 - p.db0) / 64 + 4;
    if (steps > (1u << 29)) {
      flush_classes(h, lane, acc_of(A));
      steps = 0;
    }
  }
  flush_classes(h, lane, acc_of(A));
}

// ---------------------------------------------------------- CSR after

// new_off[x] = off[x] + the net of the changed entries in rows below x
__global__ void k_new_offsets(UpdGraph g, const uint64_t* __restrict__ E, const int64_t* __restrict__ S,
                              int64_t* __restrict__ noff, const uint32_t* __restrict__ u) {
  if (u[U_ERR]) return;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x, nE = u[U_NE];
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x <= g.n; x += stride)
    noff[x] = g.off[x] + S[lower_key(E, 0, nE, (uint64_t)x << (g.rb + 4))];
}

// The entries after the batch, by place: changed entry e stands at Q = P[e] +
// S[e] (an inserted or reflagged entry; a deleted one gives its place to what
// follows), and between two of them the old entries move by one shift. A tile
// of places finds its changed entries by two searches and stages them in LDS;
// a thread writes four ids and their flag byte. (By old entry, with the flags as
// bytes and a pass to pack them: 1.0 ms per 100,000 updates on 90 M entries;
// now 0.28.)
constexpr int CT = 4096, CSTAGE = 1024;
__global__ void __launch_bounds__(UT) k_upd_copy(UpdGraph g, const uint64_t* __restrict__ E,
                                                 const uint32_t* __restrict__ P, const int64_t* __restrict__ S,
                                                 int32_t* __restrict__ nnbr, uint8_t* __restrict__ nflg,
                                                 const uint32_t* __restrict__ u) {
  __shared__ int64_t range[2];
  __shared__ int32_t sq[CSTAGE];   // place in the tile (before it: -1)
  __shared__ int64_t ss[CSTAGE];   // shift of the entries after it
  __shared__ int32_t sid[CSTAGE];  // id of an inserted entry, else -1
  __shared__ uint8_t sf[CSTAGE];   // flag of the entry at its place, 0 for a deleted one
  if (u[U_ERR]) return;
  const int64_t nE = u[U_NE], nn = g.nnz + S[nE];
  const uint64_t cmask = (1ull << g.rb) - 1;
  auto Q = [&](int64_t e) { return (int64_t)P[e] + S[e]; };
  for (int64_t t0 = (int64_t)blockIdx.x * CT; t0 < nn; t0 += (int64_t)gridDim.x * CT) {
    const int64_t t1 = min(t0 + (int64_t)CT, nn);
    __syncthreads();
    if (threadIdx.x < 2) {
      // the last changed entry at or before the tile's first and last place
      const int64_t j = threadIdx.x ? t1 - 1 : t0;
      int64_t lo = 0, hi = nE;
      while (lo < hi) {
        const int64_t m = (lo + hi) >> 1;
        if (Q(m) <= j) lo = m + 1; else hi = m;
      }
      range[threadIdx.x] = lo - 1;
    }
    __syncthreads();
    // changed entries e0 .. e1: e0 (if any) at or before the first place
    const int64_t e0 = max(range[0], (int64_t)0), e1 = range[1];
    const int64_t ne = e1 - e0 + 1;
    const bool staged = ne <= CSTAGE;
    auto load = [&](int64_t e, int64_t& q, int64_t& sh, int32_t& id, uint32_t& f) {
      const uint64_t x = E[e];
      f = (uint32_t)x & 3u;
      q = Q(e);
      sh = S[e] + net_of((uint32_t)x & 15u);
      id = (x >> 2 & 3u) == 0 ? (int32_t)(x >> 4 & cmask) : -1;
    };
    if (staged)
      for (int64_t e = threadIdx.x; e < ne; e += UT) {
        int64_t q, sh;
        int32_t id;
        uint32_t f;
        load(e0 + e, q, sh, id, f);
        sq[e] = q < t0 ? -1 : (int32_t)(q - t0);
        ss[e] = sh;
        sid[e] = id;
        sf[e] = (uint8_t)f;
      }
    __syncthreads();
    for (int64_t j = t0 + 4 * threadIdx.x; j < t1; j += 4 * UT) {
      // the last changed entry at or before place j, k after it
      int64_t k = 0, hi = ne;  // entries e0 .. e0 + k - 1 stand at or before j
      while (k < hi) {
        const int64_t m = (k + hi) >> 1;
        if ((staged ? t0 + sq[m] : Q(e0 + m)) <= j) k = m + 1; else hi = m;
      }
      int32_t id[4];
      uint32_t byte = 0;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t jj = j + r;
        id[r] = 0;
        if (jj >= t1) continue;
        while (k < ne && (staged ? t0 + sq[k] : Q(e0 + k)) <= jj) ++k;
        int64_t q = -1, sh = 0;
        int32_t nid = -1;
        uint32_t f = 0;
        if (k > 0) {
          if (staged) {
            q = t0 + sq[k - 1];
            sh = ss[k - 1];
            nid = sid[k - 1];
            f = sf[k - 1];
          } else {
            load(e0 + k - 1, q, sh, nid, f);
          }
        }
        const bool here = q == jj && f != 0;  // an inserted or a reflagged entry
        if (here && nid >= 0) {
          id[r] = nid;
        } else {
          const int64_t o = jj - sh;
          id[r] = g.nbr[o];
          if (!here) f = entry_flag(g.flg, o);
        }
        byte |= f << (2 * r);
      }
      if (j + 4 <= t1) __builtin_memcpy(nnbr + j, id, 16);
      else
        for (int r = 0; r < 4 && j + r < t1; ++r) nnbr[j + r] = id[r];
      nflg[j >> 2] = (uint8_t)byte;
    }
  }
}

// The accumulators' copies summed, then the counts: what the host reads.
__global__ void k_upd_done(const unsigned long long* __restrict__ acc, const uint32_t* __restrict__ u,
                           const int64_t* __restrict__ S, uint64_t* __restrict__ out) {
  const int i = threadIdx.x;
  if (i < UPD_ACC) {
    uint64_t t = 0;
    for (int k = 0; k < UPD_COPIES; ++k) t += acc[k * UPD_ACC + i];
    out[i] = t;
  }
  if (i == 0) {
    out[UPD_ACC] = u[U_ERR];
    out[UPD_ACC + 1] = u[U_NE];
    out[UPD_ACC + 2] = u[U_ERR] ? 0 : (uint64_t)S[u[U_NE]];
  }
}

__global__ void k_zero32(uint32_t* p, int64_t m) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) p[i] = 0;
}

}  // namespace

int census_update(int64_t n, int64_t nnz, const int64_t* off, const int32_t* nbr, const uint8_t* flg, int64_t k,
                  const int32_t* src, const int32_t* dst, const uint8_t* ins, const uint64_t* cin, uint64_t* cout,
                  int64_t* noff, int32_t* nnbr, uint8_t* nflg, int64_t* nnz_new, int64_t* changed_pairs,
                  hipStream_t s) {
  if (n < 0 || n >= ((int64_t)1 << 30)) return fail(TRIAD_EINVAL, "n must be in [0, 2^30)");
  if (nnz < 0 || nnz >= ((int64_t)1 << 32)) return fail(TRIAD_EINVAL, "nnz must be in [0, 2^32)");
  if (k < 0 || k >= ((int64_t)1 << 31)) return fail(TRIAD_EINVAL, "the update count must be in [0, 2^31)");
  if (!off || !cin || !cout || (nnz > 0 && (!nbr || !flg)) || (k > 0 && (!src || !dst || !ins)))
    return fail(TRIAD_EINVAL, "NULL pointer argument");
  const bool new_csr = noff != nullptr;
  if (new_csr && (!nnz_new || !nnbr || !nflg)) return fail(TRIAD_EINVAL, "NULL pointer for the new CSR");
  DeviceInfo di;
  if (int st = device_info(&di)) return st;
  Scratch scratch(s, 0, true);
  const int rb = std::max(1, 64 - __builtin_clzll((unsigned long long)std::max<int64_t>(n, 1)));
  const UpdGraph g{n, nnz, off, nbr, flg, rb};
  const int64_t N = 2 * k;  // keys, and at most as many changed entries
  constexpr int ZERO = 2 * UPD_COPIES * UPD_ACC + U_WORDS;
  uint32_t* zero = nullptr;
  uint64_t *out = nullptr, *E = nullptr, *queue = nullptr;
  uint32_t* P = nullptr;
  int64_t* S = nullptr;
  ALLOC(zero, ZERO);
  ALLOC(out, UPD_ACC + 3);
  ALLOC(P, N);
  ALLOC(S, N + 1);
  // a pair has further parts for every UPD_PART entries of its shorter row, and at
  // most nnz / UPD_PART rows are that long
  const int64_t longs = nnz / UPD_PART, room = std::min(std::min(UPD_QUEUE, N * UPD_PARTS), longs * longs);
  ALLOC(queue, room);
  unsigned long long* acc = (unsigned long long*)zero;
  uint32_t* u = zero + 2 * UPD_COPIES * UPD_ACC;
  k_zero32<<<2, 256, 0, s>>>(zero, ZERO);
  if (k <= UPD_SMALL) {
    ALLOC(E, N);
    k_upd_small<<<1, SMALL_T, 0, s>>>(g, (int)k, src, dst, ins, E, P, S, u);
  } else {
    uint64_t *ka = nullptr, *kb = nullptr;
    uint32_t *chg = nullptr, *cpos = nullptr, *pos = nullptr;
    uint8_t* st8 = nullptr;
    ALLOC(ka, N);
    ALLOC(kb, N);
    ALLOC(chg, N);
    ALLOC(cpos, N);
    ALLOC(pos, N);
    ALLOC(st8, N);
    k_upd_keys<<<grid_of(k, 256, 65536), 256, 0, s>>>(g, k, src, dst, ins, ka, u);
    // by (row, column, direction); operations keep their batch order within an arc
    if (int st = radix_sort_u64(&ka, &kb, N, 1, 2 + 2 * rb, scratch, s)) return st;
    k_upd_state<<<grid_of(N, 256, 65536), 256, 0, s>>>(g, ka, N, chg, st8, pos, u);
    if (int st = scan_u32(chg, N, cpos, u + U_NE, scratch, s)) return st;
    E = kb;  // (the sort is done with it)
    k_upd_emit<<<grid_of(N, 256, 65536), 256, 0, s>>>(ka, N, chg, cpos, st8, pos, E, P, S, u);
    if (int st = scan_i64(S, N, S, scratch, s)) return st;
  }
  DeltaArgs a{g, E, {}, acc, u, queue, (uint32_t)room};
  for (int c = 0; c < 64; ++c) a.lut[c >> 4] |= (uint64_t)classify_code((unsigned)c) << (4 * (c & 15));
  if (k > 0) {
    const unsigned waves4 = (unsigned)grid_of(N * 64, UT, di.cus * 8);
    k_upd_rows<<<waves4, UT, 0, s>>>(a);
    k_upd_pairs<false><<<waves4, UT, 0, s>>>(a);
    k_upd_pairs<true><<<(unsigned)grid_of(room * 64, UT, di.cus * 8), UT, 0, s>>>(a);
  }
  if (new_csr) {
    k_new_offsets<<<grid_of(n + 1, 256, 65536), 256, 0, s>>>(g, E, S, noff, u);
    if (nnz + N > 0) k_upd_copy<<<grid_of(nnz + N, CT, di.cus * 16), UT, 0, s>>>(g, E, P, S, nnbr, nflg, u);
  }
  k_upd_done<<<1, 64, 0, s>>>(acc, u, S, out);
  HIPCHK(hipGetLastError());
  uint64_t oh[UPD_ACC + 3];
  HIPCHK(hipMemcpyAsync(oh, out, sizeof oh, hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  const uint32_t eh = (uint32_t)oh[UPD_ACC];
  if (eh) return fail(status_from_bits(eh), eh & ERR_RANGE ? "update endpoint outside [0, n) or kind not 0/1"
                                                           : "update on a self-loop");
  // the census after the batch
  uint64_t d[16];
  for (int t = 0; t < 16; ++t) d[t] = oh[t];
  d[2] += (uint64_t)n * (uint64_t)((int64_t)oh[SUMS_MUT] / 2);
  open_wedges(d);
  uint64_t res[17];
  unsigned __int128 sum = 0;
  for (int t = 1; t < 16; ++t) {
    res[t] = cin[t] + d[t];
    sum += res[t];
  }
  uint64_t clo, chi;
  choose3(n, &clo, &chi);
  const unsigned __int128 nul = (((unsigned __int128)chi << 64) | clo) - sum;
  res[0] = (uint64_t)nul;
  res[16] = (uint64_t)(nul >> 64);
  if (new_csr) *nnz_new = nnz + (int64_t)oh[UPD_ACC + 2];
  std::memcpy(cout, res, sizeof res);
  if (changed_pairs) *changed_pairs = (int64_t)oh[UPD_ACC + 1] / 2;
  return res[16] ? TRIAD_OK_003_WRAPPED : TRIAD_OK;
}

}  // namespace triad

using namespace triad;

extern "C" int triad_census_update(int64_t n, int64_t nnz, const int64_t* d_offsets, const int32_t* d_nbrs,
                                   const uint8_t* d_flags, int64_t nupd, const int32_t* d_src, const int32_t* d_dst,
                                   const uint8_t* d_insert, const uint64_t census_in[17], uint64_t census_out[17],
                                   int64_t* d_offsets_new, int32_t* d_nbrs_new, uint8_t* d_flags_new,
                                   int64_t* nnz_new, int64_t* changed_pairs, void* hip_stream) {
  return census_update(n, nnz, d_offsets, d_nbrs, d_flags, nupd, d_src, d_dst, d_insert, census_in, census_out,
                       d_offsets_new, d_nbrs_new, d_flags_new, nnz_new, changed_pairs, (hipStream_t)hip_stream);
}
