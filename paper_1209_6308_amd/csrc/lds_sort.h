// Sorting in LDS by one workgroup, for kernels of this library. Internal; not
// part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace triad {

// inclusive sum over the lanes of a wavefront
__device__ __forceinline__ uint32_t wave_scan(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);  // row_shr:1, 2, 4, 8
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);  // row_bcast:15, 31
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);
  return x;
}

// Rank of each lane's key among the equal digits before it in the wavefront,
// after those counted in cnt (the wavefront's own), which takes these in.
__device__ __forceinline__ uint32_t match_rank(uint32_t d, uint32_t* cnt, uint64_t below, uint64_t above) {
  uint32_t lo = 0, hi = 0;  // lanes whose digit differs from this lane's
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    uint32_t t = (uint32_t)__builtin_amdgcn_sbfe((int)d, b, 1);
    asm("" : "+v"(t));  // compared as it is (otherwise the bit is shifted out a second time)
    const uint64_t mb = __ballot(t != 0);
    lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)mb, t, 0xF0 | (0xCC ^ 0xAA));  // lo | (mb ^ t)
    hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(mb >> 32), t, 0xF0 | (0xCC ^ 0xAA));
  }
  const uint64_t m = ~((uint64_t)hi << 32 | lo);
  // every lane of a digit group reads the running count, then the group's
  // highest lane advances it (LDS operations of one wavefront run in order)
  const uint32_t pos = cnt[d] + (uint32_t)__popcll(m & below);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  if ((m & above) == 0) cnt[d] = pos + 1;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  return pos;
}

// Counts of W wavefronts (cnt[W][256]) -> first places, digit by digit from 0
// (or from first[digit], written by this thread) and wavefront by wavefront.
// Returns the digit's total (of thread t < 256 for digit t).
template <int W>
__device__ __forceinline__ uint32_t digit_starts(uint32_t (*cnt)[256], uint32_t* sh, const uint32_t* first) {
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  uint32_t c = 0, x = 0;
  if (t < 256) {
#pragma unroll
    for (int q = 0; q < W; ++q) c += cnt[q][t];
    x = wave_scan(c);
    if (lane == 63) sh[w] = x;
  }
  __syncthreads();
  if (t < 256) {
    uint32_t run = x - c;
    for (int q = 0; q < w; ++q) run += sh[q];
    if (first) run = first[t];
#pragma unroll
    for (int q = 0; q < W; ++q) {
      const uint32_t v = cnt[q][t];
      cnt[q][t] = run;
      run += v;
    }
  }
  __syncthreads();
  return c;
}

// Sorts len <= T * R keys from in to s (LDS) on their low `bits` bits, least
// significant digits first; the first pass may rank in any order. A wavefront
// takes 64 keys in each of ceil(len / T) rounds; the places past len hold the
// highest key and stay behind the others (s[0, len) is what counts).
template <int T, int R>
__device__ __forceinline__ void lds_sort(uint32_t* s, uint32_t (*cnt)[256], uint32_t* sh,
                                         const uint32_t* __restrict__ in, uint32_t len, int bits) {
  constexpr int W = T / 64;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const uint64_t below = (1ull << lane) - 1, above = ~below << 1;
  const int nr = (int)((len + T - 1) / T);
  const uint32_t i0 = (uint32_t)(w * nr * 64 + lane), last = (uint32_t)((1ull << bits) - 1);
  static_assert(T * R <= 65536 && R % 2 == 0, "places of 16 bits, two a register");
  uint32_t key[R], pos[R / 2];
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (r < nr) key[r] = i0 + r * 64 < len ? in[i0 + r * 64] : last;
  const int P = (bits + 7) / 8;
  int lo = 0;
  for (int p = 0; p < P; ++p) {
    const int hi = bits * (p + 1) / P, wd = hi - lo;
    static_assert(W * 256 == 4 * T, "one 16-byte store a thread");
    reinterpret_cast<uint4*>(cnt)[t] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    if (p == 0) {
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (r < nr) {
          const uint32_t q = atomicAdd(&cnt[w][__builtin_amdgcn_ubfe(key[r], 0, wd)], 1u);
          pos[r / 2] = r & 1 ? pos[r / 2] | q << 16 : q;
        }
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (r < nr) {
          key[r] = s[i0 + r * 64];
          const uint32_t q = match_rank(__builtin_amdgcn_ubfe(key[r], lo, wd), cnt[w], below, above);
          pos[r / 2] = r & 1 ? pos[r / 2] | q << 16 : q;
        }
    }
    __syncthreads();
    digit_starts<W>(cnt, sh, nullptr);
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (r < nr) {
        const uint32_t q = r & 1 ? pos[r / 2] >> 16 : pos[r / 2] & 0xFFFFu;
        s[cnt[w][__builtin_amdgcn_ubfe(key[r], lo, wd)] + q] = key[r];
      }
    __syncthreads();
    lo = hi;
  }
}

}  // namespace triad
