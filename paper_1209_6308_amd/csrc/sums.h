// Row sums and open wedges: the parts of a census that follow from each vertex's
// neighbour counts. Internal; not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace triad {

constexpr int SUMS_MUT = 16;  // counter of the entries with both arcs (each mutual edge twice)

// Sums of one row's neighbour counts (o: arcs out only, i: in only, m: both)
// into class sums: pairs of neighbours by centre, and n - d(u) - d(v) per
// edge (the n of a one-way edge taken at its tail, of a mutual one at the end).
struct RowSums {
  uint64_t c[9] = {};  // 012 102 021D 021U 021C 111D 111U 201, entries with both arcs
  __device__ __forceinline__ void row(uint64_t n, uint64_t o, uint64_t i, uint64_t m) {
    const uint64_t d = o + i + m;
    c[0] += n * o - d * (o + i);
    c[1] -= d * m;
    c[2] += o * (o - 1) / 2;  // (o = 0: 0 * ... = 0)
    c[3] += i * (i - 1) / 2;
    c[4] += o * i;
    c[5] += i * m;
    c[6] += o * m;
    c[7] += m * (m - 1) / 2;
    c[8] += m;
  }
  static __device__ __forceinline__ int slot(int k) {
    return k == 0 ? 1 : k == 1 ? 2 : k == 7 ? 10 : k == 8 ? SUMS_MUT : k + 1;
  }
  // a graph of a batch keeps the mutual count in the place of 003
  static __device__ __forceinline__ int batch_slot(int k) { return k == 8 ? 0 : slot(k); }
};

// From the sums of all rows and the triangle classes (8, 9, 11 .. 15) to the
// classes: a triangle's three pairs of neighbours are adjacent, so each class of
// triangle takes its own pairs out of the pair sums; 012 and 102 get the common
// neighbours that n - d(u) - d(v) subtracted twice. Linear: differences too.
__host__ __device__ __forceinline__ void open_wedges(uint64_t* c) {
  c[3] -= c[8] + c[11];
  c[4] -= c[8] + c[12];
  c[5] -= c[8] + 3 * c[9] + c[13];
  c[6] -= 2 * c[11] + c[13] + c[14];
  c[7] -= 2 * c[12] + c[13] + c[14];
  c[10] -= c[14] + 3 * c[15];
  const uint64_t one = c[11] + c[12] + c[13];
  c[1] += 3 * (c[8] + c[9]) + 2 * one + c[14];
  c[2] += one + 2 * c[14] + 3 * c[15];
}

}  // namespace triad
