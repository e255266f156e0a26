// How a workgroup of a persistent GEMV launch starts: finding the GEMVs its
// waves begin in, and bringing in the activations they share.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "batch.h"
#include "device_common.h"

namespace bitcos_dev {

typedef unsigned piece_t __attribute__((ext_vector_type(4)));  // 16 bytes

// The last descriptors of the table that begin at or before units U and V
// (uniform).  64 descriptors are compared at a time, one per lane: a binary
// search waits for a load from device memory at each of its steps.
struct DescPair {
  int u, v;
};
__device__ __forceinline__ DescPair first_descs(const bitcos::GemvDesc* table, int count, int64_t U, int64_t V) {
  typedef const __attribute__((address_space(1))) bitcos::GemvDesc GDesc;
  const int lane = threadIdx.x & 63;
  // A copy of the table's address for the lanes' own loads: used for both, it
  // ends in VGPRs and every descriptor field after it too.
  const bitcos::GemvDesc* tv = table;
  asm("" : "+v"(tv));
  const auto begins = [&](int lo, int n, int step) {
    const int i = lane * step;
    return i < n ? ((GDesc*)tv)[lo + i].unit_begin : INT64_MAX;
  };
  const int step0 = (count + 63) >> 6;
  const int64_t b0 = begins(0, count, step0);
  const auto find = [&](int64_t unit) {
    int lo = 0, n = count, step = step0;
    int64_t b = b0;
    for (;;) {  // descriptor lo begins at or before the unit; the last such one is among the n from there
      const int c = __builtin_popcountll(__builtin_amdgcn_ballot_w64(b <= unit)) - 1;
      lo += c * step;
      n = min(step, n - c * step);
      if (n <= 1) return __builtin_amdgcn_readfirstlane(lo);
      step = (n + 63) >> 6;
      b = begins(lo, n, step);
    }
  };
  return {find(U), find(V)};
}

// A wave's share [begin, end) of a launch's units: consecutive workgroups take
// consecutive shares, as equal as whole units allow, and so do the waves of
// each.  A launch of few units so keeps a wave or two busy on every CU rather
// than a few full ones, whose waves wait for each other's issue slots (4096 x
// 4096 int8 with the faster table build: 7.5 -> 6.3 us), and a large launch has
// no wave with more than one unit above the others' (Qwen3-8B-like int8 set of
// 8 layers 91.1 -> 86.8 us).
template <class I>
struct UnitRange {
  I first;       // the workgroup's first unit
  I begin, end;  // the wave's
};
template <int WAVES, class I>
__device__ __forceinline__ UnitRange<I> unit_range(I total, int wv) {
  const I b = static_cast<I>(blockIdx.x), g = static_cast<I>(gridDim.x);
  const I q = total / g, r = total % g;  // the first r workgroups take one unit more
  const I first = b * q + (b < r ? b : r);
  const I n = q + (b < r ? 1 : 0);
  // n wv / WAVES without a product of n, which may take all of I's bits.
  const I nq = n / WAVES;
  const int nr = static_cast<int>(n % WAVES);
  const auto cut = [&](int w) { return first + nq * w + nr * w / WAVES; };
  return {first, cut(wv), cut(wv + 1)};
}

// Activations of the GEMV that a workgroup starts on, fetched once for all of
// its waves.  A lane keeps the activations of its consecutive units, so a
// wave that reads them itself touches another cache line with every lane of
// every load, about one lane a cycle: 12 waves x 16 loads of 16 bytes held a
// CU's address unit for some 12000 cycles of every launch (4096 x 4096 int8
// GEMV: 12.3 us, with this 7.4 us).  Here every thread gathers a few pieces
// of 16 bytes while the tables are built; they go through LDS in
// [piece][segment] order, which the lanes read without conflicts.  Where the
// buffer of ROOM pieces is too small for all, they go in rounds.
//   PER: pieces of a row segment; SEG: segments of a row; NT: threads.
template <int PER, int SEG, int NT, int ROOM>
struct FirstX {
  static constexpr int kPieces = PER * SEG;
  static constexpr int kMine = (kPieces + NT - 1) / NT;
  static constexpr int kAtOnce = PER < ROOM / SEG ? PER : ROOM / SEG;  // pieces of a segment per round
  static constexpr int kRounds = (PER + kAtOnce - 1) / kAtOnce;
  static_assert(ROOM >= SEG, "one piece of every segment fits");
  piece_t v[kMine];

  // Pieces past the end of x (ragged tiles) read zero.
  __device__ __forceinline__ void fetch(rsrc_t rx, int tid) {
#pragma unroll
    for (int t = 0; t < kMine; ++t) {
      const uint32_t i = static_cast<uint32_t>(tid + t * NT);
      const uint32_t off = i < static_cast<uint32_t>(kPieces) ? (i % SEG) * (16u * PER) + 16u * (i / SEG) : kOOB;
      v[t] = __builtin_bit_cast(piece_t, __builtin_amdgcn_raw_buffer_load_b128(rx, off, 0, 0));
    }
  }

  // All threads call; segment j's activations into xr (PER pieces in order) where `take`.
  template <int A, int B>
  __device__ __forceinline__ void share(piece_t* buf, int tid, int j, bool take, uint32_t (&xr)[A][B]) const {
    static_assert(A * B == 4 * PER, "activations of a segment");
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
#pragma unroll
      for (int t = 0; t < kMine; ++t) {
        const int i = tid + t * NT - r * kAtOnce * SEG;
        if (i >= 0 && i < kAtOnce * SEG && i < kPieces - r * kAtOnce * SEG) buf[i] = v[t];
      }
      __syncthreads();
      if (take) {
#pragma unroll
        for (int d = 0; d < kAtOnce; ++d) {
          const int p = r * kAtOnce + d;
          if (p < PER) {
            const piece_t q = buf[d * SEG + j];
#pragma unroll
            for (int i = 0; i < 4; ++i) xr[(4 * p + i) / B][(4 * p + i) % B] = q[i];
          }
        }
      }
      __syncthreads();
    }
  }
};

}  // namespace bitcos_dev
