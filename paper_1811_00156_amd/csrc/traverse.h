// Tree traversal building blocks shared by prediction (predict.hip) and the
// out-of-bag and held-out scoring (oob.hip): a workgroup's rows staged in the
// LDS, and the walk of a tree whose first nodes are in the LDS.
#pragma once

#include "device.h"
#include "internal.h"

namespace aiwc {

// LDS bytes between staged rows: an odd number of 4-byte words, so that lanes
// reading one column of consecutive rows hit 64 different banks.
__host__ __device__ inline int32_t staged_stride(int32_t C) {
  const int32_t w = (C + 3) / 4;
  return 4 * (w | 1);
}

// Copies nr rows of C codes into dst (staged_stride(C) bytes apart): rows
// r0 .. r0 + nr of the matrix, or those named by list[r0 .. r0 + nr).  The
// bytes are read in their order in memory (4 at a time when the first row is
// 4-byte aligned, which a caller's slice need not be), not row by row per lane:
// 65-byte rows read one per lane touch a cache line per lane and load.  Eight
// loads are in flight per thread (4096 rows x 64 columns, 500 trees: 70 us, 79 with
// one).
// (nr * C < 2^24 and C <= 255, so the reciprocal below divides exactly.)
template <int BLOCK>
__device__ __forceinline__ void stage_rows(uint8_t* dst, const uint8_t* __restrict__ codes, int32_t C,
                                           const int32_t* __restrict__ list, int64_t r0, int32_t nr) {
  const uint32_t total = (uint32_t)nr * (uint32_t)C;
  const uint32_t inv = C > 1 ? (uint32_t)(0x100000000ull / (uint32_t)C) + 1u : 0u;
  const uint32_t st = (uint32_t)staged_stride(C);
  const uint8_t* src = codes + r0 * C;
  constexpr uint32_t U = 8;
  uint32_t bytes = 0;  // those copied four at a time
  if (!list && (reinterpret_cast<uintptr_t>(src) & 3u) == 0) {
    bytes = total & ~3u;
    for (uint32_t f0 = 4u * threadIdx.x; f0 < bytes; f0 += 4u * BLOCK * U) {
      uint32_t w[U];
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t f = f0 + 4u * BLOCK * u;
        w[u] = f < bytes ? *reinterpret_cast<const uint32_t*>(src + f) : 0u;
      }
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t f = f0 + 4u * BLOCK * u;
        if (f >= bytes) break;
        uint32_t row = C > 1 ? __umulhi(f, inv) : f;
        uint32_t col = f - row * (uint32_t)C;
#pragma unroll
        for (uint32_t b = 0; b < 4u; ++b) {
          dst[row * st + col] = (uint8_t)(w[u] >> (8 * b));
          if (++col == (uint32_t)C) {
            col = 0;
            ++row;
          }
        }
      }
    }
  }
  for (uint32_t f0 = bytes + threadIdx.x; f0 < total; f0 += BLOCK * U) {
    uint8_t v[U];
    uint32_t at[U];
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      const uint32_t f = f0 + BLOCK * u;
      const uint32_t row = C > 1 ? __umulhi(f, inv) : f;
      const uint32_t col = f - row * (uint32_t)C;
      at[u] = row * st + col;
      v[u] = f >= total ? 0 : list ? codes[(int64_t)list[r0 + row] * C + col] : src[f];
    }
#pragma unroll
    for (uint32_t u = 0; u < U; ++u)
      if (f0 + BLOCK * u < total) dst[at[u]] = v[u];
  }
}

// The leaf words that K walks reach: row k's staged codes at rows + off[k], down
// the tree whose nodes are tn[k] in global memory and whose first m (breadth
// first, so its upper levels) are at top[k] in the LDS; a walk whose `on` is false
// gets a leaf of value 0.  The walks are interleaved, so that their dependent
// reads overlap: first through the LDS part, then, for those that left it,
// through the rest.
template <int K>
__device__ __forceinline__ void walk_trees(const uint64_t* const (&top)[K], uint32_t m, const uint64_t* const (&tn)[K],
                                           const uint8_t* rows, const uint32_t (&off)[K], const bool (&on)[K],
                                           uint64_t (&v)[K]) {
  constexpr uint64_t kNoLeaf = (uint64_t)kLeafCol;  // a leaf of value 0
  uint32_t nx[K];
  bool open = false, deep = false;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    v[k] = on[k] ? top[k][0] : kNoLeaf;
    nx[k] = 0;
    open |= node_col(v[k]) != kLeafCol;
  }
  while (open) {
    open = false;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const uint32_t c = node_col(v[k]);
      if (c != kLeafCol) {
        const uint32_t next = node_left(v[k]) + (rows[off[k] + c] > node_bin(v[k]) ? 1u : 0u);
        if (next < m) {
          v[k] = top[k][next];
          open = true;
        } else {
          v[k] = kNoLeaf;
          nx[k] = next;
          deep = true;
        }
      }
    }
  }
  if (!deep) return;
#pragma unroll
  for (int k = 0; k < K; ++k)
    if (nx[k]) v[k] = tn[k][nx[k]];
  while (deep) {
    deep = false;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const uint32_t c = node_col(v[k]);
      if (c != kLeafCol) {
        v[k] = tn[k][node_left(v[k]) + (rows[off[k] + c] > node_bin(v[k]) ? 1u : 0u)];
        deep = true;
      }
    }
  }
}

}  // namespace aiwc
