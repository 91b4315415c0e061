// A forest's node arrays for the host, on gfx950: trees [0, n_trees) of a slice,
// each from its own slot of the node pool, unpacked from their node words into
// contiguous arrays (node 0 of tree t at off[t]), so that the host takes each
// array with one copy.  Taking every tree's words and weights with copies of
// their own and unpacking them on the host took 13.7 ms for 500 trees of 2220
// rows, nearly all of it the 1000 copies; now 2.5 ms with the binding.
#include "device.h"
#include "internal.h"

namespace aiwc {
namespace {

__global__ __launch_bounds__(256) void k_unpack(const uint64_t* __restrict__ nodes, const uint32_t* __restrict__ node_N,
                                                const int64_t* __restrict__ node_base, const int64_t* __restrict__ off,
                                                uint8_t* __restrict__ col, uint8_t* __restrict__ bin,
                                                int32_t* __restrict__ left, int64_t* __restrict__ q,
                                                int32_t* __restrict__ N) {
  const int32_t t = (int32_t)blockIdx.x;
  const int64_t o = off[t], cnt = off[t + 1] - o, base = node_base[t];
  for (int64_t i = (int64_t)blockIdx.y * 256 + threadIdx.x; i < cnt; i += (int64_t)gridDim.y * 256) {
    const uint64_t v = nodes[base + i];
    const bool leaf = node_col(v) == kLeafCol;
    if (col) col[o + i] = (uint8_t)node_col(v);
    if (bin) bin[o + i] = leaf ? 0u : (uint8_t)node_bin(v);
    if (left) left[o + i] = leaf ? -1 : (int32_t)node_left(v);
    if (q) q[o + i] = leaf ? node_q(v) : 0;
    if (N) N[o + i] = (int32_t)node_N[base + i];
  }
}

}  // namespace

void launch_unpack(const uint64_t* nodes, const uint32_t* node_N, const int64_t* node_base, const int64_t* off,
                   int32_t n_trees, uint8_t* col, uint8_t* bin, int32_t* left, int64_t* q, int32_t* N, hipStream_t s) {
  // a few workgroups per CU, however few the trees
  const unsigned per_tree = (unsigned)std::max(1, 4 * device_info().cus / n_trees);
  k_unpack<<<dim3((unsigned)n_trees, per_tree), 256, 0, s>>>(nodes, node_N, node_base, off, col, bin, left, q, N);
  AIWC_HIP(hipGetLastError());
}

}  // namespace aiwc
