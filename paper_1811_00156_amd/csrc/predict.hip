// Batched prediction by tree traversal on gfx950.
//
// A row goes left where its code in the node's column is <= the node's bin, else
// right; the leaf values of its trees add up as exact int64.  Many rows: a
// workgroup per (row block, tree chunk), rows and the trees' upper levels in
// the LDS; partial sums of different chunks meet in a 64-bit integer atomic
// add, which is exact in any order.  Fewer: a row per thread with codes and nodes
// where they are, lanes of a row, or workgroups of a row (predict_route).
#include <map>
#include <mutex>

#include "device.h"
#include "internal.h"
#include "traverse.h"

namespace aiwc {
namespace {

// The per-row int64 sums of the allocation-free prediction entry point live in
// this fixed array, one copy per GPU, held until the process ends.  Host code
// never uses its name as an address: the address of each device's copy comes
// from hipGetSymbolAddress (noalloc_predict_scratch).
__device__ __align__(256) unsigned long long scratch[kNoAllocPredictRows];

// Prediction of many rows.  A workgroup stages its rows' codes in the LDS (one
// row per thread) and walks its chunk of trees one after the other; each tree's
// first TP * kPredBlock nodes are staged too, G trees at a time, fetched into
// registers while the previous ones are walked.  Below them a row's reads scatter over the tree, one
// cache line each: with one tree at a time, and the chunks of an XCD taken in
// turn by all of its workgroups, an XCD's L2 holds the trees in use.  Before,
// codes and nodes were both gathered from memory (200000 rows x 65 columns, 500
// trees of 200000 rows: 9.7 ms, the address unit 84 % busy and 5.1e8 cache lines
// missing the L2); now 1.9 to 2.0 ms, bound by the latency of the dependent reads, so
// that workgroups are small (256 threads waited less at the barriers than 512 or
// 1024: 1.9, 2.3 and 2.5 ms) and one row per thread with up to 32 waves per CU
// beats two or four rows with fewer waves (2.9 and 4.3 ms).
constexpr int kPredBlock = 256;

template <int TP, int G>
__global__ __launch_bounds__(kPredBlock) void k_traverse(TreesView F, int32_t tree_begin, int32_t tree_end,
                                                         int32_t chunk, int32_t n_chunks, int32_t n_rb, int32_t R,
                                                         const uint8_t* __restrict__ codes, int64_t n, int32_t C,
                                                         unsigned long long* __restrict__ sum, double* __restrict__ y,
                                                         double trees, int accumulate) {
  extern __shared__ __align__(16) uint8_t lds[];
  constexpr uint32_t M = TP * kPredBlock;
  uint64_t* top = reinterpret_cast<uint64_t*>(lds);
  uint8_t* rows = lds + 8 * M * G;
  // workgroup b runs on XCD b % 8: with n_chunks a multiple of 8 an XCD's
  // workgroups take the row blocks of one chunk, then those of its next one
  const int32_t b = (int32_t)blockIdx.x;
  int32_t ci, rb;
  if (n_chunks % 8 == 0) {
    ci = (b / 8) / n_rb * 8 + b % 8;
    rb = (b / 8) % n_rb;
  } else {
    ci = b % n_chunks;
    rb = b / n_chunks;
  }
  const int64_t r0 = (int64_t)rb * R;
  const int32_t nr = (int32_t)min((int64_t)R, n - r0);
  const int32_t t0 = tree_begin + ci * chunk;
  const int32_t t1 = min(tree_end, t0 + chunk);
  if (nr <= 0 || t0 >= t1) return;
  const uint32_t tid = threadIdx.x;
  uint64_t pf[G][TP];
  auto fetch = [&](int32_t t) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const bool in = t + g < t1;
      const uint64_t* tn = F.nodes + (in ? F.node_base[t + g] : 0);
      const uint32_t nn = in ? min((uint32_t)F.n_nodes[t + g], M) : 0u;
#pragma unroll
      for (int u = 0; u < TP; ++u) pf[g][u] = tid + u * kPredBlock < nn ? tn[tid + u * kPredBlock] : 0ull;
    }
  };
  fetch(t0);
  stage_rows<kPredBlock>(rows, codes, C, nullptr, r0, nr);
  const bool in_row = (int32_t)tid < nr;
  const uint32_t ro = tid * (uint32_t)staged_stride(C);
  int64_t acc = 0;
  for (int32_t t = t0; t < t1; t += G) {
    __syncthreads();  // the previous trees are walked (and, at first, the rows are staged)
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int u = 0; u < TP; ++u) top[g * M + tid + u * kPredBlock] = pf[g][u];
    __syncthreads();
    if (t + G < t1) fetch(t + G);
    uint64_t v[G];
    bool on[G];
    uint32_t off[G];
    const uint64_t* tops[G];
    const uint64_t* tn[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      on[g] = in_row && t + g < t1;
      off[g] = ro;
      tops[g] = top + g * M;
      tn[g] = F.nodes + (t + g < t1 ? F.node_base[t + g] : 0);
    }
    walk_trees<G>(tops, M, tn, rows, off, on, v);
#pragma unroll
    for (int g = 0; g < G; ++g) acc += node_q(v[g]);
  }
  if (!in_row) return;
  const int64_t r = r0 + tid;
  if (accumulate) {
    atomicAdd(&sum[r], (unsigned long long)acc);
  } else {
    if (sum) sum[r] = (unsigned long long)acc;
    if (y) y[r] = ((double)acc * 0x1p-32) / trees;
  }
}

// Prediction of few rows: one workgroup per row, a tree per thread, the whole
// answer in one launch.  Both children of a node are adjacent, so they are
// fetched together as soon as the node is known, while its column's code is
// looked up: a level costs one memory latency.  With D > 0 the rows are the
// (kernel, device) pairs of a device selection: row r has kernel r / D's C - 1
// feature codes and the device code r % D.  A thread walks K trees at a time; when
// gridDim.y workgroups share a row its trees are dealt out among them, and their
// sums meet in sum[r], which starts at 0.
constexpr int kRowBlock = 512;
struct alignas(8) NodePair {
  uint64_t l, r;
};

template <int K>
__global__ __launch_bounds__(kRowBlock) void k_traverse_row(TreesView F, int32_t tree_begin, int32_t tree_end,
                                                            const uint8_t* __restrict__ codes, int32_t C, int32_t D,
                                                            unsigned long long* __restrict__ sum,
                                                            double* __restrict__ y, double trees) {
  __shared__ uint8_t row[256];
  __shared__ int64_t part[kRowBlock / kWave];
  const int64_t r = blockIdx.x;
  const int32_t tid = (int32_t)threadIdx.x;
  int64_t acc = 0;
  const uint64_t* tn[K];
  uint64_t v[K];
  auto open_trees = [&](int32_t t) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const bool in = t + k * kRowBlock < tree_end;
      tn[k] = F.nodes + (in ? F.node_base[t + k * kRowBlock] : 0);
      v[k] = in ? tn[k][0] : (uint64_t)kLeafCol;
    }
  };
  int32_t t = tree_begin + (int32_t)blockIdx.y * (K * kRowBlock) + tid;
  open_trees(t);
  if (tid < C) {
    if (D > 0)
      row[tid] = tid < C - 1 ? codes[r / D * (C - 1) + tid] : (uint8_t)(r % D);
    else
      row[tid] = codes[r * C + tid];
  }
  __syncthreads();
  while (t < tree_end) {
    bool open = true;
    while (open) {
      open = false;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const uint32_t c = node_col(v[k]);
        if (c != kLeafCol) {
          const NodePair p = *reinterpret_cast<const NodePair*>(tn[k] + node_left(v[k]));
          v[k] = row[c] > node_bin(v[k]) ? p.r : p.l;
          open = true;
        }
      }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) acc += node_q(v[k]);
    t += K * kRowBlock * (int32_t)gridDim.y;
    open_trees(t);
  }
  acc = (int64_t)wave_sum((uint64_t)acc);
  if (lane_id() == 0) part[tid / kWave] = acc;
  __syncthreads();
  if (tid == 0) {
    int64_t s = 0;
    for (int w = 0; w < kRowBlock / kWave; ++w) s += part[w];
    if (gridDim.y > 1) {
      atomicAdd(&sum[r], (unsigned long long)s);
    } else {
      if (sum) sum[r] = (unsigned long long)s;
      if (y) y[r] = ((double)s * 0x1p-32) / trees;
    }
  }
}

// Prediction in between: 2^lg lanes per row, each with every 2^lg-th tree, codes and
// nodes where they are, the whole answer in one launch.
__global__ __launch_bounds__(kPredBlock) void k_traverse_lanes(TreesView F, int32_t tree_begin, int32_t tree_end,
                                                               int32_t lg, const uint8_t* __restrict__ codes,
                                                               int64_t n, int32_t C,
                                                               unsigned long long* __restrict__ sum,
                                                               double* __restrict__ y, double trees) {
  const int64_t g = (int64_t)blockIdx.x * kPredBlock + threadIdx.x;
  const int64_t r = g >> lg;
  const int32_t slot = (int32_t)(g & ((1 << lg) - 1)), step = 1 << lg;
  const uint8_t* row = codes + min(r, n - 1) * C;
  constexpr int K = 2;
  int64_t acc = 0;
  for (int32_t t = tree_begin + slot; t < tree_end; t += K * step) {
    const uint64_t* tn[K];
    uint64_t v[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const bool in = t + k * step < tree_end;
      tn[k] = F.nodes + (in ? F.node_base[t + k * step] : 0);
      v[k] = in ? tn[k][0] : (uint64_t)kLeafCol;
    }
    bool open = true;
    while (open) {
      open = false;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const uint32_t c = node_col(v[k]);
        if (c != kLeafCol) {
          const NodePair p = *reinterpret_cast<const NodePair*>(tn[k] + node_left(v[k]));
          v[k] = row[c] > node_bin(v[k]) ? p.r : p.l;
          open = true;
        }
      }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) acc += node_q(v[k]);
  }
  for (int d = step >> 1; d >= 1; d >>= 1) acc += __shfl_xor((long long)acc, d, kWave);
  if (slot == 0 && r < n) {
    if (sum) sum[r] = (unsigned long long)acc;
    if (y) y[r] = ((double)acc * 0x1p-32) / trees;
  }
}

// Prediction of some rows by trees that are small, or too few pairs of rows and trees
// to pay for staging: a row per thread and a chunk of the trees per workgroup, codes
// and nodes where they are, two trees at a time.  (700 rows x 1100 trees of 34 leaves:
// 23 us, 35 with the rows and upper levels staged; 8000 x 122 of 75: 25 and 29.)
__global__ __launch_bounds__(kPredBlock) void k_traverse_direct(TreesView F, int32_t tree_begin, int32_t tree_end,
                                                                int32_t chunk, int32_t n_chunks,
                                                                const uint8_t* __restrict__ codes, int64_t n,
                                                                int32_t C, unsigned long long* __restrict__ sum,
                                                                double* __restrict__ y, double trees) {
  const int32_t t0 = tree_begin + (int32_t)(blockIdx.x % (unsigned)n_chunks) * chunk, t1 = min(tree_end, t0 + chunk);
  const int64_t r = (int64_t)(blockIdx.x / (unsigned)n_chunks) * kPredBlock + threadIdx.x;
  if (r >= n || t0 >= t1) return;
  const uint8_t* row = codes + r * C;
  constexpr int K = 2;
  int64_t acc = 0;
  for (int32_t t = t0; t < t1; t += K) {
    const uint64_t* tn[K];
    uint64_t v[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const bool in = t + k < t1;
      tn[k] = F.nodes + (in ? F.node_base[t + k] : 0);
      v[k] = in ? tn[k][0] : (uint64_t)kLeafCol;
    }
    bool open = true;
    while (open) {
      open = false;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const uint32_t c = node_col(v[k]);
        if (c != kLeafCol) {
          const NodePair p = *reinterpret_cast<const NodePair*>(tn[k] + node_left(v[k]));
          v[k] = row[c] > node_bin(v[k]) ? p.r : p.l;
          open = true;
        }
      }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) acc += node_q(v[k]);
  }
  if (n_chunks > 1) {
    atomicAdd(&sum[r], (unsigned long long)acc);
  } else {
    if (sum) sum[r] = (unsigned long long)acc;
    if (y) y[r] = ((double)acc * 0x1p-32) / trees;
  }
}

__global__ void k_zero_i64(unsigned long long* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0ull;
}

// yhat = (P * 2^-32) / num.trees: an exact scaling then one rounded division.
__global__ void k_finalize(const int64_t* sum, int64_t n, double trees, double* y) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    y[i] = ((double)sum[i] * 0x1p-32) / trees;
}

// Row i * D + d of the expanded matrix = kernel i's feature codes + device d.
__global__ void k_expand_devices(const uint8_t* feat, int64_t m, int32_t C, int32_t D, uint8_t* out) {
  const int64_t total = m * D * C;
  for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < total; g += (int64_t)gridDim.x * blockDim.x) {
    const int64_t row = g / C;
    const int32_t j = (int32_t)(g % C);
    const int64_t i = row / D;
    out[g] = j < C - 1 ? feat[i * (C - 1) + j] : (uint8_t)(row % D);
  }
}

// Fastest device per kernel: the smallest predicted time, the lowest id on ties.
__global__ void k_argmin_devices(const double* times, int64_t m, int32_t D, int32_t* best) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x) {
    const double* t = times + i * D;
    int32_t b = 0;
    for (int32_t d = 1; d < D; ++d)
      if (t[d] < t[b]) b = d;
    best[i] = b;
  }
}

// Sec. VI's scheduler criterion, one thread per kernel: for every device pair
// i < j the predicted choice is i when times[i] <= times[j] (lowest id on a
// tie), else j; it is right when the chosen device's true time is strictly the
// smaller.  Pairs with equal true times are not counted.  The fastest device is
// hit when the predicted best (smallest prediction, lowest id on ties) has the
// smallest true time.  Only comparisons: exact.
__global__ void k_rank_accuracy(const double* times, const double* truth, int64_t m, int32_t D, int32_t* correct,
                                int32_t* counted, int32_t* hit) {
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < m; k += (int64_t)gridDim.x * blockDim.x) {
    const double* p = times + k * D;
    const double* t = truth + k * D;
    int32_t c = 0, n = 0, best = 0;
    double tmin = t[0];
    for (int32_t i = 0; i < D; ++i) {
      const double pi = p[i], ti = t[i];
      if (pi < p[best]) best = i;
      tmin = ti < tmin ? ti : tmin;
      for (int32_t j = i + 1; j < D; ++j) {
        const double tj = t[j];
        if (ti == tj) continue;
        ++n;
        const bool pick_i = pi <= p[j];
        c += (pick_i ? ti < tj : tj < ti) ? 1 : 0;
      }
    }
    if (correct) correct[k] = c;
    if (counted) counted[k] = n;
    if (hit) hit[k] = t[best] == tmin ? 1 : 0;
  }
}

}  // namespace

void launch_rank_accuracy(const double* times, const double* truth, int64_t m, int32_t D, int32_t* correct,
                          int32_t* counted, int32_t* hit, hipStream_t s) {
  if (m <= 0) return;
  const int b = (int)std::max<int64_t>(1, std::min<int64_t>(4096, (m + 255) / 256));
  k_rank_accuracy<<<b, 256, 0, s>>>(times, truth, m, D, correct, counted, hit);
  AIWC_HIP(hipGetLastError());
}

// The route by the (row, tree) pairs and the leaves of a tree, from which the reads
// that share no cache line cost more.  One launch instead of three is worth 8 us, so
// few pairs take a workgroup per row, which reads another tree with every lane, or
// lanes of a row; several workgroups per row where it has more trees than one fetches
// soon.  Then a row per thread, which staging beats from the last limit on.  The
// limits are those of the fastest route over 13000 predictions (1 to 200000 rows, 1
// to 2000 trees of 1 to 126000 leaves, 3 to 80 columns).  Limits by the training rows
// alone, calibrated on deep trees and without the row per thread, had left 1 in 14
// behind that kernel, by up to 1.7 times.  For instance (us, by route): 300 trees of
// 75 leaves, 700 rows: a workgroup per row 11, lanes 17, a row per thread 21, staged
// 22; 3000 rows: 37, 25, 26, 26; 8000 rows: 92, 74, 43, 42; of 5000 leaves, 100 rows:
// 15, 53, 22, 24; 1500 rows: 65, 66, 38, 31.
struct RouteLimits {
  int32_t leaves;     // of trees with fewer leaves than this, in units of 1024 pairs:
  int32_t row, row2;  // a workgroup per row up to 1024 rows and 512 trees, and 1024
  int32_t rows;       // the same for up to 4096 rows and 512 trees, counted as 192 at least
  int32_t parts;      // several workgroups per row, more than 512 trees
  int32_t lanes[5];   // lanes of a row up to 32, 64, 128, 320 and 512 trees
  int32_t direct;     // a row per thread
};
constexpr RouteLimits kRouteLimits[] = {
    {1, 512, 512, 1024, 512, {1700, 1700, 1700, 1700, 1700}, INT32_MAX},  // a root alone
    {4, 512, 512, 1024, 512, {1700, 1700, 1700, 1700, 1700}, 16384},
    {16, 512, 704, 1024, 512, {2000, 2000, 2000, 1448, 1024}, 4096},
    {64, 512, 512, 1024, 352, {1200, 1448, 1448, 1024, 512}, 1200},
    {256, 352, 352, 512, 256, {1200, 860, 704, 704, 0}, 1024},
    {1024, 352, 256, 352, 256, {704, 512, 512, 224, 0}, 512},
    {4096, 256, 224, 64, 208, {512, 352, 304, 128, 0}, 256},
    {16384, 128, 0, 64, 128, {512, 208, 64, 0, 0}, 256},
    {65536, 128, 0, 64, 128, {256, 176, 0, 0, 0}, 192},
    {INT32_MAX, 91, 0, 64, 128, {256, 128, 0, 0, 0}, 128}};

PredictRoute predict_route(const TreesView& F, int64_t n, int32_t n_trees, int32_t C, bool sums) {
  const RouteLimits* L = kRouteLimits;
  while (F.leaves >= L->leaves) ++L;
  const int64_t pairs = (n * n_trees + 1023) / 1024;
  // the pairs that one launch of a workgroup per row or lanes is held against: sums
  // alone take two launches otherwise, not three, so it saves half as much (18858 rows
  // x 22 trees of 790 leaves: lanes 23 us, a row per thread 19)
  const int64_t by_row = sums ? 3 * pairs / 2 : pairs, by_lanes = sums ? 2 * pairs : pairs;
  // trees grown on many rows lie far apart in memory, whatever their leaves (66183
  // rows, 1946 leaves, 547 rows x 453 trees: a workgroup per row 35 us, staged 27;
  // 23836 rows, 3575 leaves, 2364 x 92: lanes 28 us, a row per thread 22)
  const bool far = F.train_rows > 8192;
  const int group = n_trees <= 32 ? 0 : n_trees <= 64 ? 1 : n_trees <= 128 ? 2 : n_trees <= 320 ? 3 : 4;
  const bool lanes = n_trees <= 512 && by_lanes <= L->lanes[group] && !(far && group > 1 && F.leaves >= 1024);
  if (n <= 1024) {
    const int32_t row = far ? std::min(L->row, 176) : L->row;
    if (by_row <= (n_trees <= kRowBlock ? row : n_trees <= 2 * kRowBlock ? L->row2 : 0)) return PredictRoute::kRow;
  } else if (lanes) {
    return PredictRoute::kLanes;
  } else if (n <= 4096 && n_trees <= kRowBlock && n * std::max(n_trees, 192) / 1024 <= (sums ? 2 * L->rows / 3 : L->rows)) {
    return PredictRoute::kRow;
  }
  if (n <= 4096 && n_trees > kRowBlock && pairs <= L->parts) return PredictRoute::kRowParts;
  if (lanes) return PredictRoute::kLanes;
  // (wide rows of the smallest trees: staging reads them in order)
  const int wide = F.leaves < 1 || F.leaves >= 16 || C <= 24 ? 0 : C <= 48 ? 1 : 2;
  return pairs <= L->direct >> wide ? PredictRoute::kDirect : PredictRoute::kMany;
}

namespace {
void launch_row(const TreesView& F, int32_t tree_begin, int32_t tree_end, const uint8_t* codes, int64_t n, int32_t C,
                int32_t D, int64_t* sum, double* y, int32_t num_trees, int32_t parts, hipStream_t s) {
  const auto k = parts > 1 ? k_traverse_row<1> : k_traverse_row<2>;
  k<<<dim3((unsigned)n, (unsigned)parts), kRowBlock, 0, s>>>(F, tree_begin, tree_end, codes, C, D,
                                                             reinterpret_cast<unsigned long long*>(sum), y,
                                                             (double)num_trees);
  AIWC_HIP(hipGetLastError());
}

void zero_sums(int64_t* sum, int64_t n, hipStream_t s) {
  const int zb = (int)std::min<int64_t>(1024, (n + 255) / 256);
  k_zero_i64<<<zb, 256, 0, s>>>(reinterpret_cast<unsigned long long*>(sum), n);
  AIWC_HIP(hipGetLastError());
}

void finalize_sums(const int64_t* sum, int64_t n, int32_t num_trees, double* y, hipStream_t s) {
  const int fb = (int)std::min<int64_t>(1024, (n + 255) / 256);
  k_finalize<<<fb, 256, 0, s>>>(sum, n, (double)num_trees, y);
  AIWC_HIP(hipGetLastError());
}
}  // namespace

void launch_select_device(const TreesView& F, int32_t tree_begin, int32_t tree_end, const uint8_t* feature_codes,
                          int64_t m, int32_t C, int32_t n_devices, int32_t num_trees, uint8_t* expanded, int64_t* sum,
                          double* times, int32_t* best, hipStream_t s) {
  const int64_t rows = m * n_devices;
  if (predict_route(F, rows, tree_end - tree_begin, C, false) == PredictRoute::kRow) {
    launch_row(F, tree_begin, tree_end, feature_codes, rows, C, n_devices, nullptr, times, num_trees, 1, s);
  } else {
    const int eb = (int)std::max<int64_t>(1, std::min<int64_t>(4096, (rows * C + 255) / 256));
    k_expand_devices<<<eb, 256, 0, s>>>(feature_codes, m, C, n_devices, expanded);
    AIWC_HIP(hipGetLastError());
    launch_predict(F, tree_begin, tree_end, expanded, rows, C, sum, times, num_trees, s);
  }
  const int ab = (int)std::max<int64_t>(1, std::min<int64_t>(1024, (m + 255) / 256));
  k_argmin_devices<<<ab, 256, 0, s>>>(times, m, n_devices, best);
  AIWC_HIP(hipGetLastError());
}

int64_t* noalloc_predict_scratch() {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = 0;
  AIWC_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) fail(AIWC_RF_EINVAL, "device ordinal beyond the allocation-free table");
  std::lock_guard<std::mutex> g(mu);
  if (!addr[dev]) {
    // this device is current: its own copy of the array, at its own address
    void* p = nullptr;
    AIWC_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    addr[dev] = p;
  }
  return static_cast<int64_t*>(addr[dev]);
}

void allow_lds(const void* kernel) {
  static std::mutex mu;
  static std::map<std::pair<const void*, int>, bool> done;
  int dev = 0;
  AIWC_HIP(hipGetDevice(&dev));
  std::lock_guard<std::mutex> g(mu);
  bool& d = done[{kernel, dev}];
  if (d) return;
  AIWC_HIP(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)device_info().lds_per_block));
  d = true;
}

namespace {

// Launch of k_traverse: the row blocks, and the tree chunks that the CUs get
// through soonest, in times of a tree's walk: a workgroup takes its chunk's trees
// (four walked together about 1.6) and about 1.5 for staging its rows, `slots`
// workgroups run at a time, and more than one chunk costs two more launches and
// an atomic per row and chunk.
template <int TP, int G>
void traverse_many(const TreesView& F, int32_t tree_begin, int32_t tree_end, const uint8_t* codes, int64_t n,
                   int32_t C, int64_t* sum, double* y, int32_t num_trees, hipStream_t s) {
  const int32_t T = tree_end - tree_begin;
  const int64_t n_rb = (n + kPredBlock - 1) / kPredBlock;
  const int32_t R = (int32_t)((n + n_rb - 1) / n_rb);
  const size_t lds = (size_t)8 * TP * G * kPredBlock + (size_t)R * staged_stride(C);
  const int64_t per_cu = std::max<int64_t>(1, std::min<int64_t>(2048 / kPredBlock, (int64_t)(device_info().lds_per_block / lds)));
  const int64_t slots = per_cu * device_info().cus;
  int32_t n_chunks = 1;
  double best = 0.0;
  for (int32_t c = 1; c <= std::min(T, 2048); c += c < 8 ? 1 : 8) {
    const double rounds = (double)((n_rb * c + slots - 1) / slots);
    const int32_t per = (T + c - 1) / c;
    const double walks = G == 1 ? (double)per : 1.6 * (double)((per + G - 1) / G);
    const double t = rounds * (1.5 + walks) + (c > 1 ? 4.0 + 0.004 * c : 0.0);
    if (c == 1 || t < best) {
      best = t;
      n_chunks = c;
    }
  }
  const int32_t chunk = (T + n_chunks - 1) / n_chunks;
  if (n_chunks % 8 != 0) n_chunks = (T + chunk - 1) / chunk;
  const int accumulate = n_chunks > 1 ? 1 : 0;
  if (accumulate) zero_sums(sum, n, s);
  if (lds > 65536) allow_lds(reinterpret_cast<const void*>(k_traverse<TP, G>));
  k_traverse<TP, G><<<(unsigned)(n_rb * n_chunks), kPredBlock, lds, s>>>(
      F, tree_begin, tree_end, chunk, n_chunks, (int32_t)n_rb, R, codes, n, C,
      reinterpret_cast<unsigned long long*>(sum), y, (double)num_trees, accumulate);
  AIWC_HIP(hipGetLastError());
  if (accumulate && y) finalize_sums(sum, n, num_trees, y, s);
}

}  // namespace

void launch_predict(const TreesView& F, int32_t tree_begin, int32_t tree_end, const uint8_t* codes, int64_t n,
                    int32_t C, int64_t* sum, double* y, int32_t num_trees, hipStream_t s) {
  if (n <= 0) return;
  const PredictRoute route = predict_route(F, n, tree_end - tree_begin, C, !y);
  if (route == PredictRoute::kRow) {
    launch_row(F, tree_begin, tree_end, codes, n, C, 0, sum, y, num_trees, 1, s);
    return;
  }
  if (route == PredictRoute::kRowParts) {
    zero_sums(sum, n, s);
    launch_row(F, tree_begin, tree_end, codes, n, C, 0, sum, nullptr, num_trees,
               (tree_end - tree_begin + kRowBlock - 1) / kRowBlock, s);
    if (y) finalize_sums(sum, n, num_trees, y, s);
    return;
  }
  if (route == PredictRoute::kLanes) {
    int32_t lg = 0;
    while (lg < 6 && (1 << lg) < tree_end - tree_begin) ++lg;
    k_traverse_lanes<<<(unsigned)(((n << lg) + kPredBlock - 1) / kPredBlock), kPredBlock, 0, s>>>(
        F, tree_begin, tree_end, lg, codes, n, C, reinterpret_cast<unsigned long long*>(sum), y, (double)num_trees);
    AIWC_HIP(hipGetLastError());
    return;
  }
  if (route == PredictRoute::kDirect) {
    // about four workgroups per CU, the chunks of an XCD's workgroups the same
    const int32_t T = tree_end - tree_begin;
    const int64_t n_rb = (n + kPredBlock - 1) / kPredBlock, target = 4LL * device_info().cus;
    int64_t n_chunks = std::max<int64_t>(1, std::min<int64_t>(T, (target + n_rb - 1) / n_rb));
    if (n_chunks > 1) n_chunks = std::min<int64_t>(T, (n_chunks + 7) / 8 * 8);
    const int32_t chunk = (int32_t)((T + n_chunks - 1) / n_chunks);
    n_chunks = (T + chunk - 1) / chunk;
    if (n_chunks > 1) zero_sums(sum, n, s);
    k_traverse_direct<<<(unsigned)(n_rb * n_chunks), kPredBlock, 0, s>>>(
        F, tree_begin, tree_end, chunk, (int32_t)n_chunks, codes, n, C, reinterpret_cast<unsigned long long*>(sum), y,
        (double)num_trees);
    AIWC_HIP(hipGetLastError());
    if (n_chunks > 1 && y) finalize_sums(sum, n, num_trees, y, s);
    return;
  }
  // 256 or 512 of a tree's nodes in the LDS: the fewer, the more workgroups fit
  // a CU; trees of a training set above 100000 rows outgrow an XCD's L2, where
  // a level less read from it pays (200000 rows predicted by 200 trees of 64000
  // training rows: 650 us with 256 nodes, 718 with 512; of 128000: 874 and 799).
  // Small trees are walked four at a time: a barrier per tree and a short walk
  // leave little to overlap (200000 rows x 250 trees of 300 training rows: 651 us
  // one at a time, 500 four; of 2220 rows 567 and 504; of 30000, which share the
  // L2, 924 and 1141), but for few pairs one at a time leaves more workgroups
  // (3000 rows x 175 trees of 7669 rows 28 us, 34 four; 6000 x 200 of 3500 37 and
  // 41; 6000 x 300 of 2220 46 and 45).
  if (F.train_rows <= 8192 && n * (tree_end - tree_begin) > (int64_t)1 << 20)
    traverse_many<1, 4>(F, tree_begin, tree_end, codes, n, C, sum, y, num_trees, s);
  else if (F.train_rows <= 100000)
    traverse_many<1, 1>(F, tree_begin, tree_end, codes, n, C, sum, y, num_trees, s);
  else
    traverse_many<2, 1>(F, tree_begin, tree_end, codes, n, C, sum, y, num_trees, s);
}

}  // namespace aiwc
