// Out-of-bag error on gfx950 (the tuning objective of Sec. III-B and Sec. III-C).
//
// Every training row of a forest is predicted by the trees whose bootstrap
// sample left it out (the in-bag bitmaps written by the fit), as an exact int64
// sum of leaf values and a tree count; its out-of-bag prediction is then
// (sum * 2^-32) / count, like the forest mean.  The squared and absolute errors
// are reduced per forest in a fixed order (wave butterflies, then workgroups in
// index order), so the result does not depend on scheduling.
#include "device.h"
#include "internal.h"
#include "traverse.h"

namespace aiwc {
namespace {

constexpr int kOobBlock = 256;

// Leaf sums and tree counts of a forest's rows: its training rows, each under
// the trees that left it out (OOB), or its held-out rows under every tree.
// A workgroup takes R rows of a forest and a chunk of its trees: the rows' codes
// and their running sums lie in the LDS, and each wave takes trees of its own, or
// `split` waves (a power of two) each tree, a part of the rows each.
// It lists the rows that the tree left out (a bitmap word per 64 rows), so that
// every lane walks a row of it, K rows per lane at a time, with the tree's first
// nodes in the wave's part of the LDS.  One thread per row and forest walking
// every tree in turn, codes and nodes gathered from memory, took 11.7 ms for 2000
// trees on 2220 rows (nine workgroups) and 19.5 ms for the tuning grid's 1700
// forests; now 0.06 and 7.2 ms, bound by the latency of the walk's dependent reads
// (128 nodes per tree in the LDS; 256 and 512 cost waves: 1.2 and 1.6 times as long).
constexpr int kScoreWaves = 8;
constexpr uint32_t kScoreTop = 128;

template <bool OOB>
__global__ __launch_bounds__(kScoreWaves* kWave) void k_score(
    const uint64_t* __restrict__ nodes, const TreeTask* __restrict__ tasks, const int64_t* __restrict__ node_base,
    const int32_t* __restrict__ n_nodes, const uint64_t* __restrict__ inbag, const int32_t* __restrict__ row_list,
    const OobForest* __restrict__ forests, const uint8_t* __restrict__ codes, int32_t C, int32_t R, int32_t n_chunks,
    int32_t split, unsigned long long* __restrict__ sum, int32_t* __restrict__ count) {
  extern __shared__ __align__(16) uint8_t lds[];
  constexpr int BLOCK = kScoreWaves * kWave, K = 2;
  const OobForest F = forests[blockIdx.y];
  const int32_t r0 = (int32_t)blockIdx.x * R;
  const int32_t nr = min(R, F.n_train - r0);
  const int32_t chunk = (F.num_trees + n_chunks - 1) / n_chunks;
  const int32_t t0 = (int32_t)blockIdx.z * chunk, t1 = min(F.num_trees, t0 + chunk);
  if (nr <= 0 || (t0 >= t1 && t0 > 0)) return;
  const int tid = (int)threadIdx.x, wid = tid / kWave, lane = (int)lane_id();
  const uint32_t st = (uint32_t)staged_stride(C);
  uint64_t* s_sum = reinterpret_cast<uint64_t*>(lds);                       // [R]
  uint64_t* top = s_sum + R + (size_t)wid * kScoreTop;                          // [kScoreTop] of each wave
  uint32_t* s_cnt = reinterpret_cast<uint32_t*>(s_sum + R + (size_t)kScoreWaves * kScoreTop);  // [R]
  uint16_t* list = reinterpret_cast<uint16_t*>(s_cnt + R) + (size_t)wid * (OOB ? R : 0);
  uint8_t* rows = reinterpret_cast<uint8_t*>(s_cnt + R) + (OOB ? (size_t)2 * kScoreWaves * R : 0);
  stage_rows<BLOCK>(rows, codes, C, F.train_off >= 0 ? row_list + F.train_off : nullptr, r0, nr);
  for (int i = tid; i < nr; i += BLOCK) {
    s_sum[i] = 0;
    s_cnt[i] = 0;
  }
  __syncthreads();
  // bitmap words of these rows (at most 64), and this wave's part of them
  const int nw = (nr + kWave - 1) / kWave, per = (nw + split - 1) / split;
  const int w0 = min(nw, wid % split * per), w1 = min(nw, w0 + per);
  for (int32_t t = t0 + wid / split; t < t1; t += kScoreWaves / split) {
    const int64_t task = F.first_task + t;
    uint32_t n_rows = (uint32_t)max(0, min(nr, kWave * w1) - kWave * w0);
    if constexpr (OOB) {
      const int64_t bits = tasks[task].inbag_off;
      if (bits < 0) continue;  // no bootstrap: every row is in bag
      const uint64_t word = lane < nw ? inbag[bits + r0 / kWave + lane] : ~0ull;
      n_rows = 0;
      for (int i = w0; i < w1; ++i) {
        uint64_t out = ~read_lane(word, i);
        if (64 * i + 64 > nr) out &= ~0ull >> (64 * i + 64 - nr);
        if ((out >> lane) & 1ull) list[n_rows + (uint32_t)__popcll(out & ((1ull << lane) - 1ull))] = (uint16_t)(64 * i + lane);
        n_rows += (uint32_t)__popcll(out);
      }
    }
    const uint64_t* tn = nodes + node_base[task];
    const uint32_t nn = min((uint32_t)n_nodes[task], kScoreTop);
    for (uint32_t i = lane; i < nn; i += kWave) top[i] = tn[i];
    wave_lds_sync();
    for (uint32_t j0 = 0; j0 < n_rows; j0 += K * kWave) {
      uint32_t row[K], off[K];
      bool on[K];
      uint64_t v[K];
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const uint32_t j = j0 + (uint32_t)(k * kWave + lane);
        on[k] = j < n_rows;
        row[k] = on[k] ? (OOB ? list[j] : (uint32_t)(kWave * w0) + j) : 0u;
        off[k] = row[k] * st;
      }
      const uint64_t* const tops[K] = {top, top};
      const uint64_t* const trees[K] = {tn, tn};
      walk_trees<K>(tops, kScoreTop, trees, rows, off, on, v);
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (on[k]) {
          atomicAdd((unsigned long long*)&s_sum[row[k]], (unsigned long long)node_q(v[k]));
          if (OOB) atomicAdd(&s_cnt[row[k]], 1u);
        }
    }
    wave_lds_sync();
  }
  __syncthreads();
  for (int i = tid; i < nr; i += BLOCK) {
    const int64_t o = F.row_off + r0 + i;
    if (n_chunks > 1) {
      atomicAdd(&sum[o], (unsigned long long)s_sum[i]);
      if (OOB) atomicAdd(&count[o], (int32_t)s_cnt[i]);
    } else {
      sum[o] = s_sum[i];
      if (OOB) count[o] = (int32_t)s_cnt[i];
    }
    // a held-out prediction is the forest mean: every tree counts
    if (!OOB && t0 == 0) count[o] = F.num_trees;
  }
}

__global__ void k_zero_scores(unsigned long long* sum, int32_t* count, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    sum[i] = 0ull;
    if (count) count[i] = 0;
  }
}

// Per workgroup: sums of squared error, absolute error and rows with a
// prediction (count > 0).
__global__ __launch_bounds__(kOobBlock) void k_oob_partial(const int64_t* __restrict__ sum,
                                                           const int32_t* __restrict__ count,
                                                           const int32_t* __restrict__ train_rows,
                                                           const OobForest* __restrict__ forests,
                                                           const double* __restrict__ y, double* __restrict__ partial) {
  __shared__ double s_sq[kOobBlock / kWave], s_ab[kOobBlock / kWave], s_m[kOobBlock / kWave];
  const OobForest F = forests[blockIdx.y];
  const int64_t i = (int64_t)blockIdx.x * kOobBlock + threadIdx.x;
  double sq = 0.0, ab = 0.0, m = 0.0;
  if (i < F.n_train) {
    const int32_t c = count[F.row_off + i];
    if (c > 0) {
      const int64_t row = F.train_off >= 0 ? train_rows[F.train_off + i] : i;
      const double pred = ((double)sum[F.row_off + i] * 0x1p-32) / (double)c;
      const double e = pred - y[row];
      sq = e * e;
      ab = fabs(e);
      m = 1.0;
    }
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    sq += __shfl_xor(sq, d, kWave);
    ab += __shfl_xor(ab, d, kWave);
    m += __shfl_xor(m, d, kWave);
  }
  const int wid = threadIdx.x / kWave;
  if (lane_id() == 0) {
    s_sq[wid] = sq;
    s_ab[wid] = ab;
    s_m[wid] = m;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double a = 0.0, b = 0.0, c = 0.0;
    for (int w = 0; w < kOobBlock / kWave; ++w) {
      a += s_sq[w];
      b += s_ab[w];
      c += s_m[w];
    }
    double* out = partial + 3 * ((int64_t)blockIdx.y * gridDim.x + blockIdx.x);
    out[0] = a;
    out[1] = b;
    out[2] = c;
  }
}

// Per forest: mean squared error, mean absolute error, rows counted.
__global__ void k_oob_final(const double* partial, int32_t n_forests, int32_t blocks, double* result) {
  const int32_t f = blockIdx.x * blockDim.x + threadIdx.x;
  if (f >= n_forests) return;
  double a = 0.0, b = 0.0, c = 0.0;
  for (int32_t k = 0; k < blocks; ++k) {
    const double* p = partial + 3 * ((int64_t)f * blocks + k);
    a += p[0];
    b += p[1];
    c += p[2];
  }
  result[3 * f + 0] = c > 0.0 ? a / c : 0.0;
  result[3 * f + 1] = c > 0.0 ? b / c : 0.0;
  result[3 * f + 2] = c;
}

void launch_errors(const int32_t* row_list, const OobForest* forests, int32_t n_forests, int32_t max_n,
                   const double* y, const int64_t* sum, const int32_t* count, double* partial, double* result,
                   hipStream_t s) {
  const int32_t blocks = std::max(1, (max_n + kOobBlock - 1) / kOobBlock);
  k_oob_partial<<<dim3((unsigned)blocks, (unsigned)n_forests), kOobBlock, 0, s>>>(sum, count, row_list, forests, y,
                                                                               partial);
  AIWC_HIP(hipGetLastError());
  k_oob_final<<<(n_forests + 255) / 256, 256, 0, s>>>(partial, n_forests, blocks, result);
  AIWC_HIP(hipGetLastError());
}

// Launch of k_score over `total` rows of n_forests forests, the largest of max_n
// rows and max_trees trees.
template <bool OOB>
void launch_score(const TreesView& T, const TreeTask* tasks, const uint64_t* inbag, const int32_t* row_list,
                  const OobForest* forests, int32_t n_forests, int32_t max_n, int32_t max_trees, int64_t total,
                  const uint8_t* codes, int32_t C, int64_t* sum, int32_t* count, hipStream_t s) {
  const ScoreShape S = score_shape(OOB, n_forests, max_n, max_trees, C, device_info().cus, device_info().lds_per_block);
  const int32_t n_chunks = S.chunks;
  if (n_chunks > 1) {
    const int zb = (int)std::max<int64_t>(1, std::min<int64_t>(1024, (total + 255) / 256));
    k_zero_scores<<<zb, 256, 0, s>>>(reinterpret_cast<unsigned long long*>(sum), OOB ? count : nullptr, total);
    AIWC_HIP(hipGetLastError());
  }
  k_score<OOB><<<dim3((unsigned)S.row_blocks, (unsigned)n_forests, (unsigned)n_chunks), kScoreWaves * kWave, S.lds, s>>>(
      T.nodes, tasks, T.node_base, T.n_nodes, inbag, row_list, forests, codes, C, S.rows, n_chunks, S.split,
      reinterpret_cast<unsigned long long*>(sum), count);
  AIWC_HIP(hipGetLastError());
}
}  // namespace

// A wave walks its rows 128 at a time (two per lane): a workgroup takes 128 held-out
// rows, or 512 training rows, of which a tree left a third out (the tuning grid's
// out-of-bag scores, the whole call: 6.8 ms with 512 rows, 7.9 with 256, 8.4 with 1024).  Waves
// that would have no tree of their own share one: eight waves a single tree's rows,
// four the rows of two.  And while the launch has less than eight waves per CU
// with a tree to walk, a workgroup takes half the rows.  Always 512 rows and a wave
// per tree left most of the chip idle for few trees (the whole call: 10000 held-out
// rows x 1 tree 111 us, so 77; x 40 trees 118 and 88; 100000 x 1 154 and 121; 100000
// x 16 241 and 196; out of bag 10000 x 1 92 and 77).
// More chunks of the trees fill the CUs when forests and row blocks do not.
ScoreShape score_shape(bool oob, int64_t n_forests, int64_t max_n, int64_t max_trees, int32_t C, int64_t cus,
                       size_t lds_per_block) {
  ScoreShape S;
  const int64_t row_bytes = staged_stride(C) + 12 + (oob ? 2 * kScoreWaves : 0), tops = (int64_t)kScoreWaves * kScoreTop * 8;
  // at most a third of the LDS, so that three workgroups (24 waves) fit a CU
  const int64_t room = ((int64_t)lds_per_block / 3 - tops) / row_bytes / kWave * kWave;
  S.split = 1;
  while (S.split < kScoreWaves && 2 * S.split * max_trees <= kScoreWaves) S.split *= 2;
  int64_t most = std::min<int64_t>(oob ? 512 : std::min(512, 128 * S.split), room);
  while (most > kWave && (max_n + most - 1) / most * n_forests * max_trees * S.split < 8 * cus)
    most = (most / 2 + kWave - 1) / kWave * kWave;
  while (S.split * kWave > most) S.split /= 2;
  const int64_t n_rb = (max_n + most - 1) / most;
  const int64_t R = ((max_n + n_rb - 1) / n_rb + kWave - 1) / kWave * kWave;
  S.rows = (int32_t)R;
  S.row_blocks = (int32_t)n_rb;
  S.lds = (size_t)(R * row_bytes + tops);
  const int64_t per_cu = std::max<int64_t>(1, std::min<int64_t>(32 / kScoreWaves, (int64_t)(lds_per_block / S.lds)));
  const int64_t slots = per_cu * cus, wgs = n_rb * n_forests;
  int64_t n_chunks = std::min<int64_t>((2 * slots + wgs - 1) / wgs, (max_trees + kScoreWaves - 1) / kScoreWaves);
  S.chunks = (int32_t)std::max<int64_t>(1, n_chunks);
  return S;
}

void launch_oob(const TreesView& T, const TreeTask* tasks, const uint64_t* inbag, const int32_t* train_rows,
                const OobForest* forests, int32_t n_forests, int32_t max_n_train, int32_t max_trees, int64_t total,
                const uint8_t* codes, int32_t C, const double* y, int64_t* sum, int32_t* count, double* partial,
                double* result, hipStream_t s) {
  launch_score<true>(T, tasks, inbag, train_rows, forests, n_forests, max_n_train, max_trees, total, codes, C, sum,
                     count, s);
  launch_errors(train_rows, forests, n_forests, max_n_train, y, sum, count, partial, result, s);
}

void launch_heldout(const TreesView& T, const int32_t* test_rows, const OobForest* forests, int32_t n_forests,
                    int32_t max_n_test, int32_t max_trees, int64_t total, const uint8_t* codes, int32_t C,
                    const double* y, int64_t* sum, int32_t* count, double* partial, double* result, hipStream_t s) {
  launch_score<false>(T, nullptr, nullptr, test_rows, forests, n_forests, max_n_test, max_trees, total, codes, C, sum,
                      count, s);
  launch_errors(test_rows, forests, n_forests, max_n_test, y, sum, count, partial, result, s);
}

}  // namespace aiwc
