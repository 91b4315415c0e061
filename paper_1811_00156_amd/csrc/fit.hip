// Forest fitting on gfx950: one workgroup (k_grow) or one wave of a workgroup of
// sixteen (k_grow_teams) grows one tree at a time, level by level, pulling trees
// from a device-side queue until every tree of every forest in the launch is grown.
//
// Per tree (Sec. III-B: a random-forest regression tree with num.trees, mtry and
// min.node.size; the readings of the unspecified steps are listed in the public
// header):
//   1. bootstrap: n_train Philox draws -> multiplicity per training row, then the
//      in-bag rows are packed into 64-bit entries (row, weight, y_fp);
//   2. for each level, one thread per open node applies the leaf rules
//      (min.node.size, purity) and draws the node's mtry candidate columns; the
//      split search over every (candidate column, bin) is then tiered by the
//      node's number of in-bag rows:
//        - small (<= 64 rows): one row per lane in a segment of 4..64 lanes,
//          every candidate column's codes gathered at once, the left sums of
//          each lane's split found from the segment's rows staged in LDS (by matrix
//          instructions in k_grow_teams), the rows of a split placed at once;
//        - large (<= huge limit): one wave per (node, up to four columns), one LDS
//          histogram of packed (N, S) per column and a wave prefix scan over bins;
//        - wide (above a tuned size): the whole workgroup takes a batch of such
//          nodes at once; each row's entry is read once and its codes in all
//          candidate columns are gathered by one thread, into packed (N, S)
//          LDS histograms of every node and candidate column of the batch;
//          one wave per (node, column) then scans;
//      every split maximises S_L^2/N_L + S_R^2/N_R; ties keep the lowest
//      (column, bin);
//   3. split nodes get breadth-first child ids from a workgroup scan, node words
//      are written, and the in-bag entries are partitioned into the children's
//      segments of the other entry buffer (wave-aggregated cursor atomics).
// All sums are integers and the only floating point is the binary64 score, so
// the order in which rows are visited never changes a result.
// "The tuning grid" whose times stand in this file is one launch of 1700 forests x
// 256 trees (2220 rows x 35 columns of 64 bins, 10 folds x mtry 1 to 34 x five
// min.node.size); it takes 201 to 217 ms now, by the frame's seed, and the times
// that are compared with each other are of one frame.
#include <limits.h>

#include <type_traits>

#include <cstring>
#include <map>
#include <mutex>
#include <tuple>

#include "device.h"
#include "internal.h"

namespace aiwc {
namespace {

// kSplitDone: split and already partitioned by the wave that searched it (nodes
// of at most kSegMax rows); kSplit: a large or wide node decided to split in
// the child-id step, its rows still to be partitioned (never stored)
constexpr uint8_t kLeaf = 0, kSmall = 1, kBig = 2, kHuge = 3, kSplit = 4, kSplitDone = 5;
// Nodes with at most kSegMax in-bag rows are searched with their rows in a
// lane segment of width 4, 8, 16, 32 or 64 (the smallest that holds them).
constexpr uint32_t kSegMax = 64;
constexpr int kSegClasses = 5;
constexpr int kMaxBins = 256;

// A searched node as the split-search tasks see it (filled when the node is
// classified, so a task needs one dependent load to find its rows).
struct NodeDesc {
  uint32_t k;      // index of the node within its level
  uint32_t start;  // first entry of its segment
  uint32_t len;    // in-bag rows
  uint32_t N;      // bootstrap weight
  int64_t S;       // sum of weight * y_fp
};

struct Rec {
  double score;
  int64_t SL;
  uint32_t NL;
  uint32_t colbin;  // column << 8 | bin
};

// Per-workgroup global scratch.  The per-level arrays come in two copies (the
// level being grown and the next one), selected by the level parity without
// indexing, so that every pointer stays in scalar registers.
struct Level2 {
  uint64_t* buf;
  uint32_t* mstart;
  uint32_t* mend;
  uint32_t* mN;
  int64_t* mS;
  uint64_t* mQ;
};

// A node's candidate list takes mtry bytes rounded up to 16 (the padding
// repeats the last candidate), so that it can be read with 16-byte loads.
__host__ __device__ inline int cand_stride(int mtry) { return (mtry + 15) & ~15; }

// A split node's partition state, by its rank among the level's split nodes:
// the next free slots from the left and from the right of its entry range, and
// the left side's sum of w y^2.
struct Cursor {
  uint32_t L, R;
  uint64_t q;
};

struct Scratch {
  uint32_t* draws;
  Level2 L0, L1;
  uint8_t* status;
  uint8_t* cand;     // level node k's candidate columns at k * cand_stride(mtry), ascending, padded
  uint32_t* btask;   // large node j's candidate i at j * mtry + i: column | bin count << 8
  uint8_t* dcol;  // small split node k's decision: column, bin, left weight and sum
  uint8_t* dbin;
  uint32_t* dNL;
  int64_t* dSL;
  uint32_t* ridx;  // large node k: its index among the level's large (or wide) nodes
  uint32_t* dcnt;  // small split node k: entries that went left
  uint64_t* dQL;   // small split node k: left side's sum of w y^2
  Cursor* cur;    // by split rank, when a level's do not fit the LDS
  uint4* chunks;  // partition work per 64-entry chunk: first entry, the node's end, split rank, column | bin << 8
  NodeDesc* seg[kSegClasses];  // small nodes by segment width 4 << class
  NodeDesc* big;
  NodeDesc* huge;
  Rec* recs;  // large node j's task t at j * mtry + t; wide node h's at (n_big + h) * mtry + i
  // entry p of a wide node: its row's codes in the node's candidate columns, at
  // p * cand_stride(mtry) + i (written by the wide batches, read by the partition
  // instead of the row's code line); null when the launch has no wide phase
  uint8_t* side;
  // the level at which the trees of a group of tasks part, as its split
  // searches left it (kept while each member grows on from it): this level's
  // entries and node sums, the next level's entries (the small nodes' rows,
  // placed by their searches), and the per-node search results and records;
  // null when the launch has no groups
  struct Parted {
    Level2 L;
    uint64_t* nbuf;
    uint8_t *status, *dcol, *dbin;
    uint32_t *ridx, *dNL, *dcnt;
    int64_t* dSL;
    uint64_t* dQL;
    Rec* recs;
    uint8_t* side;
  } SN;
};

__host__ __device__ inline size_t carve(Scratch* s, uintptr_t base, int64_t n_cap, int32_t mtry_max, bool wide,
                                        bool grouped) {
  size_t off = 0;
  auto take = [&](size_t bytes) -> uintptr_t {
    const size_t o = off;
    off = (off + bytes + 255) & ~size_t(255);
    return base + o;
  };
  const size_t n = (size_t)n_cap;
  // large and huge nodes hold more than kSegMax rows each
  const size_t n_large = n / (kSegMax + 1) + 1;
  s->draws = reinterpret_cast<uint32_t*>(take(4 * n));
  Level2* lv[2] = {&s->L0, &s->L1};
  for (int b = 0; b < 2; ++b) {
    lv[b]->buf = reinterpret_cast<uint64_t*>(take(8 * n));
    lv[b]->mstart = reinterpret_cast<uint32_t*>(take(4 * n));
    lv[b]->mend = reinterpret_cast<uint32_t*>(take(4 * n));
    lv[b]->mN = reinterpret_cast<uint32_t*>(take(4 * n));
    lv[b]->mS = reinterpret_cast<int64_t*>(take(8 * n));
    lv[b]->mQ = reinterpret_cast<uint64_t*>(take(8 * n));
  }
  s->status = reinterpret_cast<uint8_t*>(take(n));
  s->cand = reinterpret_cast<uint8_t*>(take(n * (size_t)cand_stride(mtry_max)));
  s->dcol = reinterpret_cast<uint8_t*>(take(n));
  s->dbin = reinterpret_cast<uint8_t*>(take(n));
  s->dNL = reinterpret_cast<uint32_t*>(take(4 * n));
  s->dSL = reinterpret_cast<int64_t*>(take(8 * n));
  // a split node holds at least two rows, so a level has at most n/2 of them
  // and at most n/64 + n/2 chunks
  s->cur = reinterpret_cast<Cursor*>(take(sizeof(Cursor) * (n / 2 + 1)));
  s->dcnt = reinterpret_cast<uint32_t*>(take(4 * n));
  s->ridx = reinterpret_cast<uint32_t*>(take(4 * n));
  s->dQL = reinterpret_cast<uint64_t*>(take(8 * n));
  s->chunks = reinterpret_cast<uint4*>(take(sizeof(uint4) * (n / 64 + n / 2 + 2)));
  // class c holds nodes of more than 2 << c rows (c >= 1)
  for (int c = 0; c < kSegClasses; ++c)
    s->seg[c] = reinterpret_cast<NodeDesc*>(take(sizeof(NodeDesc) * (n / (1 + (c ? (2u << c) : 0)) + 1)));
  s->big = reinterpret_cast<NodeDesc*>(take(sizeof(NodeDesc) * n_large));
  s->huge = reinterpret_cast<NodeDesc*>(take(sizeof(NodeDesc) * n_large));
  s->recs = reinterpret_cast<Rec*>(take(sizeof(Rec) * n_large * (size_t)mtry_max));
  s->btask = reinterpret_cast<uint32_t*>(take(sizeof(uint32_t) * n_large * (size_t)mtry_max));
  s->side = wide ? reinterpret_cast<uint8_t*>(take(n * (size_t)cand_stride(mtry_max))) : nullptr;
  s->SN = Scratch::Parted{};
  if (grouped) {
    s->SN.L.buf = reinterpret_cast<uint64_t*>(take(8 * n));
    s->SN.L.mstart = reinterpret_cast<uint32_t*>(take(4 * n));
    s->SN.L.mend = reinterpret_cast<uint32_t*>(take(4 * n));
    s->SN.L.mN = reinterpret_cast<uint32_t*>(take(4 * n));
    s->SN.L.mS = reinterpret_cast<int64_t*>(take(8 * n));
    s->SN.L.mQ = reinterpret_cast<uint64_t*>(take(8 * n));
    s->SN.nbuf = reinterpret_cast<uint64_t*>(take(8 * n));
    s->SN.status = reinterpret_cast<uint8_t*>(take(n));
    s->SN.dcol = reinterpret_cast<uint8_t*>(take(n));
    s->SN.dbin = reinterpret_cast<uint8_t*>(take(n));
    s->SN.ridx = reinterpret_cast<uint32_t*>(take(4 * n));
    s->SN.dNL = reinterpret_cast<uint32_t*>(take(4 * n));
    s->SN.dcnt = reinterpret_cast<uint32_t*>(take(4 * n));
    s->SN.dSL = reinterpret_cast<int64_t*>(take(8 * n));
    s->SN.dQL = reinterpret_cast<uint64_t*>(take(8 * n));
    s->SN.recs = reinterpret_cast<Rec*>(take(sizeof(Rec) * n_large * (size_t)mtry_max));
    s->SN.side = wide ? reinterpret_cast<uint8_t*>(take(n * (size_t)cand_stride(mtry_max))) : nullptr;
  }
  return off;
}

// Per-wave LDS: one histogram of packed (N, S) bins over at most 256 bins.
// The small-node methods reuse the area for their staged weights, sums and
// codes (up to 4864 bytes).
struct WaveHist {
  uint64_t hv[kMaxBins];
  uint8_t stage[4864 - 8 * kMaxBins];
};

struct GrowArgs {
  const uint8_t* codes;
  int32_t C;
  const uint8_t* codes_p;  // the same codes, rows padded to Cp bytes (one cache line holds whole rows)
  int32_t Cp;
  // the copy the searches and the partition gather codes from: the dense rows
  // while the training set's codes fit an L2 comfortably, else the padded ones
  const uint8_t* rcodes;
  int32_t rC;
  const int32_t* n_bins;
  const int64_t* y_fp;
  const int32_t* train_rows;
  const TreeTask* tasks;
  int32_t n_tasks;
  // groups of tasks that differ only in min.node.size: group g's members are
  // tasks group_task[group_first[g] .. group_first[g + 1]), by min.node.size
  // ascending; null: every task is a group of its own, in task order
  const int32_t* group_task;
  const int32_t* group_first;
  int32_t n_groups;
  uint64_t* nodes;
  uint32_t* node_N;
  int32_t* n_nodes;
  int64_t* work;  // per task (kWorkWords each): searched rows, searched nodes, partitioned rows, levels, LDS bin adds
  uint64_t* inbag;
  uint32_t* queue;
  uint32_t* status;
  uint8_t* scratch;
  int64_t n_cap;
  int32_t mtry_max;
  int32_t huge_min;  // nodes with more rows than this are searched in workgroup-wide batches
  int32_t wide_sums;  // 1: the small-node searches add 64-bit sums even when weights fit a byte
  int32_t bstride;   // bins per column histogram in the workgroup-wide layout
  int32_t big_cols;    // candidate columns per large-node task (1 .. 4)
  int32_t big_stride;  // bins per column histogram of a large-node task
  size_t scratch_stride;
  uint32_t union_bytes;  // dynamic LDS
  uint32_t wave_bytes;   // per-wave area of the split-search tasks
  // teams in one workgroup: rows of the code matrix in the LDS, the bytes it
  // takes there, and each team's bytes (union_bytes and its Shared)
  uint32_t lcode_rows, lcode_bytes, team_bytes;
};

__device__ __forceinline__ uint32_t rfl(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// A value that is the same in every lane, in scalar registers.
template <typename T>
__device__ __forceinline__ T uniform(const T& v) {
  static_assert(sizeof(T) % 4 == 0, "whole words");
  uint32_t w[sizeof(T) / 4];
  __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
  for (int i = 0; i < (int)(sizeof(T) / 4); ++i) w[i] = rfl(w[i]);
  T r;
  __builtin_memcpy(&r, w, sizeof(T));
  return r;
}

__device__ __forceinline__ NodeDesc load_desc(const NodeDesc* p) {
  return NodeDesc{gload(&p->k), gload(&p->start), gload(&p->len), gload(&p->N), gload(&p->S)};
}

// A team of BLOCK threads grows a tree: the workgroup, or (BLOCK = 64) one wave,
// of which a workgroup may hold several.
template <int BLOCK>
__device__ __forceinline__ int team_tid() {
  return BLOCK == kWave ? (int)lane_id() : (int)threadIdx.x;
}
template <int BLOCK>
__device__ __forceinline__ void team_sync() {
  if constexpr (BLOCK == kWave) {
    // the wave's earlier memory operations, in LDS and in global memory, are
    // complete before its later ones: no other wave is waited for
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  } else {
    __syncthreads();
  }
}

// Team exclusive scan of one u32 per thread; `total` receives the sum.
template <int BLOCK>
__device__ __forceinline__ uint32_t block_exscan(uint32_t v, uint32_t* tmp, uint32_t& total) {
  constexpr int NW = BLOCK / kWave;
  const int lane = (int)lane_id(), wid = threadIdx.x / kWave;
  if constexpr (NW == 1) {
    const uint32_t incl = wave_incl_scan_u32(v);
    total = read_lane(incl, kWave - 1);
    return incl - v;
  }
  const uint32_t incl = wave_incl_scan_u32(v);
  if (lane == kWave - 1) tmp[wid] = incl;
  __syncthreads();
  if (wid == 0) {
    const uint32_t t = lane < NW ? tmp[lane] : 0u;
    const uint32_t ti = wave_incl_scan_u32(t);
    if (lane < NW) tmp[lane] = ti - t;
    if (lane == NW - 1) tmp[NW] = ti;
  }
  __syncthreads();
  const uint32_t res = tmp[wid] + incl - v;
  total = tmp[NW];
  __syncthreads();
  return res;
}

// The same for one u64 per thread (two counts packed in its halves).
template <int BLOCK>
__device__ __forceinline__ uint64_t block_exscan64(uint64_t v, uint64_t* tmp, uint64_t& total) {
  constexpr int NW = BLOCK / kWave;
  const int lane = (int)lane_id(), wid = threadIdx.x / kWave;
  if constexpr (NW == 1) {
    const uint64_t incl = wave_incl_scan<uint64_t>(v);
    total = read_lane(incl, kWave - 1);
    return incl - v;
  }
  const uint64_t incl = wave_incl_scan<uint64_t>(v);
  if (lane == kWave - 1) tmp[wid] = incl;
  __syncthreads();
  if (wid == 0) {
    const uint64_t t = lane < NW ? tmp[lane] : 0ull;
    const uint64_t ti = wave_incl_scan<uint64_t>(t);
    if (lane < NW) tmp[lane] = ti - t;
    if (lane == NW - 1) tmp[NW] = ti;
  }
  __syncthreads();
  const uint64_t res = tmp[wid] + incl - v;
  total = tmp[NW];
  __syncthreads();
  return res;
}

template <int BLOCK, typename T>
__device__ __forceinline__ T block_sum(T v, T* tmp) {
  constexpr int NW = BLOCK / kWave;
  const int lane = (int)lane_id(), wid = threadIdx.x / kWave;
  v = wave_sum(v);
  if constexpr (NW == 1) return v;
  if (lane == 0) tmp[wid] = v;
  __syncthreads();
  T s = 0;
  for (int i = 0; i < NW; ++i) s += tmp[i];
  __syncthreads();
  return s;
}

// The mtry candidate columns of node `node` of tree `tree`, drawn by one
// thread: a partial Fisher-Yates shuffle of 0..C-1 driven by draws k = 0 ..
// mtry-1 of the stream (seed, tag 1, node, tree); position k swaps with
// k + floor(r_k (C-k) / 2^64).  `perm` is this thread's C-entry LDS row
// (stride `pst` bytes between entries).  The chosen columns are written
// ascending to `out`, and, when `bt` is given, column | bin count << 8 to
// bt[0 .. mtry) (`nb`: the bin counts, in LDS).
__device__ __forceinline__ void draw_candidates(uint8_t* perm, int pst, uint64_t seed, uint32_t node, uint32_t tree, int C, int mtry,
                                uint8_t* out, uint32_t* bt, const uint16_t* nb) {
  for (int c = 0; c < C; ++c) perm[c * pst] = (uint8_t)c;
  uint64_t m0 = 0, m1 = 0, m2 = 0, m3 = 0;
  for (int b = 0; 4 * b < mtry; ++b) {
    const U64x4 r = philox4x64_10((uint64_t)b, kTagMtry, node, tree, seed, 0);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int k = 4 * b + w;
      if (k < mtry) {
        const int j = k + (int)scale_draw(r.w[w], (uint32_t)(C - k));
        const uint8_t vk = perm[k * pst], vj = perm[j * pst];
        perm[k * pst] = vj;
        perm[j * pst] = vk;
        const uint64_t bit = 1ull << (vj & 63);
        switch (vj >> 6) {
          case 0: m0 |= bit; break;
          case 1: m1 |= bit; break;
          case 2: m2 |= bit; break;
          default: m3 |= bit; break;
        }
      }
    }
  }
  int i = 0;
  uint32_t last = 0;
  auto put = [&](uint32_t c) {
    out[i] = (uint8_t)c;
    if (bt) bt[i] = c | ((uint32_t)nb[c] << 8);
    ++i;
    last = c;
  };
  for (uint64_t m = m0; m; m &= m - 1) put((uint32_t)__builtin_ctzll(m));
  for (uint64_t m = m1; m; m &= m - 1) put(64u + (uint32_t)__builtin_ctzll(m));
  for (uint64_t m = m2; m; m &= m - 1) put(128u + (uint32_t)__builtin_ctzll(m));
  for (uint64_t m = m3; m; m &= m - 1) put(192u + (uint32_t)__builtin_ctzll(m));
  for (; i < cand_stride(mtry); ++i) out[i] = (uint8_t)last;
}

// A row's codes, read by column: in the workgroup's LDS copy of the code matrix
// (LC) or in global memory.
template <bool LC>
struct RowCodes;
template <>
struct RowCodes<false> {
  const uint8_t* p;
  __device__ __forceinline__ uint32_t operator[](uint32_t c) const { return gload(p + c); }
};
template <>
struct RowCodes<true> {
  const __attribute__((address_space(3))) uint8_t* p;
  __device__ __forceinline__ uint32_t operator[](uint32_t c) const { return p[c]; }
};

template <bool LC>
struct Ctx {
  const GrowArgs* a;
  const TreeTask* T;
  const uint8_t* lcodes;  // LC: the code matrix in the LDS, rows of C bytes
  const double* recip;    // reciprocals of the weights below kRecip, in the LDS
  __device__ __forceinline__ RowCodes<LC> row(uint32_t r) const {
    if constexpr (LC)
      return {(const __attribute__((address_space(3))) uint8_t*)(lcodes + __umul24(r, (uint32_t)a->C))};
    else
      return {a->rcodes + (size_t)r * a->rC};
  }
  Scratch sc;
  const uint64_t* buf;  // this level's entries
  uint64_t* nbuf;       // the next level's entries
  const uint32_t* mstart;
  const uint32_t* mend;
  const uint32_t* mN;
  const int64_t* mS;
  const uint64_t* mQ;
};

// Small nodes (at most kSegMax rows): a wave takes P = 64 / W nodes whose rows
// fit a segment of W lanes, one row per lane.  For each candidate position i
// (node k's i-th column, ascending) every lane takes the split at its own
// row's code: the left sums come from the W rows of its segment staged in
// LDS, the segment keeps the best (max score, then lowest bin), and across
// columns a strictly greater score is needed, so ties keep the lowest column.
// The segment's first lane then decides the node; the children's sums come
// from one more segment reduction over the winning column.
// Packed bin of the workgroup-wide and rank histograms: N * 2^45 + S in one unsigned
// 64-bit word.  With N <= 2^18 and |S| <= 2^40 (the fixed-point budget) a bin,
// and every prefix sum of bins, lies in [0, 2^64) and decodes exactly; a bin
// is empty iff its word is 0.  One LDS atomic adds a row to a bin.
__device__ __forceinline__ uint64_t pack_ns(uint32_t w, int64_t wy) { return ((uint64_t)w << 45) + (uint64_t)wy; }
__device__ __forceinline__ uint32_t packed_n(uint64_t v) { return (uint32_t)((v + (1ull << 44)) >> 45); }
__device__ __forceinline__ int64_t packed_s(uint64_t v, uint32_t n) { return (int64_t)(v - ((uint64_t)n << 45)); }

// Light nodes weigh below kRecip: their split scores divide by reciprocals from a
// table in the LDS (div_recip).  Most of the gain comes with the first entries, and
// each takes 8 bytes of every workgroup's LDS from the code matrix or from the
// resident one-wave workgroups (128, 192, 256, 320 entries: the tuning grid 205.0
// 202.3 201.1 200.7 ms, 2000 trees on 2220 rows 2.06 2.00 1.95 1.95, 500 on 200000
// rows 60.6 59.6 59.2 59.1; with 320 a CU held 19 one-wave workgroups, not 20).
constexpr int kRecip = 256;

template <int THREADS>
__device__ __forceinline__ void fill_recip(double* recip) {
  for (int i = threadIdx.x; i < kRecip; i += THREADS) recip[i] = i ? 1.0 / (double)i : 0.0;
}

// The score of a light node's split (|S| < kRecip 2^22 < 2^31: both sides'
// sums convert exactly; Sd, Nd: the node's sum and weight).  A split that leaves
// a side empty scores the parent's S^2 / N (the table's entry 0 is 0), which
// never beats the parent, so callers need not leave it out.
__device__ __forceinline__ double light_score(const double* recip, int32_t SL, uint32_t NL, uint32_t N, double Sd,
                                              double Nd) {
  const double rl = recip[NL], rr = recip[N - NL];
  const double a = (double)SL, b = Sd - a, nl = (double)NL, nr = Nd - nl;
  return div_recip(a * a, nl, rl) + div_recip(b * b, nr, rr);
}

// Prefix sums of a light node's bins (light_word), as two 32-bit words.
__device__ __forceinline__ uint64_t scan_light(uint64_t h) {
  return ((uint64_t)wave_incl_scan_u32((uint32_t)(h >> 32)) << 32) | wave_incl_scan_u32((uint32_t)h);
}

// The wave's best split of (score, key), one per lane: the largest score, then
// the smallest key; scores are -1 (none) or not negative.  Every lane returns it.
__device__ __forceinline__ ArgMax wave_best(double score, int32_t key) {
  double m = score;
  m = max_step0<kDppRowShr1>(m);
  m = max_step0<kDppRowShr2>(m);
  m = max_step0<kDppRowShr4>(m);
  m = max_step0<kDppRowShr8>(m);
  m = max_step0<kDppRowBcast15>(m);
  m = max_step0<kDppRowBcast31>(m);
  ArgMax r;
  r.score = __builtin_bit_cast(double, read_lane(__builtin_bit_cast(uint64_t, m), kWave - 1));
  uint64_t at = __ballot(score == r.score);
  if (at == 0) return ArgMax{-1.0, INT_MAX, 0};
  r.lane = __builtin_ctzll(at);
  r.key = read_lane(key, r.lane);
  for (at &= at - 1; at; at &= at - 1) {
    const int l = __builtin_ctzll(at);
    const int32_t k = read_lane(key, l);
    if (k < r.key) {
      r.key = k;
      r.lane = l;
    }
  }
  return r;
}

// The end of a small node's search, for the W lanes of its segment (one row
// each, lane `sbase + r`): the left child's weight, sum and sum of w y^2 from
// segment reductions, and the node's rows placed into its children's segments
// of the next level (left ones first, in lane order, then the right ones), so
// that the partition skips it; the segment's first lane writes the decision.
template <int W, bool LC>
__device__ __forceinline__ void small_finish(const Ctx<LC>& x, uint32_t k, bool node_ok, int r, int sbase, bool split,
                                             uint32_t col, uint32_t bin, bool valid, bool left, uint64_t e,
                                             uint32_t start) {
  const uint32_t w = entry_w(e);
  const int64_t y = entry_y(e);
  const int64_t wy = (int64_t)w * y;
  uint64_t acc, QL;
  if constexpr (W == kWave) {
    acc = wave_sum(left ? pack_ns(w, wy) : 0ull);
    QL = wave_sum(left ? (uint64_t)(wy * y) : 0ull);
  } else {
    acc = seg_sum<W>(left ? pack_ns(w, wy) : 0ull);
    QL = seg_sum<W>(left ? (uint64_t)(wy * y) : 0ull);
  }
  const uint32_t NL = packed_n(acc);
  const int64_t SL = packed_s(acc, NL);
  const uint64_t seg = (W == kWave ? ~0ull : ((1ull << W) - 1ull)) << sbase;
  const uint64_t lm = __ballot(left) & seg, rm = __ballot(split && valid && !left) & seg;
  const uint64_t below = (1ull << lane_id()) - 1ull;
  const uint32_t nl = (uint32_t)__popcll(lm);
  if (split && valid)
    x.nbuf[start + (left ? (uint32_t)__popcll(lm & below) : nl + (uint32_t)__popcll(rm & below))] = e;
  if (node_ok && r == 0) {
    if (split) {
      x.sc.dcol[k] = (uint8_t)col;
      x.sc.dbin[k] = (uint8_t)bin;
      x.sc.dNL[k] = NL;
      x.sc.dSL[k] = SL;
      x.sc.dcnt[k] = nl;
      x.sc.dQL[k] = QL;
      x.sc.status[k] = kSplitDone;
    } else {
      x.sc.status[k] = kLeaf;
    }
  }
  wave_lds_sync();
}

// Left sums of the split at `code` over a segment of W rows staged as byte
// planes (the group of rows 4j..4j+3 takes 32 bytes: word 0 their weights,
// words 1..4 bytes 0..3 of their w y), four rows at a time: byte b of `ind`
// marks row b's code <= `code`, then dot products with the planes.  C7 (every
// code below 128): 128 + code - c stays in [1, 255] in each byte, so no borrow
// crosses the bytes and its bit 7 is the comparison; `ind` keeps that bit in
// place (byte 0x80: 128 unsigned, -128 signed), so the sums come out times 128
// (the signed top plane's times -128) and one exact shift at the end divides it
// out.  Otherwise per 16-bit half 256 + code - c stays in [1, 511] and its high
// byte (0 or 1) is the comparison: bytes 0 and 2 of the codes are compared in
// place, bytes 1 and 3 moved down by a byte permute, and a second permute
// gathers the four high bytes.
template <int W, bool C7, bool B3>
__device__ __forceinline__ void byte_plane_sums(uint32_t code, const uint32_t* seg_codes, const uint8_t* seg_planes,
                                                uint32_t& NL, int64_t& SL) {
  static_assert(!C7 || B3, "the search with four byte planes takes any code");
  const uint32_t kk = C7 ? (code + 0x80u) * 0x01010101u : code * 0x00010001u + 0x01000100u;
  uint32_t aN = 0, a0 = 0, a1 = 0;
  int32_t a2 = 0, a3 = 0;
#pragma unroll 4
  for (int b4 = 0; b4 < W / 4; ++b4) {
    const uint32_t c4 = seg_codes[b4];
    uint32_t ind;
    if constexpr (C7) {
      ind = (kk - c4) & 0x80808080u;
    } else {
      const uint32_t d02 = kk - (c4 & 0x00FF00FFu);
      const uint32_t d13 = kk - __builtin_amdgcn_perm(0u, c4, 0x0c030c01u);  // bytes 1, 3 of c4 to 0, 2
      ind = __builtin_amdgcn_perm(d02, d13, 0x03070105u);  // bytes 1, 3 of each difference, interleaved
    }
    const uint4 pl = *reinterpret_cast<const uint4*>(seg_planes + b4 * 32);
    aN = __builtin_amdgcn_udot4(ind, pl.x, aN, false);
    a0 = __builtin_amdgcn_udot4(ind, pl.y, a0, false);
    a1 = __builtin_amdgcn_udot4(ind, pl.z, a1, false);
    if constexpr (B3) {
      // w y in 24 bits: byte 2 is its signed top byte
      a2 = __builtin_amdgcn_sdot4((int32_t)ind, (int32_t)pl.w, a2, false);
    } else {
      const uint32_t p3 = *reinterpret_cast<const uint32_t*>(seg_planes + b4 * 32 + 16);
      a2 = (int32_t)__builtin_amdgcn_udot4(ind, pl.w, (uint32_t)a2, false);
      a3 = __builtin_amdgcn_sdot4((int32_t)ind, (int32_t)p3, a3, false);
    }
  }
  if constexpr (C7) {
    // every accumulator is a multiple of 128 (at most 128 * 255 * 32): byte
    // plane j's sum times 2^(8 j) is a_j / 128 * 2^(8 j), the signed top
    // plane's negated
    NL = aN >> 7;
    SL = (int64_t)(a0 >> 7) + ((int64_t)a1 << 1) - ((int64_t)a2 << 9);
  } else {
    NL = aN;
    if constexpr (B3)
      SL = (int64_t)a0 + ((int64_t)a1 << 8) + ((int64_t)a2 << 16);
    else
      SL = (int64_t)a0 + ((int64_t)a1 << 8) + ((int64_t)(uint32_t)a2 << 16) + ((int64_t)a3 << 24);
  }
}

// Left sums of a candidate's splits for the whole wave by matrix instructions:
// for every lane the sums, over its segment's W rows whose code is at most its
// own row's, of the rows' weights and of their w y.  A 16 x 16 x 64 product of
// signed bytes contracts the wave's 64 rows: its A operand holds the rows' digits
// (staged once per task, negated), its B operand the comparisons, and its
// accumulator's layout gives lane 16 q + j rows 4 q .. 4 q + 3 of column j, the
// four digit sums of that lane's own split.
//   A: lane 16 b + i holds row i's bytes for the wave's rows 16 b .. 16 b + 15;
//      row 4 q + p is digit p of the rows that quarter q's lanes sum over.
//   B: lane 16 b + j holds column j's comparisons with the rows 16 b .. 16 b + 15:
//      W <= 16: its own row's code against its own segment (the quarter's other
//      segments 0); W = 32: two products, with rows j and 16 + j of its node, each
//      with the A rows of the quarters it is for.
// Digits: word 0 the weight (at most 127), words 1..3 (4) the balanced base-256
// digits of w y.  A comparison is the byte 0x80 = -128, so a sum comes out
// times 128 and one exact shift divides that out.
// Against the dot products above it drops the LDS reads of the planes and, of
// the VALU instructions per candidate, two thirds for W = 32 (48 -> 16) and half
// for W = 8 and 16: the tuning grid's launch issues 11 % fewer VALU and 31 %
// fewer LDS instructions.  It holds eight registers more through the candidate
// loop, which only the kernel of k_grow_teams has to spare: there the grid takes
// 261 ms with it and 280 without; kernels of 96 and 80 registers spill for it and
// lose (the grid 287 -> 292 ms, 2000 trees on 2220 rows 2.29 -> 2.36 ms).
typedef int v4i_t __attribute__((ext_vector_type(4)));

// Bit 7 of each byte: the byte of c4 is at most `code`, whose broadcasts are kb
// (all four bytes) and kh (kb with bit 7 set).  C7 (every code below 128): 128 +
// code - c stays in [1, 255] in each byte, so no borrow crosses the bytes and its
// bit 7 is the comparison.  Otherwise the low seven bits are compared that way
// and bit 7 decides where it differs.
template <bool C7>
__device__ __forceinline__ uint32_t bytes_le(uint32_t c4, uint32_t kb, uint32_t kh) {
  if constexpr (C7) return kh - c4;
  const uint32_t t = kh - (c4 & 0x7F7F7F7Fu);
  return (kb & ~c4) | (~(kb ^ c4) & t);
}

template <int W>
struct SegDigits {
  static constexpr int H = W == 32 ? 2 : 1;  // products per candidate
  v4i_t a[H];
};

// A operands of digits 0..3, from the staged digit planes (plane p's byte of the
// wave's row r at planes + 64 p + r); TOP: of digit 4 alone, in its first row.
template <int W, bool TOP>
__device__ __forceinline__ SegDigits<W> seg_digits(const uint8_t* planes, int lane) {
  const int b = lane >> 4, q = (lane >> 2) & 3, p = lane & 3;
  const v4i_t v = *reinterpret_cast<const v4i_t*>(planes + 64 * (TOP ? 4 : p) + 16 * b);
  SegDigits<W> d;
#pragma unroll
  for (int h = 0; h < d.H; ++h) {
    const bool mine = (W == 32 ? q == (b & 2) + h : q == b) && (!TOP || p == 0);
#pragma unroll
    for (int u = 0; u < 4; ++u) d.a[h][u] = mine ? v[u] : 0;
  }
  return d;
}

// B3: three digits of w y, and light nodes only (`light` is not looked at).
template <int W, bool C7, bool B3>
__device__ __forceinline__ void matrix_sums(const SegDigits<W>& A, const uint8_t* planes, const uint8_t* col_codes,
                                            uint32_t code, int lane, uint32_t& NL, int64_t& SL, bool light) {
  static_assert(!C7 || B3, "the search with four digits takes any code");
  constexpr uint32_t kTop = 0x80808080u;
  v4i_t acc = {0, 0, 0, 0}, acc4 = {0, 0, 0, 0};
  if constexpr (W <= 16) {
    const uint32_t kb = __builtin_amdgcn_perm(0u, code, 0u), kh = kb | kTop;
    const uint32_t* seg = reinterpret_cast<const uint32_t*>(col_codes + (lane & ~(W - 1)));
    uint32_t c[W / 4];
#pragma unroll
    for (int u = 0; u < W / 4; ++u) c[u] = bytes_le<C7>(seg[u], kb, kh);
    v4i_t bm;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      // word u belongs to the quarter's segment 4 u / W
      const uint32_t m = W == 16 || (lane & 15) / W == 4 * u / W ? kTop : 0u;
      bm[u] = (int)(c[u % (W / 4)] & m);
    }
    acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(A.a[0], bm, acc, 0, 0, 0);
    if constexpr (!B3)
      acc4 = __builtin_amdgcn_mfma_i32_16x16x64_i8(seg_digits<W, true>(planes, lane).a[0], bm, acc4, 0, 0, 0);
  } else {
    const uint4 c4 = *reinterpret_cast<const uint4*>(col_codes + (lane & 0x30));
    SegDigits<W> A4;
    if constexpr (!B3) A4 = seg_digits<W, true>(planes, lane);
#pragma unroll
    for (int h = 0; h < SegDigits<W>::H; ++h) {
      const uint32_t kb = __builtin_amdgcn_perm(0u, col_codes[(lane & 0x20) + 16 * h + (lane & 15)], 0u);
      const uint32_t kh = kb | kTop;
      const v4i_t bm = {(int)(bytes_le<C7>(c4.x, kb, kh) & kTop), (int)(bytes_le<C7>(c4.y, kb, kh) & kTop),
                        (int)(bytes_le<C7>(c4.z, kb, kh) & kTop), (int)(bytes_le<C7>(c4.w, kb, kh) & kTop)};
      acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(A.a[h], bm, acc, 0, 0, 0);
      if constexpr (!B3) acc4 = __builtin_amdgcn_mfma_i32_16x16x64_i8(A4.a[h], bm, acc4, 0, 0, 0);
    }
  }
  // every accumulator is a multiple of 128
  NL = (uint32_t)(acc[0] >> 7);
  if (B3 || light) {  // the sum fits 32 bits (its terms need not: they wrap)
    uint32_t v = (uint32_t)(acc[1] >> 7) + ((uint32_t)acc[2] << 1) + ((uint32_t)acc[3] << 9);
    if constexpr (!B3) v += (uint32_t)acc4[0] << 17;
    SL = (int32_t)v;
  } else {
    SL = (int64_t)(acc[1] >> 7) + (int64_t)acc[2] * 2 + (int64_t)acc[3] * 512 + (int64_t)acc4[0] * 131072;
  }
}

template <int W, bool LC>
__device__ __forceinline__ void small_task(const Ctx<LC>& x, const NodeDesc* list, uint32_t t, uint32_t n_list, WaveHist& wl) {
  const GrowArgs& a = *x.a;
  const int mtry = x.T->mtry;
  const int lane = (int)lane_id();
  constexpr int P = kWave / W;
  const int g = lane / W, r = lane % W, sbase = g * W;
  // (the segments past the list's end repeat its last node without rows)
  const uint32_t idx = t * (uint32_t)P + (uint32_t)g;
  const bool node_ok = idx < n_list;
  const NodeDesc d = load_desc(list + min(idx, n_list - 1u));
  const uint32_t k = d.k, start = d.start, len = node_ok ? d.len : 0u, N = d.N;
  const int64_t S = d.S;
  const bool valid = (uint32_t)r < len;
  const uint64_t e = valid ? gload(x.buf + start + r) : 0ull;
  const uint32_t row = entry_row(e);
  const uint32_t w = valid ? entry_w(e) : 0u;
  const int64_t y = entry_y(e);
  const int64_t wy = (int64_t)w * y;
  uint8_t* area = reinterpret_cast<uint8_t*>(&wl);
  uint8_t* s_codes = area + 512;  // [64 columns][64 lanes]
  // The rows' weights and w y, staged in the first 512 bytes.  When every weight
  // of the wave is small (bootstrap multiplicities nearly always are), as signed
  // digits for the matrix products (MX, weights up to 127: 64 bytes of -w, then
  // 64 of each balanced base-256 digit of -w y) or as byte planes for the dot
  // products (weights up to 255: the group of rows 4j..4j+3 takes 32 bytes, word 0
  // their weights and words 1..4 bytes 0..3 of their w y, two's complement).
  // |w y| < 2^30 takes four digits or bytes, three when every w y of the wave
  // fits 24 bits.  Otherwise packed (w, w y) words, one per row.
  constexpr bool MX = LC;
  const bool bytes_ok = !a.wide_sums && __ballot(w > (MX ? 127u : 255u)) == 0ull;
  const uint32_t u = 0x80808080u - (uint32_t)(int32_t)wy;  // digit j of -w y is byte j of u less 128
  const bool b3 = MX ? __ballot(u >> 24 != 0x80u) == 0ull
                     : __ballot(wy < -(int64_t)(1 << 23) || wy >= (int64_t)(1 << 23)) == 0ull;
  // every column's codes fit 7 bits (at most 128 bins)
  const bool codes7 = a.bstride <= 128;
  // every node of the wave is light: its sums fit 32 bits
  const bool light = __ballot(N >= (uint32_t)kRecip) == 0ull;
  const double Sd = i64_to_f64(S), Nd = (double)N;
  uint8_t* planes = area;
  uint64_t* s_pv = reinterpret_cast<uint64_t*>(area);
  SegDigits<W> A;
  if (bytes_ok) {
    if constexpr (MX) {
      const uint32_t dg = u ^ 0x80808080u;
      planes[lane] = (uint8_t)(0u - w);
      planes[64 + lane] = (uint8_t)dg;
      planes[128 + lane] = (uint8_t)(dg >> 8);
      planes[192 + lane] = (uint8_t)(dg >> 16);
      planes[256 + lane] = (uint8_t)(dg >> 24);
    } else {
      const uint32_t wy32 = (uint32_t)(int32_t)wy;
      uint8_t* gp = planes + (lane >> 2) * 32 + (lane & 3);
      gp[0] = (uint8_t)w;
      gp[4] = (uint8_t)wy32;
      gp[8] = (uint8_t)(wy32 >> 8);
      gp[12] = (uint8_t)(wy32 >> 16);
      gp[16] = (uint8_t)(wy32 >> 24);
    }
  } else {
    s_pv[lane] = pack_ns(w, wy);
  }
  if constexpr (MX) {
    wave_lds_sync();
    A = seg_digits<W, false>(planes, lane);  // (unused with packed words)
  }
  const RowCodes<LC> rowp = x.row(row);
  const uint8_t* cand = x.sc.cand + (size_t)k * cand_stride(mtry);

  // each lane keeps its own best split (score, candidate index, bin) over the
  // candidates in order; one segment arg-max at the end picks the node's
  double best = -1.0;
  uint32_t best_ib = 0xFFFFFFFFu;  // candidate index << 8 | bin
  const uint64_t* seg_pv = s_pv + sbase;
  // the candidates of a chunk, with every form of the sums and scores
  auto general_search = [&](int i0, int nc) {
    for (int i = 0; i < nc; ++i) {
      const uint8_t* col_codes = s_codes + i * kWave;
      const uint32_t code = col_codes[lane];
      // left sums of the split at this lane's code: the segment's rows with a code <= it
      uint32_t NL;
      int64_t SL;
      const uint32_t* seg_codes = reinterpret_cast<const uint32_t*>(col_codes + sbase);
      if (bytes_ok) {
        if constexpr (MX)
          matrix_sums<W, false, false>(A, planes, col_codes, code, lane, NL, SL, light);
        else
          byte_plane_sums<W, false, false>(code, seg_codes, planes + (sbase >> 2) * 32, NL, SL);
      } else {
        uint64_t acc = 0;  // packed left sums
#pragma unroll 2
        for (int b4 = 0; b4 < W / 4; ++b4) {
          const uint32_t c4 = seg_codes[b4];
#pragma unroll
          for (int u = 0; u < 4; ++u) acc += ((c4 >> (8 * u)) & 0xFFu) <= code ? seg_pv[4 * b4 + u] : 0ull;
        }
        NL = packed_n(acc);
        SL = packed_s(acc, NL);
      }
      // (a lane without a row holds row 0's code: a split like any other of its
      // node, equal to that of the highest code not above it)
      double sc = -1.0;
      if (light)
        sc = light_score(x.recip, (int32_t)SL, NL, N, Sd, Nd);
      else if (valid && NL < N)
        sc = split_score(SL, NL, S - SL, N - NL);
      if (sc > best) {
        best = sc;
        best_ib = ((uint32_t)(i0 + i) << 8) | code;
      }
    }
  };
  for (int i0 = 0; i0 < mtry; i0 += kWave) {
    const int nc = min(kWave, mtry - i0);
    // gather the row's codes in every candidate column of this chunk at once:
    // sixteen candidates per 16-byte load, sixteen gathers in flight.  Every
    // lane loads and stores without a branch: a lane without a row reads row 0
    // (entry 0), whose codes no sum uses (its weight and w y are zero), and a
    // position past the list reads its padding, the last candidate again, into a
    // slot no candidate reads (g0 + u < 64: inside the 64-column staging area).
    for (int g0 = 0; g0 < nc; g0 += 16) {
      const uint4 c16 = gload16(cand + i0 + g0);
      const uint32_t cw[4] = {c16.x, c16.y, c16.z, c16.w};
      uint32_t cd[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        cd[u] = rowp[(cw[u >> 2] >> (8 * (u & 3))) & 0xFFu];
      }
#pragma unroll
      for (int u = 0; u < 16; ++u) s_codes[(g0 + u) * kWave + lane] = (uint8_t)cd[u];
    }
    wave_lds_sync();
    // the common case (sums of three digits or bytes over light nodes) has loops
    // of its own, and the general one the widest form alone: with a branch on each
    // of its conditions in one loop the tuning grid took 223 ms, so 215
    if (bytes_ok && b3 && light) {
      auto search = [&](auto c7) {
#pragma unroll 1
        for (int i = 0; i < nc; ++i) {
          const uint8_t* col_codes = s_codes + i * kWave;
          const uint32_t code = col_codes[lane];
          uint32_t NL;
          int64_t SL;
          constexpr bool C7 = decltype(c7)::value;
          if constexpr (MX)
            matrix_sums<W, C7, true>(A, planes, col_codes, code, lane, NL, SL, true);
          else
            byte_plane_sums<W, C7, true>(code, reinterpret_cast<const uint32_t*>(col_codes + sbase),
                                         planes + (sbase >> 2) * 32, NL, SL);
          const double sc = light_score(x.recip, (int32_t)SL, NL, N, Sd, Nd);
          if (sc > best) {
            best = sc;
            best_ib = ((uint32_t)(i0 + i) << 8) | code;
          }
        }
      };
      if (codes7)
        search(std::true_type{});
      else
        search(std::false_type{});
    } else {
      general_search(i0, nc);
    }
    wave_lds_sync();
  }
  // segment arg-max: the largest score, then the lowest candidate, then the lowest bin
  seg_argmax<W>(best, best_ib);
  const bool split = node_ok && best >= 0.0 && best - parent_score(S, N) > 0.0;
  const uint32_t col = split ? cand[best_ib >> 8] : 0u, bin = best_ib & 0xFF;
  const bool left = split && valid && rowp[col] <= bin;
  small_finish<W, LC>(x, k, node_ok, r, sbase, split, col, bin, valid, left, e, start);
}

// Nodes of 33..64 rows: one node per wave, one row per lane.  Per candidate
// column the rows' packed (w, w y) are added into the column's LDS bins, a wave
// prefix scan over the bins turns them into left sums, and every lane scores the
// split at its own row's code (lanes sharing a code score the same split).  A
// light node of columns of at most 64 bins keeps its prefix sums in registers
// (one bin per lane) and each lane takes the one at its own code by a cross-lane
// read; wider columns write them back to LDS.  The loop of the common case has no
// branches and takes two candidates at a time, whose waits overlap: the tuning
// grid's launch 215 -> 201 ms, the leave-one-kernel-out fit (148 bins) 26.0 ->
// 24.3 ms.
template <bool LC>
__device__ __forceinline__ void rank_task(const Ctx<LC>& x, const NodeDesc* list, uint32_t t, uint32_t n_list, WaveHist& wl) {
  const GrowArgs& a = *x.a;
  const int mtry = x.T->mtry;
  const int lane = (int)lane_id();
  if (t >= n_list) return;
  const NodeDesc d = uniform(load_desc(list + t));
  const uint32_t k = d.k, start = d.start, len = d.len, N = d.N;
  const int64_t S = d.S;
  const bool valid = (uint32_t)lane < len;
  const uint64_t e = valid ? gload(x.buf + start + lane) : 0ull;
  const uint32_t w = valid ? entry_w(e) : 0u;
  const int64_t y = entry_y(e);
  const int64_t wy = (int64_t)w * y;
  const bool light = N < (uint32_t)kRecip;
  const uint64_t pv = light ? light_word(w, wy) : pack_ns(w, wy);
  const double Sd = i64_to_f64(S), Nd = (double)N;
  const RowCodes<LC> rowp = x.row(entry_row(e));
  const uint8_t* cand = x.sc.cand + (size_t)k * cand_stride(mtry);
  uint8_t* area = reinterpret_cast<uint8_t*>(&wl);
  uint64_t* hb = reinterpret_cast<uint64_t*>(area);  // [2][256] packed bins, then prefix sums
  uint8_t* s_cand = area + 4096;                     // [mtry]
  uint8_t* s_bm1 = area + 4352;                      // [mtry]: each candidate's bin count - 1
  for (int i = lane; i < mtry; i += kWave) {
    const uint32_t c = gload(cand + i);
    s_cand[i] = (uint8_t)c;
    if (!LC) s_bm1[i] = (uint8_t)(gload(a.n_bins + c) - 1);
  }
  // both buffers start zeroed: four bins per lane each
  *reinterpret_cast<uint4*>(hb + 4 * lane) = make_uint4(0u, 0u, 0u, 0u);
  *reinterpret_cast<uint4*>(hb + 4 * lane + 2) = make_uint4(0u, 0u, 0u, 0u);
  *reinterpret_cast<uint4*>(hb + 256 + 4 * lane) = make_uint4(0u, 0u, 0u, 0u);
  *reinterpret_cast<uint4*>(hb + 256 + 4 * lane + 2) = make_uint4(0u, 0u, 0u, 0u);
  wave_lds_sync();

  // each lane keeps the best of the splits it scores (the one at its own code,
  // for every candidate) as (score, candidate index << 8 | bin); one arg-max at
  // the end
  double best = -1.0;
  int32_t best_ib = INT_MAX;
  // U candidates at a time, in buffers of their own; lane l owns bins [l Q, l Q +
  // Q), Q the same for every column (the lanes past a column's bins read zeros).
  // A wave's LDS operations are in order, so a buffer is read and cleared, and
  // added to again, without waits between.  A lane without a row holds row 0's
  // codes: splits like any other of the node.
  const int Q = a.bstride / kWave;
  auto step = [&](auto is_light, auto one_bin, auto nu, int i, const uint32_t (&code)[2]) {
    constexpr bool LIGHT = decltype(is_light)::value, ONE = decltype(one_bin)::value;
    constexpr int U = decltype(nu)::value;
    auto scan = [](uint64_t v) { return LIGHT ? scan_light(v) : wave_incl_scan<uint64_t>(v); };
    if (valid) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        atomicAdd((unsigned long long*)&hb[u * kMaxBins + code[u]], (unsigned long long)pv);
    }
    wave_lds_sync();
    uint64_t V[U];  // left sums of the split at this lane's code
    if constexpr (ONE) {
      // the prefix sums stay in registers: each lane takes the one at its own
      // code by a cross-lane read
      uint64_t h[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        h[u] = hb[u * kMaxBins + lane];
        hb[u * kMaxBins + lane] = 0ull;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) V[u] = lane_pick64(scan(h[u]), code[u]);
    } else {
      uint64_t h[U][4], v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        v[u] = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          h[u][c] = c < Q ? hb[u * kMaxBins + lane * Q + c] : 0ull;
          v[u] += h[u][c];
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        uint64_t run = scan(v[u]) - v[u];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          run += h[u][c];
          if (c < Q) hb[u * kMaxBins + lane * Q + c] = run;
        }
      }
      wave_lds_sync();
#pragma unroll
      for (int u = 0; u < U; ++u) V[u] = hb[u * kMaxBins + code[u]];
      wave_lds_sync();
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (c < Q) hb[u * kMaxBins + lane * Q + c] = 0ull;
    }
    wave_lds_sync();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      double sc = -1.0;
      if constexpr (LIGHT) {
        const uint32_t NL = (uint32_t)(V[u] >> 32);
        sc = light_score(x.recip, light_sum(NL, (uint32_t)V[u]), NL, N, Sd, Nd);
      } else {
        const uint32_t NL = packed_n(V[u]);
        const int64_t SL = packed_s(V[u], NL);
        if (NL > 0 && NL < N) sc = split_score(SL, NL, S - SL, N - NL);
      }
      if (sc > best) {
        best = sc;
        best_ib = ((i + u) << 8) | (int32_t)code[u];
      }
    }
  };
  // the candidates' codes are fetched one step ahead
  auto search = [&](auto is_light, auto one_bin, auto nu) {
    constexpr int U = decltype(nu)::value;
    uint32_t next[2] = {rowp[rfl(s_cand[0])], rowp[rfl(s_cand[min(1, mtry - 1)])]};
    int i = 0;
#pragma unroll 1
    for (; i + U <= mtry; i += U) {
      const uint32_t code[2] = {next[0], next[1]};
      if constexpr (U == 1)
        next[0] = next[1];
      else
        next[0] = rowp[rfl(s_cand[min(i + 2, mtry - 1)])];
      next[1] = rowp[rfl(s_cand[min(i + U + 1, mtry - 1)])];
      step(is_light, one_bin, nu, i, code);
    }
    if (i < mtry) step(is_light, one_bin, std::integral_constant<int, 1>{}, i, next);
  };
  if (light && Q == 1) {
    search(std::true_type{}, std::true_type{}, std::integral_constant<int, 2>{});
  } else if constexpr (LC) {
    if (light)
      search(std::true_type{}, std::false_type{}, std::integral_constant<int, 2>{});
    else
      search(std::false_type{}, std::false_type{}, std::integral_constant<int, 1>{});
  } else {
    // one candidate at a time, within the registers that the other kernels can
    // spare, its bins read to its own count (with the loop above 2000 trees on 2220
    // rows of 148 bins take 2.28 ms and 500 on 200000 rows 65.8; with this one
    // 2.07 and 63.0)
    uint32_t code_next = rowp[rfl(s_cand[0])];
#pragma unroll 1
    for (int i = 0; i < mtry; ++i) {
      const uint32_t code = code_next;
      const int B = (int)rfl(s_bm1[i]) + 1, q = (B + kWave - 1) / kWave, b0 = lane * q;
      if (i + 1 < mtry) code_next = rowp[rfl(s_cand[i + 1])];
      uint64_t* hv = hb + (i & 1) * kMaxBins;
      if (valid) atomicAdd((unsigned long long*)&hv[code], (unsigned long long)pv);
      wave_lds_sync();
      // the other buffer holds the previous candidate's prefix sums, which every
      // lane has read: cleared while this one is scanned
      if (i > 0) {
        uint64_t* ho = hb + ((i - 1) & 1) * kMaxBins;
        *reinterpret_cast<uint4*>(ho + 4 * lane) = make_uint4(0u, 0u, 0u, 0u);
        *reinterpret_cast<uint4*>(ho + 4 * lane + 2) = make_uint4(0u, 0u, 0u, 0u);
      }
      uint64_t h[4];
      uint64_t loc = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        h[u] = u < q && b0 + u < B ? hv[b0 + u] : 0ull;
        loc += h[u];
      }
      uint64_t v = (light ? scan_light(loc) : wave_incl_scan<uint64_t>(loc)) - loc;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        v += h[u];
        if (u < q && b0 + u < B) hv[b0 + u] = v;
      }
      wave_lds_sync();
      const uint64_t V = hv[code];  // (a lane without a row has row 0's code: below B)
      double sc = -1.0;
      if (light) {
        const uint32_t NL = (uint32_t)(V >> 32);
        sc = light_score(x.recip, light_sum(NL, (uint32_t)V), NL, N, Sd, Nd);
      } else if (valid) {
        const uint32_t NL = packed_n(V);
        const int64_t SL = packed_s(V, NL);
        if (NL < N) sc = split_score(SL, NL, S - SL, N - NL);
      }
      if (sc > best) {
        best = sc;
        best_ib = (i << 8) | (int32_t)code;
      }
    }
  }
  const ArgMax am = wave_best(best, best_ib);
  const bool split = am.score >= 0.0 && am.score - parent_score(S, N) > 0.0;
  const uint32_t col = split ? (uint32_t)s_cand[am.key >> 8] : 0u, bin = (uint32_t)am.key & 0xFF;
  const bool left = split && valid && rowp[col] <= bin;
  small_finish<kWave, LC>(x, k, true, lane, 0, split, col, bin, valid, left, e, start);
}

// Scan one column's histogram of packed bins (B <= 256 bins) with a wave: lane
// l owns bins [l q, l q + q) with q = ceil(B / 64) (so a 64-bin column takes one
// bin per lane); prefix sums give the left side of every split b <= B-2.
// Returns the wave's best (max score, lowest bin) in every lane; the left sums
// oNL, oSL of that split are valid in lane `am.lane`.
__device__ __forceinline__ ArgMax scan_packed(const uint64_t* hv, int B, uint32_t N, int64_t S, uint32_t& oNL,
                                              int64_t& oSL) {
  const int lane = (int)lane_id();
  if (B <= kWave) {  // one bin per lane
    const uint64_t h = lane < B ? hv[lane] : 0ull;
    const uint64_t v = wave_incl_scan<uint64_t>(h);
    double lbest = -1.0;
    oNL = 0;
    oSL = 0;
    // an empty bin repeats the previous split, which already won any tie
    if (h != 0 && lane <= B - 2) {
      const uint32_t NL = packed_n(v);
      if (NL < N) {
        const int64_t SL = packed_s(v, NL);
        lbest = split_score(SL, NL, S - SL, N - NL);
        oNL = NL;
        oSL = SL;
      }
    }
    return wave_argmax_lane_ordered(lbest, lbest >= 0.0 ? lane : INT_MAX);
  }
  const int q = (B + kWave - 1) / kWave;
  const int b0 = lane * q;
  uint64_t h[4];
  uint64_t loc = 0;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    h[u] = u < q && b0 + u < B ? hv[b0 + u] : 0ull;
    loc += h[u];
  }
  uint64_t v = wave_incl_scan<uint64_t>(loc) - loc;
  double lbest = -1.0;
  int32_t lbin = INT_MAX;
  oNL = 0;
  oSL = 0;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int b = b0 + u;
    // an empty bin repeats the previous split, which already won any tie
    if (u >= q || h[u] == 0) continue;
    v += h[u];
    const uint32_t NL = packed_n(v);
    if (b <= B - 2 && NL < N) {
      const int64_t SL = packed_s(v, NL);
      const double s = split_score(SL, NL, S - SL, N - NL);
      if (s > lbest) {
        lbest = s;
        lbin = b;
        oNL = NL;
        oSL = SL;
      }
    }
  }
  // lane l's bins precede lane l+1's: the lowest lane with the best score holds
  // the lowest best bin
  return wave_argmax_lane_ordered(lbest, lbin);
}

// Large nodes: one wave per (node, up to four consecutive candidate columns),
// one LDS histogram per column: the node's entries are read once for all of
// them, a step ahead, and the columns' code gathers overlap.  The node and its
// columns are the same in every lane, and kept in scalar registers as such
// (column g's id and bin count are lane g's, read across): with loops over
// vector counts and one copy of the scan per column the grid took 235 ms, the
// 200000-row fit 66.4; now 223 and 63.2.
template <bool LC>
__device__ __forceinline__ void big_task(const Ctx<LC>& x, uint32_t j, int ci0, WaveHist& L) {
  constexpr int G = 4;
  const GrowArgs& a = *x.a;
  const int lane = (int)lane_id();
  const int mtry = x.T->mtry;
  const int gn = min(a.big_cols, mtry - ci0);  // columns of this task
  const int gs = a.big_stride;
  const NodeDesc d = uniform(load_desc(x.sc.big + j));
  const uint32_t start = d.start, end = start + d.len, N = d.N;
  const int64_t S = d.S;
  const uint32_t* btp = x.sc.btask + (size_t)j * mtry + ci0;
  const uint32_t btl = gload(btp + min(lane, gn - 1));  // lane g: column g's id and bin count
  uint32_t bt[G];
#pragma unroll
  for (int g = 0; g < G; ++g) bt[g] = read_lane(btl, g) & 0xFFu;
  uint64_t* hv = L.hv;
  for (int b = lane; b < gn * gs; b += kWave) hv[b] = 0;
  wave_lds_sync();
  // each lane keeps the best split of its bins over the task's columns, and the
  // wave's best of all is the task's record
  double best = -1.0;
  int32_t key = INT_MAX;  // column of the task << 8 | bin
  uint32_t bNL = 0;
  int64_t bSL = 0;
  auto search = [&](auto is_light) {
    constexpr bool LIGHT = decltype(is_light)::value;
    // two rows per lane in flight: entries, then their codes in every column,
    // then the atomics (a lane past the node's end repeats its last entry)
    constexpr int U = 2;
    uint64_t en[U];
#pragma unroll
    for (int u = 0; u < U; ++u) en[u] = gload(x.buf + min(start + (uint32_t)(u * kWave + lane), end - 1u));
    for (uint32_t p = start; p < end; p += U * kWave) {
      uint64_t e[U];
      uint32_t code[U][G];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        e[u] = en[u];
        en[u] = gload(x.buf + min(p + (uint32_t)((U + u) * kWave + lane), end - 1u));
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const RowCodes<LC> rp = x.row(entry_row(e[u]));
#pragma unroll
        for (int g = 0; g < G; ++g) code[u][g] = g < gn ? rp[bt[g] & 0xFFu] : 0u;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (p + (uint32_t)(u * kWave + lane) < end) {
          const uint32_t w = entry_w(e[u]);
          const int32_t y = (int32_t)entry_y(e[u]);
          const uint64_t v = LIGHT ? light_word(w, (int32_t)w * y) : pack_ns(w, (int64_t)w * y);
#pragma unroll
          for (int g = 0; g < G; ++g)
            if (g < gn) atomicAdd((unsigned long long*)&hv[g * gs + (int)code[u][g]], (unsigned long long)v);
        }
      }
    }
    wave_lds_sync();
    const double Sd = i64_to_f64(S), Nd = (double)N;
    auto score = [&](uint64_t v, int32_t k) {
      uint32_t NL;
      int64_t SL;
      double sc = -1.0;
      if constexpr (LIGHT) {
        NL = (uint32_t)(v >> 32);
        SL = light_sum(NL, (uint32_t)v);
        sc = light_score(x.recip, (int32_t)SL, NL, N, Sd, Nd);
      } else {
        NL = packed_n(v);
        SL = packed_s(v, NL);
        if (NL > 0 && NL < N) sc = split_score(SL, NL, S - SL, N - NL);
      }
      if (sc > best) {
        best = sc;
        key = k;
        bNL = NL;
        bSL = SL;
      }
    };
    auto scan = [](uint64_t v) { return LIGHT ? scan_light(v) : wave_incl_scan<uint64_t>(v); };
#pragma unroll 1
    for (int g = 0; g < gn; ++g) {
      const uint32_t btg = read_lane(btl, g);
      // lane l owns bins [l q, l q + q): an empty bin repeats the split before it,
      // which wins the tie
      const int B = (int)(btg >> 8), q = (B + kWave - 1) / kWave, b0 = lane * q;
      const uint64_t* hg = hv + g * gs;
      if (q == 1) {
        score(scan(lane < B ? hg[lane] : 0ull), (g << 8) | lane);
      } else {
        uint64_t h[4];
        uint64_t loc = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          h[u] = u < q && b0 + u < B ? hg[b0 + u] : 0ull;
          loc += h[u];
        }
        uint64_t v = scan(loc) - loc;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (u >= q) break;
          v += h[u];
          score(v, (g << 8) | (b0 + u));
        }
      }
    }
  };
  if (N < (uint32_t)kRecip)
    search(std::true_type{});
  else
    search(std::false_type{});
  const ArgMax am = wave_best(best, key);
  if (lane == am.lane) {
    Rec r;
    r.score = am.score;
    r.SL = bSL;
    r.NL = bNL;
    r.colbin = am.score >= 0.0 ? (read_lane(btl, am.key >> 8) & 0xFFu) << 8 | (uint32_t)(am.key & 0xFF) : 0u;
    x.sc.recs[(size_t)j * mtry + (uint32_t)ci0 / (uint32_t)a.big_cols] = r;
  }
  wave_lds_sync();
}

// A split decision: the column and bin, and the left child's weight and sum.
struct Decision {
  bool split;
  uint32_t col, bin, NL;
  int64_t SL;
  uint32_t cand;  // the split column's position among the node's candidates
};

// Decide a large or wide node from its records (columns ascending: keep the first
// strictly greater score).
__device__ __forceinline__ Decision decide_from_recs(const Rec* recs, int n_recs, int64_t S, uint32_t N) {
  double best = -1.0;
  int bi = -1;
  for (int i = 0; i < n_recs; ++i) {
    const double s = recs[i].score;
    if (s > best) {
      best = s;
      bi = i;
    }
  }
  Decision d{false, 0u, 0u, 0u, 0, 0u};
  if (bi >= 0 && best - parent_score(S, N) > 0.0) {
    const Rec r = recs[bi];
    d = Decision{true, r.colbin >> 8, r.colbin & 0xFFu, r.NL, r.SL, (uint32_t)bi};
  }
  return d;
}

constexpr int kWideMax = 8;  // nodes per workgroup-wide batch
constexpr int kTeams = 16;   // one-wave teams of a workgroup that holds the code matrix

struct SharedWide {
  // two wide batches (the one being searched and the next): node j's first
  // entry, rows, first chunk, weight, sum, and its candidates at
  // j * round_up(mtry, 8) + i
  uint32_t wstart[2][kWideMax], wlen[2][kWideMax], wcpre[2][kWideMax], wN[2][kWideMax];
  int64_t wS[2][kWideMax];
  alignas(8) uint8_t cand[2][256];
};
struct SharedNarrow {};

// A team's state in the LDS.
template <int BLOCK, bool WIDE>
struct Shared : std::conditional<WIDE, SharedWide, SharedNarrow>::type {
  // (one wave scans and sums without them)
  uint32_t tmp[BLOCK == kWave ? 1 : BLOCK / kWave + 1];
  uint64_t tmp64[BLOCK == kWave ? 1 : BLOCK / kWave + 1];
  uint64_t red[BLOCK == kWave ? 1 : BLOCK / kWave];
  uint32_t cnt[3 + kSegClasses];  // [1] large, [2] wide, [3..] small nodes per segment width
  uint32_t task;
  uint32_t next_task;  // the split-search tasks' queue head
  // the group being grown: its members' task indices, min.node.size, node
  // slots and in-bag bitmaps, and the level at which their trees part (first
  // node id, node count, next free id, entry buffer, levels grown, large and
  // wide nodes)
  int32_t gk, vi;  // members; the member being grown, -1 while their trees agree
  int64_t vmin, vbase;  // its min.node.size and node slot
  int32_t gtask[kGroupMax];
  int32_t gmin[kGroupMax];
  int64_t gbase[kGroupMax];
  int64_t ginbag[kGroupMax];
  uint32_t n_inbag;
  uint32_t f_lo, f_cnt, f_next, f_cur, f_levels, f_big, f_huge;
  uint32_t part;    // this level holds a node that is a leaf for some members only
  uint32_t resume;  // the member grows on from the decisions of the parting level
};

// Metadata of wide batch `bi` (nodes list[0 .. nb)) into buffer bi & 1.
template <int BLOCK>
__device__ __forceinline__ void wide_setup(const Ctx<false>& x, const NodeDesc* list, int nb, int bi, Shared<BLOCK, true>& sh) {
  const int mtry = x.T->mtry, tid = threadIdx.x, q = bi & 1;
  if (tid < nb) {
    const NodeDesc d = list[tid];
    uint32_t first = 0;
    for (int j = 0; j < tid; ++j) first += (list[j].len + kWave - 1) / kWave;
    sh.wstart[q][tid] = d.start;
    sh.wlen[q][tid] = d.len;
    sh.wcpre[q][tid] = first;
    sh.wN[q][tid] = d.N;
    sh.wS[q][tid] = d.S;
  }
  // candidates padded to 8 per node (with the node's last one), read 8 at a time
  const int cst = (mtry + 7) & ~7;
  for (int i = tid; i < nb * cst; i += BLOCK)
    sh.cand[q][i] = x.sc.cand[(size_t)list[i / cst].k * cand_stride(mtry) + min(i % cst, mtry - 1)];
}

// The wide nodes of a level, nb at a time.  Node j of a batch has its rows cut
// into chunks of 64, one wave per chunk, so the candidate columns are uniform
// across a wave.  Each lane reads its row's entry once and, when a row has at
// most 80 codes, the first 80 bytes of its padded code row with five 16-byte
// loads; the
// candidate codes are picked from registers and each is added to the packed
// bin of its (node, column) histogram (hc columns at a time when they do not
// all fit the LDS).  One wave per (node, column) then scans, writes the
// column's record (decided with the other nodes' after the phase) and zeroes
// the bins it read, while the next batch's metadata is staged.
template <int BLOCK>
__device__ __forceinline__ void wide_phase(const Ctx<false>& x, const NodeDesc* list, uint32_t n_wide, int nb_max, int hc, uint32_t rec_base,
                           uint8_t* lds, Shared<BLOCK, true>& sh) {
  constexpr int NW = BLOCK / kWave;
  const GrowArgs& a = *x.a;
  const int mtry = x.T->mtry;
  const int bs = a.bstride;
  const int cst = (mtry + 7) & ~7;
  const size_t sst = (size_t)cand_stride(mtry);
  const int tid = threadIdx.x, wid = tid / kWave, lane = (int)lane_id();
  uint64_t* H = reinterpret_cast<uint64_t*>(lds);
  const bool row_regs = a.C <= 80;
  // the histograms start zeroed; each scan zeroes what it read
  for (uint32_t i = 2 * tid; i < a.union_bytes / 8; i += 2 * BLOCK)
    *reinterpret_cast<uint4*>(H + i) = make_uint4(0u, 0u, 0u, 0u);
  wide_setup<BLOCK>(x, list, (int)min((uint32_t)nb_max, n_wide), 0, sh);
  __syncthreads();
  int bi = 0;
  for (uint32_t h0 = 0; h0 < n_wide; h0 += (uint32_t)nb_max, ++bi) {
    const int nb = (int)min((uint32_t)nb_max, n_wide - h0);
    const NodeDesc* bl = list + h0;
    const int q = bi & 1;
    uint32_t cpre[kWideMax];  // first chunk of node j (uniform)
    uint32_t n_chunks = 0;
#pragma unroll
    for (int j = 0; j < kWideMax; ++j) {
      cpre[j] = n_chunks;
      n_chunks += j < nb ? (bl[j].len + kWave - 1) / kWave : 0u;
    }
    // node of chunk ch: the number of later nodes' first chunks <= ch
    auto node_of = [&](uint32_t ch) {
      int j = 0;
#pragma unroll
      for (int jj = 1; jj < kWideMax; ++jj) j += (jj < nb && ch >= cpre[jj]) ? 1 : 0;
      return j;
    };
    for (int c0 = 0; c0 < mtry; c0 += hc) {
      const int nc = min(hc, mtry - c0);
      for (uint32_t ch = (uint32_t)wid; ch < n_chunks; ch += NW) {
        const int j = node_of(ch);
        const uint32_t r = (ch - sh.wcpre[q][j]) * kWave + (uint32_t)lane;
        const bool valid = r < sh.wlen[q][j];
        uint64_t v = 0;
        uint32_t row = 0;
        // this entry's slot of the candidate codes the partition reads back
        uint8_t* side_row = x.sc.side + (size_t)(sh.wstart[q][j] + r) * sst;
        if (valid) {
          const uint64_t e = x.buf[sh.wstart[q][j] + r];
          const uint32_t w = entry_w(e);
          v = pack_ns(w, (int64_t)w * entry_y(e));
          row = entry_row(e);
        }
        const uint8_t* cj = sh.cand[q] + j * cst + c0;
        uint64_t* Hj = H + (size_t)j * nc * bs;
        if (row_regs) {
          // five unconditional loads: the padded copy has 64 bytes of slack after
          // its last row, and a lane without a row reads row 0
          uint32_t rw[20];
          const uint4* rp = reinterpret_cast<const uint4*>(a.codes_p + (size_t)row * a.Cp);
#pragma unroll
          for (int u = 0; u < 5; ++u) {
            const uint4 t = rp[u];
            rw[4 * u] = t.x;
            rw[4 * u + 1] = t.y;
            rw[4 * u + 2] = t.z;
            rw[4 * u + 3] = t.w;
          }
          for (int i0 = 0; i0 < nc; i0 += 8) {
            const uint64_t c8 = *reinterpret_cast<const uint64_t*>(cj + i0);
            const uint32_t lo = rfl((uint32_t)c8), hi = rfl((uint32_t)(c8 >> 32));
            uint32_t sv0 = 0, sv1 = 0;  // the eight codes, for the partition
#pragma unroll
            for (int u = 0; u < 8; ++u) {
              const uint32_t col = ((u < 4 ? lo : hi) >> (8 * (u & 3))) & 0xFFu;
              const uint32_t code = (rw[col >> 2] >> (8 * (col & 3))) & 0xFFu;
              if (u < 4)
                sv0 |= code << (8 * u);
              else
                sv1 |= code << (8 * (u - 4));
              if (valid && i0 + u < nc)
                atomicAdd((unsigned long long*)&Hj[(i0 + u) * bs + (int)code], (unsigned long long)v);
            }
            if (valid) *reinterpret_cast<uint2*>(side_row + c0 + i0) = make_uint2(sv0, sv1);
          }
        } else {
          const uint8_t* rp = a.rcodes + (size_t)row * a.rC;
          for (int i0 = 0; i0 < nc; i0 += 8) {
            const uint64_t c8 = *reinterpret_cast<const uint64_t*>(cj + i0);
            uint32_t cd[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) cd[u] = valid ? rp[(uint32_t)(c8 >> (8 * u)) & 0xFFu] : 0u;
#pragma unroll
            for (int u = 0; u < 8; ++u)
              if (valid && i0 + u < nc)
                atomicAdd((unsigned long long*)&Hj[(i0 + u) * bs + (int)cd[u]], (unsigned long long)v);
            if (valid)
              *reinterpret_cast<uint2*>(side_row + c0 + i0) =
                  make_uint2(cd[0] | cd[1] << 8 | cd[2] << 16 | cd[3] << 24, cd[4] | cd[5] << 8 | cd[6] << 16 | cd[7] << 24);
          }
        }
      }
      __syncthreads();
      for (int t = wid; t < nb * nc; t += NW) {
        const int j = t / nc, i = t % nc;
        const int c = sh.cand[q][j * cst + c0 + i];
        const int B = a.n_bins[c];
        uint64_t* hv = H + (size_t)t * bs;
        uint32_t NL;
        int64_t SL;
        const ArgMax am = scan_packed(hv, B, sh.wN[q][j], sh.wS[q][j], NL, SL);
        if (lane == am.lane) {
          Rec rc;
          rc.score = am.score;
          rc.SL = SL;
          rc.NL = NL;
          rc.colbin = ((uint32_t)c << 8) | (uint32_t)(am.score >= 0.0 ? am.key : 0);
          x.sc.recs[(size_t)(rec_base + h0 + j) * mtry + c0 + i] = rc;
        }
        // zero the column's bins, four per lane (the scan's reads are done)
        if (4 * lane < B) *reinterpret_cast<uint4*>(hv + 4 * lane) = make_uint4(0u, 0u, 0u, 0u);
        if (4 * lane + 2 < B) *reinterpret_cast<uint4*>(hv + 4 * lane + 2) = make_uint4(0u, 0u, 0u, 0u);
      }
      // the next batch's metadata goes to the other buffer meanwhile
      if (c0 + hc >= mtry && h0 + (uint32_t)nb_max < n_wide)
        wide_setup<BLOCK>(x, list + h0 + nb_max, (int)min((uint32_t)nb_max, n_wide - h0 - nb_max), bi + 1, sh);
      __syncthreads();
    }
  }
}

// One wave per chunk of 64 entries of a split node: the lanes that go left take
// consecutive slots from the left cursor in lane order, the others from the
// right cursor, one atomic each; the left side's sum of w y^2 is added up on
// the way.  Rows of leaves are not touched again.  Four chunks per wave are in
// flight at a time, so that their dependent loads (chunk, entry, code)
// overlap.  `cur` is in LDS or in global memory (inlined once for each).
template <int BLOCK, bool WIDE, bool LC>
__device__ __forceinline__ void partition_level(const Ctx<LC>& x, uint64_t* __restrict__ out, Cursor* cur,
                                                uint32_t n_chunks) {
  constexpr int NW = BLOCK / kWave;
  constexpr int UP = 4;
  const int lane = (int)lane_id();
  const size_t sst = (size_t)cand_stride(x.T->mtry);
  for (uint32_t c0 = (uint32_t)team_tid<BLOCK>() / kWave; c0 < n_chunks; c0 += UP * NW) {
    uint32_t rk[UP], col[UP], bin[UP], sci[UP], pos[UP];
    uint64_t e[UP];
    bool mv[UP], go_left[UP];
#pragma unroll
    for (int u = 0; u < UP; ++u) {
      const uint32_t ch = c0 + (uint32_t)(u * NW);
      const uint4 cw = ch < n_chunks ? x.sc.chunks[ch] : make_uint4(0u, 0u, 0u, 0u);
      const uint32_t p0 = rfl(cw.x), en = rfl(cw.y), cb = rfl(cw.w);
      rk[u] = rfl(cw.z);
      col[u] = cb & 0xFFu;
      bin[u] = (cb >> 8) & 0xFFu;
      sci[u] = cb >> 16;
      pos[u] = p0 + (uint32_t)lane;
      mv[u] = pos[u] < en;
      e[u] = mv[u] ? x.buf[pos[u]] : 0ull;
    }
    // the split column's code: beside the entry when a wide batch searched the
    // node (candidate index + 1 in the chunk word), else from the row's codes
#pragma unroll
    for (int u = 0; u < UP; ++u) {
      uint32_t code = 0;
      if (mv[u]) {
        if constexpr (WIDE)
          code = sci[u] ? x.sc.side[(size_t)pos[u] * sst + (sci[u] - 1u)]
                        : x.row(entry_row(e[u]))[col[u]];
        else
          code = x.row(entry_row(e[u]))[col[u]];
      }
      go_left[u] = mv[u] && code <= bin[u];
    }
#pragma unroll
    for (int u = 0; u < UP; ++u) {
      if (c0 + (uint32_t)(u * NW) >= n_chunks) break;
      const uint64_t lm = __ballot(go_left[u]), rm = __ballot(mv[u] && !go_left[u]);
      const uint64_t below = (1ull << lane) - 1ull;
      uint32_t bl = 0, br = 0;
      if (lane == 0) {
        const uint32_t nl = (uint32_t)__popcll(lm), nr = (uint32_t)__popcll(rm);
        if (nl) bl = atomicAdd(&cur[rk[u]].L, nl);
        if (nr) br = atomicSub(&cur[rk[u]].R, nr) - nr;
      }
      bl = read_lane(bl, 0);
      br = read_lane(br, 0);
      if (mv[u]) out[go_left[u] ? bl + (uint32_t)__popcll(lm & below) : br + (uint32_t)__popcll(rm & below)] = e[u];
      const int64_t y = entry_y(e[u]);
      const uint64_t q = wave_sum(go_left[u] ? (uint64_t)((int64_t)entry_w(e[u]) * y * y) : 0ull);
      if (lane == 0 && q != 0) atomicAdd((unsigned long long*)&cur[rk[u]].q, (unsigned long long)q);
    }
  }
}

// A tree's bootstrap: n draws with replacement, draw i = floor(r_i n / 2^64) for
// the words r_i of the Philox stream (seed, tag 0, 0, tree); f(b, rows) gets the
// four draws of block b, those past the n-th as ~0.
template <int BLOCK, typename F>
__device__ __forceinline__ void bootstrap_draws(const TreeTask& T, int64_t n, F f) {
  const int64_t nblk = (n + 3) / 4;
  for (int64_t b = team_tid<BLOCK>(); b < nblk; b += BLOCK) {
    const U64x4 r = philox4x64_10((uint64_t)b, kTagBootstrap, 0, (uint64_t)T.tree, T.seed, 0);
    uint32_t d[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) d[w] = 4 * b + w < n ? (uint32_t)scale_draw(r.w[w], (uint32_t)n) : ~0u;
    f(b, make_uint4(d[0], d[1], d[2], d[3]));
  }
}

// The trees of one group: K tasks that differ only in min.node.size (sh.gtask,
// by min.node.size ascending; a lone task is a group of one), T being the
// first.  Their trees agree node for node down to the first level holding an
// open node whose leaf rule depends on min.node.size (more weight than the
// smallest value, at most the largest, and not pure), since every other step
// (bootstrap, candidate draws by node id, searches, child ids) is the same.
// Those levels, and the split searches of the parting level itself, are done
// once, with the smallest value (every node open for some member is searched,
// and a search does not depend on min.node.size).  The parting level's state
// is then put aside as the searches left it, and each member in turn grows its
// own tree on from its decisions: the nodes of at most its min.node.size are
// made leaves, the shared levels' node words are copied into its slot.  The
// work counters count the work done: the shared levels, searches included,
// count for the group's first member.
// WIDE: the launch may hold nodes above the wide limit (the kernel without
// the wide-batch phase is compiled separately, so that small training sets
// keep its leaner register allocation).  GROUPED: the launch has groups (the
// kernels of launches without compile the group logic out, which keeps their
// register allocation as it was).
// LC: the code matrix is in the LDS, at lcodes.  nbins: the columns' bin counts,
// in the LDS.
template <int BLOCK, bool WIDE, bool GROUPED, bool LC>
__device__ __forceinline__ void grow_group(const GrowArgs& a, const TreeTask& T, const Scratch& sc, uint8_t* lds,
                                           Shared<BLOCK, WIDE>& sh, const uint16_t* nbins, const double* recip,
                                           const uint8_t* lcodes) {
  constexpr int NW = BLOCK / kWave;
  const int tid = team_tid<BLOCK>(), wid = tid / kWave, lane = (int)lane_id();
  const int64_t n = T.n_train;
  const int32_t* train = T.train_off >= 0 ? a.train_rows + T.train_off : nullptr;
  const int mtry = T.mtry;

  // 1. bootstrap multiplicities, counted in the LDS union area (free until the
  // first level), as many rows at a time as it holds.  When that takes more than
  // one pass the draws are written out once and read by each pass: counters in
  // global memory, an atomic through the L2 per draw, made the launch of 500
  // trees of 200000 rows 63.1 ms, the seven passes make it 59.0.  Below 2^16 draws
  // no count exceeds 16 bits, which leaves one-wave teams a single pass for the
  // tuning grid's 2000 rows (201.0 ms; 205.6 with two passes of 32-bit counters).
  uint32_t* const cnt = reinterpret_cast<uint32_t*>(lds);
  const uint32_t h = n < (1 << 16) ? 1u : 0u;  // 16-bit counters, two to a word
  const int64_t span = (int64_t)((a.union_bytes / 4u) << h) & ~(int64_t)(kWave - 1);
  uint4* const draws = reinterpret_cast<uint4*>(sc.draws);
  if (T.bootstrap && n > span) bootstrap_draws<BLOCK>(T, n, [&](int64_t b, uint4 d) { draws[b] = d; });
  // in-bag entries and root sums; each thread takes eight rows per pass,
  // strided by the block, so a pass costs one workgroup scan (the order of the
  // entries is free: every later sum over them is exact)
  uint32_t n_inbag = 0;
  uint64_t N0 = 0, Q0 = 0;
  int64_t S0 = 0;
  constexpr int R = 8;
  for (int64_t lo = 0; lo < n; lo += span) {
    const int64_t hi = min(n, lo + span);
    const uint32_t rows = (uint32_t)(hi - lo), off = (uint32_t)lo;
    if (T.bootstrap) {
      for (uint32_t i = (uint32_t)tid; i << h < rows; i += BLOCK) cnt[i] = 0u;
      team_sync<BLOCK>();
      const auto count1 = [&](uint32_t i) {
        if (i < rows) atomicAdd(&cnt[i >> h], 1u << ((i & h) << 4));
      };
      const auto count = [&](int64_t, uint4 d) {
        count1(d.x - off);
        count1(d.y - off);
        count1(d.z - off);
        count1(d.w - off);
      };
      if (n > span) {
        const int64_t nblk = (n + 3) / 4;
        for (int64_t b = tid; b < nblk; b += BLOCK) count(b, draws[b]);
      } else {
        bootstrap_draws<BLOCK>(T, n, count);
      }
      team_sync<BLOCK>();
    }
    for (int64_t base = lo; base < hi; base += (int64_t)R * BLOCK) {
      uint32_t c[R];
      uint32_t mine = 0;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int64_t i = base + (int64_t)r * BLOCK + tid;
        const uint32_t j = (uint32_t)(i - lo);
        c[r] = i >= hi ? 0u : !T.bootstrap ? 1u : h ? cnt[j >> 1] >> ((j & 1) << 4) & 0xFFFFu : cnt[j];
        mine += c[r] > 0 ? 1u : 0u;
        // in-bag bitmap: this wave's 64 consecutive rows form one word
        const uint64_t bits = __ballot(c[r] > 0);
        const int64_t wbase = base + (int64_t)r * BLOCK + (int64_t)(tid / kWave) * kWave;
        if (lane_id() == 0 && T.inbag_off >= 0 && wbase < hi) {
          if (GROUPED)
            for (int v = 0; v < sh.gk; ++v) a.inbag[sh.ginbag[v] + wbase / kWave] = bits;
          else
            a.inbag[T.inbag_off + wbase / kWave] = bits;
        }
      }
      uint32_t total;
      uint32_t pos = block_exscan<BLOCK>(mine, sh.tmp, total) + n_inbag;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (c[r] > 0) {
          const int64_t i = base + (int64_t)r * BLOCK + tid;
          const uint32_t row = train ? (uint32_t)train[i] : (uint32_t)i;
          const int64_t y = a.y_fp[row];
          sc.L0.buf[pos++] = entry_pack(row, c[r], y);
          N0 += c[r];
          S0 += (int64_t)c[r] * y;
          Q0 += (uint64_t)((int64_t)c[r] * y * y);
        }
      }
      n_inbag += total;
    }
    team_sync<BLOCK>();
  }
  N0 = block_sum<BLOCK, uint64_t>(N0, sh.red);
  S0 = (int64_t)block_sum<BLOCK, uint64_t>((uint64_t)S0, sh.red);
  Q0 = block_sum<BLOCK, uint64_t>(Q0, sh.red);
  if (tid == 0) {
    sc.L0.mstart[0] = 0;
    sc.L0.mend[0] = n_inbag;
    sc.L0.mN[0] = (uint32_t)N0;
    sc.L0.mS[0] = S0;
    sc.L0.mQ[0] = Q0;
  }
  if (tid < 3 + kSegClasses) sh.cnt[tid] = 0;
  if (tid == 0) {
    sh.next_task = NW;
    sh.n_inbag = n_inbag;
    sh.vi = sh.gk > 1 ? -1 : 0;
    sh.vmin = sh.gmin[0];
    sh.vbase = sh.gbase[0];
    sh.part = 0;
    sh.resume = 0;
  }
  team_sync<BLOCK>();

  // threads that draw candidates each own a C-byte row of the LDS union area
  const int n_draw = min(BLOCK, (int)(a.union_bytes / (uint32_t)a.C));
  const uint32_t draw_q = ((uint32_t)n_draw * (uint32_t)a.C + 15u) & ~15u;  // the draw queue, after the rows
  // (the member being grown, its min.node.size and node slot are kept in the
  // LDS, which spares registers across the level loop)
  uint32_t level_lo = 0, level_cnt = 1, next_id = 1;
  int cur = 0;
  uint64_t work_rows = 0, work_nodes = 0, work_part = 0, levels = 0, work_hist = 0;
  for (;;) {
    while (level_cnt > 0) {
      const Level2 C = cur ? sc.L1 : sc.L0;  // this level
      const Level2 X = cur ? sc.L0 : sc.L1;  // the next level
      const Ctx<LC> x{&a, &T, lcodes, recip, sc, C.buf, X.buf, C.mstart, C.mend, C.mN, C.mS, C.mQ};
      // (a) - (c) are skipped by a member that grows on from the parting level
      if (!GROUPED || !sh.resume) {
        ++levels;
        // (a) leaf rules, candidate draws, tiers (the tier counts and the task
        // queue head were reset before the level began).  A one-wave workgroup
        // queues its open nodes in the LDS after the draw rows (node and large-node
        // index, 128 entries) and draws them 64 at a time, so that a level whose
        // open nodes are sparse among its nodes runs the draws fewer times.
        const bool queue_draws = BLOCK == kWave && n_draw == kWave && draw_q + 1024u <= a.union_bytes;
        if (tid < n_draw) {
          const int64_t min_node = GROUPED ? sh.vmin : (int64_t)T.min_node;
          // while the members' trees agree: an open node of at most the largest
          // member's min.node.size is a leaf for some members only
          const int64_t m_part = GROUPED && sh.vi < 0 ? (int64_t)sh.gmin[sh.gk - 1] : -1;
          uint32_t* const qk = reinterpret_cast<uint32_t*>(lds + draw_q);
          uint32_t* const qj = qk + 128;
          uint32_t q_head = 0, q_tail = 0;
          auto draw_queued = [&](uint32_t n_q) {
            if ((uint32_t)tid < n_q) {
              const uint32_t e = (q_head + (uint32_t)tid) & 127u;
              const uint32_t k = qk[e], j1 = qj[e];
              draw_candidates(lds + tid, n_draw, T.seed, level_lo + k, (uint32_t)T.tree, a.C, mtry,
                              sc.cand + (size_t)k * cand_stride(mtry), j1 ? sc.btask + (size_t)(j1 - 1) * mtry : nullptr,
                              nbins);
            }
            q_head += n_q;
          };
          const uint32_t k_end = queue_draws ? (level_cnt + kWave - 1) / kWave * kWave : level_cnt;
          for (uint32_t k = tid; k < k_end; k += n_draw) {
            bool open = false;
            uint32_t j1 = 0;  // large node j: j + 1
            uint32_t* bt = nullptr;
            if (k < level_cnt) {
              const uint32_t N = x.mN[k];
              const int64_t S = x.mS[k];
              const uint64_t Q = x.mQ[k];
              const uint32_t st = x.mstart[k];
              const uint32_t len = x.mend[k] - st;
              if ((int64_t)N <= min_node || node_is_pure(N, S, Q)) {
                sc.status[k] = kLeaf;
              } else {
                open = true;
                if (GROUPED && (int64_t)N <= m_part) sh.part = 1u;
                work_rows += len;
                ++work_nodes;
                // nodes above 32 rows add each row to an LDS bin per candidate column
                if (len > 32) work_hist += (uint64_t)len * (uint64_t)mtry;
                if (len <= kSegMax) {
                  const int cls = len <= 4 ? 0 : len <= 8 ? 1 : len <= 16 ? 2 : len <= 32 ? 3 : 4;
                  sc.status[k] = kSmall;
                  NodeDesc* list = cls == 0   ? sc.seg[0]
                                   : cls == 1 ? sc.seg[1]
                                   : cls == 2 ? sc.seg[2]
                                   : cls == 3 ? sc.seg[3]
                                              : sc.seg[4];
                  list[atomicAdd(&sh.cnt[3 + cls], 1u)] = NodeDesc{k, st, len, N, S};
                } else if (!WIDE || (int32_t)len <= a.huge_min) {
                  sc.status[k] = kBig;
                  const uint32_t j = atomicAdd(&sh.cnt[1], 1u);
                  sc.big[j] = NodeDesc{k, st, len, N, S};
                  sc.ridx[k] = j;
                  j1 = j + 1;
                  bt = sc.btask + (size_t)j * mtry;  // each (node, column) task's column and bin count
                } else {
                  sc.status[k] = kHuge;
                  const uint32_t h = atomicAdd(&sh.cnt[2], 1u);
                  sc.huge[h] = NodeDesc{k, st, len, N, S};
                  sc.ridx[k] = h;
                }
              }
            }
            if (queue_draws) {
              const uint64_t om = __ballot(open);
              if (open) {
                const uint32_t e = (q_tail + (uint32_t)__popcll(om & ((1ull << lane) - 1ull))) & 127u;
                qk[e] = k;
                qj[e] = j1;
              }
              q_tail += (uint32_t)__popcll(om);
              wave_lds_sync();
              if (q_tail - q_head >= (uint32_t)kWave) {
                draw_queued(kWave);
                wave_lds_sync();
              }
            } else if (open) {
              draw_candidates(lds + tid, n_draw, T.seed, level_lo + k, (uint32_t)T.tree, a.C, mtry,
                              sc.cand + (size_t)k * cand_stride(mtry), bt, nbins);
            }
          }
          if (queue_draws && q_tail > q_head) draw_queued(q_tail - q_head);
        }
        team_sync<BLOCK>();
        const uint32_t n_big = sh.cnt[1], n_huge = sh.cnt[2];
        // (b) wide nodes, in batches, with the whole workgroup
        if (WIDE && n_huge > 0) {
          const int per_node = mtry * a.bstride * 8;
          int nb = 1, hc = mtry;
          if (per_node <= (int)a.union_bytes)
            nb = min(min(kWideMax, 256 / ((mtry + 7) & ~7)), (int)a.union_bytes / per_node);
          // (records of wide node j go after the large nodes', at n_big + j)
          else  // column chunks of a multiple of 8 (the LDS holds at least 8 columns)
            hc = max(8, (int)a.union_bytes / (a.bstride * 8) / 8 * 8);
          if constexpr (WIDE) wide_phase<BLOCK>(x, sc.huge, n_huge, nb, hc, n_big, lds, sh);
        }
        // (c) large-node columns and small-node segments, one wave each; a wave
        // takes its next task from the queue head when it starts one (their costs
        // differ widely, so a fixed deal would leave waves idle at the barrier)
        {
          const uint32_t per_big = (uint32_t)((mtry + a.big_cols - 1) / a.big_cols);
          const uint32_t n_big_tasks = n_big * per_big;
          uint32_t first[kSegClasses + 1];
          first[0] = n_big_tasks;
          for (int c = 0; c < kSegClasses; ++c) {
            const uint32_t per_wave = (uint32_t)(kWave >> (2 + c));
            first[c + 1] = first[c] + (sh.cnt[3 + c] + per_wave - 1) / per_wave;
          }
          WaveHist& wl = *reinterpret_cast<WaveHist*>(lds + (size_t)wid * a.wave_bytes);
          for (uint32_t t = wid; t < first[kSegClasses];) {
            uint32_t t_next = 0;
            if (lane == 0) t_next = atomicAdd(&sh.next_task, 1u);
            if (t < n_big_tasks)
              big_task<LC>(x, t / per_big, (int)(t % per_big) * a.big_cols, wl);
            else if (t < first[1])
              small_task<4, LC>(x, sc.seg[0], t - first[0], sh.cnt[3], wl);
            else if (t < first[2])
              small_task<8, LC>(x, sc.seg[1], t - first[1], sh.cnt[4], wl);
            else if (t < first[3])
              small_task<16, LC>(x, sc.seg[2], t - first[2], sh.cnt[5], wl);
            else if (t < first[4])
              small_task<32, LC>(x, sc.seg[3], t - first[3], sh.cnt[6], wl);
            else
              rank_task<LC>(x, sc.seg[4], t - first[4], sh.cnt[7], wl);
            t = read_lane(t_next, 0);
          }
        }
        team_sync<BLOCK>();
        if (GROUPED && sh.part) {
          // the members' trees part at this level: put its searched state aside
          // (the open nodes' entries lie in [0, n_inbag)); the first member goes on
          const uint32_t ni = sh.n_inbag;
          for (uint32_t i = tid; i < ni; i += BLOCK) {
            sc.SN.L.buf[i] = C.buf[i];
            sc.SN.nbuf[i] = X.buf[i];
          }
          for (uint32_t k = tid; k < level_cnt; k += BLOCK) {
            sc.SN.L.mstart[k] = C.mstart[k];
            sc.SN.L.mend[k] = C.mend[k];
            sc.SN.L.mN[k] = C.mN[k];
            sc.SN.L.mS[k] = C.mS[k];
            sc.SN.L.mQ[k] = C.mQ[k];
            sc.SN.status[k] = sc.status[k];
            sc.SN.ridx[k] = sc.ridx[k];
            sc.SN.dcol[k] = sc.dcol[k];
            sc.SN.dbin[k] = sc.dbin[k];
            sc.SN.dNL[k] = sc.dNL[k];
            sc.SN.dSL[k] = sc.dSL[k];
            sc.SN.dcnt[k] = sc.dcnt[k];
            sc.SN.dQL[k] = sc.dQL[k];
          }
          for (uint32_t i = tid; i < (n_big + n_huge) * (uint32_t)mtry; i += BLOCK) sc.SN.recs[i] = sc.recs[i];
          if (WIDE && n_huge > 0) {
            const uint4* src = reinterpret_cast<const uint4*>(sc.side);
            uint4* dst = reinterpret_cast<uint4*>(sc.SN.side);
            for (uint32_t i = tid; i < ni * (uint32_t)cand_stride(mtry) / 16u; i += BLOCK) dst[i] = src[i];
          }
          team_sync<BLOCK>();  // (every thread has read the flag)
          if (tid == 0) {
            sh.part = 0;
            sh.vi = 0;
            sh.f_lo = level_lo;
            sh.f_cnt = level_cnt;
            sh.f_next = next_id;
            sh.f_cur = (uint32_t)cur;
            sh.f_levels = (uint32_t)levels;
            sh.f_big = n_big;
            sh.f_huge = n_huge;
          }
        }
      }
      const uint32_t n_big = sh.cnt[1];
      // (d) the large and wide nodes' decisions from their records (the wide
      // nodes' records follow the large nodes'), then (e) breadth-first child
      // ids, node words, children's sums and cursors, and the partition's chunks
      // of 64 entries of every split node that is not placed yet.  The cursors
      // live in the LDS union area (free until the next level) when the level's
      // nodes fit it, else in scratch.
      const bool lds_cur = level_cnt <= a.union_bytes / (uint32_t)sizeof(Cursor);
      const int64_t base_node = GROUPED ? sh.vbase : T.node_base;
      Cursor* lcur = reinterpret_cast<Cursor*>(lds);
      uint32_t n_split = 0, n_chunks = 0;
      for (uint32_t b0 = 0; b0 < level_cnt; b0 += BLOCK) {
        const uint32_t k = b0 + tid;
        const bool in = k < level_cnt;
        uint8_t stk = in ? sc.status[k] : kLeaf;
        Decision dc{false, 0u, 0u, 0u, 0, 0u};
        // a wide node's rows carry their candidate codes (candidate index + 1 in
        // the partition's chunk word; 0 = read the row's code)
        uint32_t side_ci = 0;
        if (stk == kBig || stk == kHuge) {
          // a large node has a record per task, a wide one per candidate column
          const uint32_t ri = sc.ridx[k] + (stk == kHuge ? n_big : 0u);
          const int n_recs = stk == kHuge ? mtry : (mtry + a.big_cols - 1) / a.big_cols;
          dc = decide_from_recs(sc.recs + (size_t)ri * mtry, n_recs, x.mS[k], x.mN[k]);
          if (WIDE && stk == kHuge) side_ci = dc.cand + 1u;
          stk = dc.split ? kSplit : kLeaf;
        } else if (stk == kSplitDone) {
          dc = Decision{true, sc.dcol[k], sc.dbin[k], sc.dNL[k], sc.dSL[k], 0u};
        }
        const bool split = stk == kSplit || stk == kSplitDone;
        // (the small nodes' rows were placed by their searches)
        const uint32_t nch = stk == kSplit ? (x.mend[k] - x.mstart[k] + kWave - 1) / kWave : 0u;
        // split ranks in the low half, chunk offsets in the high half
        uint64_t tot;
        const uint64_t ex = block_exscan64<BLOCK>((split ? 1ull : 0ull) | ((uint64_t)nch << 32), sh.tmp64, tot);
        const uint32_t total = (uint32_t)tot, ctotal = (uint32_t)(tot >> 32);
        const uint32_t r = (uint32_t)ex + n_split;
        const uint32_t cfirst = (uint32_t)(ex >> 32) + n_chunks;
        // (the bounds below hold by construction; the guards keep a broken
        // invariant from writing outside the scratch arrays)
        if (nch > 0 && (uint64_t)cfirst + nch <= (uint64_t)(a.n_cap / 64 + a.n_cap / 2 + 2)) {
          const uint32_t st = x.mstart[k], en = x.mend[k], cb = dc.col | (dc.bin << 8) | (side_ci << 16);
          for (uint32_t c = 0; c < nch; ++c) sc.chunks[cfirst + c] = make_uint4(st + c * kWave, en, r, cb);
        }
        if (in) {
          const uint32_t node = level_lo + k;
          const uint32_t N = x.mN[k];
          const int64_t S = x.mS[k];
          if (split && (int64_t)2 * r + 1 >= a.n_cap) {
            atomicOr(a.status, kStatusCapacity);
          } else if (split) {
            const uint32_t left = next_id + 2 * r;
            if ((int64_t)left + 1 < T.capacity) {
              a.nodes[base_node + node] = node_split(dc.col, dc.bin, left);
            } else {
              atomicOr(a.status, kStatusCapacity);
            }
            const uint32_t st = x.mstart[k], en = x.mend[k];
            work_part += en - st;
            // a placed node's boundary is known; its cursor is marked done
            const bool done = stk == kSplitDone;
            const Cursor c0{done ? 0xFFFFFFFFu : st, en, 0ull};
            if (lds_cur)
              lcur[r] = c0;
            else
              sc.cur[r] = c0;
            if (done) {
              const uint32_t b = st + sc.dcnt[k];
              const uint64_t QL = sc.dQL[k];
              X.mend[2 * r] = b;
              X.mstart[2 * r + 1] = b;
              X.mQ[2 * r] = QL;
            }
            const uint32_t NL = dc.NL;
            const int64_t SL = dc.SL;
            X.mstart[2 * r] = st;
            X.mN[2 * r] = NL;
            X.mS[2 * r] = SL;
            X.mend[2 * r + 1] = en;
            X.mN[2 * r + 1] = N - NL;
            X.mS[2 * r + 1] = S - SL;
            // the right side's: the parent's, less the left side's when known
            X.mQ[2 * r + 1] = x.mQ[k] - (done ? sc.dQL[k] : 0ull);
          } else {
            a.nodes[base_node + node] = node_leaf(leaf_value(N, S));
          }
          a.node_N[base_node + node] = N;
        }
        n_split += total;
        n_chunks += ctotal;
      }
      team_sync<BLOCK>();
      if ((int64_t)next_id + 2 * (int64_t)n_split > T.capacity ||
          (int64_t)n_chunks > a.n_cap / 64 + a.n_cap / 2 + 2) {
        // cannot happen for consistent inputs: every child holds an in-bag row
        if (tid == 0) atomicOr(a.status, kStatusCapacity);
        next_id = (uint32_t)T.capacity;
        break;
      }
      // (f) partition the entries of split nodes into their children's segments
      if (lds_cur)
        partition_level<BLOCK, WIDE, LC>(x, X.buf, lcur, n_chunks);
      else
        partition_level<BLOCK, WIDE, LC>(x, X.buf, sc.cur, n_chunks);
      team_sync<BLOCK>();
      // (g) the boundary between each pair of children, and their sums of w y^2
      for (uint32_t r = tid; r < n_split; r += BLOCK) {
        const Cursor c = lds_cur ? lcur[r] : sc.cur[r];
        if (c.L == 0xFFFFFFFFu) continue;  // placed by its search
        X.mend[2 * r] = c.L;
        X.mstart[2 * r + 1] = c.L;
        X.mQ[2 * r] = c.q;
        X.mQ[2 * r + 1] -= c.q;
      }
      // the next level's tier counts and task queue head
      if (tid < 3 + kSegClasses) sh.cnt[tid] = 0;
      if (tid == 0) {
        sh.next_task = NW;
        if (GROUPED) sh.resume = 0;
      }
      team_sync<BLOCK>();
      level_lo = next_id;
      level_cnt = 2 * n_split;
      next_id += 2 * n_split;
      cur ^= 1;
    }
    // the tree of member max(vi, 0) is complete
    work_rows = block_sum<BLOCK, uint64_t>(work_rows, sh.red);
    work_nodes = block_sum<BLOCK, uint64_t>(work_nodes, sh.red);
    work_part = block_sum<BLOCK, uint64_t>(work_part, sh.red);
    work_hist = block_sum<BLOCK, uint64_t>(work_hist, sh.red);
    const int vi = GROUPED ? sh.vi : 0, K = GROUPED ? sh.gk : 1;
    const int64_t base_node = GROUPED ? sh.vbase : T.node_base;
    const int v0 = vi < 0 ? 0 : vi;
    // without a parting level every member's tree is the first one's
    const int v1 = vi < 0 ? K : vi + 1;
    for (int v = v0; v < v1; ++v) {
      if (v > v0) {
        const int64_t b = sh.gbase[v];
        for (uint32_t i = tid; i < next_id; i += BLOCK) {
          a.nodes[b + i] = a.nodes[base_node + i];
          a.node_N[b + i] = a.node_N[base_node + i];
        }
      }
      if (tid == 0) {
        const int64_t ti = GROUPED ? sh.gtask[v] : sh.gtask[0];
        a.n_nodes[ti] = (int32_t)next_id;
        int64_t* wk = a.work + kWorkWords * ti;
        const bool first = v == v0;
        wk[0] = first ? (int64_t)work_rows : 0;
        wk[1] = first ? (int64_t)work_nodes : 0;
        wk[2] = first ? (int64_t)work_part : 0;
        wk[3] = (int64_t)levels;
        wk[4] = first ? (int64_t)work_hist : 0;
      }
    }
    if (vi < 0 || vi + 1 == K) break;
    // member vi + 1 grows on from the parting level's decisions: its searched
    // state restored, the nodes of at most its min.node.size made leaves, the
    // shared levels' node words copied into its slot
    const int64_t nbase = sh.gbase[vi + 1], m_v = sh.gmin[vi + 1];
    level_lo = sh.f_lo;
    level_cnt = sh.f_cnt;
    next_id = sh.f_next;
    cur = (int)sh.f_cur;
    levels = sh.f_levels;
    work_rows = work_nodes = work_part = work_hist = 0;
    {
      const uint32_t f_big = sh.f_big, f_huge = sh.f_huge;
      const int64_t b0 = sh.gbase[0];
      for (uint32_t i = tid; i < level_lo; i += BLOCK) {
        a.nodes[nbase + i] = a.nodes[b0 + i];
        a.node_N[nbase + i] = a.node_N[b0 + i];
      }
      const Level2 C = cur ? sc.L1 : sc.L0;
      const Level2 X = cur ? sc.L0 : sc.L1;
      const uint32_t ni = sh.n_inbag;
      for (uint32_t i = tid; i < ni; i += BLOCK) {
        C.buf[i] = sc.SN.L.buf[i];
        X.buf[i] = sc.SN.nbuf[i];
      }
      for (uint32_t k = tid; k < level_cnt; k += BLOCK) {
        const uint32_t N = sc.SN.L.mN[k];
        C.mstart[k] = sc.SN.L.mstart[k];
        C.mend[k] = sc.SN.L.mend[k];
        C.mN[k] = N;
        C.mS[k] = sc.SN.L.mS[k];
        C.mQ[k] = sc.SN.L.mQ[k];
        const uint8_t st = sc.SN.status[k];
        sc.status[k] = (int64_t)N <= m_v ? kLeaf : st;
        sc.ridx[k] = sc.SN.ridx[k];
        sc.dcol[k] = sc.SN.dcol[k];
        sc.dbin[k] = sc.SN.dbin[k];
        sc.dNL[k] = sc.SN.dNL[k];
        sc.dSL[k] = sc.SN.dSL[k];
        sc.dcnt[k] = sc.SN.dcnt[k];
        sc.dQL[k] = sc.SN.dQL[k];
      }
      for (uint32_t i = tid; i < (f_big + f_huge) * (uint32_t)mtry; i += BLOCK) sc.recs[i] = sc.SN.recs[i];
      if (WIDE && f_huge > 0) {
        const uint4* src = reinterpret_cast<const uint4*>(sc.SN.side);
        uint4* dst = reinterpret_cast<uint4*>(sc.side);
        for (uint32_t i = tid; i < ni * (uint32_t)cand_stride(mtry) / 16u; i += BLOCK) dst[i] = src[i];
      }
      team_sync<BLOCK>();  // (every thread has read the member index)
      if (tid < 3 + kSegClasses) sh.cnt[tid] = tid == 1 ? f_big : tid == 2 ? f_huge : 0u;
    }
    if (tid == 0) {
      sh.next_task = NW;
      sh.vi = vi + 1;
      sh.vmin = m_v;
      sh.vbase = nbase;
      sh.resume = 1;
    }
    team_sync<BLOCK>();
  }
  (void)wid;
}

// A team's loop over the queue of task groups, with scratch area `area`.
template <int BLOCK, bool WIDE, bool GROUPED, bool LC>
__device__ __forceinline__ void grow_queue(const GrowArgs& a, uint32_t area, uint8_t* lds, Shared<BLOCK, WIDE>& sh,
                                           const uint16_t* nbins, const double* recip, const uint8_t* lcodes) {
  const int tid = team_tid<BLOCK>();
  Scratch sc;
  carve(&sc, reinterpret_cast<uintptr_t>(a.scratch) + a.scratch_stride * area, a.n_cap, a.mtry_max, WIDE, GROUPED);
  for (;;) {
    if (tid == 0) sh.task = atomicAdd(a.queue, 1u);
    team_sync<BLOCK>();
    const uint32_t g = sh.task;
    if (g >= (uint32_t)a.n_groups) return;
    // the group's members (the host keeps a group within kGroupMax tasks)
    const int32_t gf = GROUPED ? a.group_first[g] : (int32_t)g;
    const int K = GROUPED ? min(a.group_first[g + 1] - gf, kGroupMax) : 1;
    if (tid == 0) sh.gk = K;
    if (tid < K) {
      const int32_t ti = GROUPED ? a.group_task[gf + tid] : (int32_t)g;
      sh.gtask[tid] = ti;
      sh.gmin[tid] = a.tasks[ti].min_node;
      sh.gbase[tid] = a.tasks[ti].node_base;
      sh.ginbag[tid] = a.tasks[ti].inbag_off;
    }
    team_sync<BLOCK>();
    const TreeTask T = uniform(a.tasks[rfl((uint32_t)sh.gtask[0])]);
    grow_group<BLOCK, WIDE, GROUPED, LC>(a, T, sc, lds, sh, nbins, recip, lcodes);
    team_sync<BLOCK>();
  }
}

// OCC waves per SIMD (at most 512 / OCC VGPRs): the persistent kernel is bound
// by latency, so resident waves can matter more than the registers it spills;
// the kernel with the wide phase keeps four, the other is built for 4, 5 and 6.
template <int BLOCK, bool WIDE, int OCC, bool GROUPED>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(OCC))) void k_grow(GrowArgs a) {
  extern __shared__ __align__(16) uint8_t lds[];
  __shared__ Shared<BLOCK, WIDE> sh;
  __shared__ uint16_t nbins[256];
  __shared__ double recip[kRecip];
  // a code at or above its column's bin count (flagged by the prepare kernel,
  // which ran before on this stream) would index past a histogram: grow nothing
  // and let the fit report EINVAL
  if (__atomic_load_n(a.status, __ATOMIC_RELAXED) & kStatusBadCode) return;
  for (int c = threadIdx.x; c < a.C; c += BLOCK) nbins[c] = (uint16_t)a.n_bins[c];
  fill_recip<BLOCK>(recip);
  team_sync<BLOCK>();
  grow_queue<BLOCK, WIDE, GROUPED, false>(a, blockIdx.x, lds, sh, nbins, recip, nullptr);
}

// Trees of a deep queue over a small code matrix: a workgroup holds the matrix in
// its LDS, and each of its waves is a team of its own, growing one tree after the
// other.  The waves never wait for one another.  Gathering a row's codes from
// memory took a cache lookup per lane (the tuning grid's launch: 1.3e11, 67 % of
// the address unit's cycles) and its latency at every candidate; from the LDS
// the lookups fall to 2.7e10.  One matrix for sixteen waves leaves each 4.9 KB of
// the 160 KB (2220 rows x 35 columns) and 128 registers at four waves per SIMD,
// against 96 registers and five waves for one-wave workgroups (twelve teams
// at 168 registers: 302 ms).  Grid 287 -> 261 ms, leave-one-kernel-out 33.7 ->
// 32.2 ms, with the small nodes' sums by matrix instructions.
template <bool GROUPED>
__global__ __launch_bounds__(kTeams* kWave) __attribute__((amdgpu_waves_per_eu(kTeams / 4))) void k_grow_teams(GrowArgs a) {
  extern __shared__ __align__(16) uint8_t lds[];
  if (__atomic_load_n(a.status, __ATOMIC_RELAXED) & kStatusBadCode) return;  // (as in k_grow)
  const int tid = (int)threadIdx.x, team = (int)rfl((uint32_t)tid / kWave);
  uint8_t* lcodes = lds;
  double* recip = reinterpret_cast<double*>(lds + a.lcode_bytes);
  uint16_t* nbins = reinterpret_cast<uint16_t*>(recip + kRecip);
  for (int c = tid; c < a.C; c += kTeams * kWave) nbins[c] = (uint16_t)a.n_bins[c];
  const uint32_t total = a.lcode_rows * (uint32_t)a.C;
  for (uint32_t i = (uint32_t)tid; i < total; i += kTeams * kWave) lcodes[i] = a.codes[i];
  fill_recip<kTeams * kWave>(recip);
  __syncthreads();
  uint8_t* own = reinterpret_cast<uint8_t*>(nbins + 256) + (size_t)team * a.team_bytes;
  auto& sh = *reinterpret_cast<Shared<kWave, false>*>(own + a.union_bytes);
  grow_queue<kWave, false, GROUPED, true>(a, blockIdx.x * (uint32_t)kTeams + (uint32_t)team, own, sh, nbins, recip,
                                          lcodes);
}

// The grow kernel of this translation unit for a launch shape (block, wide
// phase, waves per SIMD): the kernels for launches with task groups are built
// in a unit of their own (which includes this file with AIWC_GROW_GROUPED set),
// so that the two sets compile in parallel.
#ifndef AIWC_GROW_GROUPED
#define AIWC_GROW_GROUPED 0
#endif
template <int BLOCK>
const void* grow_kernel(bool wide, int occ) {
  constexpr bool G = AIWC_GROW_GROUPED != 0;
  if constexpr (BLOCK < 192) {
    // one- and two-wave workgroups serve deep queues of small trees only
    if (wide) fail(AIWC_RF_EINVAL, "the workgroup-wide phase needs at least 192 threads per workgroup");
  } else {
    if (wide) return reinterpret_cast<const void*>(k_grow<BLOCK, true, 4, G>);
  }
  switch (occ) {
    case 5: return reinterpret_cast<const void*>(k_grow<BLOCK, false, 5, G>);
    case 6: return reinterpret_cast<const void*>(k_grow<BLOCK, false, 6, G>);
    default: return reinterpret_cast<const void*>(k_grow<BLOCK, false, 4, G>);
  }
}

const void* grow_kernel_block(int block, bool wide, int occ, bool teams) {
  if (teams) {
    constexpr bool G = AIWC_GROW_GROUPED != 0;
    return reinterpret_cast<const void*>(k_grow_teams<G>);
  }
  switch (block) {
    case 64: return grow_kernel<64>(wide, occ);
    case 128: return grow_kernel<128>(wide, occ);
    case 192: return grow_kernel<192>(wide, occ);
    case 256: return grow_kernel<256>(wide, occ);
    case 512: return grow_kernel<512>(wide, occ);
    case 1024: return grow_kernel<1024>(wide, occ);
    default: fail(AIWC_RF_EINVAL, "unsupported grow block size");
  }
}

#if AIWC_GROW_GROUPED
}  // namespace

const void* grow_kernel_grouped(int block, bool wide, int occ, bool teams) {
  return grow_kernel_block(block, wide, occ, teams);
}

}  // namespace aiwc
#else

__global__ void k_init(uint32_t* status, uint32_t* queue) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    if (status) *status = 0;
    if (queue) *queue = 0;
  }
}

// y -> y_fp = rint(y * 2^16) with range check, and every code < its column's bin count.
__global__ void k_prepare(const uint8_t* codes, int64_t n, int32_t C, const int32_t* n_bins, const double* y,
                          int64_t* y_fp, uint8_t* codes_p, int32_t Cp, uint32_t* status) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  uint32_t bad = 0;
  for (int64_t i = g; i < n; i += stride) {
    const double v = y[i];
    if (!(fabs(v) <= 64.0)) {
      bad |= kStatusBadY;
      y_fp[i] = 0;
    } else {
      y_fp[i] = (int64_t)rint(v * 65536.0);
    }
  }
  const int64_t total = n * C;
  for (int64_t i = g; i < total; i += stride)
    if ((int32_t)codes[i] >= n_bins[i % C]) bad |= kStatusBadCode;
  // the padded copy: row i at i * Cp, zeros after column C - 1
  const int64_t total_p = n * Cp;
  for (int64_t i = g; i < total_p; i += stride) {
    const int64_t row = i / Cp;
    const int32_t c = (int32_t)(i - row * Cp);
    codes_p[i] = c < C ? codes[row * C + c] : 0u;
  }
  if (bad) atomicOr(status, bad);
}

__global__ void k_set_i32(int32_t* p, int32_t v) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *p = v;
}

// Dynamic LDS of the grow kernel: the per-wave histograms, or the packed
// histograms of a batch of wide nodes, or the candidate-draw rows, whichever is
// largest (the three are used in different phases of a level).
struct Layout {
  uint32_t lds_bytes;    // dynamic LDS of a workgroup
  uint32_t lcode_bytes, team_bytes;  // with teams: the code matrix, and a team's union and Shared
  uint32_t union_bytes;
  uint32_t wave_bytes;
  int32_t bstride;
  int32_t big_stride;  // bins per large-node column histogram (a multiple of 4)
  int32_t big_cols;    // large-node columns per wave task (the wave area holds that many histograms)
};

Layout grow_layout(const GrowConfig& cfg, int32_t mtry_max, int32_t C, int64_t n) {
  Layout L{};
  L.bstride = (std::max(cfg.bins_max, 1) + 63) / 64 * 64;
  L.big_stride = (std::max(cfg.bins_max, 1) + 3) / 4 * 4;
  // a wave's histogram, or the staging of its small-node task (the rank task's
  // two bin buffers and candidates take 4096 + mtry bytes)
  const size_t wb = std::max(sizeof(WaveHist), (size_t)4096 + (size_t)mtry_max);
  L.wave_bytes = (uint32_t)((wb + 255) / 256 * 256);
  L.big_cols = (int32_t)std::min<size_t>(4, L.wave_bytes / (8 * (size_t)L.big_stride));
  const size_t waves = (size_t)(cfg.block / kWave) * L.wave_bytes;
  const size_t draw = (size_t)std::min(cfg.block, 256) * (size_t)C;
  size_t wide = 0;
  if (grow_has_wide_phase(cfg)) {
    // by default a quarter of the 128 KiB per 256 threads, so that the
    // workgroups that fit a CU still do
    const size_t want = cfg.wide_bytes > 0 ? (size_t)cfg.wide_bytes : (size_t)cfg.block * 128;
    wide = std::max(std::max(waves, want), (size_t)8 * L.bstride * 8);
  }
  L.union_bytes = (uint32_t)std::max(std::max(waves, wide), draw);
  L.lds_bytes = L.union_bytes;
  // teams: the one-wave shape of deep queues, when the code matrix and every
  // team's area fit the LDS together
  if (cfg.block == kWave && cfg.occupancy == 5 && !grow_has_wide_phase(cfg) && cfg.wg_per_cu == 0) {
    const size_t lcodes = ((size_t)n * C + 255) / 256 * 256;
    const size_t uni = ((size_t)L.union_bytes + 15) / 16 * 16;
    const size_t team = uni + (sizeof(Shared<kWave, false>) + 15) / 16 * 16;
    const size_t total = lcodes + kRecip * sizeof(double) + 512 + kTeams * team;
    if (total <= device_info().lds_per_block) {
      L.lds_bytes = (uint32_t)total;
      L.lcode_bytes = (uint32_t)lcodes;
      L.union_bytes = (uint32_t)uni;
      L.team_bytes = (uint32_t)team;
    }
  }
  return L;
}

const void* grow_kernel_for(const GrowConfig& cfg, const Layout& L, bool grouped) {
  const bool wide = grow_has_wide_phase(cfg), teams = L.team_bytes > 0;
  return grouped ? grow_kernel_grouped(cfg.block, wide, cfg.occupancy, teams)
                 : grow_kernel_block(cfg.block, wide, cfg.occupancy, teams);
}
int grow_threads(const GrowConfig& cfg, const Layout& L) { return L.team_bytes > 0 ? kTeams * kWave : cfg.block; }

int occupancy(const void* kernel, int block, uint32_t lds) {
  int nb = 0;
  AIWC_HIP(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  AIWC_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kernel, block, lds));
  return nb;
}

}  // namespace

void launch_init(uint32_t* d_status, uint32_t* d_queue, hipStream_t s) {
  k_init<<<1, 64, 0, s>>>(d_status, d_queue);
  AIWC_HIP(hipGetLastError());
}

void launch_set_i32(int32_t* p, int32_t v, hipStream_t s) {
  k_set_i32<<<1, 64, 0, s>>>(p, v);
  AIWC_HIP(hipGetLastError());
}

size_t grow_scratch_bytes(int64_t n_cap, int32_t mtry_max, bool wide, bool grouped) {
  Scratch s;
  return carve(&s, 0, n_cap, mtry_max, wide, grouped);
}

void launch_prepare(const uint8_t* codes, int64_t n, int32_t C, const int32_t* d_n_bins, const double* y,
                    int64_t* y_fp, uint8_t* codes_p, uint32_t* d_status, hipStream_t s) {
  const int64_t work = n * padded_cols(C);
  const int blocks = (int)std::max<int64_t>(1, std::min<int64_t>(2048, (work + 255) / 256));
  k_prepare<<<blocks, 256, 0, s>>>(codes, n, C, d_n_bins, y, y_fp, codes_p, padded_cols(C), d_status);
  AIWC_HIP(hipGetLastError());
}

int grow_teams(const GrowConfig& cfg, int32_t mtry_max, int32_t C, int64_t n) {
  return grow_layout(cfg, mtry_max, C, n).team_bytes > 0 ? kTeams : 1;
}

int grow_grid_size(const GrowConfig& cfg, int64_t n_tasks, int32_t mtry_max, int32_t C, int64_t n, bool grouped) {
  const Layout L = grow_layout(cfg, mtry_max, C, n);
  if (L.lds_bytes > device_info().lds_per_block) fail(AIWC_RF_EINVAL, "grow kernel LDS exceeds the device limit");
  int per_cu = occupancy(grow_kernel_for(cfg, L, grouped), grow_threads(cfg, L), L.lds_bytes);
  if (per_cu < 1) fail(AIWC_RF_ENOMEM, "grow kernel does not fit the device (LDS or registers)");
  if (cfg.wg_per_cu > 0) per_cu = std::min(per_cu, cfg.wg_per_cu);
  const int64_t slots = (int64_t)device_info().cus * per_cu, teams = L.team_bytes > 0 ? kTeams : 1;
  return (int)std::max<int64_t>(1, std::min<int64_t>(slots, (n_tasks + teams - 1) / teams));
}

namespace {

GrowArgs grow_args(const GrowConfig& cfg, const Layout& L, const GrowLaunch& g, int32_t C, const int32_t* d_n_bins,
                   const int64_t* y_fp, uint32_t* d_status, int32_t mtry_max) {
  GrowArgs a;
  a.codes = g.codes;
  a.C = C;
  a.codes_p = g.codes_p;
  a.Cp = padded_cols(C);
  const bool dense = g.n_cap * (int64_t)C <= (int64_t)1 << 20;
  a.rcodes = dense ? g.codes : g.codes_p;
  a.rC = dense ? C : a.Cp;
  a.n_bins = d_n_bins;
  a.y_fp = y_fp;
  a.train_rows = g.train_rows;
  a.tasks = g.tasks;
  a.n_tasks = g.n_tasks;
  a.group_task = g.group_task;
  a.group_first = g.group_first;
  a.n_groups = g.group_first ? g.n_groups : g.n_tasks;
  a.nodes = g.nodes;
  a.node_N = g.node_N;
  a.n_nodes = g.n_nodes;
  a.work = g.work;
  a.inbag = g.inbag;
  a.queue = g.queue;
  a.status = d_status;
  a.scratch = g.scratch;
  a.n_cap = g.n_cap;
  a.mtry_max = mtry_max;
  a.huge_min = cfg.huge_min;
  a.wide_sums = cfg.wide_sums ? 1 : 0;
  a.scratch_stride = grow_scratch_bytes(g.n_cap, mtry_max, grow_has_wide_phase(cfg), g.group_first != nullptr);
  a.lcode_rows = (uint32_t)g.n;
  a.lcode_bytes = L.lcode_bytes;
  a.team_bytes = L.team_bytes;
  a.union_bytes = L.union_bytes;
  a.wave_bytes = L.wave_bytes;
  a.bstride = L.bstride;
  a.big_stride = L.big_stride;
  a.big_cols = cfg.big_cols > 0 ? std::min(cfg.big_cols, L.big_cols) : L.big_cols;
  return a;
}

int prepare_blocks(int64_t n, int32_t C) {
  const int64_t work = n * padded_cols(C);
  return (int)std::max<int64_t>(1, std::min<int64_t>(2048, (work + 255) / 256));
}

// Executable graphs of fused fits, one per launch shape: the status and queue
// reset, the prepare kernel and the grow launch as three kernel nodes.  A later
// fit of the same shape only replaces the nodes' arguments, once the graph's
// previous launch has finished.
struct GraphKey {
  int device;
  const void* kernel;
  int block, grid, prep_blocks;
  uint32_t lds;
  bool operator<(const GraphKey& o) const {
    return std::tie(device, kernel, block, grid, prep_blocks, lds) <
           std::tie(o.device, o.kernel, o.block, o.grid, o.prep_blocks, o.lds);
  }
};
struct GraphEntry {
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  hipGraphNode_t init = nullptr, prep = nullptr, grow = nullptr;
  hipEvent_t last = nullptr;  // recorded after the latest launch
  uint64_t used = 0;
};
constexpr size_t kMaxGraphs = 16;

std::mutex& graph_mu() {
  static std::mutex* m = new std::mutex();
  return *m;
}
std::map<GraphKey, GraphEntry>& graph_cache() {
  static auto* c = new std::map<GraphKey, GraphEntry>();  // kept until exit
  return *c;
}

hipKernelNodeParams node_params(const void* fn, int grid, int block, uint32_t lds, void** args) {
  hipKernelNodeParams p;
  std::memset(&p, 0, sizeof(p));
  p.func = const_cast<void*>(fn);
  p.gridDim = dim3((unsigned)grid);
  p.blockDim = dim3((unsigned)block);
  p.sharedMemBytes = lds;
  p.kernelParams = args;
  p.extra = nullptr;
  return p;
}

}  // namespace

int effective_big_cols(const GrowConfig& cfg, int32_t mtry_max, int32_t C) {
  const Layout L = grow_layout(cfg, mtry_max, C, 0);
  return cfg.big_cols > 0 ? std::min(cfg.big_cols, L.big_cols) : L.big_cols;
}

void launch_grow(const GrowConfig& cfg, const GrowLaunch& g, int32_t C, const int32_t* d_n_bins, const int64_t* y_fp,
                 uint32_t* d_status, int32_t mtry_max, int grid, hipStream_t s) {
  const Layout L = grow_layout(cfg, mtry_max, C, g.n);
  GrowArgs a = grow_args(cfg, L, g, C, d_n_bins, y_fp, d_status, mtry_max);
  const void* kernel = grow_kernel_for(cfg, L, g.group_first != nullptr);
  void* args[] = {&a};
  AIWC_HIP(hipLaunchKernel(kernel, dim3((unsigned)grid), dim3((unsigned)grow_threads(cfg, L)), args, L.lds_bytes, s));
  AIWC_HIP(hipGetLastError());
}

bool launch_fit_graph(const GrowConfig& cfg, const GrowLaunch& g, const uint8_t* codes, int64_t n, int32_t C,
                      const int32_t* d_n_bins, const double* y, int64_t* y_fp, uint32_t* d_status, int32_t mtry_max,
                      int grid, hipStream_t s) {
  const Layout L = grow_layout(cfg, mtry_max, C, g.n);
  GrowArgs a = grow_args(cfg, L, g, C, d_n_bins, y_fp, d_status, mtry_max);
  const void* kernel = grow_kernel_for(cfg, L, g.group_first != nullptr);
  const int threads = grow_threads(cfg, L);
  const int pb = prepare_blocks(n, C);
  int32_t Cp = padded_cols(C);
  uint32_t* queue = g.queue;
  uint8_t* codes_p = g.codes_p;
  void* init_args[] = {&d_status, &queue};
  void* prep_args[] = {const_cast<uint8_t**>(&codes), &n, &C, const_cast<int32_t**>(&d_n_bins),
                       const_cast<double**>(&y), &y_fp, &codes_p, &Cp, &d_status};
  void* grow_args_v[] = {&a};
  const hipKernelNodeParams p_init = node_params(reinterpret_cast<const void*>(k_init), 1, 64, 0, init_args);
  const hipKernelNodeParams p_prep = node_params(reinterpret_cast<const void*>(k_prepare), pb, 256, 0, prep_args);
  const hipKernelNodeParams p_grow = node_params(kernel, grid, threads, L.lds_bytes, grow_args_v);
  int dev = 0;
  AIWC_HIP(hipGetDevice(&dev));
  const GraphKey key{dev, kernel, threads, grid, pb, L.lds_bytes};
  static uint64_t clock = 0;
  std::lock_guard<std::mutex> lk(graph_mu());
  auto& cache = graph_cache();
  auto it = cache.find(key);
  const bool reused = it != cache.end();
  if (reused) {
    GraphEntry& e = it->second;
    AIWC_HIP(hipEventSynchronize(e.last));  // its previous launch read the old arguments
    AIWC_HIP(hipGraphExecKernelNodeSetParams(e.exec, e.init, &p_init));
    AIWC_HIP(hipGraphExecKernelNodeSetParams(e.exec, e.prep, &p_prep));
    AIWC_HIP(hipGraphExecKernelNodeSetParams(e.exec, e.grow, &p_grow));
  } else {
    if (cache.size() >= kMaxGraphs) {  // drop the least recently used shape
      auto old = cache.begin();
      for (auto j = cache.begin(); j != cache.end(); ++j)
        if (j->second.used < old->second.used) old = j;
      (void)hipEventSynchronize(old->second.last);
      (void)hipGraphExecDestroy(old->second.exec);
      (void)hipGraphDestroy(old->second.graph);
      (void)hipEventDestroy(old->second.last);
      cache.erase(old);
    }
    GraphEntry e;
    try {
      AIWC_HIP(hipGraphCreate(&e.graph, 0));
      AIWC_HIP(hipGraphAddKernelNode(&e.init, e.graph, nullptr, 0, &p_init));
      AIWC_HIP(hipGraphAddKernelNode(&e.prep, e.graph, &e.init, 1, &p_prep));
      AIWC_HIP(hipGraphAddKernelNode(&e.grow, e.graph, &e.prep, 1, &p_grow));
      AIWC_HIP(hipGraphInstantiate(&e.exec, e.graph, nullptr, nullptr, 0));
      AIWC_HIP(hipEventCreateWithFlags(&e.last, hipEventDisableTiming));
    } catch (...) {
      if (e.exec) (void)hipGraphExecDestroy(e.exec);
      if (e.graph) (void)hipGraphDestroy(e.graph);
      throw;
    }
    it = cache.emplace(key, e).first;
  }
  GraphEntry& e = it->second;
  e.used = ++clock;
  AIWC_HIP(hipGraphLaunch(e.exec, s));
  AIWC_HIP(hipEventRecord(e.last, s));
  return reused;
}

}  // namespace aiwc
#endif
