// Quantile binning of the AIWC feature matrix on gfx950.
//
// Each feature column is turned into order-preserving u32 keys and sorted in
// chunks of up to 8192 by a radix sort in the LDS.  The thresholds are the
// column's distinct values (when there are at most max_bins of them: the chunks'
// distinct values, merged) or its order statistics s[floor(k n / B) - 1], each
// found by one wave that bisects all sorted chunks at once, a chunk per lane.  A
// feature's code is then the number of its column's thresholds strictly below
// it, found by binary search.  The device id is its own code column.
#include "device.h"
#include "internal.h"

namespace aiwc {
namespace {

constexpr int kChunk = 8192;  // most keys sorted per workgroup in LDS (32 KiB)
constexpr int kSortBlock = 1024;
constexpr int kSortWaves = kSortBlock / kWave;
// 2^18 rows make at most 32 chunks: one per lane of a selecting wave
static_assert(AIWC_RF_MAX_ROWS / kChunk <= kWave, "a chunk per lane");

// Order-preserving key of a float (-0.0 folded onto +0.0).
__device__ __forceinline__ uint32_t float_key(float f) {
  if (f == 0.0f) f = 0.0f;
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_float(uint32_t k) {
  const uint32_t u = (k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k;
  return __uint_as_float(u);
}

// keys[j][i] for i < n_pad; padding sorts last.  A 64 x 64 tile goes through the
// LDS, so that both the rows of X and the columns of keys are touched in order
// (200000 x 64: 126 us with X read by column, now 22).
__global__ __launch_bounds__(256) void k_make_keys(const float* __restrict__ X, int64_t n, int32_t p, int64_t n_pad,
                                                   uint32_t* __restrict__ keys, uint32_t* status) {
  __shared__ uint32_t tile[64][65];
  const int64_t i0 = (int64_t)blockIdx.x * 64;
  const int32_t j0 = (int32_t)blockIdx.y * 64, lane = (int32_t)(threadIdx.x & 63), w = (int32_t)(threadIdx.x >> 6);
  uint32_t bad = 0;
  for (int r = w; r < 64; r += 4) {
    uint32_t k = 0xFFFFFFFFu;
    if (i0 + r < n && j0 + lane < p) {
      const float x = X[(i0 + r) * p + j0 + lane];
      if (isnan(x)) bad |= kStatusBadFeature;
      k = float_key(x);
    }
    tile[r][lane] = k;
  }
  __syncthreads();
  for (int c = w; c < 64 && j0 + c < p; c += 4) keys[(int64_t)(j0 + c) * n_pad + i0 + lane] = tile[lane][c];
  if (bad) atomicOr(status, bad);
}

// Sum of tmp[0 .. this wave).
__device__ __forceinline__ uint32_t waves_before(const uint32_t* tmp) {
  const int lane = (int)lane_id(), wid = (int)__builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t v = lane < kSortWaves ? tmp[lane] : 0u;
  return read_lane(wave_incl_scan_u32(v) - v, wid);
}

// Sorts the workgroup's K * kSortBlock keys, ascending: wave w's keys are w K 64 +
// 64 i + lane.  Four stable passes of 8 bits; in a pass each wave ranks its keys
// among the equal digits before them (the lanes of equal digit from eight
// ballots, the wave's earlier keys from its digit counts in the LDS), one scan
// of the counts of all waves gives every (digit, wave) its first place, and the
// keys are placed through the LDS.  A bitonic network took 91 passes over the
// chunk.  s: K * kSortBlock words, cnt: kCounts (a digit's counts of all waves, so
// that the scan runs over (digit, wave), one word apart from the next digit's to
// spread the banks).
constexpr int kDigitStride = kSortWaves + 1, kCounts = 256 * kDigitStride;
static_assert(kSortBlock == 64 * kSortWaves && kSortWaves == 16, "four counts per thread");
template <int K>
__device__ __forceinline__ void block_sort(uint32_t (&k)[K], uint32_t* s, uint32_t* cnt, uint32_t* tmp) {
  const int tid = (int)threadIdx.x, lane = (int)lane_id(), wid = tid / kWave;
  const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll 1
  for (int shift = 0; shift < 32; shift += 8) {
    for (int i = tid; i < kCounts; i += kSortBlock) cnt[i] = 0;
    __syncthreads();
    uint32_t rank[K];
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const uint32_t dgt = (k[i] >> shift) & 0xFFu;
      uint32_t p0 = ~0u, p1 = ~0u;  // the lanes that agree in every bit
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        const uint32_t t = (uint32_t)((int32_t)(dgt << (31 - b)) >> 31);
        const uint64_t m = __ballot(t != 0u);
        p0 &= ~((uint32_t)m ^ t);
        p1 &= ~((uint32_t)(m >> 32) ^ t);
      }
      const uint64_t peers = ((uint64_t)p1 << 32) | p0;
      uint32_t* c = cnt + dgt * kDigitStride + wid;
      const uint32_t before = *c;
      rank[i] = before + (uint32_t)__popcll(peers & below);
      wave_lds_sync();
      if ((peers & below) == 0) *c = before + (uint32_t)__popcll(peers);
      wave_lds_sync();
    }
    __syncthreads();
    // exclusive scan of the 4096 counts, four per thread
    uint32_t* c4 = cnt + tid / 4 * kDigitStride + tid % 4 * 4;
    const uint4 v = make_uint4(c4[0], c4[1], c4[2], c4[3]);
    const uint32_t mine = v.x + v.y + v.z + v.w;
    const uint32_t incl = wave_incl_scan_u32(mine);
    if (lane == kWave - 1) tmp[wid] = incl;
    __syncthreads();
    uint32_t off = incl - mine + waves_before(tmp);
    c4[0] = off;
    c4[1] = off + v.x;
    c4[2] = off + v.x + v.y;
    c4[3] = off + v.x + v.y + v.z;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < K; ++i) s[cnt[((k[i] >> shift) & 0xFFu) * kDigitStride + wid] + rank[i]] = k[i];
    __syncthreads();
    if (shift < 24) {
#pragma unroll
      for (int i = 0; i < K; ++i) k[i] = s[wid * K * kWave + i * kWave + lane];
      __syncthreads();
    }
  }
}

// The distinct values of the sorted s[0 .. len), len <= K * kSortBlock, the first
// `most` of them to out in order; returns their number (the same in every thread).
template <int K>
__device__ __forceinline__ uint32_t block_distinct(const uint32_t* s, int32_t len, uint32_t* out, uint32_t most,
                                                   uint32_t* tmp) {
  const int tid = (int)threadIdx.x, lane = (int)lane_id(), wid = tid / kWave;
  uint64_t m[K];
  uint32_t mine = 0;
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const int32_t g = wid * K * kWave + i * kWave + lane;
    m[i] = __ballot(g < len && (g == 0 || s[g] != s[g - 1]));
    mine += (uint32_t)__popcll(m[i]);
  }
  __syncthreads();
  if (lane == 0) tmp[wid] = mine;
  __syncthreads();
  uint32_t at = waves_before(tmp);
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const uint32_t o = at + (uint32_t)__popcll(m[i] & ((1ull << lane) - 1ull));
    if (((m[i] >> lane) & 1ull) && o < most) out[o] = s[wid * K * kWave + i * kWave + lane];
    at += (uint32_t)__popcll(m[i]);
  }
  const uint32_t v = lane < kSortWaves ? tmp[lane] : 0u;
  return wave_sum(v);
}

// A column's thresholds and bin count: its m distinct values (in `all`) but the
// largest when there are at most max_bins, else its order statistics value(0 ..
// max_bins - 2), ascending: the first of each run of equal ones, below the
// column's largest key.
template <typename Value>
__device__ __forceinline__ void write_thresholds(uint32_t m, int32_t max_bins, const uint32_t* all, uint32_t vmax,
                                                 Value value, float* t, int32_t* n_bins, uint32_t* tmp) {
  const int tid = (int)threadIdx.x, lane = (int)lane_id(), wid = tid / kWave;
  if (m <= (uint32_t)max_bins) {
    if (tid < 255) t[tid] = (uint32_t)tid + 1u < m ? key_float(all[tid]) : 0.0f;
    if (tid == 0) *n_bins = (int32_t)m;
    return;
  }
  const bool in = tid < max_bins - 1;
  const uint32_t v = in ? value(tid) : 0u;
  const bool keep = in && v < vmax && (tid == 0 || value(tid - 1) != v);
  const uint64_t km = __ballot(keep);
  if (wid < 4 && lane == 0) tmp[wid] = (uint32_t)__popcll(km);
  __syncthreads();
  const uint32_t total = tmp[0] + tmp[1] + tmp[2] + tmp[3];
  uint32_t at = (uint32_t)__popcll(km & ((1ull << lane) - 1ull));
  for (int w = 0; w < min(wid, 4); ++w) at += tmp[w];
  if (keep) t[at] = key_float(v);
  if (tid < 255 && (uint32_t)tid >= total) t[tid] = 0.0f;
  if (tid == 0) *n_bins = (int32_t)total + 1;
}

// Sorts chunk blockIdx.x of column blockIdx.y in place and lists its distinct
// values, up to kMaxDistinct of them; a column of one chunk (ONE) gets its
// thresholds at once.
constexpr uint32_t kMaxDistinct = 257;
template <int K, bool ONE>
__global__ __launch_bounds__(kSortBlock) void k_sort_chunks(uint32_t* __restrict__ keys, int64_t n, int64_t n_pad,
                                                            int32_t max_bins, uint32_t* __restrict__ distinct,
                                                            uint32_t* __restrict__ n_distinct, int32_t* n_bins,
                                                            float* thresholds) {
  __shared__ uint32_t s[K * kSortBlock];
  __shared__ uint32_t cnt[kCounts];
  __shared__ uint32_t tmp[kSortWaves];
  const int tid = (int)threadIdx.x, lane = (int)lane_id(), wid = tid / kWave;
  const int64_t c = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  uint32_t* col = keys + (int64_t)blockIdx.y * n_pad + (int64_t)blockIdx.x * (K * kSortBlock);
  uint32_t k[K];
#pragma unroll
  for (int i = 0; i < K; ++i) k[i] = col[wid * K * kWave + i * kWave + lane];
  const int32_t len = (int32_t)min((int64_t)K * kSortBlock, n - (int64_t)blockIdx.x * (K * kSortBlock));
  if (K == 1 && ONE && len <= 256) {
    // few keys: each one's place is the number of keys before it
    s[tid] = k[0];
    __syncthreads();
    uint32_t at = 0;
    if (tid < len) {
      for (int32_t j = 0; j < len; ++j) at += (s[j] < k[0] || (s[j] == k[0] && j < tid)) ? 1u : 0u;
    }
    __syncthreads();
    if (tid < len) s[at] = k[0];
    __syncthreads();
  } else {
    block_sort<K>(k, s, cnt, tmp);
  }
  if constexpr (ONE) {
    uint32_t* all = cnt;  // (the sort is done with its counts)
    const uint32_t m = block_distinct<K>(s, len, all, kMaxDistinct, tmp);
    __syncthreads();
    write_thresholds(m, max_bins, all, s[len - 1], [&](int r) { return s[(r + 1) * n / max_bins - 1]; },
                     thresholds + (int64_t)blockIdx.y * 255, n_bins + blockIdx.y, tmp);
  } else {
#pragma unroll
    for (int i = 0; i < K; ++i) col[i * kSortBlock + tid] = s[i * kSortBlock + tid];
    const uint32_t m = block_distinct<K>(s, len, distinct + c * kMaxDistinct, kMaxDistinct, tmp);
    if (tid == 0) n_distinct[c] = m;
  }
}

// Order statistics: wave t of column blockIdx.y finds the key of rank floor(k n /
// B) - 1, k = t + 1, among the column's sorted chunks, lane c holding chunk c.
// Key bits are decided from the top: the keys below the prefix with the bit set
// are counted by a bisection of each chunk's remaining range.   200000 x 64, 255 ranks: 120 us, bound by
// the address unit (a cache line per chunk and step); it and the chunk sort (132
// us) take the place of a bitonic sort of the whole columns (1370 us).
__global__ __launch_bounds__(256) void k_select(const uint32_t* __restrict__ keys, int64_t n, int64_t n_pad,
                                                int32_t chunk, int32_t n_chunks, int32_t max_bins,
                                                uint32_t* __restrict__ stat) {
  const int lane = (int)lane_id();
  const int k = (int)(blockIdx.x * 4 + threadIdx.x / kWave) + 1;
  if (k >= max_bins) return;
  const uint32_t* col = keys + (int64_t)blockIdx.y * n_pad;
  int64_t idx64 = ((int64_t)k * n) / max_bins - 1;
  if (idx64 < 0) return;  // fewer rows than bins: the column is lossless
  uint32_t idx = (uint32_t)idx64;
  const uint32_t* ch = col + (int64_t)lane * chunk;
  uint32_t lo = 0, hi = lane < n_chunks ? (uint32_t)min((int64_t)chunk, n - (int64_t)lane * chunk) : 0u;
  // the keys at the range's ends, known from the bisection that set them
  uint32_t first = lo < hi ? ch[lo] : 0u, last = lo < hi ? ch[hi - 1] : 0u;
  uint32_t prefix = 0;
  for (int b = 31; b >= 0; --b) {
    const uint32_t T = prefix | (1u << b);
    // l: the first key not below T; vb, va: the keys before and at it
    uint32_t l = lo, h = hi, vb = first, va = first;
    if (lo < hi && first < T) {
      va = last;
      if (last < T) {
        l = hi;
        vb = last;
      } else {
        h = hi - 1;  // its key is not below T; lo's is
        ++l;
        while (l < h) {
          const uint32_t mid = (l + h) >> 1, v = ch[mid];
          if (v < T) {
            l = mid + 1;
            vb = v;
          } else {
            h = mid;
            va = v;
          }
        }
      }
    }
    const uint32_t zeros = wave_sum(l - lo);
    if (idx < zeros) {
      hi = l;
      last = vb;
    } else {
      idx -= zeros;
      lo = l;
      first = va;
      prefix = T;
    }
    const uint64_t left = __ballot(lo < hi);
    // one key left, or one chunk: the rank within it is known
    if (__popcll(left) == 1) {
      const int c = __builtin_ctzll(left);
      prefix = col[(int64_t)c * chunk + read_lane(lo, c) + idx];
      break;
    }
  }
  if (lane == 0) stat[(int64_t)blockIdx.y * 256 + k - 1] = prefix;
}

// Thresholds of one column of several chunks (one workgroup per column) from the
// chunks' distinct values or the order statistics.
__global__ __launch_bounds__(kSortBlock) void k_thresholds(const uint32_t* __restrict__ keys, int64_t n, int64_t n_pad,
                                                           int32_t chunk, int32_t n_chunks, int32_t max_bins,
                                                           const uint32_t* __restrict__ distinct,
                                                           const uint32_t* __restrict__ n_distinct,
                                                           const uint32_t* __restrict__ stat, int32_t* n_bins,
                                                           float* thresholds) {
  __shared__ uint32_t s[kChunk];
  __shared__ uint32_t cnt[kCounts];
  __shared__ uint32_t all[kMaxDistinct + 1];
  __shared__ uint32_t tmp[kSortWaves];
  __shared__ uint32_t s_most;
  const int j = blockIdx.x, lane = (int)lane_id(), wid = (int)threadIdx.x / kWave;
  const uint32_t* nd = n_distinct + (int64_t)j * n_chunks;
  const uint32_t* dl = distinct + (int64_t)j * n_chunks * kMaxDistinct;
  if (wid == 0) {  // the most distinct values of any chunk
    uint32_t m = lane < n_chunks ? nd[lane] : 0u;
    for (int d = 32; d >= 1; d >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, d, kWave));
    if (lane == 0) s_most = m;
  }
  __syncthreads();
  uint32_t m = s_most;  // the column's distinct values, or more than max_bins
  if (m <= (uint32_t)max_bins) {
    // at most 32 x 256 values: sorted again, and their distinct ones listed
    constexpr int K = kChunk / kSortBlock;
    uint32_t k[K];
    uint32_t total = 0;
#pragma unroll
    for (int i = 0; i < K; ++i) k[i] = 0xFFFFFFFFu;
    for (int c = 0; c < n_chunks; ++c) total += nd[c];
#pragma unroll
    for (int i = 0; i < K; ++i) {
      uint32_t g = (uint32_t)(wid * K * kWave + i * kWave + lane);
      if (g < total) {
        int c = 0;
        while (g >= nd[c]) g -= nd[c++];
        k[i] = dl[(int64_t)c * kMaxDistinct + g];
      }
    }
    block_sort<K>(k, s, cnt, tmp);
    m = block_distinct<K>(s, (int32_t)total, all, kMaxDistinct, tmp);
  }
  __syncthreads();
  // the column's largest key: the last of its chunks' last ones
  uint32_t vmax = 0;
  for (int c = 0; c < n_chunks; ++c) {
    const int64_t last = min((int64_t)(c + 1) * chunk, n) - 1;
    vmax = max(vmax, keys[(int64_t)j * n_pad + last]);
  }
  write_thresholds(m, max_bins, all, vmax, [&](int r) { return stat[(int64_t)j * 256 + r]; },
                   thresholds + (int64_t)j * 255, n_bins + j, tmp);
}

// code(x) = #{thresholds < x}; column p = device id.  A workgroup codes R rows in
// up to kEncodeCols columns, whose thresholds it holds in the LDS, padded with
// +inf to one less than a power of two that holds the largest column's, so that
// the search takes the same steps for every column; the odd row of words puts a
// step's reads of neighbouring columns into different banks.
constexpr int kEncodeCols = 64;
__global__ __launch_bounds__(256) void k_encode(const float* __restrict__ X, const int32_t* __restrict__ dev,
                                                int64_t n, int32_t p, int32_t n_devices, int32_t R,
                                                const int32_t* __restrict__ n_bins,
                                                const float* __restrict__ thresholds, uint8_t* __restrict__ codes,
                                                uint32_t* status) {
  extern __shared__ float s_thr[];  // [columns][2 top + 1], at most 257 words a row
  const int32_t C = p + 1, j0 = (int32_t)blockIdx.y * kEncodeCols, nc = min(kEncodeCols, p - j0);
  const int64_t i0 = (int64_t)blockIdx.x * R;
  const int32_t nr = (int32_t)min((int64_t)R, n - i0), tid = (int32_t)threadIdx.x;
  uint32_t bad = 0;
  int32_t most = 1;  // bins of the largest column
  for (int32_t c = 0; c < nc; ++c) most = max(most, n_bins[j0 + c]);
  int32_t lg = 0;  // a search of lg steps tells 2^lg codes apart
  while ((1 << lg) < most) ++lg;
  const int32_t st = (1 << lg) + 1;
  for (int32_t e = tid; e < nc << lg; e += 256) {
    const int32_t c = e >> lg, k = e & ((1 << lg) - 1);
    s_thr[c * st + k] = k < n_bins[j0 + c] - 1 ? thresholds[(int64_t)(j0 + c) * 255 + k] : INFINITY;
  }
  if (blockIdx.y == 0) {
    for (int32_t r = tid; r < nr; r += 256) {
      const int32_t d = dev[i0 + r];
      const bool ok = d >= 0 && d < n_devices;
      if (!ok) bad |= kStatusBadDevice;
      codes[(i0 + r) * C + p] = ok ? (uint8_t)d : 0u;
    }
  }
  __syncthreads();
  const uint32_t inv = nc > 1 ? (uint32_t)(0x100000000ull / (uint32_t)nc) + 1u : 0u;
  const uint32_t total = (uint32_t)nr * (uint32_t)nc;
  for (uint32_t e = (uint32_t)tid; e < total; e += 256) {
    const uint32_t r = nc > 1 ? __umulhi(e, inv) : e, c = e - r * (uint32_t)nc;
    const float x = X[(i0 + r) * p + j0 + c];
    if (isnan(x)) bad |= kStatusBadFeature;
    const float* t = s_thr + c * (uint32_t)st;
    uint32_t at = 0;
    for (uint32_t d = 1u << lg >> 1; d > 0; d >>= 1) at += t[at + d - 1] < x ? d : 0u;
    codes[(i0 + r) * C + j0 + c] = (uint8_t)at;
  }
  if (bad) atomicOr(status, bad);
}

// The same for few values, one per thread, the thresholds read where they are.
__global__ __launch_bounds__(256) void k_encode_few(const float* __restrict__ X, const int32_t* __restrict__ dev,
                                                    int64_t n, int32_t p, int32_t n_devices,
                                                    const int32_t* __restrict__ n_bins,
                                                    const float* __restrict__ thresholds,
                                                    uint8_t* __restrict__ codes, uint32_t* status) {
  const uint32_t C = (uint32_t)p + 1u, g = blockIdx.x * 256u + threadIdx.x;
  if (g >= (uint32_t)n * C) return;
  const uint32_t i = g / C, j = g - i * C;
  uint32_t bad = 0, code = 0;
  if (j == (uint32_t)p) {
    const int32_t d = dev[i];
    if (d < 0 || d >= n_devices)
      bad = kStatusBadDevice;
    else
      code = (uint32_t)d;
  } else {
    const float x = X[(int64_t)i * p + j];
    if (isnan(x)) bad = kStatusBadFeature;
    const float* t = thresholds + (int64_t)j * 255;
    uint32_t hi = (uint32_t)n_bins[j] - 1u;  // count of thresholds below x lies in [code, hi]
    while (code < hi) {
      const uint32_t mid = (code + hi) >> 1;
      if (t[mid] < x)
        code = mid + 1;
      else
        hi = mid;
    }
  }
  codes[g] = (uint8_t)code;
  if (bad) atomicOr(status, bad);
}

template <int K, bool ONE>
void sort_chunks(uint32_t* keys, int64_t n, int64_t n_pad, int32_t p, int32_t max_bins, uint32_t* distinct,
                 uint32_t* n_distinct, int32_t* n_bins, float* thresholds, hipStream_t s) {
  k_sort_chunks<K, ONE><<<dim3((unsigned)(n_pad / (K * kSortBlock)), (unsigned)p), kSortBlock, 0, s>>>(
      keys, n, n_pad, max_bins, distinct, n_distinct, n_bins, thresholds);
  AIWC_HIP(hipGetLastError());
}

}  // namespace

void launch_bin_fit(const float* X, const int32_t* dev, int64_t n, int32_t p, int32_t n_devices, int32_t max_bins,
                    int32_t* d_n_bins, float* d_thresholds, uint32_t* d_status, hipStream_t s) {
  (void)dev;
  (void)n_devices;
  const int32_t chunk = n <= 1024 ? 1024 : n <= 2048 ? 2048 : n <= 4096 ? 4096 : kChunk;
  const int64_t n_chunks = (n + chunk - 1) / chunk, n_pad = n_chunks * chunk;
  DevBuf<uint32_t> keys((size_t)n_pad * p, s);
  k_make_keys<<<dim3((unsigned)(n_pad / 64), (unsigned)((p + 63) / 64)), 256, 0, s>>>(X, n, p, n_pad, keys.p, d_status);
  AIWC_HIP(hipGetLastError());
  if (n_chunks == 1) {
    const auto sort = chunk == 1024   ? sort_chunks<1, true>
                      : chunk == 2048 ? sort_chunks<2, true>
                      : chunk == 4096 ? sort_chunks<4, true>
                                      : sort_chunks<8, true>;
    sort(keys.p, n, n_pad, p, max_bins, nullptr, nullptr, d_n_bins, d_thresholds, s);
    return;
  }
  DevBuf<uint32_t> distinct((size_t)p * n_chunks * (kMaxDistinct + 1) + (size_t)p * 256, s);
  uint32_t* n_distinct = distinct.p + (size_t)p * n_chunks * kMaxDistinct;
  uint32_t* stat = n_distinct + (size_t)p * n_chunks;
  sort_chunks<8, false>(keys.p, n, n_pad, p, max_bins, distinct.p, n_distinct, nullptr, nullptr, s);
  k_select<<<dim3((unsigned)((max_bins + 2) / 4), (unsigned)p), 256, 0, s>>>(keys.p, n, n_pad, chunk, (int32_t)n_chunks,
                                                                            max_bins, stat);
  AIWC_HIP(hipGetLastError());
  k_thresholds<<<p, kSortBlock, 0, s>>>(keys.p, n, n_pad, chunk, (int32_t)n_chunks, max_bins, distinct.p, n_distinct,
                                        stat, d_n_bins, d_thresholds);
  AIWC_HIP(hipGetLastError());
}

void launch_bin_encode(const float* X, const int32_t* dev, int64_t n, int32_t p, int32_t n_devices,
                       const int32_t* d_n_bins, const float* d_thresholds, uint8_t* codes, uint32_t* d_status,
                       hipStream_t s) {
  // below 2^21 values the thresholds' way into every workgroup's LDS costs more
  // than it saves (2220 x 34 values: 15.8 us against 4.2, 22015 x 80 about equal, 200000 x 64: 84
  // against 228)
  if (n * (p + 1) < (int64_t)1 << 21) {
    k_encode_few<<<(unsigned)((n * (p + 1) + 255) / 256), 256, 0, s>>>(X, dev, n, p, n_devices, d_n_bins, d_thresholds,
                                                                     codes, d_status);
    AIWC_HIP(hipGetLastError());
    return;
  }
  // rows per workgroup: about two workgroups per CU, 16 to 512 rows
  const int64_t cols = (p + kEncodeCols - 1) / kEncodeCols, slots = 2LL * device_info().cus;
  const int32_t R = (int32_t)std::min<int64_t>(512, std::max<int64_t>(16, (n * cols + slots - 1) / slots));
  const size_t lds = (size_t)std::min(p, kEncodeCols) * 257 * sizeof(float);
  if (lds > 65536) allow_lds(reinterpret_cast<const void*>(k_encode));
  k_encode<<<dim3((unsigned)((n + R - 1) / R), (unsigned)cols), 256, lds, s>>>(X, dev, n, p, n_devices, R, d_n_bins,
                                                                            d_thresholds, codes, d_status);
  AIWC_HIP(hipGetLastError());
}

}  // namespace aiwc
