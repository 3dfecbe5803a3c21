// Mean-pooled block-score selector: Q/K block pooling, block scores and the
// exact top-k + sink + local + chunk-causal mask emission.
//
// The paper plugs any lightweight block-level pattern search in front of the
// block union (Sec. 3.1, Sec. 3.2 first paragraph); per-chunk search cost is
// first-order under chunked prefill (Sec. 2.1), so every stage here is a
// single streaming pass: pooling is HBM-bound, scores are a small fp32
// contraction on the matrix cores, selection finds the k-th score of a mask row
// in one workgroup, keys in registers.
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace ca {

// ---------------------------------------------------------------------------
// Pooling: one wavefront reduces `rows` rows of D bf16 (row stride `stride`
// elements) to their fp32 mean.  Lane l reads 16 bytes of row (l / CPR) +
// k*RPI, so each load instruction covers RPI whole rows contiguously; the
// lane adds its rows in ascending k, then the lanes holding the same chunk
// meet in a butterfly.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void add_bf16x8(float (&acc)[8], const uint4& v) {
  acc[0] += bf16_lo(v.x); acc[1] += bf16_hi(v.x);
  acc[2] += bf16_lo(v.y); acc[3] += bf16_hi(v.y);
  acc[4] += bf16_lo(v.z); acc[5] += bf16_hi(v.z);
  acc[6] += bf16_lo(v.w); acc[7] += bf16_hi(v.w);
}

template <int D>
__device__ __forceinline__ void pool_store(float (&acc)[8], float* __restrict__ out, float scale) {
  constexpr int CPR = D / 8;
  const int l = lane_id();
#pragma unroll
  for (int o = CPR; o < kWave; o <<= 1) {
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += __shfl_xor(acc[e], o, kWave);
  }
  if (l < CPR) {
    float4* dst = reinterpret_cast<float4*>(out + (l % CPR) * 8);
    dst[0] = make_float4(acc[0] * scale, acc[1] * scale, acc[2] * scale, acc[3] * scale);
    dst[1] = make_float4(acc[4] * scale, acc[5] * scale, acc[6] * scale, acc[7] * scale);
  }
}

// Any row count: one load per step of the loop.
template <int D>
__device__ __forceinline__ void pool_rows(const uint16_t* __restrict__ base, size_t stride,
                                          int rows, float* __restrict__ out, float scale) {
  constexpr int CPR = D / 8;           // 16-byte chunks per row
  constexpr int RPI = kWave / CPR;     // rows per load instruction
  const int l = lane_id();
  const int chunk = l % CPR;
  float acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.f;
  for (int r = l / CPR; r < rows; r += RPI)
    add_bf16x8(acc, *reinterpret_cast<const uint4*>(base + (size_t)r * stride + chunk * 8));
  pool_store<D>(acc, out, scale);
}

// Exactly N * RPI rows: all N loads are issued before the first add, so a
// wave keeps N 16-byte loads per lane in flight instead of one (same adds,
// same order as pool_rows).
template <int D, int N, bool NT>
__device__ __forceinline__ void pool_rows_n(const uint16_t* __restrict__ base, size_t stride,
                                            float* __restrict__ out, float scale) {
  constexpr int CPR = D / 8;
  constexpr int RPI = kWave / CPR;
  const int l = lane_id();
  const uint16_t* src = base + (size_t)(l / CPR) * stride + (l % CPR) * 8;
  uint4 v[N];
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const u32x4* const at = reinterpret_cast<const u32x4*>(src + (size_t)k * RPI * stride);
    const u32x4 x = NT ? __builtin_nontemporal_load(at) : *at;
    v[k] = make_uint4(x[0], x[1], x[2], x[3]);
  }
  float acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.f;
#pragma unroll
  for (int k = 0; k < N; ++k) add_bf16x8(acc, v[k]);
  pool_store<D>(acc, out, scale);
}

// One launch pools both operands of the scores:
//   * workgroups [0, n_q_wg): one per (b, h, i) Q-block; each wave sums a
//     quarter of the block's rows and the four partial sums meet in LDS (the
//     chunk's last Q-block may hold fewer rows; its mean is over those);
//   * the rest: 4 waves per workgroup, one K block (b, kvh, j) per wave, j in
//     [first_block, nKB_b); a sequence's last block is pooled over its rows
//     before the sequence end only.
// In the fused estimator-to-union path the launch also clears the group union
// words that the selection ORs into (clear_words, n_clear; none otherwise).
struct PoolArgs {
  const uint16_t* q;
  float* q_mean;
  int B, C, Hq, q_block, nqb, n_q_wg;
  uint64_t* clear_words;
  int n_clear;
  const uint16_t* k_pool;
  const int32_t* page_table;
  const int32_t* cached_len;
  float* k_mean;
  int Hkv, max_kv_blocks, first_block, k_tiles;   // k_tiles workgroups per (b, kvh)
};

template <int D, bool NT>
__global__ __launch_bounds__(256) void pool_kernel(const PoolArgs a) {
  __shared__ __attribute__((aligned(16))) float part[4][D];
  constexpr int RPI = kWave / (D / 8);
  for (int x = blockIdx.x * 256 + threadIdx.x; x < a.n_clear; x += gridDim.x * 256)
    a.clear_words[x] = 0ull;
  const int wv = threadIdx.x >> 6;
  if ((int)blockIdx.x < a.n_q_wg) {
    const int w = blockIdx.x;
    const int i = w % a.nqb;
    const int h = (w / a.nqb) % a.Hq;
    const int b = w / (a.nqb * a.Hq);
    const int quarter = a.q_block / 4;
    const int n_valid = a.C - i * a.q_block < a.q_block ? a.C - i * a.q_block : a.q_block;
    int rows = n_valid - wv * quarter;
    rows = rows < 0 ? 0 : (rows > quarter ? quarter : rows);
    const uint16_t* base =
        a.q + (((size_t)b * a.C + (size_t)i * a.q_block + (size_t)wv * quarter) * a.Hq + h) * D;
    const size_t stride = (size_t)a.Hq * D;
    if (rows == 8 * RPI) pool_rows_n<D, 8, false>(base, stride, part[wv], 1.0f);
    else pool_rows<D>(base, stride, rows, part[wv], 1.0f);
    __syncthreads();
    const int t = threadIdx.x;
    if (t < D)
      a.q_mean[(size_t)w * D + t] = ((part[0][t] + part[1][t]) + (part[2][t] + part[3][t])) *
                                    (1.0f / (float)n_valid);
    return;
  }
  const int kw = blockIdx.x - a.n_q_wg;
  const int bk = kw / a.k_tiles;   // b * Hkv + kvh
  const int b = bk / a.Hkv;
  const int j = a.first_block + (kw % a.k_tiles) * 4 + wv;
  const int seq = a.cached_len[b] + a.C;
  if (j >= blocks_for(seq)) return;
  const int rows = seq - kPage * j < kPage ? seq - kPage * j : kPage;
  const int page = a.page_table[(size_t)bk * a.max_kv_blocks + j];
  const uint16_t* base = a.k_pool + (size_t)page * kPage * D;
  float* out = a.k_mean + ((size_t)bk * a.max_kv_blocks + j) * D;
  if (rows == kPage) pool_rows_n<D, kPage / RPI, NT>(base, D, out, 1.0f / (float)kPage);
  else pool_rows<D>(base, D, rows, out, 1.0f / (float)rows);
}

// ---------------------------------------------------------------------------
// Scores: for one (b, kvh), the ratio*nQB pooled query rows are contiguous in
// q_mean and the matching score rows are contiguous too.  One wave computes a
// 32-row x 32-block tile with fp32 matrix instructions (v_mfma_f32_32x32x2_f32,
// fp32 products and sums); a workgroup's four waves cover 32 WR rows x 32 WJ
// blocks and share their operands through LDS.  Lane l holds row / block l % 32
// and, for k-step (t, e), element d = 8t + 4(l / 32) + e of both operands (the
// contraction over d may take the d in any order as long as both operands share
// it).  Loaded straight into registers, those operands were 32-byte pieces of
// 32 rows per load, and each wave read both of its own: 9 us at 64 rows x 2016
// blocks x 8 heads and 29 us at 128 rows x 3354 blocks x 8, where the reads
// through L2 (440 MB) set the time.  Here a wave loads whole rows, 1 KB per
// instruction, all before the first is needed.  LDS rows are padded by 16 bytes:
// the 16 lanes of a read then touch 16 different 16-byte bank slots.
// ---------------------------------------------------------------------------
typedef float f32x16 __attribute__((ext_vector_type(16)));

template <int D, int WR>
__global__ __launch_bounds__(256) void scores_kernel(const float* __restrict__ q_mean,
                                                     const float* __restrict__ k_mean,
                                                     const int32_t* __restrict__ cached_len,
                                                     float* __restrict__ scores, int Hq, int Hkv,
                                                     int nqb, int max_kv_blocks, int n_rg) {
  constexpr int NT = D / 8, WJ = 4 / WR, LD = D + 4, CPR = D / 4;
  constexpr int QR = 32 * WR, KR = 32 * WJ;              // rows of each operand
  constexpr int QL = QR * CPR / 256, KL = KR * CPR / 256;   // float4 per thread
  __shared__ __attribute__((aligned(16))) float qs[QR * LD];
  __shared__ __attribute__((aligned(16))) float ks[KR * LD];
  const int bk = blockIdx.y;
  const int b = bk / Hkv, kvh = bk % Hkv;
  const int ratio = Hq / Hkv;
  const int nrows = ratio * nqb;
  const int nc = cached_len[b] / kPage;
  const int r_wg = (blockIdx.x % n_rg) * QR, j_wg = (blockIdx.x / n_rg) * KR;
  if (j_wg >= nc) return;   // whole workgroup
  const size_t row_base = ((size_t)b * Hq + (size_t)kvh * ratio) * nqb;
  const int t = threadIdx.x;
  // rows past the end repeat the last one; their results are not stored
  float4 qv[QL], kv[KL];
#pragma unroll
  for (int m = 0; m < KL; ++m) {
    const int x = m * 256 + t, j = j_wg + x / CPR;
    kv[m] = reinterpret_cast<const float4*>(
        k_mean + ((size_t)bk * max_kv_blocks + (j < nc ? j : nc - 1)) * D)[x % CPR];
  }
#pragma unroll
  for (int m = 0; m < QL; ++m) {
    const int x = m * 256 + t, r = r_wg + x / CPR;
    qv[m] = reinterpret_cast<const float4*>(
        q_mean + (row_base + (r < nrows ? r : nrows - 1)) * D)[x % CPR];
  }
#pragma unroll
  for (int m = 0; m < KL; ++m) {
    const int x = m * 256 + t;
    *reinterpret_cast<float4*>(ks + (x / CPR) * LD + 4 * (x % CPR)) = kv[m];
  }
#pragma unroll
  for (int m = 0; m < QL; ++m) {
    const int x = m * 256 + t;
    *reinterpret_cast<float4*>(qs + (x / CPR) * LD + 4 * (x % CPR)) = qv[m];
  }
  __syncthreads();
  const int l = t & 63, wv = t >> 6, i = l & 31, h = l >> 5;
  const int r0 = r_wg + 32 * (wv % WR), j = j_wg + 32 * (wv / WR) + i;
  const float* qrow = qs + (32 * (wv % WR) + i) * LD + 4 * h;
  const float* krow = ks + (32 * (wv / WR) + i) * LD + 4 * h;
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
  for (int x = 0; x < NT; ++x) {
    const float4 qa = *reinterpret_cast<const float4*>(qrow + 8 * x);
    const float4 kb = *reinterpret_cast<const float4*>(krow + 8 * x);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(qa.x, kb.x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(qa.y, kb.y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(qa.z, kb.z, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(qa.w, kb.w, acc, 0, 0, 0);
  }
  // result v of lane l: row 8(v/4) + 4(l/32) + v%4 of the tile, block l % 32
  if (j >= nc) return;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int r = r0 + 8 * (v / 4) + 4 * h + (v % 4);
    if (r < nrows) scores[(row_base + r) * max_kv_blocks + j] = acc[v];
  }
}

// ---------------------------------------------------------------------------
// Selection: one workgroup (4 waves) per mask row (b, h, i); thread t holds the
// keys of blocks t + 256 m, m < M, in registers.  Scores become order-preserving
// uint32 keys (-0.0 folded onto +0.0).  The k-th key in the order (key
// descending, block ascending) is found in two steps:
//   * 256 buckets of equal width between the row's lowest and highest score
//     (a monotone map, so a higher bucket holds only higher keys).  Their
//     counts spread over the LDS atomics, where the leading bits of the keys
//     would put most of a row on a few counters: the radix passes over those
//     took 25 us for 4096 rows of up to 1562 blocks, most of it in the first
//     pass's contended atomics;
//   * the few keys of the bucket that holds the k-th one are ranked directly, a
//     wave per copy of the work.  A bucket of more than 64 keys (scores far from
//     evenly spread: an outlier, clusters) is cut into 256 buckets again, between
//     its own lowest and highest key; from the third time on the buckets are of
//     equal width in the keys' integer order, whose lowest and highest key always
//     part, so that the search ends.  Equal keys are told apart by block index.
//     In us for 512 rows, with radix passes over the bucket's keys instead, and
//     so: 2016 blocks, one score of 1e4 13.9, 9.4; all equal 27.5, 5.3; 5000
//     blocks in clusters 34.4, 21.4 (evenly spread scores: 6.8, 6.9).
// A block is then selected by comparing (key, index) with the k-th: the words
// come straight from wave ballots, wave v of a 256-block slab owning word
// slab/64 + v, with no ranking of ties and one barrier.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t order_key(float f) {
  uint32_t u = __float_as_uint(f);
  if (u == 0x80000000u) u = 0u;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_value(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

constexpr int kBuckets = 256;
constexpr int kRanked = kWave;   // largest bucket that is ranked directly

// From the counts of the buckets (in LDS), the one that holds the r-th element
// counted from the highest, its count, and the number of elements above it.
// Every wave computes it alone: lane l takes the buckets 255-4l .. 252-4l.
__device__ __forceinline__ void bucket_of(const int* counts, int r, int* bkt, int* above,
                                          int* count) {
  const int l = lane_id();
  const int4 h = *reinterpret_cast<const int4*>(counts + 252 - 4 * l);
  const int c[4] = {h.w, h.z, h.y, h.x};
  const int sum = c[0] + c[1] + c[2] + c[3];
  const int incl = wave_inclusive_scan(sum);
  const int lane = __builtin_ctzll(__ballot(incl >= r));   // r <= the total
  int at = __builtin_amdgcn_readlane(incl - sum, lane), e = 0;
#pragma unroll
  for (int x = 0; x < 3; ++x) {
    const int cx = __builtin_amdgcn_readlane(c[x], lane);
    if (e == x && at + cx < r) at += cx, e = x + 1;
  }
  *above = at;
  *count = __builtin_amdgcn_readlane(e == 0 ? c[0] : e == 1 ? c[1] : e == 2 ? c[2] : c[3], lane);
  *bkt = 255 - (4 * lane + e);
}

template <int M>
__global__ __launch_bounds__(256) void select_kernel(const float* __restrict__ scores,
                                                     const int32_t* __restrict__ cached_len,
                                                     uint64_t* __restrict__ masks, int Hq,
                                                     int nqb, int max_kv_blocks, int W,
                                                     int C, int q_block,
                                                     float top_frac, int sink_blocks,
                                                     int local_blocks,
                                                     unsigned long long* __restrict__ gwords,
                                                     int group_size) {
  __shared__ __attribute__((aligned(16))) int hist[2][kBuckets];
  __shared__ uint32_t red[2][4];
  __shared__ uint32_t cand_key[kRanked];
  __shared__ int cand_idx[kRanked];
  __shared__ int n_cand;
  __shared__ unsigned long long words[kMaxKvBlocks / 64];
  const int row = blockIdx.x;
  const int t = threadIdx.x;
  const int wv = t >> 6;
  const int i = row % nqb;
  const int b = row / (nqb * Hq);
  const int cl = cached_len[b];
  const int nc = cl / kPage;            // full cached blocks: the candidates
  const int nkb = blocks_for(cl + C);
  int k = 0;
  if (nc > 0) {
    k = (int)ceilf(top_frac * (float)nc);
    k = k < 0 ? 0 : (k > nc ? nc : k);
  }
  const float* s = scores + (size_t)row * max_kv_blocks;
  uint32_t key[M];
  {
    float v[M];
#pragma unroll
    for (int m = 0; m < M; ++m) v[m] = t + 256 * m < nc ? s[t + 256 * m] : 0.f;
#pragma unroll
    for (int m = 0; m < M; ++m) key[m] = order_key(v[m]);
  }
  // f(m, j) for the thread's blocks j; rounds past the row's end are skipped whole
  auto each = [&](auto f) {
#pragma unroll
    for (int m = 0; m < M; ++m)
      if ((M < 32 || 256 * m < nc) && t + 256 * m < nc) f(m, t + 256 * m);
  };
  // the k-th key and its block: everything of (key, index) up to it is taken
  uint32_t T = 0xffffffffu;   // k = 0: none
  int Jt = -1;
  if (k == nc) {              // all (or no candidates)
    T = 0u;
    Jt = nc;
  } else if (k > 0) {
    // the r-th key of those in [lo, hi] is the k-th of the row
    uint32_t lo, hi;
    int r = k;
    auto extremes = [&](auto in) {   // lowest and highest key of those with in(key)
      uint32_t l1 = 0xffffffffu, h1 = 0u;
      each([&](int m, int) {
        if (in(key[m])) {
          l1 = key[m] < l1 ? key[m] : l1;
          h1 = key[m] > h1 ? key[m] : h1;
        }
      });
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        const uint32_t l2 = __shfl_xor(l1, o, kWave), h2 = __shfl_xor(h1, o, kWave);
        l1 = l2 < l1 ? l2 : l1;
        h1 = h2 > h1 ? h2 : h1;
      }
      if (lane_id() == 0) red[0][wv] = l1, red[1][wv] = h1;
      __syncthreads();
      lo = red[0][0], hi = red[1][0];
#pragma unroll
      for (int x = 1; x < 4; ++x) {
        lo = red[0][x] < lo ? red[0][x] : lo;
        hi = red[1][x] > hi ? red[1][x] : hi;
      }
    };
    // One level of the search among the keys from lo to hi (FIRST: all keys), in
    // buckets of equal width: by value on the first two levels, where the range is
    // a positive finite number (not so with infinities or NaN: one bucket then),
    // else by the keys' order.
    auto cut = [&](auto FIRST, int level) -> bool {
      constexpr bool kFirst = decltype(FIRST)::value;
      int* const counts = hist[level & 1];
      const float base = key_value(lo), range = key_value(hi) - base;
      const bool finite = range > 0.f && range < INFINITY, by_value = kFirst || (level == 1 && finite);
      const float scale = kFirst && !finite ? 0.f : 255.99f / (by_value ? range : (float)(hi - lo));
      const uint32_t from = lo, to = hi;
      auto bucket = [&](uint32_t x) {
        const float f = (by_value ? key_value(x) - base : (float)(x - from)) * scale;
        return f >= 255.f ? 255 : (f > 0.f ? (int)f : 0);   // (NaN compares false: bucket 0)
      };
      auto member = [&](uint32_t x) { return kFirst || (x >= from && x <= to); };
      // 64 atomics on one counter are served one after another: a wave whose
      // first round falls into one bucket adds the lanes of such a round at once
      const int b0 = __builtin_amdgcn_readfirstlane(bucket(key[0]));
      if (__ballot(bucket(key[0]) != b0) != 0) {
        each([&](int m, int) {
          if (member(key[m])) atomicAdd(&counts[bucket(key[m])], 1);
        });
      } else {
        each([&](int m, int) {
          const int b = member(key[m]) ? bucket(key[m]) : -1;
          const uint64_t same = __ballot(b == b0);
          if (b >= 0 && b != b0) atomicAdd(&counts[b], 1);
          else if (b == b0 && lane_id() == __builtin_ctzll(same)) atomicAdd(&counts[b0], __popcll(same));
        });
      }
      __syncthreads();
      int bkt, above, count;
      bucket_of(counts, r, &bkt, &above, &count);
      r -= above;
      if (count > kRanked) {
        // the next level's counters: their last reader was a level ago
        hist[(level + 1) & 1][t] = 0;
        extremes([&](uint32_t x) { return member(x) && bucket(x) == bkt; });
        return false;
      }
      each([&](int m, int j) {
        if (member(key[m]) && bucket(key[m]) == bkt) {
          const int at = atomicAdd(&n_cand, 1);
          cand_key[at] = key[m];
          cand_idx[at] = j;
        }
      });
      __syncthreads();
      const int l = lane_id() < count ? lane_id() : count - 1;
      const uint32_t ck = cand_key[l];
      const int ci = cand_idx[l];
      int rank = 0;   // candidates before this one
      for (int x = 0; x < count; ++x) {
        const uint32_t xk = __builtin_amdgcn_readlane(ck, x);
        const int xi = __builtin_amdgcn_readlane(ci, x);
        rank += (xk > ck || (xk == ck && xi < ci)) ? 1 : 0;
      }
      const int at = __builtin_ctzll(__ballot(rank == r - 1));
      T = __builtin_amdgcn_readlane(ck, at);
      Jt = __builtin_amdgcn_readlane(ci, at);
      return true;
    };
    hist[0][t] = 0;
    if (t == 0) n_cand = 0;
    extremes([](uint32_t) { return true; });
    if (lo != hi && !cut(std::true_type{}, 0))
      for (int level = 1; lo != hi && !cut(std::false_type{}, level);) ++level;
    if (Jt < 0) {
      // more than 64 equal keys (or a row of one value): the r-th of them by
      // block.  Rounds of 256 blocks first, then a wave's 64, then the bit.
      T = lo;
#pragma unroll
      for (int m = 0; m < M; ++m)
        if (256 * m < nc) {
          const uint64_t word = __ballot(t + 256 * m < nc && key[m] == T);
          if (lane_id() == 0) words[4 * m + wv] = word;
        }
      __syncthreads();
      // lane l: words 4l .. 4l+3 (those of round l)
      int c[4] = {0, 0, 0, 0};
      if (256 * lane_id() < nc)
#pragma unroll
        for (int x = 0; x < 4; ++x) c[x] = __popcll(words[4 * lane_id() + x]);
      const int sum = c[0] + c[1] + c[2] + c[3], incl = wave_inclusive_scan(sum);
      const int lane = __builtin_ctzll(__ballot(incl >= r));
      int rest = r - __builtin_amdgcn_readlane(incl - sum, lane), x = 0;
#pragma unroll
      for (int y = 0; y < 3; ++y) {
        const int cy = __builtin_amdgcn_readlane(c[y], lane);
        if (x == y && rest > cy) rest -= cy, x = y + 1;
      }
      const unsigned long long word = words[4 * lane + x];
      const uint64_t hit = __ballot(((word >> lane_id()) & 1ull) && lanes_below(word) == rest - 1);
      Jt = 64 * (4 * lane + x) + __builtin_ctzll(hit);
      __syncthreads();   // the words are written anew below
    }
  }

  const int causal_end = causal_block_end(cl, C, i, q_block);
  const int sink_end = sink_blocks < nc ? sink_blocks : nc;
  const int local_begin = nc - local_blocks;
  auto emit = [&](int j, bool sel) {
    const bool forced = j < nkb && ((j < sink_end) || (j >= local_begin && j < nc) ||
                                    (j >= nc && j < causal_end));
    const uint64_t word = __ballot(sel || forced);
    if (lane_id() == 0) words[j >> 6] = word;   // j < 64 * 256
  };
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const int j = t + 256 * m;
    if (256 * m < W * 64) emit(j, j < nc && (key[m] > T || (key[m] == T && j <= Jt)));
  }
  for (int base = 256 * M; base < W * 64; base += 256) emit(base + t, false);   // past the cache
  // The row leaves in one run of words.  One word at a time, the fused path's
  // ORs into the group words (64 rows on the same 32 words at 128K, from every
  // XCD) queued behind each other: 21.9 us against 11.9 for the masks.
  __syncthreads();
  if (t < W) {
    const unsigned long long word = words[t];
    if (gwords == nullptr) {
      masks[(size_t)row * W + t] = word;
    } else if (word) {   // fused path: straight into the words of the group's table row
      const int h = (row / nqb) % Hq;
      atomicOr(gwords + ((size_t)b * (Hq / group_size) + h / group_size) * W + t, word);
    }
  }
}

// ---------------------------------------------------------------------------
// Threshold selection (the alpha / max-threshold reading): one workgroup per
// mask row keeps every cached block with s_j >= s_max + margin (the sum in
// fp32), plus the same sink, local and chunk-causal bits as select_kernel.
// ---------------------------------------------------------------------------
// Thread t holds the scores of blocks t + 256 m, m < M, in registers: one
// memory latency, where a loop over the row for the maximum and another for the
// comparison waited for one per 256 blocks (5.2 us for 256 rows of 1562 blocks,
// launch included).
template <int M>
__global__ __launch_bounds__(256) void threshold_select_kernel(
    const float* __restrict__ scores, const int32_t* __restrict__ cached_len,
    uint64_t* __restrict__ masks, int Hq, int nqb, int max_kv_blocks, int W, int C,
    int q_block, float margin, int sink_blocks, int local_blocks) {
  __shared__ float red[4];
  const int row = blockIdx.x;
  const int t = threadIdx.x;
  const int wv = t >> 6;
  const int i = row % nqb;
  const int b = row / (nqb * Hq);
  const int cl = cached_len[b];
  const int nc = cl / kPage;
  const int nkb = blocks_for(cl + C);
  const float* s = scores + (size_t)row * max_kv_blocks;
  float v[M], mx = -INFINITY;
#pragma unroll
  for (int m = 0; m < M; ++m) v[m] = t + 256 * m < nc ? s[t + 256 * m] : -INFINITY;
#pragma unroll
  for (int m = 0; m < M; ++m) mx = fmaxf(mx, v[m]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, kWave));
  if (lane_id() == 0) red[wv] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  const float thr = mx + margin;
  const int causal_end = causal_block_end(cl, C, i, q_block);
  const int sink_end = sink_blocks < nc ? sink_blocks : nc;
  const int local_begin = nc - local_blocks;
  uint64_t* mrow = masks + (size_t)row * W;
  auto emit = [&](int j, bool sel) {
    const bool forced = j < nkb && ((j < sink_end) || (j >= local_begin && j < nc) ||
                                    (j >= nc && j < causal_end));
    const uint64_t word = __ballot(sel || forced);
    const int widx = j >> 6;
    if (lane_id() == 0 && widx < W) mrow[widx] = word;
  };
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const int j = t + 256 * m;
    if (256 * m < W * 64) emit(j, j < nc && v[m] >= thr);
  }
  for (int base = 256 * M; base < W * 64; base += 256) emit(base + t, false);   // past the cache
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
constexpr size_t kLastLevelCacheBytes = 256u << 20;   // MI355X

// q == nullptr: no Q pooling; k_pool == nullptr: no K pooling.
hipError_t launch_pool(const Dims& d, const uint16_t* q, float* q_mean, const uint16_t* k_pool,
                       const int32_t* page_table, const int32_t* cached_len,
                       const int32_t* cached_len_host, int first_block, float* k_mean,
                       hipStream_t st, uint64_t* clear_words, int n_clear) {
  PoolArgs a;
  a.q = q;
  a.q_mean = q_mean;
  a.B = d.B;
  a.C = d.C;
  a.Hq = d.Hq;
  a.q_block = d.q_block;
  a.nqb = d.nqb;
  a.n_q_wg = q != nullptr ? d.B * d.Hq * d.nqb : 0;
  a.clear_words = clear_words;
  a.n_clear = n_clear;
  a.k_pool = k_pool;
  a.page_table = page_table;
  a.cached_len = cached_len;
  a.k_mean = k_mean;
  a.Hkv = d.Hkv;
  a.max_kv_blocks = d.max_kv_blocks;
  a.first_block = first_block;
  const int span = d.max_nkb - first_block;
  a.k_tiles = k_pool != nullptr && span > 0 ? (span + 3) / 4 : 0;
  const long long nwg = (long long)a.n_q_wg + (long long)a.k_tiles * d.B * d.Hkv;
  if (nwg == 0) return hipSuccess;
  if (nwg > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  // K pages that could not stay in the 256 MB last-level cache are streamed past
  // it (non-temporal).  Pooling alone in us, cached : streamed, after 800 MB of
  // other data and again at once (8 heads, D = 128):
  //   63 MB 24.7 : 17.8, 15.2 : 12.4     252 MB 75.7 : 49.5, 42.7 : 46.5
  //  131 MB 43.7 : 29.1, 25.3 : 25.2     256 MB 76.4 : 51.2, 42.8 : 48.5
  //  199 MB 61.3 : 40.4, 34.5 : 37.1     316 MB 89.7 : 61.1, 64.1 : 58.6
  // Past the cache streaming is faster either way; below it only where other data
  // went through the cache since, which the call cannot know: pages that are read
  // again at once stay cached.  A step's attention takes as long after either.
  size_t k_bytes = 0;
  for (int b = 0; b < d.B && k_pool != nullptr; ++b) {
    const int blocks = blocks_for(cached_len_host[b] + d.C) - first_block;
    if (blocks > 0) k_bytes += (size_t)blocks * d.Hkv * kPage * d.D * 2;
  }
  const bool nt = k_bytes >= kLastLevelCacheBytes;
  auto launch = [&](auto kernel) { kernel<<<(int)nwg, 256, 0, st>>>(a); };
  if (d.D == 128) nt ? launch(pool_kernel<128, true>) : launch(pool_kernel<128, false>);
  else nt ? launch(pool_kernel<64, true>) : launch(pool_kernel<64, false>);
  return hipGetLastError();
}

hipError_t launch_pool_q(const Dims& d, const uint16_t* q, float* q_mean, hipStream_t st,
                         uint64_t* clear_words, int n_clear) {
  return launch_pool(d, q, q_mean, nullptr, nullptr, nullptr, nullptr, 0, nullptr, st, clear_words,
                     n_clear);
}

hipError_t launch_pool_k(const Dims& d, const uint16_t* k_pool, const int32_t* page_table,
                         const int32_t* cached_len, const int32_t* cached_len_host,
                         int first_block, float* k_mean, hipStream_t st) {
  return launch_pool(d, nullptr, nullptr, k_pool, page_table, cached_len, cached_len_host,
                     first_block, k_mean, st, nullptr, 0);
}

hipError_t launch_scores(const Dims& d, const float* q_mean, const float* k_mean,
                         const int32_t* cached_len, float* scores, hipStream_t st) {
  if (d.max_nc <= 0) return hipSuccess;
  const int nrows = (d.Hq / d.Hkv) * d.nqb;
  // two row tiles per workgroup where there are two (half the block rows read
  // per score), else one
  const int wr = nrows > 32 ? 2 : 1, wj = 4 / wr;
  const int n_rg = (nrows + 32 * wr - 1) / (32 * wr);
  dim3 grid(n_rg * ((d.max_nc + 32 * wj - 1) / (32 * wj)), d.B * d.Hkv);
  auto launch = [&](auto kernel) {
    kernel<<<grid, 256, 0, st>>>(q_mean, k_mean, cached_len, scores, d.Hq, d.Hkv, d.nqb,
                                 d.max_kv_blocks, n_rg);
  };
  if (d.D == 128) wr == 2 ? launch(scores_kernel<128, 2>) : launch(scores_kernel<128, 1>);
  else wr == 2 ? launch(scores_kernel<64, 2>) : launch(scores_kernel<64, 1>);
  return hipGetLastError();
}

// Calls f(integral_constant M): a row of up to max_nc blocks, M per thread.  The
// rounds of a longer M are skipped or run empty: 5000 blocks took 18.8 us with 64
// keys per thread and take 13.7 with 32.
template <typename F>
static void with_keys_per_thread(int max_nc, F f) {
  if (max_nc <= 256) f(std::integral_constant<int, 1>{});
  else if (max_nc <= 1024) f(std::integral_constant<int, 4>{});
  else if (max_nc <= 2048) f(std::integral_constant<int, 8>{});
  else if (max_nc <= 4096) f(std::integral_constant<int, 16>{});
  else if (max_nc <= 8192) f(std::integral_constant<int, 32>{});
  else f(std::integral_constant<int, kMaxKvBlocks / 256>{});
}

hipError_t launch_select(const Dims& d, const float* scores, const int32_t* cached_len,
                         float top_frac, int sink_blocks, int local_blocks, uint64_t* masks,
                         hipStream_t st, uint64_t* group_words, int group_size) {
  dim3 grid(d.B * d.Hq * d.nqb);
  auto* gw = reinterpret_cast<unsigned long long*>(group_words);
  with_keys_per_thread(d.max_nc, [&](auto M) {
    select_kernel<M.value><<<grid, 256, 0, st>>>(scores, cached_len, masks, d.Hq, d.nqb,
                                                 d.max_kv_blocks, d.W, d.C, d.q_block, top_frac,
                                                 sink_blocks, local_blocks, gw, group_size);
  });
  return hipGetLastError();
}

hipError_t launch_threshold_select(const Dims& d, const float* scores, const int32_t* cached_len,
                                   float margin, int sink_blocks, int local_blocks,
                                   uint64_t* masks, hipStream_t st) {
  dim3 grid(d.B * d.Hq * d.nqb);
  with_keys_per_thread(d.max_nc, [&](auto M) {
    threshold_select_kernel<M.value><<<grid, 256, 0, st>>>(scores, cached_len, masks, d.Hq, d.nqb,
                                                           d.max_kv_blocks, d.W, d.C, d.q_block,
                                                           margin, sink_blocks, local_blocks);
  });
  return hipGetLastError();
}

}  // namespace ca
