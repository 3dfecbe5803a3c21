// Block-union tables: Q-block union + intra-group union (bitwise OR) and
// compaction of the union bitmask into CSR kv_indptr / kv_indices
// (Sec. 3.2 displayed equations; App. B.2 for the CSR pair).
//
// One launch for few rows (tables_kernel), else two, all integer-only and
// deterministic:
//   union_kernel   one workgroup per table row r = b*G + g: OR the
//                  group_size*nQB mask rows of the group word by word in LDS
//                  (ds_or_b64), clip to nKB_b, store the row's union words and
//                  its popcount;
//   compact_kernel one workgroup per row: row offset = sum of the counts of
//                  earlier rows (no atomics), one scan of the words'
//                  popcounts, then every wave writes the set block ids of
//                  words of its own, in ascending order.
#include "common.hpp"
#include "kernels.hpp"

namespace ca {

constexpr int kMaxWords = kMaxKvBlocks / 64;

__global__ __launch_bounds__(256) void union_kernel(const uint64_t* __restrict__ masks,
                                                    const int32_t* __restrict__ cached_len,
                                                    uint64_t* __restrict__ gwords,
                                                    int32_t* __restrict__ counts, int Hq,
                                                    int nqb, int W, int group_size, int G,
                                                    int C) {
  __shared__ unsigned long long acc[kMaxWords];
  __shared__ int red[4];
  const int r = blockIdx.x;
  const int b = r / G, g = r % G;
  const int t = threadIdx.x;
  const int nkb = blocks_for(cached_len[b] + C);
  for (int w = t; w < W; w += 256) acc[w] = 0ull;
  __syncthreads();
  const int rows = group_size * nqb;
  const uint64_t* src = masks + ((size_t)b * Hq + (size_t)g * group_size) * nqb * W;
  if (W <= 256 && (256 % W) == 0) {
    // fixed word per thread: OR privately, then one LDS atomic
    // 8 loads per lane in flight per round
    const int w = t % W, step = 256 / W;
    unsigned long long v = 0ull;
    for (int row0 = t / W; row0 < rows; row0 += 8 * step) {
      unsigned long long x[8];
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const int row = row0 + m * step;
        x[m] = row < rows ? src[(size_t)row * W + w] : 0ull;
      }
#pragma unroll
      for (int m = 0; m < 8; ++m) v |= x[m];
    }
    if (v) atomicOr(&acc[w], v);
  } else {
    for (int x = t; x < rows * W; x += 256) {
      const unsigned long long v = src[x];
      if (v) atomicOr(&acc[x % W], v);
    }
  }
  __syncthreads();
  int cnt = 0;
  for (int w = t; w < W; w += 256) {
    unsigned long long v = acc[w];
    const int lo = w * 64;
    if (lo >= nkb) v = 0ull;
    else if (nkb - lo < 64) v &= (~0ull >> (64 - (nkb - lo)));
    gwords[(size_t)r * W + w] = v;
    cnt += __popcll(v);
  }
  cnt = wave_sum(cnt);
  if (lane_id() == 0) red[t >> 6] = cnt;
  __syncthreads();
  if (t == 0) counts[r] = red[0] + red[1] + red[2] + red[3];
}

// Writes the set bits of one row's words, ascending, from row_start on.  The
// words' offsets come from one scan (a word per thread and round); then every
// wave writes words of its own, 64 bits by 64 lanes, with no further barrier.
// (256-block slabs with two barriers each took 4.7 us for 32 rows of 2016
// blocks, launch included.)
template <int THREADS, typename Words>
__device__ void compact_row(const Words* gw, int row_start, int32_t* __restrict__ kv_indices,
                            int W) {
  __shared__ unsigned long long words[kMaxWords];
  __shared__ int offset[kMaxWords];
  __shared__ int tot[4];
  const int t = threadIdx.x, wv = t >> 6;
  static_assert(kMaxWords == 256 && THREADS >= 256, "one word per thread, four waves");
  if (t < kMaxWords) {
    const unsigned long long v = t < W ? gw[t] : 0ull;
    const int n = __popcll(v), incl = wave_inclusive_scan(n);
    if (lane_id() == 63) tot[wv] = incl;
    words[t] = v;
    offset[t] = incl - n;
  }
  __syncthreads();
  int before[4], sum = row_start;   // start of each 64-word quarter
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    before[x] = sum;
    sum += tot[x];
  }
#pragma unroll 4
  for (int w = wv; w < W; w += THREADS / kWave) {
    const unsigned long long word = words[w];
    const int q = w >> 6;
    const int at = offset[w] + (q == 0 ? before[0] : q == 1 ? before[1] : q == 2 ? before[2] : before[3]);
    if ((word >> lane_id()) & 1ull) kv_indices[at + lanes_below(word)] = 64 * w + lane_id();
  }
}

__global__ __launch_bounds__(256) void compact_kernel(const uint64_t* __restrict__ gwords,
                                                      const int32_t* __restrict__ counts,
                                                      int32_t* __restrict__ kv_indptr,
                                                      int32_t* __restrict__ kv_indices, int W) {
  __shared__ int red[4];
  const int r = blockIdx.x;
  const int t = threadIdx.x;
  int part = 0;
  for (int x = t; x < r; x += 256) part += counts[x];
  part = wave_sum(part);
  if (lane_id() == 0) red[t >> 6] = part;
  __syncthreads();
  const int row_start = red[0] + red[1] + red[2] + red[3];
  if (t == 0) {
    if (r == 0) kv_indptr[0] = 0;
    kv_indptr[r + 1] = row_start + counts[r];
  }
  compact_row<256>(gwords + (size_t)r * W, row_start, kv_indices, W);
}

// Same, with the counts taken from the words themselves: row r starts after
// the set bits of rows 0..r-1 (the fused estimator-to-union path, whose
// words are complete only once every selection row has been ORed in).
__global__ __launch_bounds__(256) void compact_words_kernel(const uint64_t* __restrict__ gwords,
                                                            int32_t* __restrict__ kv_indptr,
                                                            int32_t* __restrict__ kv_indices,
                                                            int W) {
  __shared__ int red[8];
  const int r = blockIdx.x;
  const int t = threadIdx.x;
  int before = 0, own = 0;
  // 8 loads per lane in flight per round
  for (int x0 = t; x0 < (r + 1) * W; x0 += 8 * 256) {
    uint64_t v[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) v[m] = x0 + 256 * m < (r + 1) * W ? gwords[x0 + 256 * m] : 0ull;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const int c = __popcll(v[m]);
      if (x0 + 256 * m < r * W) before += c;
      else own += c;
    }
  }
  before = wave_sum(before);
  own = wave_sum(own);
  if (lane_id() == 0) {
    red[t >> 6] = before;
    red[4 + (t >> 6)] = own;
  }
  __syncthreads();
  const int row_start = red[0] + red[1] + red[2] + red[3];
  if (t == 0) {
    if (r == 0) kv_indptr[0] = 0;
    kv_indptr[r + 1] = row_start + red[4] + red[5] + red[6] + red[7];
  }
  compact_row<256>(gwords + (size_t)r * W, row_start, kv_indices, W);
}

// Union and compaction of few rows in one launch: workgroup r forms the union
// words of rows 0 .. r, a wave per row, from the masks themselves, keeps the
// counts of the earlier rows for its offset and the words of its own for
// compact_row.  It saves the host's second launch, which sets the time of the
// two it replaces (8.1-9 us in all).  Two lines bound it:
//   * the masks of the earlier rows are read again by every later row's
//     workgroup, (R + 1) / 2 times the masks in all: 32 rows of 524 KB (8.7 MB of
//     reads) took 11.5 us against 9.3;
//   * a wave waits for its loads one round after another: table rows of the wave
//     (R / 16) x 64-word windows x rounds of 16 loads over the mask rows.  Up to 4
//     rounds 5.6-9.3 us against 8.1-11.7 (128 mask rows of 32 words 6.1 : 8.4, 32
//     of 128 words 7.3 : 8.6, 16 of 256 words 8.5 : 10.6), with more than 16 table
//     rows up to 3 (48 rows 7.6-8.2 : 8.5-9.1; 64 rows, 4 rounds, 9.0-9.8 :
//     8.8-9.2).  Past the line one wave reads for long: 1 row of 256 x 32 words
//     8.8 : 8.3, of 512 x 32 13.9 : 9.3, of 512 x 256 90 : 46.
constexpr size_t kTablesOneLaunchReads = 4 << 20;
constexpr int kTablesThreads = 1024;
constexpr int kTablesWaves = kTablesThreads / kWave;
constexpr int kTablesRowsInFlight = 16;   // loads per round of a wave
constexpr int kTablesOneLaunchRows = 3 * kTablesWaves;

// Rounds of loads that a wave of the last workgroup waits for in turn.
static int tables_wave_rounds(int rows, int mask_rows, int W) {
  int Wp = 1;
  while (Wp < W && Wp < kWave) Wp <<= 1;
  const int per_round = kTablesRowsInFlight * (kWave / Wp);
  return ((rows + kTablesWaves - 1) / kTablesWaves) * ((W + kWave - 1) / kWave) *
         ((mask_rows + per_round - 1) / per_round);
}

static bool tables_one_launch(int rows, int mask_rows, int W, size_t mask_bytes) {
  return mask_bytes * (rows + 1) / 2 <= kTablesOneLaunchReads &&
         tables_wave_rounds(rows, mask_rows, W) <= (rows <= kTablesWaves ? 4 : 3);
}

// OR over `rows` mask rows of W words: word w of the result in lane w % 64 of
// round w / 64 (Wp = the power of two from W up, at most 64; 64 / Wp rows are
// read at once).
__device__ __forceinline__ unsigned long long or_rows(const uint64_t* __restrict__ src, int rows,
                                                      int W, int Wp, int w0) {
  const int l = lane_id(), w = w0 + (l & (Wp - 1)), step = kWave / Wp;
  unsigned long long v = 0ull;
  for (int row0 = l / Wp; row0 < rows; row0 += kTablesRowsInFlight * step) {
    unsigned long long x[kTablesRowsInFlight];
#pragma unroll
    for (int m = 0; m < kTablesRowsInFlight; ++m) {
      const int row = row0 + m * step;
      x[m] = row < rows && w < W ? src[(size_t)row * W + w] : 0ull;
    }
#pragma unroll
    for (int m = 0; m < kTablesRowsInFlight; ++m) v |= x[m];
  }
  for (int o = Wp; o < kWave; o <<= 1) {
    const unsigned lo = __shfl_xor((unsigned)v, o, kWave);
    const unsigned hi = __shfl_xor((unsigned)(v >> 32), o, kWave);
    v |= ((unsigned long long)hi << 32) | lo;
  }
  return v;
}

__global__ __launch_bounds__(kTablesThreads) void tables_kernel(
    const uint64_t* __restrict__ masks, const int32_t* __restrict__ cached_len,
    int32_t* __restrict__ kv_indptr, int32_t* __restrict__ kv_indices, int Hq, int nqb, int W,
    int group_size, int G, int C) {
  __shared__ unsigned long long own[kMaxWords];
  __shared__ int counts[kTablesOneLaunchRows];   // rows whose rounds are at most 3
  const int r = blockIdx.x, t = threadIdx.x, wv = t >> 6, l = t & 63;
  const int rows = group_size * nqb;
  int Wp = 1;
  while (Wp < W && Wp < kWave) Wp <<= 1;
  for (int x = wv; x <= r; x += kTablesWaves) {
    const int b = x / G, g = x - b * G;
    const int nkb = blocks_for(cached_len[b] + C);
    const uint64_t* src = masks + ((size_t)b * Hq + (size_t)g * group_size) * nqb * W;
    int cnt = 0;
    for (int w0 = 0; w0 < W; w0 += kWave) {
      unsigned long long v = or_rows(src, rows, W, Wp, w0);
      const int w = w0 + l, lo = 64 * w;   // lanes past the words hold copies: not counted
      if (l >= Wp || lo >= nkb) v = 0ull;
      else if (nkb - lo < 64) v &= ~0ull >> (64 - (nkb - lo));
      cnt += __popcll(v);
      if (x == r && w < W && l < Wp) own[w] = v;
    }
    cnt = wave_sum(cnt);
    if (l == 0) counts[x] = cnt;
  }
  __syncthreads();
  int row_start = 0;
  for (int x = 0; x < r; ++x) row_start += counts[x];
  if (t == 0) {
    if (r == 0) kv_indptr[0] = 0;
    kv_indptr[r + 1] = row_start + counts[r];
  }
  compact_row<kTablesThreads>(own, row_start, kv_indices, W);
}

hipError_t launch_compact_words(const Dims& d, int rows, const uint64_t* words,
                                int32_t* kv_indptr, int32_t* kv_indices, hipStream_t st) {
  compact_words_kernel<<<rows, 256, 0, st>>>(words, kv_indptr, kv_indices, d.W);
  return hipGetLastError();
}

// Block-sparse arm at matched tables (Sec. 4.4): the union of execution group
// g(h) as the mask row of every (b, h, Q-block i), limited to the blocks that
// Q-block i can see causally (up to the block holding its last query).  One
// workgroup per (b, h, i) row; words from the group rows written by
// union_kernel.
__global__ __launch_bounds__(256) void expand_union_kernel(const uint64_t* __restrict__ gwords,
                                                           const int32_t* __restrict__ cached_len,
                                                           uint64_t* __restrict__ rwords,
                                                           int32_t* __restrict__ counts, int Hq,
                                                           int nqb, int W, int group_size,
                                                           int q_block, int C) {
  __shared__ int red[4];
  const int r = blockIdx.x;                 // (b*Hq + h)*nqb + i
  const int i = r % nqb;
  const int h = (r / nqb) % Hq;
  const int b = r / (nqb * Hq);
  const int G = Hq / group_size;
  const int t = threadIdx.x;
  const int lim = causal_block_end(cached_len[b], C, i, q_block);
  const uint64_t* src = gwords + ((size_t)b * G + h / group_size) * W;
  int cnt = 0;
  for (int w = t; w < W; w += 256) {
    unsigned long long v = src[w];
    const int lo = w * 64;
    if (lo >= lim) v = 0ull;
    else if (lim - lo < 64) v &= (~0ull >> (64 - (lim - lo)));
    rwords[(size_t)r * W + w] = v;
    cnt += __popcll(v);
  }
  cnt = wave_sum(cnt);
  if (lane_id() == 0) red[t >> 6] = cnt;
  __syncthreads();
  if (t == 0) counts[r] = red[0] + red[1] + red[2] + red[3];
}

// The per-row words follow the group-row workspace at the next 8-byte boundary
// (the group-row part ends with one int32 count per row).
static size_t union_rows_offset(const Dims& d, int group_size) {
  return (tables_ws_bytes(d, group_size) + 7) & ~(size_t)7;
}

size_t union_rows_ws_bytes(const Dims& d, int group_size) {
  const size_t R = (size_t)d.B * d.Hq * d.nqb;
  return union_rows_offset(d, group_size) + R * d.W * sizeof(uint64_t) + R * sizeof(int32_t);
}

hipError_t launch_union_rows(const Dims& d, const uint64_t* masks, const int32_t* cached_len,
                             int group_size, int32_t* kv_indptr, int32_t* kv_indices, void* ws,
                             hipStream_t st) {
  const int G = d.Hq / group_size;
  const int RG = d.B * G;
  const int R = d.B * d.Hq * d.nqb;
  uint64_t* gwords = static_cast<uint64_t*>(ws);
  int32_t* gcounts = reinterpret_cast<int32_t*>(gwords + (size_t)RG * d.W);
  uint64_t* rwords = reinterpret_cast<uint64_t*>(
      static_cast<char*>(ws) + union_rows_offset(d, group_size));
  int32_t* rcounts = reinterpret_cast<int32_t*>(rwords + (size_t)R * d.W);
  union_kernel<<<RG, 256, 0, st>>>(masks, cached_len, gwords, gcounts, d.Hq, d.nqb, d.W,
                                   group_size, G, d.C);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  expand_union_kernel<<<R, 256, 0, st>>>(gwords, cached_len, rwords, rcounts, d.Hq, d.nqb, d.W,
                                         group_size, d.q_block, d.C);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  compact_kernel<<<R, 256, 0, st>>>(rwords, rcounts, kv_indptr, kv_indices, d.W);
  return hipGetLastError();
}

size_t tables_ws_bytes(const Dims& d, int group_size) {
  const size_t R = (size_t)d.B * (d.Hq / group_size);
  return R * d.W * sizeof(uint64_t) + R * sizeof(int32_t);
}

hipError_t launch_tables(const Dims& d, const uint64_t* masks, const int32_t* cached_len,
                         int group_size, int32_t* kv_indptr, int32_t* kv_indices, void* ws,
                         hipStream_t st) {
  const int G = d.Hq / group_size;
  const int R = d.B * G;
  const size_t mask_bytes = (size_t)d.B * d.Hq * d.nqb * d.W * sizeof(uint64_t);
  if (tables_one_launch(R, group_size * d.nqb, d.W, mask_bytes)) {
    tables_kernel<<<R, kTablesThreads, 0, st>>>(masks, cached_len, kv_indptr, kv_indices, d.Hq,
                                                d.nqb, d.W, group_size, G, d.C);
    return hipGetLastError();
  }
  uint64_t* gwords = static_cast<uint64_t*>(ws);
  int32_t* counts = reinterpret_cast<int32_t*>(gwords + (size_t)R * d.W);
  union_kernel<<<R, 256, 0, st>>>(masks, cached_len, gwords, counts, d.Hq, d.nqb, d.W,
                                  group_size, G, d.C);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  compact_kernel<<<R, 256, 0, st>>>(gwords, counts, kv_indptr, kv_indices, d.W);
  return hipGetLastError();
}

}  // namespace ca
