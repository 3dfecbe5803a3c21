// Internal launcher interface between the C ABI (api.hip) and the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ca {

// Validated problem sizes, derived once on the host.
struct Dims {
  int B, Hq, Hkv, D, page, q_block, C, max_kv_blocks;
  int nqb;           // ceil(C / q_block)
  int W;             // mask words per row
  int max_nc;        // max_b full cached blocks, floor(cached_len_b / page)
  int max_nkb;       // max_b blocks of the sequence, ceil((cached_len_b + C) / page)
};

// Q-block and K-block pooling in one launch (q or k_pool may be nullptr to
// skip that part); clear_words[0, n_clear) are zeroed by the same launch.
hipError_t launch_pool(const Dims& d, const uint16_t* q, float* q_mean, const uint16_t* k_pool,
                       const int32_t* page_table, const int32_t* cached_len,
                       const int32_t* cached_len_host, int first_block, float* k_mean,
                       hipStream_t st, uint64_t* clear_words = nullptr, int n_clear = 0);
hipError_t launch_pool_q(const Dims& d, const uint16_t* q, float* q_mean, hipStream_t st,
                         uint64_t* clear_words = nullptr, int n_clear = 0);
hipError_t launch_pool_k(const Dims& d, const uint16_t* k_pool, const int32_t* page_table,
                         const int32_t* cached_len, const int32_t* cached_len_host,
                         int first_block, float* k_mean, hipStream_t st);
hipError_t launch_scores(const Dims& d, const float* q_mean, const float* k_mean,
                         const int32_t* cached_len, float* scores, hipStream_t st);
// With group_words set, the selected rows are ORed into the (b, group) union
// words (cleared beforehand) instead of being stored as masks.
hipError_t launch_select(const Dims& d, const float* scores, const int32_t* cached_len,
                         float top_frac, int sink_blocks, int local_blocks, uint64_t* masks,
                         hipStream_t st, uint64_t* group_words = nullptr, int group_size = 1);
hipError_t launch_threshold_select(const Dims& d, const float* scores, const int32_t* cached_len,
                                   float margin, int sink_blocks, int local_blocks,
                                   uint64_t* masks, hipStream_t st);

size_t tables_ws_bytes(const Dims& d, int group_size);
hipError_t launch_tables(const Dims& d, const uint64_t* masks, const int32_t* cached_len,
                         int group_size, int32_t* kv_indptr, int32_t* kv_indices, void* ws,
                         hipStream_t st);
// CSR from per-row union words (each row's count is its words' popcount).
hipError_t launch_compact_words(const Dims& d, int rows, const uint64_t* words,
                                int32_t* kv_indptr, int32_t* kv_indices, hipStream_t st);
// Block-sparse rows (b, h, Q-block i) holding the union of the group of h,
// causally limited to Q-block i (the block-sparse arm at matched tables).
size_t union_rows_ws_bytes(const Dims& d, int group_size);
hipError_t launch_union_rows(const Dims& d, const uint64_t* masks, const int32_t* cached_len,
                             int group_size, int32_t* kv_indptr, int32_t* kv_indices, void* ws,
                             hipStream_t st);

// Table layouts the attention kernel understands.
constexpr int kTablesPerGroup = 0;   // row b*G + g, entries translated by page_table
constexpr int kTablesPerQTile = 1;   // row (b*Hq + h)*n_qtiles + tile (block-sparse arm)
constexpr int kTablesPacked = 2;     // per-group rows; page of entry p is p (copy arm)

// ---------------------------------------------------------------------------
// Equal shares of a launch's pages, one per CU: the arithmetic of the balanced
// attention launch (plain integers, the same on host and device).
//
// For a query tile t, the table rows r = 0 .. R-1 laid end to end form a line
// of length T(t), row r on [A_r, A_r + o + w_r): o is what a piece's start and
// end cost, in entries, and w_r the number of the row's entries the tile can
// see if the row lists the chunk's own blocks (at least 1, so that every row
// has a piece that writes its output, and never more than the true count, so
// that no piece is left out; the piece holding the last of them runs on to the
// row's end and drops what the tile cannot see).  XCD x takes the slab
// [x T/8, (x+1) T/8) of the line, and its 32 CUs share the n < 32 tiles' slabs:
// a slab is cut into s_main = 32 / n main segments of equal length and, when
// n * s_main < 32, a shorter last one.  CU i*n + t runs main segment i of tile
// t.  The m = 32 - n*s_main < n CUs left over share the last segments of all
// tiles, laid end to end and cut into m equal parts (so a tile's last segment
// is cut at most once more); a last segment is as long as makes a part and the
// cost of its pieces equal to a main segment and its piece.  All tiles of a
// segment walk the same entries in step, which the XCD's 4 MB L2 needs for long
// rows.
//
// Where a cut meets a row it takes effect at an even entry (the kernel
// pipelines pairs of pages), or not at all when it falls on the row's first o
// or so near an end that the short piece would cost more than it moves: the
// row then starts, or ends, with the cut (ShareRow).  Interval J of a tile's
// line lies between its cuts J-1 and J.  A row's pieces are the intervals j0 ..
// j0+P-1 that meet it, in entry order (one between two cuts that take effect at
// the same entry is empty).
// ---------------------------------------------------------------------------
constexpr int kAttnXcds = 8;         // MI355X: 8 dies of 32 CUs, one L2 each
constexpr int kAttnCusPerXcd = 32;
constexpr int kSharesMaxRows = 64;   // one table row per lane

struct AttnShares {
  bool on = false;
  int n = 1;               // query tiles
  int s_main = 1;          // main segments per slab
  int left = 0;            // CUs left over (m above)
  int overhead = 0;        // cost of a piece's start and end, in entries
  int query_tile = 0;      // chunk queries per tile
  int slots_per_slab = 0;  // intervals of one slab over all tiles
  bool first_by_row = true;   // slots of rows' first pieces: see PieceList
  int slots = 0;           // partial results a launch can store
  int slot_rows = 0;       // rows of a slot: a tile's 16-row fragments that hold a query
};

// a / b for a quotient below 2^20 (one step of correction on the float one).
__host__ __device__ __forceinline__ unsigned share_div(unsigned a, unsigned b) {
#if defined(__HIP_DEVICE_COMPILE__)
  unsigned q = (unsigned)((float)a * __builtin_amdgcn_rcpf((float)b));
  int r = (int)(a - q * b);
  if (r < 0) --q, r += (int)b;
  if (r >= (int)b) ++q;
  return q;
#else
  return a / b;
#endif
}

// Cuts of tile t's line, of length T: interval i < per of slab x begins at
// share_cut(x, i).
struct ShareLine {
  unsigned T, S;
  unsigned last;    // length of a slab's last segment (0: there is none)
  unsigned inner;   // where in it another cut lies (0: there is none)
  unsigned per;     // intervals per slab
};

// The left-over CU that begins inside the last segment of tile t, or begins
// with the next tile's.
__host__ __device__ __forceinline__ unsigned share_next_left(const AttnShares& s, unsigned t) {
  return share_div(t * s.left, s.n) + 1;
}

__host__ __device__ __forceinline__ ShareLine share_line(const AttnShares& s, unsigned T, unsigned t) {
  ShareLine l = {T, (unsigned)s.s_main, 0, 0, (unsigned)s.s_main};
  if (s.left > 0) {
    // main + overhead = (n / m) last + pieces * overhead, where a left-over CU
    // has n / m pieces, and one more when its part begins inside a tile;
    // s_main * main + last = T / 8
    const int m = s.left, n = s.n, begun = n % m != 0 ? m - 1 : 0;
    const int room = (int)(T / kAttnXcds) * m - s.s_main * s.overhead * (n + begun - m);
    if (room > 0) l.last = share_div((unsigned)room, (unsigned)(s.s_main * n + m));
    if (l.last > 0) {
      ++l.per;
      const unsigned at = share_next_left(s, t) * n - t * m;   // of m parts of the segment
      if (at < (unsigned)m) {
        l.inner = share_div(l.last * at + m - 1, m);
        ++l.per;
      }
    }
  }
  return l;
}

__host__ __device__ __forceinline__ unsigned share_slab(const ShareLine& l, unsigned x) {
  return (l.T * x + kAttnXcds - 1) / kAttnXcds;
}
// Combined length of the main segments of slab [b0, b1).
__host__ __device__ __forceinline__ unsigned share_main(const ShareLine& l, unsigned b0, unsigned b1) {
  return b1 - b0 > l.last ? b1 - b0 - l.last : 0;
}

__host__ __device__ __forceinline__ unsigned share_cut(const ShareLine& l, unsigned x, unsigned i) {
  const unsigned b0 = share_slab(l, x), b1 = share_slab(l, x + 1);
  if (i >= l.per) return b1;
  const unsigned main = share_main(l, b0, b1);
  if (i > l.S) {
    const unsigned cut = b0 + main + l.inner;
    return cut < b1 ? cut : b1;
  }
  return b0 + share_div(main * i + l.S - 1, l.S);
}

// Number of cuts at or before position p (< T).
__host__ __device__ __forceinline__ unsigned share_cuts_upto(const ShareLine& l, unsigned p) {
  unsigned x = share_div(kAttnXcds * p, l.T);
  if (x < kAttnXcds - 1 && share_slab(l, x + 1) <= p) ++x;
  const unsigned b0 = share_slab(l, x), main = share_main(l, b0, share_slab(l, x + 1));
  // cut i <= p - b0  <=>  main * i <= S (p - b0)
  unsigned i = l.last > 0 ? l.S : l.S - 1;
  if (main > 0) {
    const unsigned q = share_div(l.S * (p - b0), main);
    i = q < i ? q : i;
  }
  if (l.inner > 0 && p >= b0 + main + l.inner) i = l.S + 1;
  return x * l.per + i;
}

// One row of the line: len entries, w of them counted, on [A, A + o + w).
struct ShareRow {
  int A, w, len, o;
  __host__ __device__ __forceinline__ int near() const { return w / 4 < o ? w / 4 : o; }   // too short for a piece
  // The first and the last position at which a cut divides the row.
  __host__ __device__ __forceinline__ int first() const { return A + o + near() + 1; }
  __host__ __device__ __forceinline__ int last() const { return A + o + w - near() - 1; }
  __host__ __device__ __forceinline__ bool meets(int lo, int hi) const { return hi >= first() && lo <= last(); }
  // The entry at which a cut at or after first() takes effect.
  __host__ __device__ __forceinline__ int entry(int cut) const {
    const int e = (cut - A - o + 1) & ~1;
    return e < len ? e : len;
  }
};

// The pieces of one (row, tile).
struct PieceList {
  int j0, pieces, per_slab, tile;
  // Slot of piece o's partial result.  An interval holds at most one piece
  // that continues a row, and one that begins a row which goes on after it; a
  // row's first piece is also the only one of its (row, tile), whichever is
  // the smaller number.
  __host__ __device__ __forceinline__ int slot(int o, int row_tile, const AttnShares& s) const {
    const int first = kAttnXcds * s.slots_per_slab;
    if (o == 0 && s.first_by_row) return first + row_tile;
    const int J = j0 + o, x = J / per_slab, i = J - x * per_slab;
    const int in_slab = i <= s.s_main
                            ? i * s.n + tile
                            : s.n * (s.s_main + 1) + (int)share_next_left(s, tile) - 1;
    return (o == 0 ? first : 0) + x * s.slots_per_slab + in_slab;
  }
};

// Entries of a row of `len` entries that query tile t can see (the line's w).
__host__ __device__ __forceinline__ int share_visible(int len, int cached_len, int C, int t, int query_tile, int page) {
  const int q_end = (t + 1) * query_tile < C ? (t + 1) * query_tile : C;
  const int unseen = (cached_len + C - 1) / page - (cached_len + q_end - 1) / page;
  return len - unseen > 1 ? len - unseen : 1;
}

// ---------------------------------------------------------------------------
// Which launch an attention call takes (num_splits = 0).  The tables are on the
// GPU, so the choice goes by the sizes and the expected table lengths; a result's
// validity never depends on it.
// ---------------------------------------------------------------------------
constexpr int kAttnCus = kAttnXcds * kAttnCusPerXcd;
constexpr int kAttnTileRows = 256, kAttnHalfTileRows = 128;   // (head, query) rows per workgroup
constexpr int kMaxUniformSplits = 16;   // of the automatic choice

// Cached blocks that a row's table is expected to list: the paper's executed
// density after both unions is 0.30 on long contexts; short ones keep more (the
// forced blocks and the union of few top blocks per row: nearly all of 16).
inline double expected_listed(int cached_blocks) {
  const double n = 16 + 0.3 * cached_blocks;
  return n < cached_blocks ? n : cached_blocks;
}

// Uniform splits of `base` tiles that fill the `resident` workgroups of the GPU.
inline int attn_uniform_splits(int base, int resident, int max_nkb) {
  if (base >= resident) return 1;
  int s = (resident + base - 1) / base;
  const int by_len = max_nkb / 4 > 1 ? max_nkb / 4 : 1;
  if (s > by_len) s = by_len;
  return s < kMaxUniformSplits ? s : kMaxUniformSplits;
}

// Sizes of an attention call as the choice sees them.
struct AttnSize {
  int rows;                 // table rows (b, group)
  int tiles, half_tiles;    // query tiles per row, whole and half
  int query_tile;           // chunk queries of a whole tile
  int tile_rows;            // rows of a whole tile that hold a query
  int splits;               // uniform splits
  double longest, line;     // expected entries of the longest row and of all rows
  double full;              // pages per CU that whole tiles walk
  double unseen, unseen_half;   // entries that a whole or half tile does not see, on average
  double xcd_share;         // pages of the XCD with the most half tiles, over the average
  bool dense;
};

inline AttnSize attn_size(int batch, int groups, int group_size, int C, int page,
                          const int* cached_len, bool dense) {
  AttnSize z{};
  z.rows = batch * groups;
  z.dense = dense;
  const int qt = z.query_tile = kAttnTileRows / group_size, qt_half = kAttnHalfTileRows / group_size;
  z.tiles = (C + qt - 1) / qt;
  z.half_tiles = qt_half > 0 && kAttnHalfTileRows % group_size == 0 ? (C + qt_half - 1) / qt_half : 0;
  z.tile_rows = group_size * (C < qt ? C : qt);
  z.unseen = (z.tiles - 1) * (qt / (double)page) / 2;
  z.unseen_half = (z.half_tiles - 1) * (qt_half / (double)page) / 2;
  int max_nkb = 0;
  auto entries = [&](int b) {
    const int nc = cached_len[b] / page, nkb = (cached_len[b] + C - 1) / page + 1;
    max_nkb = nkb > max_nkb ? nkb : max_nkb;
    return dense ? nkb : nkb - nc + expected_listed(nc);
  };
  for (int b = 0; b < batch; ++b) {
    const double len = entries(b);
    z.longest = len > z.longest ? len : z.longest;
    z.line += groups * len;
    z.full += groups * z.tiles * (len - z.unseen) / kAttnCus;
  }
  z.splits = attn_uniform_splits(z.rows * z.tiles, kAttnCus, max_nkb);
  // Half tiles of row r run on XCD r % 8 where the rows spread evenly, else the XCDs
  // take the rows in order, an eighth of the launch each; a launch that is not a
  // multiple of 8 workgroups is dealt out one by one.  Only the choice where whole
  // tiles fill the GPU asks.
  z.xcd_share = 1;
  const long long rows = z.rows;
  if (rows * z.tiles < kAttnCus || rows * z.half_tiles % kAttnXcds != 0 || groups % kAttnXcds == 0)
    return z;
  double load[kAttnXcds] = {}, most = 0, all = 0;
  for (int b = 0; b < batch; ++b) {
    const double len = entries(b), pages = len > z.unseen_half + 1 ? len - z.unseen_half : 1;
    const long long r0 = (long long)b * groups, r1 = r0 + groups;
    for (int x = 0; x < kAttnXcds; ++x) {
      // of rows r0 .. r1-1: how many are x modulo 8, or lie in the x-th eighth
      const long long lo = x * rows > r0 * kAttnXcds ? x * rows : r0 * kAttnXcds;
      const long long hi = (x + 1) * rows < r1 * kAttnXcds ? (x + 1) * rows : r1 * kAttnXcds;
      const double held = rows % kAttnXcds == 0
                              ? (r1 + kAttnXcds - 1 - x) / kAttnXcds - (r0 + kAttnXcds - 1 - x) / kAttnXcds
                              : hi > lo ? (hi - lo) / (double)kAttnXcds : 0;
      load[x] += pages * held;
    }
  }
  for (double x : load) {
    most = x > most ? x : most;
    all += x;
  }
  z.xcd_share = most * kAttnXcds / all;
  return z;
}

// Times in us of the launches where the whole tiles leave CUs idle.  The constants
// were fitted to the choice that they make, over 2900 random sizes with every launch
// timed (1-8 sequences, 0-130K cached, 1-3000 tokens, 4-64 heads, listed at 0.15-0.5
// or dense, one GPU): 22 of them then take over 3% longer than with uniform splits
// and the XCD cut alone (at most 1.25 times), 0.855 of the time in the mean.
//   half tiles: a start, and the longest row at the rate of a workgroup that is
//     alone on its CU, or (more tiles than CUs) the longest and the shortest tile
//     of a row side by side;
//   equal shares: a start and the merge launch, the CU's pages, the more pieces
//     the more tiles, and the partial results of the rows that hold a query;
//   uniform splits: the same with pieces of the longest row, or where the pieces
//     outnumber the CUs about one piece more than the average; the merge of more
//     than 8 pieces goes through them twice.
struct AttnTimes {
  double half, shares, uniform;
};
inline AttnTimes attn_times(const AttnSize& z, int head_dim) {
  const bool d64 = head_dim == 64;
  const double base = z.rows * (double)z.tiles / kAttnCus, held = z.tile_rows / (double)kAttnTileRows;
  const double alone = (d64 ? 0.6 : 0.88) * z.longest;
  const double paired = z.rows * (long long)z.half_tiles <= kAttnCus
                            ? 0 : (d64 ? 0.9 : 1.2) * (z.longest - z.unseen_half);
  const double piece = z.longest / z.splits;
  const double walked = base * z.splits <= 1 ? piece : z.full + (d64 ? 1.0 : 0.7) * piece;
  AttnTimes t;
  t.half = (d64 ? 8 : 11.5) + (alone > paired ? alone : paired);
  t.shares = d64 ? 16.5 + 1.1 * z.full + 10 * base + 4.5 * held
                 : 25.5 + 1.4 * z.full + 18 * base + 5.5 * held;
  t.uniform = d64 ? 12.5 + 1.0 * walked + 7.5 * base * z.splits * held + (z.splits > 8 ? 8 : 0)
                  : 17.5 + 1.4 * walked + 13 * base * z.splits * held + (z.splits > 8 ? 9 : 0);
  return t;
}

// Equal shares can be laid out, and every CU has at least 4 expected pages (below
// that they take as long as the best other launch in the median, 0.65 to 1.4 of it
// from size to size).
inline bool attn_shares_fit(const AttnSize& z) {
  return z.rows <= kSharesMaxRows && z.tiles < kAttnCusPerXcd &&
         z.line * z.tiles / kAttnCus >= 4.0;
}

enum class AttnChoice { kHalfTiles, kShares, kOther };   // kOther: the XCD cut or uniform splits
// fit: equal shares can be laid out and the workspace holds them; z.splits: the
// uniform splits that it holds.
inline AttnChoice attn_choice(const AttnSize& z, int head_dim, bool fit) {
  const long long tiles = (long long)z.rows * z.tiles;
  if (tiles >= kAttnCus) {
    // Whole tiles fill the GPU.  By the part of the pages that the causal triangle
    // takes off the first tiles, medians over 112 of those sizes:
    //                          < 0.03  0.03-  0.06-  0.09-  0.12-  0.18-  0.25-
    //   half tiles : XCD cut     1.01   0.98   0.96   0.91   0.92   0.89   0.89
    //   equal shares : XCD cut   0.69   0.82   1.00   1.09   1.08   1.07   1.11
    // Copying each page for half the rows costs half tiles 3% at 128K.  They are not
    // cut, so that rows of different lengths leave some XCDs idle: with 1.13-1.54
    // times the average on one XCD 0.61-0.98 (11 sizes, one 1.03), with 1.99-2.7
    // times 0.93-1.42.
    // Equal shares gain what other launches leave idle, about the longest row's
    // pages in every round of tiles less the average: 0.37-1.0 of their time from
    // 24 pages (20 of 21 sizes), 0.93-1.12 below (11 sizes, median 1.04), the
    // 0.93 in four rounds, where the XCD cut makes twice their pieces.
    const bool much = z.rows * z.unseen >= 0.09 * z.line;
    if (much && z.half_tiles > 0 && z.xcd_share < 1.75) return AttnChoice::kHalfTiles;
    const long long rounds = (tiles + kAttnCus - 1) / kAttnCus;
    return fit && !much && (rounds >= 3 || z.longest * rounds - z.full >= 24)
               ? AttnChoice::kShares : AttnChoice::kOther;
  }
  // rows of at most 7 blocks, or no workspace: no cut, and half tiles walk a page in
  // 0.6-0.9 us where whole ones take 1.0-1.4
  if (z.splits == 1 && z.half_tiles > 0) return AttnChoice::kHalfTiles;
  const AttnTimes t = attn_times(z, head_dim);
  // Equal shares, but where uniform splits give every CU one piece only if they are
  // shorter: those are as even by expectation.  Real tables differ from row to row,
  // which outweighs what more pieces cost on long rows: with at most 8 rows (one per
  // XCD) from about 64 pages per CU (rows 10% apart: 0.96-1.06 of the time at 40-51
  // pages, 0.87-0.95 at 83), with more rows from about 100 (15% apart: 1.0-1.11 at
  // 41-95 pages, 1.0 at 130 and 210).
  const bool one_each = tiles * z.splits == kAttnCus;
  const bool uneven = !z.dense && z.full >= (z.rows <= kAttnXcds ? 64 : 100);
  const bool shares = fit && (!one_each || t.shares < t.uniform || uneven);
  // 6% for the fit's error: the cut launches lose less where they are wrong
  if (z.half_tiles > 0 && 1.06 * t.half < (shares ? t.shares : t.uniform))
    return AttnChoice::kHalfTiles;
  return shares ? AttnChoice::kShares : AttnChoice::kOther;
}

// The shares of a launch (attn_shares_fit).
inline AttnShares attn_shares(const AttnSize& z, int C, int head_dim) {
  AttnShares s;
  const int n = z.tiles;
  s.on = true;
  // one tile: its rows packed, so that a tile's rows end with the last query
  s.query_tile = n == 1 ? C : z.query_tile;
  // A piece costs 11 to 15 us, about 8 pages of 1.6 us (D = 128), and less counts
  // on short shares, which lose more by rounding to it than the pieces cost.  In us
  // at costs of 4, 6, 8 and 12 pages (the one taken in brackets):
  //     37 tokens over 65536           [40.2]  43.6   43.2   49.7
  //    300 over 20000                   69.0  [53.4]  55.4   59.8   (taken: 5, 53.4)
  //   1451 over 50001                  340.7  331.3  [322.5] 334.2
  //    512 over 129024                 261.7  260.5  [260.2] 260.0
  //   1024 over 30720 and 12345, D = 64 161.9 [160.1] 162.8  162.9
  //     64 over 16384, dense, D = 64    [27.2]  28.8   32.4   32.3
  const int most = head_dim == 64 ? 6 : 8;
  const double o = z.line * n / kAttnCus / (head_dim == 64 ? 8 : 3);
  s.overhead = o < 4 ? 4 : o > most ? most : (int)o;
  s.n = n;
  s.s_main = kAttnCusPerXcd / n;
  s.left = kAttnCusPerXcd - n * s.s_main;
  s.slots_per_slab = n * s.s_main + (s.left > 0 ? n + s.left : 0);
  s.first_by_row = z.rows * n < kAttnXcds * s.slots_per_slab;
  s.slots = kAttnXcds * s.slots_per_slab +
            (s.first_by_row ? z.rows * n : kAttnXcds * s.slots_per_slab);
  s.slot_rows = (z.tile_rows + 15) & ~15;
  return s;
}

// V page layouts of the pool (ca_problem.v_layout).
constexpr int kVTokenMajor = 0;   // [P, page, D], like the K pages
constexpr int kVTransposed = 1;   // [P, D, page]

// Attention over per-group tables (dense = identity tables, no table read).
struct AttnLaunch {
  const uint16_t* q;
  const uint16_t* k_pool;
  const uint16_t* v_pool;
  const int32_t* page_table;
  const int32_t* kv_indptr;
  const int32_t* kv_indices;
  const int32_t* cached_len;
  uint16_t* out;
  float* lse;
  int group_size;
  float sm_scale;
  int splits;        // >= 1
  void* ws;          // partials when splits > 1 (+ cuts and counters: XCD split)
  bool dense;
  int table_mode = kTablesPerGroup;
  long long packed_pages = 0;
  // splits == 2 with the cut of every table row chosen so that the 8 XCDs
  // carry equal loads (needs B * G % 8 == 0 and attn_xcd_ws_bytes of ws)
  bool xcd_balanced = false;
  int v_layout = kVTokenMajor;
  AttnShares shares;   // shares.on: balanced launch (attn_shares_ws_bytes of ws)
  // 128 rows per workgroup, two workgroups per CU, so that the causal triangle evens
  // out and no row is cut; splits == 1 (attention.hip: pair_tiles)
  bool half_tiles = false;
};
size_t attn_shares_ws_bytes(const Dims& d, int group_size, const AttnShares& s);
int attn_rows_per_workgroup(int table_mode);             // (head, query) rows per workgroup
int attn_query_tile(int group_size, int table_mode);     // chunk queries per workgroup
int attn_base_workgroups(const Dims& d, int group_size, int table_mode);
int attn_resident_workgroups(int table_mode);            // workgroups the GPU holds at once
size_t attn_ws_bytes(const Dims& d, int splits);
size_t attn_xcd_ws_bytes(const Dims& d, int group_size);
hipError_t launch_attention(const Dims& d, const AttnLaunch& a, hipStream_t st);
hipError_t launch_gather(const Dims& d, const uint16_t* k_pool, const uint16_t* v_pool,
                         const int32_t* page_table, const int32_t* kv_indptr,
                         const int32_t* kv_indices, int group_size, long long capacity_pages,
                         uint16_t* k_packed, uint16_t* v_packed, hipStream_t st);

}  // namespace ca
