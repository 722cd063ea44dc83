// tvq_spans.h -- how an attention call is split over workgroups: the plan that the host makes and
// the rule by which the kernels give the columns to the sequences.  Plain arithmetic, compiled
// into the library and, by itself, into the host tests.
//
// A workgroup takes a span of whole tiles of one (sequence, KV head).  The spans of all sequences
// are the n_part columns of one list per head, in batch order.
//   spare == 0  sequence b holds columns b per_seq .. b per_seq + per_seq - 1 and uses the first
//               per_seq of them (contexts known to the host) or span_floor(T_b) of them (contexts
//               that are device data): nothing to look up but its own context.
//   spare > 0   (contexts on the device) sequence b holds span_count(T_b) consecutive columns:
//               span_floor(T_b) + floor(T_b spare / sum T), while its spans stay at or above
//               2^min_log2 tiles.  Every workgroup counts the same way.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define TVQ_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define TVQ_HOST_DEVICE inline
#endif

namespace tvq {

constexpr uint32_t kSpanWaves = 4;       // waves of a workgroup: a span of T tiles keeps them
                                         // busy from T = 4 on
constexpr int64_t kMaxWaveTokens = 4096; // most tokens of a wave
constexpr int64_t kMaxWaveBlocks = 63;   // and pool blocks: a wave may start inside a block and
                                         // holds the ids of 64 in its lanes
constexpr int64_t kMaxSpareBatch = 4096; // most sequences that share columns: the lookup holds
                                         // 64 sequences per lane (seq_columns)

TVQ_HOST_DEVICE uint32_t span_floor(uint32_t T, uint32_t max_span) {
  return T <= max_span ? 1u : (T + max_span - 1) / max_span;
}

// Columns of a sequence of T tiles, `total` tiles in all.  T * spare is exact in fp64 (spare is at
// most a few times the workgroups of a launch), and its quotient cannot round up to an integer
// above it, so the counts add up to at most the sum of the floors + spare.  A span is at most
// max(2^min_log2, ceil(total / spare)) tiles, n_part / spare times an even share.
TVQ_HOST_DEVICE uint32_t span_count(uint32_t T, uint32_t total, uint32_t spare, uint32_t max_span,
                                    uint32_t min_log2) {
  const uint32_t c = span_floor(T, max_span);
  const uint32_t more = (uint32_t)((double)T * (double)spare / (double)total);
  const uint32_t most = (T + (1u << min_log2) - 1) >> min_log2;
  const uint32_t n = c + more < most ? c + more : most;
  return n > c ? n : c;
}

// Column and KV head of workgroup `unit` (passes aside).  Where the contexts differ the columns go
// first, a column's heads side by side, so that the columns of a long sequence lie together and
// go round all XCDs and compute units.  Ordered by head first, they were n_part apart for the
// heads, a multiple of the XCDs and of an XCD's places as a rule, and met on the same compute
// units.  8 KV heads, d = 128, us a layer, heads first / columns first: 2 sequences of 8,192
// tokens among 126 of 1,000, a column each 442 / 264; 4 of 8,192 among 512 506 / 330; 16 of 8,193
// to 32,770 222 / 201; 64 of 75 to 300 26 / 19.  Equal contexts keep the heads first: neighbours
// then read neighbouring records (8 sequences of 8,195 tokens, d = 64, six layers: 171 / 172.6).
struct UnitOf {
  uint32_t column, head;
};
TVQ_HOST_DEVICE UnitOf unit_of(uint32_t unit, uint32_t heads, uint32_t n_part,
                               bool columns_first) {
  const uint32_t div = columns_first ? heads : n_part;
  const uint32_t q = unit / div, r = unit - q * div;
  return columns_first ? UnitOf{q, r} : UnitOf{r, q};
}

struct AttnSplit {
  int64_t chunk, n_chunks;                       // of the workspace rule
  int64_t n_part, per_seq, spare, max_span, min_log2;
};

// The split of a call; n_part = 0: no columns, a wave takes a whole row.  rows: (sequence, KV head, pass over the query heads); vpw: tokens of a
// tile; block_tokens: of a paged pool (the contexts are then device data and t_end bounds them),
// 0 for a contiguous cache (every context is t_end); slots: waves that the device holds at once.
//
// Workspace rule: the rows split into equal chunks so that there is about one per wave slot, of
// whole tile pairs, at least four tiles and at most kMaxWaveTokens tokens.  The workspace holds a
// partial per query head and chunk; the columns never number more.
//
// Columns.  A launch of as many workgroups as the device holds runs in one go, and where the rows
// divide it well that is the fastest.  Where they do not, or the contexts differ much, finer
// columns let the device even the work out as places fall free.  Each costs a start, about 1.4
// tiles' time, and a partial, so short spans are not cut further.  us a layer on 1,024 places
// (d = 128, 8 KV heads, 32 query heads), one go / finer; "chunks" is a wave per chunk of the
// workspace rule, which four waves of a workgroup make coarser:
//   equal contexts of 4,096 tokens: 65 sequences 188 / 160 (chunks 163), 98: 235 / 226 (229),
//   129: 331 / 297 (335); of 1,500 tokens: 65 sequences 74 / 64 (68); of 512: 65 sequences 29 / 30
//   paged, 65 sequences of 4,096: 198 / 164 (166), 96: 221 / 230 (229)
//   paged, 1,025 to 4,100 tokens: 33 sequences 60 / 63 (80), 40: 70 / 69 (83), 48: 89 / 80 (107),
//   64: 117 / 103 (142), 100: 164 / 160 (202)
//   paged, a column a sequence / and a half: 128 of 1,025 to 4,100 186 / 190 (244), 128 of 4,096
//   275 / 279 (290), 2 of 8,192 and 126 of 1,000 264 / 102 (258)
// A wave per row, where there are rows for the wave slots and the contexts are short: a row then
// costs one wave's start instead of four, and nothing is summed over waves; but the longest row
// is one wave's.  us a layer, a workgroup / a wave per row (chunks), 8 KV heads:
//   twice as many rows as slots, d = 64, 64 query heads, 512 paged sequences: 2 to 8 tokens 44 / 19
//   (34), 25 to 100 51 / 32 (44), 250 to 1,000 182 / 174 (178)
//   as many, d = 128, 32 query heads, 512 sequences: 8 tokens 23 / 12 (23), 100: 43 / 38 (46);
//   paged, 16 of 500 among 512 of 40: 33 / 71 (78); 600 of 500: 168 / 181 (184)
//   half as many: 30 tokens 14 / 11 (17), 60: 16 / 16 (22), paged, 100 to 400: 44 / 59 (54); a
//   quarter: 30 tokens 7.5 / 9.4 (13.5)
inline AttnSplit attn_split(int64_t batch, int64_t heads, int64_t n_pass, int64_t t_end,
                            int64_t block_tokens, int64_t vpw, int64_t slots) {
  AttnSplit s;
  const auto at_least = [](int64_t a, int64_t b) { return a > b ? a : b; };
  const auto at_most = [](int64_t a, int64_t b) { return a < b ? a : b; };
  const auto ceil_div = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  const int64_t rows = batch * heads * n_pass;
  const int64_t max_chunk = block_tokens > 0
                                ? at_most(kMaxWaveTokens, kMaxWaveBlocks * block_tokens)
                                : kMaxWaveTokens;
  const int64_t step = 2 * vpw;
  const int64_t even = ceil_div(t_end, at_least(1, slots / rows));
  s.chunk = at_most(at_least(ceil_div(even, step) * step, 4 * vpw), max_chunk / step * step);
  s.n_chunks = ceil_div(t_end, s.chunk);

  const int64_t tiles = ceil_div(t_end, vpw);
  if (2 * rows >= slots && tiles <= (rows >= 2 * slots ? 32 : rows >= slots ? 8 : 4)) {
    s.n_part = s.spare = s.max_span = s.min_log2 = 0;
    s.per_seq = 1;
    return s;
  }
  s.max_span = kSpanWaves * (max_chunk / vpw);
  s.min_log2 = 2;                                                  // a tile per wave
  const int64_t need = ceil_div(tiles, s.max_span);                // columns of a full context
  const int64_t most = at_most(ceil_div(tiles, kSpanWaves), s.n_chunks);
  const int64_t places = at_least(1, slots / kSpanWaves);          // workgroups at once
  const int64_t per_head = places / (heads * n_pass);              // columns of a head in one go
  if (block_tokens == 0) {
    // one go unless it leaves more than a fifth of its places empty; then four, of at least 24
    // tiles each
    int64_t c = at_least(need, at_most(per_head / batch, most));
    const int64_t goes = ceil_div(rows * c, places);
    if (rows * c * 5 < goes * places * 4)
      c = at_least(c, at_most(at_most(ceil_div(4 * places, rows), tiles / 24), most));
    s.per_seq = c;
    s.n_part = batch * c;
    s.spare = 0;
    return s;
  }
  // Contexts that differ: one go while the sequences are at most a quarter of its columns (a span
  // is then at most 4/3 of an even share), else two.  From a sequence per column on, the device
  // evens whole sequences out; half a column more for each splits those of twice the mean and up.
  int64_t n = at_most(per_head, batch * most);
  if (batch < per_head && 4 * batch > per_head) {
    s.min_log2 = 5;
    n = at_least(n, at_most(2 * per_head, batch * at_most(tiles / 32, most)));
  } else if (batch >= per_head && batch <= 2 * per_head && tiles >= 64) {
    s.min_log2 = 5;
    n = at_most(batch + batch / 2, batch * most);
  }
  s.n_part = at_least(batch * need, n);
  s.spare = s.n_part - batch * need;
  if (batch > kMaxSpareBatch || s.spare == 0) {
    s.n_part = batch * need;
    s.spare = 0;
  }
  s.per_seq = need;
  return s;
}

}  // namespace tvq
