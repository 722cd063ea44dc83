/* The split of an attention call (csrc/tvq_spans.h), compiled for the host: attn_split and the
 * column counts of a batch, for the checks in test_attention_spans.py. */
#include "../../paper_2603_27467_amd/csrc/tvq_spans.h"

extern "C" void split(int64_t batch, int64_t heads, int64_t n_pass, int64_t t_end,
                      int64_t block_tokens, int64_t vpw, int64_t slots, int64_t* out) {
  const tvq::AttnSplit s =
      tvq::attn_split(batch, heads, n_pass, t_end, block_tokens, vpw, slots);
  const int64_t v[7] = {s.chunk, s.n_chunks, s.n_part, s.per_seq, s.spare, s.max_span, s.min_log2};
  for (int i = 0; i < 7; ++i) out[i] = v[i];
}

extern "C" void counts(const uint32_t* tiles, int64_t batch, uint32_t spare, uint32_t max_span,
                       uint32_t min_log2, uint32_t* out) {
  uint32_t total = 0;
  for (int64_t b = 0; b < batch; ++b) total += tiles[b];
  if (total == 0) total = 1;
  for (int64_t b = 0; b < batch; ++b)
    out[b] = spare == 0 ? tvq::span_floor(tiles[b], max_span)
                        : tvq::span_count(tiles[b], total, spare, max_span, min_log2);
}

extern "C" void unit(uint32_t u, uint32_t heads, uint32_t n_part, int columns_first,
                     uint32_t* column_and_head) {
  const tvq::UnitOf of = tvq::unit_of(u, heads, n_part, columns_first != 0);
  column_and_head[0] = of.column;
  column_and_head[1] = of.head;
}
