// Which kernel takes the chunk rows of a varlen call, and in which form, from
// what the host knows of the call (plain C++, so that it also runs on the host
// alone).
#pragma once

#include <stdint.h>

namespace pa {

// Query rows of a prefill item with `blocks` 16-row blocks in each of its 8 waves.
constexpr int kPfWaves = 8;
constexpr int kPfBlocksMax = 2;
constexpr int pf_rows(int blocks) { return 16 * blocks * kPfWaves; }

// 16-row blocks per wave of the prefill kernel (2, or 1: twice the items of half
// the rows) for a call of `rows` query rows in `seqs` sequences on `cus` CUs.
//
// With no more items of 128 rows than CUs, all run at once and the longest
// item's chain of steps is the call's time: a step with one block per wave has
// half the products and half the softmax's vector work, at the same staging.
// 32 query heads over 8: one chunk of 700 rows 31.1 us with 256-row items and
// 22.5 with 128, 1,000 rows 38.5 and 28.8, 8 of 60-100 rows on 0-1,000 tokens
// 39.8 and 29.3; one KV head of 8 query heads, 2,048 rows on 1,000 tokens 97.6
// and 70.4.  Past the line items wait for a second round, or share a CU: one
// chunk of 1,030 rows 40.5 and 47.5, 1,500 rows 52.7 and 73.3, 2,000 rows on
// 2,000 tokens 127 and 146, 20 of 60-90 rows on 0-2,000 tokens 69.7 and 87.0.
// The host knows no lengths: `seqs` chunks of `rows` positions in all have at
// most this many blocks.
constexpr int prefill_blocks(int s, int H_kv, int rows, int seqs, int cus) {
  const int pb = pf_rows(1) / s;  // positions per item
  return ((int64_t)rows + (int64_t)(pb - 1) * seqs) / pb * H_kv <= cus ? 1 : kPfBlocksMax;
}

// A call's chunks as the host can know them: the sequences that are not decode
// rows, taken as the fewest and longest that `rows`, `seqs` and `max_q` allow,
// each on the longest context.
struct ChunkCall {
  int s, H_kv, rows, seqs, max_q, max_ctx;
  constexpr int64_t excess() const { return rows > seqs ? rows - seqs : 1; }
  constexpr int64_t chunks() const { return (excess() + max_q - 2) / (max_q - 1); }  // (max_q > 1)
  constexpr int64_t chunk_rows() const { return excess() + chunks() < rows ? excess() + chunks() : rows; }
};

// Microseconds of the two kernels that can take bf16 head_dim 64 chunks,
// fitted to 503 measured calls (H_kv 1 to 8, s 1 to 8, 1 to 64 chunks of 2 to
// 300 rows on 0 to 30,000 tokens).
//
// Split-K: workgroups of one row, one KV head and up to 2,048 keys, 4.1 s us each
// where few run, then as many rounds as they need, or the rate of its VALU fold
// and (few query heads per KV head, long contexts) of K/V out of the last-level
// cache.  Its workgroups go to the 8 XCDs in turn, so an even number of splits
// puts the short last ones on the same XCDs, and a call takes as long as if they
// were full.
constexpr double split_us(const ChunkCall& c, int cus) {
  const int64_t splits = ((int64_t)c.max_ctx + 2047) / 2048;
  const double keys = splits % 2 == 0 ? splits * 2048.0 : c.max_ctx < 256 ? 256.0 : c.max_ctx;
  const double groups = (double)c.chunk_rows() * c.H_kv;
  const int64_t rounds = (c.chunk_rows() * c.H_kv * splits + cus - 1) / cus;
  const double one = 0.002 * c.s * (keys < 2048 ? keys : 2048.0);
  const double waves = one * (rounds > 1 ? 0.85 * rounds : 1.0);
  const double fold = groups * keys * 1e-6 * (4 * c.s + 3 + 0.27 * (c.H_kv * 256e-6 * c.max_ctx));
  return 9.5 + (waves > fold ? waves : fold);
}
// Prefill: the chain of an item's steps of 64 keys, two per trip of its loop.
constexpr double prefill64_us(const ChunkCall& c, int cus) {
  const double steps = 2.0 * (((int64_t)c.max_ctx + 127) / 128);
  const int blocks = prefill_blocks(c.s, c.H_kv, c.rows, c.seqs, cus);
  if (blocks == 1) return 5.2 + 1.15 * steps;
  const int64_t pb = pf_rows(blocks) / c.s, each = (c.chunk_rows() + c.chunks() - 1) / c.chunks();
  const double per_cu = (double)c.H_kv * c.chunks() * ((each + pb - 1) / pb) / cus;
  return (5.2 + 2.05 * steps) * (per_cu > 1 ? per_cu : 1.0);
}

// Whether bf16 head_dim 64 chunks take the split-K kernel.  Few rows on a long
// context leave the prefill kernel with one chain per KV head on a few CUs: 2
// rows on 30,000 tokens, 8 KV heads of 4 query heads, 33 us on the split-K kernel
// and 541 on the prefill kernel, 48 rows on 4,000 tokens 51 and 79, 8 rows on
// 1,000 tokens 18 and 24; 100 rows on 4,000 tokens 99 and 81, on 30,000 776 and
// 541.  The estimates are within about 10 % near the line, so the split-K kernel,
// which took these calls before, keeps that much on its side.
constexpr bool chunks64_to_split(const ChunkCall& c, int cus) {
  return c.max_q > 1 && split_us(c, cus) < 1.1 * prefill64_us(c, cus);
}

}  // namespace pa
