// Which (row, split) an attention workgroup owns, and the grid that goes with it.  It follows from the block indices without
// a division: a division by a run-time number is some forty dependent instructions, and two of them stood in front of a wave's
// first load.  One row a grid row, its splits side by side; in the order that keeps the splits of a row on one XCD (workgroup
// number b runs on XCD b % 8) eight rows a grid row.  Counts that do not fit that (`linear`) are divided as before.
// And how many (row, chunk) workgroups go into one launch, and the workgroups of a prune's rows.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pe {

struct PlaceGrid {
  uint32_t x, y;
  bool xcd, linear;
  uint32_t inv_heads;  // row / num_kv_heads is the upper half of row * inv_heads (0: one head)
};

// false: no such grid (no rows, or more workgroups than a launch takes)
inline bool place_grid(int num_seqs, int num_kv_heads, int splits, bool xcd_map, PlaceGrid* g) {
  const int64_t rows = (int64_t)num_seqs * num_kv_heads, total = rows * splits;
  if (total <= 0 || total > 0x7fffffffLL) return false;
  g->xcd = xcd_map && rows % 8 == 0;
  const int64_t grid_rows = g->xcd ? rows / 8 : rows;
  // a grid has at most 65535 rows; the quotient is exact as long as row * num_kv_heads < 2^32
  g->linear = grid_rows > 65535 || rows * num_kv_heads >= (1LL << 32);
  g->x = (uint32_t)(g->linear ? total : g->xcd ? 8 * splits : splits);
  g->y = (uint32_t)(g->linear ? 1 : grid_rows);
  g->inv_heads = num_kv_heads > 1 ? (uint32_t)((1ull << 32) / (uint32_t)num_kv_heads + 1) : 0u;
  return true;
}

// (row, chunk) pairs of several sequences in launches of fewer than 2^32 threads: f(first sequence, sequences, first chunk, chunks) for
// each of them until one gives false.  A launch covers all chunks of its sequences or some chunks of all its sequences.
template <typename F>
inline bool launch_pieces(int num_seqs, int rows_per_seq, int chunks, int threads, F f) {
  const int64_t most = ((1LL << 32) - 1) / threads;
  if (rows_per_seq > most) return false;
  const int64_t seqs = most / rows_per_seq < num_seqs ? most / rows_per_seq : num_seqs;
  for (int64_t s0 = 0; s0 < num_seqs; s0 += seqs) {
    const int64_t ns = num_seqs - s0 < seqs ? num_seqs - s0 : seqs, some = most / (ns * rows_per_seq);
    for (int64_t c0 = 0; c0 < chunks; c0 += some)
      if (!f((int)s0, (int)ns, (int)c0, (int)(chunks - c0 < some ? chunks - c0 : some))) return false;
  }
  return true;
}

// Prefill prune: into how many workgroups (the logarithm) a row goes whose selection and copy are one launch; -1: two launches, one
// workgroup a row that selects, and one for every 1024 tokens of it that copies.  `token_bytes`: K and V of a token and head, read and
// written.  The host knows how many tokens there are and how long the longest row is, not how long the others are.
//
// As many (a power of two) as the compute units have room for with one each, but none with less than one pass of its copy.  Whole prunes,
// half as many / so / twice as many, us: 8 x 4096 tokens of D = 64 23.9 / 23.0 / 24.2, 16 of 2048 to 16384 138.9 / 127.1 / 127.4, 2 of 20000
// to 32768 62.9 / 60.1 / 73.0 (each of them selects: beyond one a compute unit they take turns); one of 1000 with half a pass 10.3, with one
// 10.2, with two 10.9.
//
// One launch saves the second one and the second reading of the scores, some 4 us.  It costs where a long row's share is copied by one
// compute unit (58 GB/s) while the others have nothing to do.  So a share has to be (two launches / one, us, 8 heads of D = 128)
//   - no more than 640 KiB (16 of 2048 to 16384, 1024 kept, 512 KiB 141 / 137; 17 x 4096, 256 kept 64.6 / 64.5, 1024 kept, 1 MiB, 82.5 /
//     86.9; one of 32768 beside 31 of 512, 16384 kept, 16 MiB, 155 / 410);
//   - or no more than a workgroup of the second of two launches copies: 1024 tokens, less what goes of a row of full or of average length
//     (64 x 1000, 1024 kept 157 / 153; 4 x 4096, 4096 kept 42 / 36); or three times what it copies of an average row, where the workgroups
//     of full rows, of which the tokens make total / longest, are four ninths of the compute units or more: two launches then have few
//     workgroups too, of unequal shares (24 x 2 heads of 3927 to 7783, 3776 kept 85.1 / 73.6, 20 x 2 74.5 / 66.3, 12 of 2048 to 6000, 2048
//     kept 99.4 / 89.8, 6 of 4096 to 8192, 4096 kept 92.1 / 82.0, 9 x 4096, 2048 kept 74.9 / 72.0; at three eighths, three of 16384 beside five
//     of 512, 8192 kept, 113 / 127; at four times, 9 x 8192, 4096 kept 129.8 / 133.1);
//   - or the workgroups of full rows have to be five eighths of all and occupy five eighths of the compute units, and all of them be whole
//     rounds of these, but for a tenth (32 x 16384, 8192 kept 805 / 802; 31 x 4 heads of 5265 to 17104, 3520 kept, 160 of 248 workgroups
//     233 / 227; 20 of 16384 beside eleven of 512, 8192 kept, as many, 521 / 564, but 16 of them 426 / 504; 17 x 8192, 136 workgroups, 229 /
//     251; 24 x 8192, 192, 4096 kept 307 / 315; 33 x 4096, 264, 4096 kept 341 / 396; 60 of D = 64 of 370 to 9893, 7808 kept, 176 of 480
//     workgroups 294 / 352).
// (On the slower side of these lines: fp32, 13 of 3400 to 18500, 5248 kept, in two 465 / 448; four of 16384 beside four of 512, 8192 kept, in
// one 130 / 140.)
// Rows of more than 8192 tokens of which less than a sixteenth of the average row is kept have little to copy, and the counting in front
// of it takes the launch's time or more: one of 30335 tokens, 1120 kept 19.6 / 23.1, nine of up to 28254, 320 kept 59.2 / 62.1, 8 x 32768,
// 1024 kept 198 / 199; a tenth: 21 of up to 8274, 1024 kept 62.2 / 57.3.  Longer rows than 32768 are held in LDS too, by one compute unit.
inline int prune_log2_parts(int num_seqs, int num_kv_heads, int64_t total_tokens, int max_seqlen, int budget, int token_bytes,
                            int compute_units) {
  const int64_t rows = (int64_t)num_seqs * num_kv_heads, cus = compute_units, average = total_tokens / num_seqs;
  if (max_seqlen > 32768 || (max_seqlen > 8192 && (int64_t)budget * 16 < average)) return -1;
  const int64_t most = max_seqlen < budget ? max_seqlen : budget;
  int log2_parts = 0;
  while (rows << (log2_parts + 1) <= cus && most >> (log2_parts + 1) >= 65536 / token_bytes) ++log2_parts;
  const int64_t share = (most + (1 << log2_parts) - 1) >> log2_parts;
  if (share * token_bytes <= 640 << 10) return log2_parts;
  const int64_t of_full = 1024 * most / max_seqlen, of_average = average > budget ? 1024 * (int64_t)budget / average : average;
  const int64_t chunk = of_average < 1024 ? of_average : 1024;
  const int64_t groups = rows << log2_parts, full = (total_tokens / max_seqlen * num_kv_heads) << log2_parts;
  if (share <= of_full || share <= (full * 9 >= cus * 4 ? 3 * chunk : chunk)) return log2_parts;
  return full * 8 >= cus * 5 && full * 8 >= groups * 5 && groups * 10 >= (groups + cus - 1) / cus * cus * 9 ? log2_parts : -1;
}

// Block scores: which part of its row workgroup b has, of `parts` a row.  Workgroup b runs on XCD b % 8, there on one shader engine after the
// other, and the last parts of all rows have nothing to do where the tables hold more pages than are in use: with an even number of
// parts, side by side, some of the chip had all the work (972 rows of four pages of 128 tokens, eight heads of D = 128, in tables of six,
// two parts, 452 us, now 311).  So the parts begin somewhere else in each row, by a multiplicative hash of its number, `turn` (in two steps: fp32,
// 96 x 8 rows of 209 pages of 32 tokens in tables of 315, 20 parts 900 us side by side, 994 in one step, 874 in two).  An odd number
// spreads by itself, and better where few rows are scored (26 rows of 36 pages of 128 tokens in tables of 74, 19 parts 12.6 us, hashed 17.5).
// Head-shared, the heads of a sequence begin at the same one: their tokens lie side by side (13 sequences x 8 layers x 8 heads, fp32 719 us,
// each by itself 798).
__host__ __device__ inline uint32_t score_part(uint32_t b, uint32_t row, uint32_t parts, uint32_t turn) {
  uint32_t at = b - row * parts;
  if (parts % 2u == 0u) {
    uint32_t hash = turn * 0x9e3779b1u;  // 2^32 / the golden ratio
    hash = (hash ^ hash >> 16) * 0x9e3779b1u;
    at += (uint32_t)((uint64_t)hash * parts >> 32);
  }
  return at < parts ? at : at - parts;
}

struct Place {
  int row, split, seq, head;
};

__host__ __device__ inline Place place_at(uint32_t x, uint32_t y, bool xcd, bool linear, int splits, int num_kv_heads,
                                          uint32_t inv_heads) {
  Place p;
  if (__builtin_expect(linear, 0)) {
    const uint32_t n = (uint32_t)splits, k = xcd ? x >> 3 : x;
    p.row = (int)(xcd ? (k / n) * 8 + (x & 7u) : k / n);
    p.split = (int)(k % n);
    p.seq = p.row / num_kv_heads;
  } else {
    p.split = (int)(xcd ? x >> 3 : x);
    p.row = (int)(xcd ? y * 8 + (x & 7u) : y);
    p.seq = inv_heads != 0u ? (int)((uint64_t)(uint32_t)p.row * inv_heads >> 32) : p.row;
  }
  p.head = p.row - p.seq * num_kv_heads;
  return p;
}

}  // namespace pe
