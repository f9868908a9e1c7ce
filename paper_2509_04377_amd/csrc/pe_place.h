// Which (row, split) an attention workgroup owns, and the grid that goes with it.  It follows from the block indices without
// a division: a division by a run-time number is some forty dependent instructions, and two of them stood in front of a wave's
// first load.  One row a grid row, its splits side by side; in the order that keeps the splits of a row on one XCD (workgroup
// number b runs on XCD b % 8) eight rows a grid row.  Counts that do not fit that (`linear`) are divided as before.
// And how many (row, chunk) workgroups go into one launch.
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
