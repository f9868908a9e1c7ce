// Host-side launch interfaces between the C-ABI layer (pe_api.hip) and the kernel translation units.
// Arguments are already validated by the caller: shapes are supported, pointers are non-null.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace pe {

struct ScoreArgs {
  const void* k_pool;
  const void* v_pool;
  const int32_t* block_table;
  const int32_t* seq_lens;
  float* scores;
  int num_seqs, num_kv_heads, head_dim, block_size, max_blocks;
  bool is_bf16;
  int recent = 0;  // 0: score every page; n > 0: only the n most recently filled pages of each row
  bool shared = false;  // one table row per sequence, pages [B][Hk][D]
  int budget = 0;       // > 0: score only the sequences that trigger an eviction at this budget
};
hipError_t launch_score_blocks(const ScoreArgs& a, hipStream_t stream);

struct ScoreEvictArgs {
  const void* k_pool;
  const void* v_pool;
  int32_t* block_table;
  int32_t* seq_lens;
  float* scores_out;  // may be null
  int32_t* evicted_logical;
  int32_t* freed_phys;
  int num_seqs, num_kv_heads, head_dim, block_size, max_blocks, budget;
  bool is_bf16;
};
hipError_t launch_score_evict(const ScoreEvictArgs& a, hipStream_t stream);

struct EvictArgs {
  const float* scores;
  float* scores_mut = nullptr;  // when set (== scores): delete the evicted entry from the score row as well
  int32_t* block_table;
  int32_t* seq_lens;
  int32_t* evicted_logical;
  int32_t* freed_phys;
  int num_seqs, num_kv_heads, block_size, max_blocks, budget;
  int policy = 0, protect_first = 0, protect_last = 0, share_heads = 0;
  bool shared = false;  // one table row per sequence (implies share_heads); outputs are [S]
};
hipError_t launch_evict_blocks(const EvictArgs& a, hipStream_t stream);

struct AppendArgs {
  const void* new_k;
  const void* new_v;
  void* k_pool;
  void* v_pool;
  int32_t* block_table;
  int32_t* seq_lens;
  int32_t* freed_phys;
  const int32_t* spare;
  int32_t* spare_used;
  int n_spare, num_seqs, num_kv_heads, head_dim, block_size, max_blocks;
  bool is_bf16;
  bool shared = false;  // one table row, one spare list and one freed page per sequence
  int32_t* seq_lens_out = nullptr;  // when set, the new lengths go here and seq_lens is only read
};
hipError_t launch_append_kv(const AppendArgs& a, hipStream_t stream);

struct DecodeArgs {
  const void* q;
  const void* k_pool;
  const void* v_pool;
  const int32_t* block_table;
  const int32_t* seq_lens;
  void* out;
  float* partials;  // workspace: [rows][splits][G][D + 2] fp32 (unused when splits == 1)
  float scale;
  int num_seqs, num_kv_heads, num_q_heads, head_dim, block_size, max_blocks;
  int splits;
  int xcd_map;
  int waves, depth;  // bfloat16 kernel: workgroup size in waves, tiles in flight per wave: 4 x 2, 4 x 1; D = 128,
                     // per-head layout: 8 x 2, and with up to four query heads per KV head 4 x 3 too; D = 128 with more, 8 x 1.  Vector units: 4 or 8 waves
  bool is_bf16;
  bool vector = false;  // bfloat16 on the vector units: one query head per KV head, no append in the head-shared layout
  // fused append: all null / 0 for plain attention
  const void* new_k = nullptr;
  const void* new_v = nullptr;
  int32_t* freed_phys = nullptr;
  const int32_t* spare = nullptr;
  int32_t* spare_used = nullptr;
  int32_t* seq_lens_out = nullptr;
  int n_spare = 0;
  bool shared = false;  // one table row per sequence, pages [B][Hk][D]; with fp32 plain attention only
  // Splits merged by the last of a row to arrive, without a merge launch:
  bool counted = false;      // the arrival counts in `out` are clear
  bool tagged = false;       // `out` may hold anything but `tag`, which is this launch's own
  uint64_t tag = 0;
  void* next_out = nullptr;  // output of the launch behind this one, whose counts this one is to clear
};
hipError_t launch_paged_decode(const DecodeArgs& a, hipStream_t stream);
hipError_t launch_paged_decode_bf16(const DecodeArgs& a, hipStream_t stream);  // the attention kernel alone (no merge)
size_t decode_partials_bytes(int num_seqs, int num_q_heads, int head_dim, int splits);
// The most splits of a row that are counted or tagged, and with so many query heads a KV head; up to here they are added in one order on
// every way.
constexpr int kMostArrivals = 12;
constexpr int most_arrivals(int group) { return group > 4 ? 8 : kMostArrivals; }

struct PruneArgs {
  const void* k_in;
  const void* v_in;
  const int32_t* cu_seqlens;
  void* k_pool;
  void* v_pool;
  const int32_t* block_table;
  int32_t* seq_lens_out;
  int32_t* kept_idx_out;  // may be null
  void* workspace;
  int64_t total_tokens;
  int max_seqlen, budget;
  int num_seqs, num_kv_heads, head_dim, block_size, max_blocks;
  bool is_bf16;
  bool shared = false;  // one decision per sequence (head-mean token scores), pages [B][Hk][D]
  int compute_units = 256;
};
hipError_t launch_prefill_prune(const PruneArgs& a, hipStream_t stream);
size_t prune_workspace_bytes(int num_seqs, int num_kv_heads, int64_t total_tokens, bool shared);

}  // namespace pe
