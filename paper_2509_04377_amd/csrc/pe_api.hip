// C-ABI layer of libpe (see include/pe.h): argument validation on the host, then kernel launches on
// the caller's stream.  Nothing here allocates, frees or synchronises.
#include "../../include/pe.h"

#include <atomic>
#include <chrono>
#include <mutex>

#include "pe_launch.h"

// Split partials of pe_paged_decode_static: one copy per GPU, held until the process ends.  In host code this
// name is only a handle for hipGetSymbolAddress; kernels are given the address that call returns.
static __device__ __align__(256) unsigned char scratch[PE_STATIC_SCRATCH_BYTES];

namespace {

bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

// The decode workgroup shapes that a descriptor may name.
bool decode_shape_built(int shape) { return shape == 422 || shape == 424 || shape == 432 || shape == 822; }

// PE_OK if the descriptor names a shape the kernels are built for.
int check_desc(const pe_cache_desc* d) {
  if (d == nullptr) return PE_ERR_INVALID_ARG;
  if (d->dtype != PE_F32 && d->dtype != PE_BF16) return PE_ERR_UNSUPPORTED;
  if (d->num_seqs < 1 || d->num_kv_heads < 1 || d->num_q_heads < 1 || d->max_blocks < 1 || d->num_phys_blocks < 1)
    return PE_ERR_INVALID_ARG;
  if (d->num_q_heads % d->num_kv_heads != 0) return PE_ERR_INVALID_ARG;
  if (d->num_q_heads / d->num_kv_heads > 8) return PE_ERR_UNSUPPORTED;
  if (d->head_dim != 64 && d->head_dim != 128) return PE_ERR_UNSUPPORTED;
  if (d->block_size != 16 && d->block_size != 32 && d->block_size != 64 && d->block_size != 128)
    return PE_ERR_UNSUPPORTED;
  if (d->layout != PE_LAYOUT_PER_HEAD && d->layout != PE_LAYOUT_SHARED) return PE_ERR_UNSUPPORTED;
  if (d->num_phys_blocks > 0x7fffffffLL) return PE_ERR_UNSUPPORTED;
  if ((int64_t)d->num_seqs * d->num_kv_heads > 0x7fffffffLL / 64) return PE_ERR_UNSUPPORTED;
  if (d->decode_splits < 0 || d->decode_splits > 256) return PE_ERR_INVALID_ARG;
  if (d->decode_flat_order != 0 && d->decode_flat_order != 1) return PE_ERR_INVALID_ARG;
  if (d->decode_shape != 0) {
    if (!decode_shape_built(d->decode_shape)) return PE_ERR_UNSUPPORTED;
    const bool tunable = d->dtype == PE_BF16 && d->head_dim == 128 && d->num_q_heads / d->num_kv_heads == 4 &&
                         d->layout == PE_LAYOUT_PER_HEAD;
    if (d->decode_shape != 422 && !tunable) return PE_ERR_UNSUPPORTED;
  }
  return PE_OK;
}

// Compute units of the current device, asked of the HIP runtime once per device.  Without a device (or on an
// error) the count of an MI355X is assumed; the sticky error state of the runtime is left clean.
int compute_units() {
  constexpr int kMaxDevices = 64, kDefault = 256;
  static std::atomic<int> cached[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    (void)hipGetLastError();
    return kDefault;
  }
  int n = cached[dev].load(std::memory_order_relaxed);
  if (n > 0) return n;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) {
    (void)hipGetLastError();
    return kDefault;
  }
  cached[dev].store(n, std::memory_order_relaxed);
  return n;
}

// Bytes of K and V of a row as long as its table row.
int64_t row_bytes(const pe_cache_desc* d) {
  return (int64_t)d->max_blocks * d->block_size * d->head_dim * (d->dtype == PE_BF16 ? 4 : 8);
}

// The most splits that a table row's length gives reason for.  Rows under 512 tokens are whole, up to sixteen splits are of
// 128 tokens or more (8 fp32 rows x 1024 in four 12.3 us, in eight 9.4), more than sixteen of 256 or more: the merge walks over
// the splits one by one, and a table that holds little pays for all (8 fp32 rows in a table of 4096: in sixteen 14.6 us full and
// 7.3 with 64 tokens a row, in 32 13.8 and 9.4; of 2048: in eight 13.0 and 6.3, in sixteen 10.7 and 7.2).
int64_t splits_by_length(const pe_cache_desc* d) {
  const int64_t tokens = (int64_t)d->max_blocks * d->block_size;
  if (tokens < 512) return 1;
  const int64_t fine = tokens / 128, coarse = tokens / 256;
  return fine <= 16 ? fine : coarse > 16 ? coarse : 16;
}

// Number of splits of a row, fp32.  The kernel computes about as long as it loads (the more so the more query heads share a
// KV head), several of its workgroups fit a compute unit, and one without tokens is through early; so the rule asks for an
// even deal, also of rows of unequal length.  Measured on an MI355X with full tables / ragged ones (37 tokens to all), D = 128,
// 4 query heads a KV head (8 in brackets), us:
//   - somewhat more rows than compute units, of 2048 tokens or more, in four (264 rows x 2048 94 / 72, whole 109 / 95; rows of 64
//     tokens in that table 10.3 and 7.0), shorter ones whole (320 rows x 1024 56.7 (63.0) in four, 60.9 (60.1) whole);
//   - from half to three quarters of the compute units, four: 136 rows x 4096 104 / 56 (110 / 60), in two 113 / 69 (110 / 85),
//     whole 122 / 114 (156 / 152); beyond that, two: 224 rows x 4096 146 / 94 (150 / 98), in four 152 / 83 (160 / 88), whole
//     142 / 119 (162 / 153);
//   - from a quarter to half, four or six, two workgroups a compute unit: 88 rows x 2048 35 / 25 (37 / 29), in three 41 / 30
//     (41 / 35), in two 37 / 35 (48 / 47);
//   - up to an eighth of them, two a compute unit too where pieces of 1 MiB remain (64 rows x 8192 84 / 55 (86 / 59), in four 82 /
//     67 (92 / 84); rows of 64 tokens in that table 7.6 and 6.6);
//   - else as many as leave no compute unit two workgroups: 40 rows x 2048 in six 18.6 / 17.0, in seven 22.0 / 18.4; with more
//     than four query heads as many as leave none without: 48 rows x 4096 in six (42.6 / 37.4), in five (42.3 / 40.0).
int decode_splits_f32(const pe_cache_desc* d, int64_t rows, int64_t cus) {
  if (rows >= cus) return rows > cus && rows * 10 <= cus * 13 && (int64_t)d->max_blocks * d->block_size >= 2048 ? 4 : 1;
  const int64_t fit = cus / rows;
  int64_t splits;
  if (fit == 1)
    splits = rows * 4 <= cus * 3 ? 4 : 2;
  else if (fit < 4 || (fit <= 8 && row_bytes(d) / (2 * fit) >= (1 << 20)))
    splits = 2 * fit;
  else
    splits = d->num_q_heads / d->num_kv_heads > 4 ? (cus + rows - 1) / rows : fit;
  const int64_t by_len = splits_by_length(d);
  if (splits > by_len) splits = by_len;
  return splits > 64 ? 64 : (int)splits;
}

// Number of splits of a row in the attention calls, chosen from the shape.  The host sees the length of a table row, not of
// the sequences, so a count has to pay on full rows and on rows of unequal length, and cost little where rows are short.
// bfloat16, measured on an MI355X with full tables / ragged ones (37 tokens to all) / 64 tokens in every row, D = 128, 4 query
// heads a KV head, us:
//   - somewhat more rows than compute units, of 2048 tokens or more, in four (264 rows x 2048 49.9 / 30.3 / 10.3, whole 57.7 /
//     39.2 / 5.6; 320 rows 55.7 / 34.7 / 11.1, whole 60.9 / 40.9 / 5.8; 384 rows 66.5 / 40.9 / 12.2, whole 64.2 / 44.4 / 5.9):
//     rows shorter than some 300 tokens in such a table pay for it, up to 4.5 us; shorter tables and more rows are whole;
//   - from half of the compute units on: whole where a full row takes little longer than the launch that merges splits (136 rows
//     x 2048 26 / 23 / 5; 192 x 2048 32 / 25 / 5), else in five, four or three, about three workgroups a compute unit (136 rows x
//     8192 in five 90 / 54 / 7, in two 117 / 58 / 8, whole 94 / 81 / 5; 192 in four 126 / 74 / 8, in two 128 / 88 / 9, whole 119 /
//     89 / 5; 224 in four 148 / 82 / 9, in three 146 / 93 / 8; 248 in three 160 / 99 / 8, in four 161 / 97 / 9; D = 64, 136 x 4096
//     in five 27 / 19 / 7, in two 34 / 23 / 7, whole 30 / 28 / 5);
//   - from a quarter to half of them: whole up to 1024 tokens from 7/16 on (128 rows x 1024 14.5, in two 15.0); two workgroups a
//     compute unit for rows of 4 MiB and more (96 rows x 16384 in two 121 / 98 / 7, in five 126 / 79 / 7; 128 rows in two 165 /
//     110 / 7, in four 165 / 99 / 7); else one;
//   - below, as many as leave no compute unit two workgroups (64 rows x 16384 in four 84 / 56 / 7, in eight 85 / 51 / 10).
int decode_splits(const pe_cache_desc* d) {
  if (d->decode_splits > 0) return d->decode_splits;
  const int64_t rows = (int64_t)d->num_seqs * d->num_kv_heads;
  const int64_t cus = compute_units();
  if (d->dtype == PE_F32) return decode_splits_f32(d, rows, cus);
  const int64_t tokens = (int64_t)d->max_blocks * d->block_size;
  if (rows >= cus) return rows > cus && rows * 10 <= cus * 13 && tokens >= 2048 ? 4 : 1;
  const int64_t fit = cus / rows;
  int64_t splits = fit;
  if (fit == 1) {
    if (tokens > 16 * d->head_dim) splits = rows * 5 <= cus * 3 ? 5 : rows * 8 <= cus * 7 ? 4 : 3;
  } else if (fit <= 3) {
    if (rows * 16 >= cus * 7 && tokens <= 1024) splits = 1;
    else if (row_bytes(d) >= (4 << 20)) splits = 2 * cus / rows;
  }
  const int64_t by_len = splits_by_length(d);
  if (splits > by_len) splits = by_len;
  return splits > 64 ? 64 : (int)splits;
}

// The count that a caller's buffer of `have` bytes allows: the library's own choice may fall back to one workgroup per
// compute unit in splits of 256 tokens and more, a count that the descriptor names may not.
int decode_splits_within(const pe_cache_desc* d, size_t have) {
  int splits = decode_splits(d);
  if (d->decode_splits > 0) return splits;
  const int64_t rows = (int64_t)d->num_seqs * d->num_kv_heads;
  const int64_t by_rows = (compute_units() + rows - 1) / rows;
  const int64_t by_len = (int64_t)d->max_blocks * d->block_size / 256;
  int64_t least = by_rows < by_len ? by_rows : by_len;
  if (least > 64) least = 64;
  while (splits > least && pe::decode_partials_bytes(d->num_seqs, d->num_q_heads, d->head_dim, splits) > have) --splits;
  return splits;
}

int check_workspace(const void* ws, size_t have, size_t need) {
  if (need == 0) return PE_OK;
  if (ws == nullptr || have < need || !aligned(ws, 256)) return PE_ERR_WORKSPACE;
  return PE_OK;
}

bool finite(float x) { return x == x && x - x == 0.f; }

// The part of the attention launch description that follows from the descriptor alone.
pe::DecodeArgs decode_args(const pe_cache_desc* desc, int splits) {
  pe::DecodeArgs a;
  a.num_seqs = desc->num_seqs;
  a.num_kv_heads = desc->num_kv_heads;
  a.num_q_heads = desc->num_q_heads;
  a.head_dim = desc->head_dim;
  a.block_size = desc->block_size;
  a.max_blocks = desc->max_blocks;
  a.splits = splits;
  a.xcd_map = desc->decode_flat_order ? 0 : 1;
  // bfloat16 kernel, workgroup (waves x tiles in flight per wave), measured on an MI355X:
  //   - four x one where more workgroups than compute units come, or where rows of D = 128 are split for (nearly) all of them:
  //     with half the registers several share a compute unit, and one that has no tokens holds up none (192 rows in 768 splits,
  //     full 8192 tokens / 64 tokens: 126 / 8.3 us, four x two 126 / 9.7, eight x two 126 / 12.7; with eight query heads 127 /
  //     9.9, 128 / 13.2, 130 / 16.7; 384 whole rows x 2048 64.6 / 5.9, 64.2 / 6.7, 65.2 / 8.1; D = 64 33.0 / 5.0, 34.9 / 5.8);
  //   - and where a wave has no second tile: tables of up to 64 tokens a split;
  //   - eight x two for whole rows of 1 MiB or more of D = 128, one for every compute unit (append and attention of 256 rows x 2048
  //     out of a pool of 8.6 GB 43.9, four x two and four x one 44.2; no faster with fewer rows); in the head-shared layout,
  //     whose wave-loads are runs of 256 bytes, four x one there too (45.6; with two tiles 47.2, with eight waves 47.1);
  //   - eight x one for more than four query heads a KV head where rows of D = 128 are split for three quarters of the compute units or
  //     more, in pieces of 192 tokens or more.  Up to eight splits can be counted then, as each wave has one part of the row at the end
  //     (append and attention of all layers, four x one and a merge launch / so, full | ragged | 64 tokens a row: six query heads, 80 rows x
  //     800 in three 12.1 / 10.5 | 10.6 / 9.0 | 7.1 / 6.3, eight, 64 x 1024 in four 11.5 / 10.5, 64 x 4096 in four 26.4 / 25.8 | 19.9 / 19.8 |
  //     7.2 / 6.6; fewer workgroups, 16 x 2048 in eight, four x two 9.1, so 9.5).  With a merge launch behind either form, which is what
  //     single calls in eight splits have and every one in more, eight x one is no slower: 32 rows x 2048 in eight 11.4 / 11.2, x 8192 26.6 /
  //     26.6; 28 x 2048 in nine 12.1 / 11.8, 20 x 4096 in twelve 14.2 / 13.6 | 12.5 / 12.1 | 8.2 / 8.0.  With up to four query heads, whose
  //     splits are counted with four waves, it is the same within 2 %.
  //     (Slower are some shapes whose last round is half empty with eight waves, 48 x 2048 in five 14.0 / 14.5, 40 x 4096 in six 19.1 / 19.5;
  //     others are not, 36 x 2048 in seven 13.0 / 12.7 | 13.4 / 12.7 from the second layer on: no line drawn for them.)
  //   - four x two else (136 whole rows x 2048 26.8, four x one 28.2; D = 64, 128 rows in 256 splits of 8192 82.7 and 98.2).
  const int64_t groups = (int64_t)desc->num_seqs * desc->num_kv_heads * splits;
  const int64_t cus = compute_units();
  const bool shared = desc->layout == PE_LAYOUT_SHARED;
  const bool d128 = desc->head_dim == 128;
  const bool large = d128 && splits == 1 && groups == cus && row_bytes(desc) >= (1 << 20);
  const int64_t piece = (int64_t)desc->max_blocks * desc->block_size / splits;
  const bool most = d128 && splits > 1 && groups * 4 >= cus * 3;
  const bool one_tile = (int64_t)desc->max_blocks * desc->block_size <= (int64_t)64 * splits;
  const bool eight = most && groups <= cus && desc->num_q_heads / desc->num_kv_heads > 4 && piece >= 192;
  a.waves = eight || (large && !shared) ? 8 : 4;
  a.depth = groups > cus || one_tile || most || (large && shared) ? 1 : 2;
  if (desc->decode_shape == 424) a.waves = 4, a.depth = 2;
  if (desc->decode_shape == 432) a.waves = 4, a.depth = 3;
  if (desc->decode_shape == 822) a.waves = 8, a.depth = 2;
  a.is_bf16 = desc->dtype == PE_BF16;
  a.shared = shared;
  // The vector units for bfloat16 rows that are short, of one query head per KV head (vector / matrix kernel, us a launch: D = 64,
  // 32 rows x 64 / 256 / 448 / 1024 tokens 3.7 / 4.9 / 6.2 / 6.6 and 4.1 / 5.4 / 7.0 / 7.0, 256 rows 4.1 / 5.9 / 7.8 / 12.9 and 4.8
  // / 6.1 / 8.2 / 12.9; D = 128, 128 rows x 64 / 128 / 192 / 256 3.9 / 4.8 / 5.6 / 6.5 and 4.7 / 5.2 / 6.1 / 6.4; with more rows than
  // compute units the limits lie lower: 384 rows of D = 64 x 128 / 192 / 448 5.5 / 6.6 / 10.3 and 5.6 / 6.6 / 9.9, of D = 128 x 64
  // / 128 5.2 / 7.2 and 5.8 / 7.1; in the head-shared layout the matrix kernel is ahead from 64 tokens on, 256 rows of D = 64 4.9
  // and 4.2).
  const int64_t tokens = (int64_t)desc->max_blocks * desc->block_size;
  const bool few = (int64_t)desc->num_seqs * desc->num_kv_heads <= cus;
  a.vector = a.is_bf16 && !shared && desc->num_q_heads == desc->num_kv_heads &&
             tokens <= (few ? (d128 ? 192 : 1024) : (d128 ? 64 : 128));
  // On the vector units: eight waves where no compute unit gets two workgroups, but for four query heads a KV head or fewer in pieces of 1
  // MiB and more, which stream as well with four.  Four waves / eight, us: fp32, D = 128, four rows x 256 tokens, one query head a KV head
  // 6.0 / 4.5, eight 13.4 / 9.8; 52 rows x 256 9.3 / 7.4 with four; D = 64, two query heads, four rows 4.3 / 3.7; 64 rows x 1024 in four
  // splits, four heads 13.1 / 12.5 (D = 64 8.7 / 8.0), 32 x 4096 in eight 22.6 / 22.4, with eight heads 26.9 / 24.1; 256 whole rows x 300 13.0
  // / 12.4; x 2048 77.4 / 78.8, with eight heads 86.4 / 80.7; 384 rows x 1024 62.6 / 64.9, with eight heads 63.7 / 68.3; 128 rows x 1024 of D =
  // 64 in four, eight heads, 13.5 / 14.0.  bfloat16: 64 rows x 190 of D = 64 3.5 / 3.3, 384 x 60 3.4 / 3.7.
  // Four too where a whole row has ten tiles of 4 KiB or fewer, twelve with up to four query heads: eight waves then have little or nothing
  // each (64 | 256 rows, fp32, D = 64, four heads x 30 tokens 3.7 / 3.9 | 4.6 / 4.8, x 63 4.7 / 4.7 | 5.2 / 5.5, x 111 5.4 / 5.0 | 6.2 / 5.9; D = 128,
  // one x 30 4.1 / 4.2 | 4.7 / 5.1, x 47 4.6 / 4.3 | 5.5 / 5.3; eight heads of D = 64 x 63 5.7 / 5.6 | 6.0 / 6.0, x 79 6.5 / 5.8 | 6.9 / 6.3; bfloat16,
  // D = 128 x 63 4.3 / 4.4 | 4.9 / 5.2, x 111 4.9 / 4.6 | 5.8 / 5.6).
  if (!a.is_bf16 || a.vector) {
    const bool wide = desc->num_q_heads / desc->num_kv_heads > 4;
    const bool short_row = splits == 1 && row_bytes(desc) <= (wide ? 40 : 48) << 10;
    a.waves = groups <= cus && (wide || row_bytes(desc) / splits < (1 << 20)) && !short_row ? 8 : 4;
  }
  return a;
}

// Whether the splits of a row are merged by the last of them to arrive, counted or tagged (pe_decode_common.h says where that pays).
bool splits_counted(const pe_cache_desc* d, const pe::DecodeArgs& a) {
  const int64_t groups = (int64_t)d->num_seqs * d->num_kv_heads * a.splits;
  const int heads = d->num_q_heads / d->num_kv_heads;
  const bool built = !a.is_bf16 || a.vector ? !a.shared : a.depth == 1 || (a.waves == 4 && a.depth == 2);
  return built && a.splits > 1 && a.splits <= pe::most_arrivals(heads) && heads * d->head_dim <= 128 * a.waves &&
         groups <= (a.splits > 8 ? 1 : 2) * (int64_t)compute_units();
}
bool splits_tagged(const pe_cache_desc* d, const pe::DecodeArgs& a) {
  return splits_counted(d, a) && (a.splits < 8 || (a.splits == 8 && a.waves == 4 && row_bytes(d) / 8 < (256 << 10)));
}

bool overlap(const void* a, size_t a_bytes, const void* b, size_t b_bytes) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return x < y + b_bytes && y < x + a_bytes;
}

// A launch's own tag: a counter from the time of the first call on, mixed as in SplitMix64 (Steele, Lea and Flood, 2014: its increment, shifts and
// multipliers).  No two of a process are the same (the mixing is one to one), and what lies in memory is none by chance.
uint64_t launch_tag() {
  static std::atomic<uint64_t> calls{(uint64_t)std::chrono::system_clock::now().time_since_epoch().count()};
  uint64_t x = calls.fetch_add(1, std::memory_order_relaxed) * 0x9e3779b97f4a7c15ull;
  x = (x ^ x >> 30) * 0xbf58476d1ce4e5b9ull;
  x = (x ^ x >> 27) * 0x94d049bb133111ebull;
  return x ^ x >> 31;
}

// For a call of the attention alone: tags its launch where that pays and the output can hold tags before it is written, that is, nothing
// that is read lies there.
void tag_attention(const pe_cache_desc* d, pe::DecodeArgs* a) {
  const size_t bytes = (size_t)d->num_seqs * d->num_q_heads * d->head_dim * (a->is_bf16 ? 2 : 4);
  if (!splits_tagged(d, *a) || !aligned(a->out, 8) || overlap(a->out, bytes, a->q, bytes)) return;
  a->tagged = true;
  a->tag = launch_tag();
}

}  // namespace

extern "C" {

int pe_version(void) { return 300; }  // 0.3.0: per-descriptor launch shape replaces the process-wide options

const char* pe_status_string(int status) {
  switch (status) {
    case PE_OK: return "ok";
    case PE_ERR_INVALID_ARG: return "invalid argument";
    case PE_ERR_UNSUPPORTED: return "unsupported shape or dtype";
    case PE_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case PE_ERR_HIP: return "HIP launch failed";
    default: return "unknown status";
  }
}

int pe_decode_splits(const pe_cache_desc* desc) { return check_desc(desc) == PE_OK ? decode_splits(desc) : 0; }

size_t pe_workspace_bytes(int op, const pe_cache_desc* desc, int64_t total_tokens) {
  if (check_desc(desc) != PE_OK) return 0;
  switch (op) {
    case PE_OP_PAGED_DECODE:
      return pe::decode_partials_bytes(desc->num_seqs, desc->num_q_heads, desc->head_dim, decode_splits(desc));
    case PE_OP_APPEND_PAGED_DECODE:
      return pe::decode_partials_bytes(desc->num_seqs, desc->num_q_heads, desc->head_dim, decode_splits(desc));
    case PE_OP_PREFILL_PRUNE:
      if (total_tokens < 0) return 0;
      return pe::prune_workspace_bytes(desc->num_seqs, desc->num_kv_heads, total_tokens,
                                       desc->layout == PE_LAYOUT_SHARED);
    default:
      return 0;
  }
}

namespace {
int score_blocks_impl(const pe_cache_desc* desc, const void* k_pool, const void* v_pool, const int32_t* block_table,
                      const int32_t* seq_lens, float* scores_out, int recent, void* stream, int budget = 0);
}

int pe_score_blocks(const pe_cache_desc* desc, const void* k_pool, const void* v_pool, const int32_t* block_table,
                    const int32_t* seq_lens, float* scores_out, void* workspace, size_t workspace_bytes,
                    void* stream) {
  (void)workspace;
  (void)workspace_bytes;
  return score_blocks_impl(desc, k_pool, v_pool, block_table, seq_lens, scores_out, 0, stream);
}

int pe_score_recent_blocks(const pe_cache_desc* desc, const void* k_pool, const void* v_pool,
                           const int32_t* block_table, const int32_t* seq_lens, int32_t recent,
                           float* scores_inout, void* stream) {
  if (recent < 1) return PE_ERR_INVALID_ARG;
  return score_blocks_impl(desc, k_pool, v_pool, block_table, seq_lens, scores_inout, recent, stream);
}

int pe_score_triggered_blocks(const pe_cache_desc* desc, const void* k_pool, const void* v_pool,
                              const int32_t* block_table, const int32_t* seq_lens, int32_t budget_tokens,
                              float* scores_inout, void* stream) {
  if (desc == nullptr) return PE_ERR_INVALID_ARG;
  if (budget_tokens <= 0 || desc->block_size <= 0 || budget_tokens % desc->block_size != 0) return PE_ERR_INVALID_ARG;
  return score_blocks_impl(desc, k_pool, v_pool, block_table, seq_lens, scores_inout, 0, stream, budget_tokens);
}

namespace {
int score_blocks_impl(const pe_cache_desc* desc, const void* k_pool, const void* v_pool, const int32_t* block_table,
                      const int32_t* seq_lens, float* scores_out, int recent, void* stream, int budget) {
  const int st = check_desc(desc);
  if (st != PE_OK) return st;
  if (!k_pool || !v_pool || !block_table || !seq_lens || !scores_out) return PE_ERR_INVALID_ARG;
  if (!aligned(k_pool, 16) || !aligned(v_pool, 16)) return PE_ERR_INVALID_ARG;
  pe::ScoreArgs a;
  a.k_pool = k_pool;
  a.v_pool = v_pool;
  a.block_table = block_table;
  a.seq_lens = seq_lens;
  a.scores = scores_out;
  a.num_seqs = desc->num_seqs;
  a.num_kv_heads = desc->num_kv_heads;
  a.head_dim = desc->head_dim;
  a.block_size = desc->block_size;
  a.max_blocks = desc->max_blocks;
  a.is_bf16 = desc->dtype == PE_BF16;
  a.shared = desc->layout == PE_LAYOUT_SHARED;
  a.recent = recent;
  a.budget = budget;
  return pe::launch_score_blocks(a, static_cast<hipStream_t>(stream)) == hipSuccess ? PE_OK : PE_ERR_HIP;
}
}  // namespace

int pe_prefill_prune(const pe_cache_desc* desc, const void* k_in, const void* v_in, const int32_t* cu_seqlens,
                     int64_t total_tokens, int32_t max_seqlen, int32_t budget_tokens, void* k_pool, void* v_pool,
                     const int32_t* block_table, int32_t* seq_lens_out, int32_t* kept_idx_out, void* workspace,
                     size_t workspace_bytes, void* stream) {
  const int st = check_desc(desc);
  if (st != PE_OK) return st;
  if (!cu_seqlens || !k_pool || !v_pool || !block_table || !seq_lens_out) return PE_ERR_INVALID_ARG;
  if (total_tokens < 0 || total_tokens > 0x7fffffffLL || max_seqlen < 0 || max_seqlen > total_tokens)
    return PE_ERR_INVALID_ARG;
  if (total_tokens > 0 && (!k_in || !v_in)) return PE_ERR_INVALID_ARG;
  if (budget_tokens <= 0 || budget_tokens % desc->block_size != 0) return PE_ERR_INVALID_ARG;
  {  // the longest pruned row must fit a table row: the gather indexes block_table[...][pos / B]
    const int64_t keep = max_seqlen < budget_tokens ? max_seqlen : budget_tokens;
    if ((keep + desc->block_size - 1) / desc->block_size > desc->max_blocks) return PE_ERR_INVALID_ARG;
  }
  if (!aligned(k_pool, 16) || !aligned(v_pool, 16) || !aligned(k_in, 16) || !aligned(v_in, 16))
    return PE_ERR_INVALID_ARG;
  const int ws = check_workspace(workspace, workspace_bytes,
                                 pe::prune_workspace_bytes(desc->num_seqs, desc->num_kv_heads, total_tokens,
                                                           desc->layout == PE_LAYOUT_SHARED));
  if (ws != PE_OK) return ws;
  pe::PruneArgs a;
  a.k_in = k_in;
  a.v_in = v_in;
  a.cu_seqlens = cu_seqlens;
  a.k_pool = k_pool;
  a.v_pool = v_pool;
  a.block_table = block_table;
  a.seq_lens_out = seq_lens_out;
  a.kept_idx_out = kept_idx_out;
  a.workspace = workspace;
  a.total_tokens = total_tokens;
  a.max_seqlen = max_seqlen;
  a.budget = budget_tokens;
  a.num_seqs = desc->num_seqs;
  a.num_kv_heads = desc->num_kv_heads;
  a.head_dim = desc->head_dim;
  a.block_size = desc->block_size;
  a.max_blocks = desc->max_blocks;
  a.is_bf16 = desc->dtype == PE_BF16;
  a.shared = desc->layout == PE_LAYOUT_SHARED;
  a.compute_units = compute_units();
  return pe::launch_prefill_prune(a, static_cast<hipStream_t>(stream)) == hipSuccess ? PE_OK : PE_ERR_HIP;
}

namespace {
int evict_blocks_impl(const pe_cache_desc* desc, const float* scores, float* scores_mut, int32_t* block_table,
                      int32_t* seq_lens, int32_t budget_tokens, int32_t* evicted_logical_out, int32_t* freed_phys_out,
                      void* stream, const pe_evict_opts* opts = nullptr);
}

int pe_evict_blocks_ex(const pe_cache_desc* desc, const pe_evict_opts* opts, float* scores, int32_t* block_table,
                       int32_t* seq_lens, int32_t budget_tokens, int32_t* evicted_logical_out,
                       int32_t* freed_phys_out, void* stream) {
  if (opts == nullptr) return PE_ERR_INVALID_ARG;
  if (opts->policy != PE_POLICY_LOWEST_SCORE && opts->policy != PE_POLICY_OLDEST) return PE_ERR_INVALID_ARG;
  if (opts->protect_first < 0 || opts->protect_last < 0) return PE_ERR_INVALID_ARG;
  if (opts->policy == PE_POLICY_LOWEST_SCORE && scores == nullptr) return PE_ERR_INVALID_ARG;
  if (opts->cached_scores && scores == nullptr) return PE_ERR_INVALID_ARG;
  return evict_blocks_impl(desc, scores, opts->cached_scores ? scores : nullptr, block_table, seq_lens, budget_tokens,
                           evicted_logical_out, freed_phys_out, stream, opts);
}

int pe_score_evict(const pe_cache_desc* desc, const void* k_pool, const void* v_pool, int32_t* block_table,
                   int32_t* seq_lens, int32_t budget_tokens, float* scores_out, int32_t* evicted_logical_out,
                   int32_t* freed_phys_out, void* stream) {
  const int st = check_desc(desc);
  if (st != PE_OK) return st;
  if (!k_pool || !v_pool || !block_table || !seq_lens || !evicted_logical_out || !freed_phys_out)
    return PE_ERR_INVALID_ARG;
  if (!aligned(k_pool, 16) || !aligned(v_pool, 16)) return PE_ERR_INVALID_ARG;
  if (budget_tokens <= 0 || budget_tokens % desc->block_size != 0) return PE_ERR_INVALID_ARG;
  if (desc->layout != PE_LAYOUT_PER_HEAD) return PE_ERR_UNSUPPORTED;  // needs every head's score before the argmin
  pe::ScoreEvictArgs a;
  a.k_pool = k_pool;
  a.v_pool = v_pool;
  a.block_table = block_table;
  a.seq_lens = seq_lens;
  a.scores_out = scores_out;
  a.evicted_logical = evicted_logical_out;
  a.freed_phys = freed_phys_out;
  a.num_seqs = desc->num_seqs;
  a.num_kv_heads = desc->num_kv_heads;
  a.head_dim = desc->head_dim;
  a.block_size = desc->block_size;
  a.max_blocks = desc->max_blocks;
  a.budget = budget_tokens;
  a.is_bf16 = desc->dtype == PE_BF16;
  return pe::launch_score_evict(a, static_cast<hipStream_t>(stream)) == hipSuccess ? PE_OK : PE_ERR_HIP;
}

int pe_evict_blocks(const pe_cache_desc* desc, const float* scores, int32_t* block_table, int32_t* seq_lens,
                    int32_t budget_tokens, int32_t* evicted_logical_out, int32_t* freed_phys_out, void* stream) {
  return evict_blocks_impl(desc, scores, nullptr, block_table, seq_lens, budget_tokens, evicted_logical_out,
                           freed_phys_out, stream);
}

int pe_evict_blocks_cached(const pe_cache_desc* desc, float* scores_inout, int32_t* block_table, int32_t* seq_lens,
                           int32_t budget_tokens, int32_t* evicted_logical_out, int32_t* freed_phys_out,
                           void* stream) {
  return evict_blocks_impl(desc, scores_inout, scores_inout, block_table, seq_lens, budget_tokens,
                           evicted_logical_out, freed_phys_out, stream);
}

namespace {
int evict_blocks_impl(const pe_cache_desc* desc, const float* scores, float* scores_mut, int32_t* block_table,
                      int32_t* seq_lens, int32_t budget_tokens, int32_t* evicted_logical_out, int32_t* freed_phys_out,
                      void* stream, const pe_evict_opts* opts) {
  const int st = check_desc(desc);
  if (st != PE_OK) return st;
  if ((!scores && !(opts && opts->policy == PE_POLICY_OLDEST)) || !block_table || !seq_lens || !evicted_logical_out || !freed_phys_out) return PE_ERR_INVALID_ARG;
  if (budget_tokens <= 0 || budget_tokens % desc->block_size != 0) return PE_ERR_INVALID_ARG;
  pe::EvictArgs a;
  a.scores = scores;
  a.scores_mut = scores_mut;
  a.block_table = block_table;
  a.seq_lens = seq_lens;
  a.evicted_logical = evicted_logical_out;
  a.freed_phys = freed_phys_out;
  a.num_seqs = desc->num_seqs;
  a.num_kv_heads = desc->num_kv_heads;
  a.block_size = desc->block_size;
  a.max_blocks = desc->max_blocks;
  a.budget = budget_tokens;
  a.shared = desc->layout == PE_LAYOUT_SHARED;
  if (opts != nullptr) {
    a.policy = opts->policy;
    a.protect_first = opts->protect_first;
    a.protect_last = opts->protect_last;
    a.share_heads = opts->share_heads != 0;
  }
  return pe::launch_evict_blocks(a, static_cast<hipStream_t>(stream)) == hipSuccess ? PE_OK : PE_ERR_HIP;
}
}  // namespace

int pe_paged_decode(const pe_cache_desc* desc, const void* q, const void* k_pool, const void* v_pool,
                    const int32_t* block_table, const int32_t* seq_lens, float softmax_scale, void* out,
                    void* workspace, size_t workspace_bytes, void* stream) {
  const int st = check_desc(desc);
  if (st != PE_OK) return st;
  if (!q || !k_pool || !v_pool || !block_table || !seq_lens || !out) return PE_ERR_INVALID_ARG;
  if (!aligned(k_pool, 16) || !aligned(v_pool, 16) || !aligned(q, 16)) return PE_ERR_INVALID_ARG;
  if (!finite(softmax_scale)) return PE_ERR_INVALID_ARG;
  const int splits = decode_splits_within(desc, workspace_bytes);
  const int ws = check_workspace(
      workspace, workspace_bytes,
      pe::decode_partials_bytes(desc->num_seqs, desc->num_q_heads, desc->head_dim, splits));
  if (ws != PE_OK) return ws;
  pe::DecodeArgs a = decode_args(desc, splits);
  a.q = q;
  a.k_pool = k_pool;
  a.v_pool = v_pool;
  a.block_table = block_table;
  a.seq_lens = seq_lens;
  a.out = out;
  a.partials = static_cast<float*>(workspace);
  a.scale = softmax_scale;
  tag_attention(desc, &a);
  return pe::launch_paged_decode(a, static_cast<hipStream_t>(stream)) == hipSuccess ? PE_OK : PE_ERR_HIP;
}

namespace {
// Device address of `scratch` on the current device, looked up once per device (every GPU holds its own copy of
// the array at its own address).
int static_scratch(void** out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* ptr[kMaxDevices] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return PE_ERR_HIP;
  if (dev < 0 || dev >= kMaxDevices) return PE_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(mu);
  if (ptr[dev] == nullptr) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return PE_ERR_HIP;
    ptr[dev] = p;
  }
  *out = ptr[dev];
  return PE_OK;
}
}  // namespace

int pe_paged_decode_static(const pe_cache_desc* desc, const void* q, const void* k_pool, const void* v_pool,
                           const int32_t* block_table, const int32_t* seq_lens, float softmax_scale, void* out,
                           void* stream) {
  const int st = check_desc(desc);
  if (st != PE_OK) return st;
  if (!q || !k_pool || !v_pool || !block_table || !seq_lens || !out) return PE_ERR_INVALID_ARG;
  if (!aligned(k_pool, 16) || !aligned(v_pool, 16) || !aligned(q, 16)) return PE_ERR_INVALID_ARG;
  if (!finite(softmax_scale)) return PE_ERR_INVALID_ARG;
  const int splits = decode_splits(desc);
  const size_t need = pe::decode_partials_bytes(desc->num_seqs, desc->num_q_heads, desc->head_dim, splits);
  if (need > (size_t)PE_STATIC_SCRATCH_BYTES) return PE_ERR_WORKSPACE;  // the partials would not fit the array
  void* partials = nullptr;
  if (need > 0) {
    const int sc = static_scratch(&partials);
    if (sc != PE_OK) return sc;
  }
  pe::DecodeArgs a = decode_args(desc, splits);
  a.q = q;
  a.k_pool = k_pool;
  a.v_pool = v_pool;
  a.block_table = block_table;
  a.seq_lens = seq_lens;
  a.out = out;
  // every (row, split, head) record the merge reads is written by the attention kernel of the same call (empty
  // splits write (acc, m, l) = (0, -inf, 0)), so what an earlier call left in the array never shows
  a.partials = static_cast<float*>(partials);
  a.scale = softmax_scale;
  tag_attention(desc, &a);
  return pe::launch_paged_decode(a, static_cast<hipStream_t>(stream)) == hipSuccess ? PE_OK : PE_ERR_HIP;
}

namespace {
// The output holds tags and counts before it is written: not if something that is read still lies there, or at an odd address.
bool out_is_free(const pe_cache_desc* d, int32_t layers, const void* out, const void* q, const void* new_k, const void* new_v) {
  if (d == nullptr) return false;
  const size_t head = (size_t)layers * d->num_seqs * d->head_dim * (d->dtype == PE_F32 ? 4 : 2);
  const size_t o = head * d->num_q_heads, kv = head * d->num_kv_heads;
  return aligned(out, 8) && !overlap(out, o, q, o) && !overlap(out, o, new_k, kv) && !overlap(out, o, new_v, kv);
}

// `free_out`: nothing that is read lies in `out`, and tags and counts can; `counted`: the counts there are clear (by the call for the
// layer before); next_out: where this call is to clear them for the layer behind it, or null.
int append_paged_decode(const pe_cache_desc* desc, const void* new_k, const void* new_v, const void* q, void* k_pool, void* v_pool,
                        int32_t* block_table, const int32_t* seq_lens, int32_t* seq_lens_out, int32_t* freed_phys,
                        const int32_t* spare, int32_t* spare_used, int32_t n_spare, float softmax_scale, void* out, void* workspace,
                        size_t workspace_bytes, void* stream, bool free_out, bool counted, void* next_out) {
  const int st = check_desc(desc);
  if (st != PE_OK) return st;
  if (!new_k || !new_v || !q || !k_pool || !v_pool || !block_table || !seq_lens || !seq_lens_out || !freed_phys ||
      !spare || !spare_used || !out)
    return PE_ERR_INVALID_ARG;
  if (seq_lens_out == seq_lens) return PE_ERR_INVALID_ARG;
  if (n_spare < 1) return PE_ERR_INVALID_ARG;
  if (!aligned(k_pool, 16) || !aligned(v_pool, 16) || !aligned(q, 16) || !aligned(new_k, 16) || !aligned(new_v, 16))
    return PE_ERR_INVALID_ARG;
  if (!finite(softmax_scale)) return PE_ERR_INVALID_ARG;
  const int splits = decode_splits_within(desc, workspace_bytes);
  const int ws = check_workspace(
      workspace, workspace_bytes,
      pe::decode_partials_bytes(desc->num_seqs, desc->num_q_heads, desc->head_dim, splits));
  if (ws != PE_OK) return ws;
  pe::DecodeArgs a = decode_args(desc, splits);
  a.q = q;
  a.k_pool = k_pool;
  a.v_pool = v_pool;
  a.block_table = block_table;
  a.seq_lens = seq_lens;
  a.out = out;
  a.partials = static_cast<float*>(workspace);
  a.scale = softmax_scale;
  a.new_k = new_k;
  a.new_v = new_v;
  a.freed_phys = freed_phys;
  a.spare = spare;
  a.spare_used = spare_used;
  a.seq_lens_out = seq_lens_out;
  a.n_spare = n_spare;
  if (free_out && splits_counted(desc, a)) {
    a.counted = counted;
    a.next_out = next_out;
    a.tagged = !counted && splits_tagged(desc, a);
    if (a.tagged) a.tag = launch_tag();
  }
  if (desc->layout == PE_LAYOUT_SHARED && desc->dtype == PE_F32) {
    // One table row per sequence: the workgroups of a sequence's heads would race on its page bookkeeping inside one
    // launch of the fp32 kernel, so the same effect is produced by two launches (append, then attention over the new
    // lengths).
    pe::AppendArgs ap;
    ap.new_k = new_k;
    ap.new_v = new_v;
    ap.k_pool = k_pool;
    ap.v_pool = v_pool;
    ap.block_table = block_table;
    ap.seq_lens = const_cast<int32_t*>(seq_lens);
    ap.seq_lens_out = seq_lens_out;
    ap.freed_phys = freed_phys;
    ap.spare = spare;
    ap.spare_used = spare_used;
    ap.n_spare = n_spare;
    ap.num_seqs = desc->num_seqs;
    ap.num_kv_heads = desc->num_kv_heads;
    ap.head_dim = desc->head_dim;
    ap.block_size = desc->block_size;
    ap.max_blocks = desc->max_blocks;
    ap.is_bf16 = desc->dtype == PE_BF16;
    ap.shared = true;
    if (pe::launch_append_kv(ap, static_cast<hipStream_t>(stream)) != hipSuccess) return PE_ERR_HIP;
    a.seq_lens = seq_lens_out;
    a.new_k = nullptr;
    a.new_v = nullptr;
  }
  return pe::launch_paged_decode(a, static_cast<hipStream_t>(stream)) == hipSuccess ? PE_OK : PE_ERR_HIP;
}

}  // namespace

int pe_append_paged_decode(const pe_cache_desc* desc, const void* new_k, const void* new_v, const void* q,
                           void* k_pool, void* v_pool, int32_t* block_table, const int32_t* seq_lens,
                           int32_t* seq_lens_out, int32_t* freed_phys, const int32_t* spare, int32_t* spare_used,
                           int32_t n_spare, float softmax_scale, void* out, void* workspace, size_t workspace_bytes,
                           void* stream) {
  return append_paged_decode(desc, new_k, new_v, q, k_pool, v_pool, block_table, seq_lens, seq_lens_out, freed_phys, spare, spare_used,
                             n_spare, softmax_scale, out, workspace, workspace_bytes, stream, out_is_free(desc, 1, out, q, new_k, new_v),
                             false, nullptr);
}

int pe_append_paged_decode_layers(const pe_cache_desc* desc, int32_t num_layers, const void* new_k, const void* new_v,
                                  const void* q, void* k_pool, void* v_pool, int32_t* block_table,
                                  const int32_t* seq_lens, int32_t* seq_lens_out, int32_t* freed_phys,
                                  const int32_t* spare, int32_t* spare_used, int32_t n_spare, float softmax_scale,
                                  void* out, void* workspace, size_t workspace_bytes, void* stream) {
  const int st = check_desc(desc);
  if (st != PE_OK) return st;
  if (num_layers < 1 || n_spare < 1) return PE_ERR_INVALID_ARG;
  if (!new_k || !new_v || !q || !block_table || !seq_lens || !seq_lens_out || !freed_phys || !spare || !spare_used || !out)
    return PE_ERR_INVALID_ARG;
  const bool shared = desc->layout == PE_LAYOUT_SHARED;
  const size_t elem = desc->dtype == PE_BF16 ? 2 : 4;
  const int64_t S = desc->num_seqs;
  const int64_t rows = shared ? S : S * desc->num_kv_heads;  // table rows, spare lists, freed pages per layer
  const size_t kv_bytes = (size_t)S * desc->num_kv_heads * desc->head_dim * elem;
  const size_t q_bytes = (size_t)S * desc->num_q_heads * desc->head_dim * elem;
  const bool free_out = out_is_free(desc, num_layers, out, q, new_k, new_v);
  for (int32_t l = 0; l < num_layers; ++l) {
    const int rc = append_paged_decode(
        desc, static_cast<const char*>(new_k) + l * kv_bytes, static_cast<const char*>(new_v) + l * kv_bytes,
        static_cast<const char*>(q) + l * q_bytes, k_pool, v_pool, block_table + l * rows * desc->max_blocks,
        seq_lens + l * S, seq_lens_out + l * S, freed_phys + l * rows, spare + l * rows * n_spare, spare_used + l * rows,
        n_spare, softmax_scale, static_cast<char*>(out) + l * q_bytes, workspace, workspace_bytes, stream,
        free_out, free_out && l > 0, free_out && l + 1 < num_layers ? static_cast<char*>(out) + (l + 1) * q_bytes : nullptr);
    if (rc != PE_OK) return rc;
  }
  return PE_OK;
}

int pe_append_kv(const pe_cache_desc* desc, const void* new_k, const void* new_v, void* k_pool, void* v_pool,
                 int32_t* block_table, int32_t* seq_lens, int32_t* freed_phys, const int32_t* spare,
                 int32_t* spare_used, int32_t n_spare, void* stream) {
  const int st = check_desc(desc);
  if (st != PE_OK) return st;
  if (!new_k || !new_v || !k_pool || !v_pool || !block_table || !seq_lens || !freed_phys || !spare || !spare_used)
    return PE_ERR_INVALID_ARG;
  if (n_spare < 1) return PE_ERR_INVALID_ARG;
  if (!aligned(k_pool, 16) || !aligned(v_pool, 16) || !aligned(new_k, 16) || !aligned(new_v, 16))
    return PE_ERR_INVALID_ARG;
  pe::AppendArgs a;
  a.new_k = new_k;
  a.new_v = new_v;
  a.k_pool = k_pool;
  a.v_pool = v_pool;
  a.block_table = block_table;
  a.seq_lens = seq_lens;
  a.freed_phys = freed_phys;
  a.spare = spare;
  a.spare_used = spare_used;
  a.n_spare = n_spare;
  a.num_seqs = desc->num_seqs;
  a.num_kv_heads = desc->num_kv_heads;
  a.head_dim = desc->head_dim;
  a.block_size = desc->block_size;
  a.max_blocks = desc->max_blocks;
  a.is_bf16 = desc->dtype == PE_BF16;
  a.shared = desc->layout == PE_LAYOUT_SHARED;
  return pe::launch_append_kv(a, static_cast<hipStream_t>(stream)) == hipSuccess ? PE_OK : PE_ERR_HIP;
}

}  // extern "C"
