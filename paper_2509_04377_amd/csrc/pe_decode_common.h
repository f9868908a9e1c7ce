// What the attention kernels share: their arguments, and the end of a workgroup.
//
// Small launches are bound by the chain of dependent steps before the first K/V load and behind the last one, not by traffic.
// What shortened it, measured together on an MI355X (microseconds a launch, before / after; splits include the merge launch):
// page lookups first and without a division in front of them (pe_place.h), K and V next, queries and the remaining arguments
// behind them; tiles counted without a division; no wait for the placeholder loads behind a wave's last tile (where splits are merged by the
// last to arrive there is one, see there); reductions over lane rows on the vector units, wave states read from LDS at once.  bfloat16, 64 rows of D = 64 x 1024 8.3 / 8.0, 32 rows of
// D = 128 x 4096 16.3 / 15.8, 128 rows x 1024 15.1 / 14.8; vector units, 64 rows of D = 64 x 256, one query head per KV head
// 5.3 / 4.6, fp32 with two 6.5 / 6.1.
#pragma once

#include <stddef.h>

#include "pe_device.h"
#include "pe_launch.h"
#include "pe_place.h"

namespace pe {

// Kernel arguments besides the leading ones, which are what a wave needs before its first K/V load (14 registers' worth: the
// compiler's kernel-argument preloading puts them into scalar registers before the wave starts, and the page lookup does
// not wait for a load of them.  Layer launches of the 1B shape 8.70 / 8.52 us, 8B long context 17.9 / 17.4, 8B 44.9 / 44.7).
struct DecodeParams {
  void* out;
  float* partials;
  float scale_log2e;
  // fused append (FUSED kernels only)
  int n_spare;
  const void* new_k;
  const void* new_v;
  int32_t* freed_phys;
  const int32_t* spare;
  int32_t* spare_used;
  int32_t* seq_lens_out;  // [S], must not alias seq_lens
  void* next_out;         // output of the launch behind this one, whose arrival counts are to be cleared, or null (merge_arrived)
  uint64_t tag;           // of this launch (merge_arrived)
};

// All of them as they lie in the kernel-argument segment (in order, each at its own alignment).
struct DecodeKernelArgs {
  const int32_t* seq_lens;
  const int32_t* block_table;
  const void *q, *k_pool, *v_pool;
  int num_kv_heads, max_blocks;
  uint32_t inv_heads, shape;
  DecodeParams p;
};

// The kernels' parameters.  decode_params() below reads the last one out of the argument segment by itself, so a kernel must have
// these and no others (launch_decode takes no other), and the struct must lie as the segment does.
using DecodeKernel = void (*)(const int32_t* seq_lens, const int32_t* block_table, const void* q, const void* k_pool,
                              const void* v_pool, int num_kv_heads, int max_blocks, uint32_t inv_heads, uint32_t shape,
                              DecodeParams p);

// Where a kernel's last argument lies in the segment: each one at the next multiple of its own alignment.
template <typename... A>
constexpr size_t last_argument_offset(void (*)(A...)) {
  size_t at = 0, end = 0;
  ((at = (end + alignof(A) - 1) / alignof(A) * alignof(A), end = at + sizeof(A)), ...);
  return at;
}
static_assert(last_argument_offset(DecodeKernel(nullptr)) == offsetof(DecodeKernelArgs, p), "decode_params() reads elsewhere");

inline hipError_t launch_decode(DecodeKernel kernel, dim3 blocks, dim3 threads, hipStream_t stream, const DecodeKernelArgs& k) {
  hipLaunchKernelGGL(kernel, blocks, threads, 0, stream, k.seq_lens, k.block_table, k.q, k.k_pool, k.v_pool, k.num_kv_heads,
                     k.max_blocks, k.inv_heads, k.shape, k.p);
  return hipGetLastError();
}

// `shape`: log2 of the page size, query heads per KV head, order of the workgroups, splits
constexpr uint32_t kShapeXcd = 128u, kShapeLinear = 256u;
__host__ __device__ inline int shape_log2_block(uint32_t shape) { return (int)(shape & 7u); }
__host__ __device__ inline int shape_group(uint32_t shape) { return (int)(shape >> 3 & 15u); }
__host__ __device__ inline int shape_splits(uint32_t shape) { return (int)(shape >> 9); }

inline bool decode_kernel_args(const DecodeArgs& a, DecodeKernelArgs* k, dim3* blocks) {
  PlaceGrid g;
  if (!place_grid(a.num_seqs, a.num_kv_heads, a.splits, a.xcd_map != 0, &g)) return false;
  int log2_block = 0;
  while ((1 << log2_block) < a.block_size) ++log2_block;
  *blocks = dim3(g.x, g.y);
  *k = DecodeKernelArgs{a.seq_lens, a.block_table, a.q, a.k_pool, a.v_pool, a.num_kv_heads, a.max_blocks, g.inv_heads,
                        (uint32_t)log2_block | (uint32_t)(a.num_q_heads / a.num_kv_heads) << 3 | (g.xcd ? kShapeXcd : 0u) |
                            (g.linear ? kShapeLinear : 0u) | (uint32_t)a.splits << 9,
                        DecodeParams{a.out, a.partials, a.scale * 1.4426950408889634f, a.n_spare, a.new_k, a.new_v, a.freed_phys,
                                     a.spare, a.spare_used, a.seq_lens_out, a.next_out, a.tag}};
  return true;
}

__device__ __forceinline__ Place decode_place(uint32_t shape, int num_kv_heads, uint32_t inv_heads) {
  return place_at(blockIdx.x, blockIdx.y, (shape & kShapeXcd) != 0, (shape & kShapeLinear) != 0, shape_splits(shape),
                  num_kv_heads, inv_heads);
}

// The other arguments.  They are asked for behind a wave's first page lookup: scalar loads come back in any order, so that
// the wait for the lookup would wait for them too.  (Their address is made to depend on `behind`, something that the lookup
// gave: the compiler otherwise moves loads of arguments to the top.)
__device__ __forceinline__ DecodeParams decode_params(int behind) {
  uint64_t args = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(DecodeKernelArgs, p);
  asm("" : "+s"(args) : "s"(behind));
  const auto* a = reinterpret_cast<const __attribute__((address_space(4))) DecodeParams*>(args);
  return DecodeParams{a->out,   a->partials,   a->scale_log2e, a->n_spare,    a->new_k,
                      a->new_v, a->freed_phys, a->spare,       a->spare_used, a->seq_lens_out, a->next_out, a->tag};
}

// Two neighbouring elements of the output in one store, at any boundary of their own size.
struct __attribute__((packed, aligned(2))) Bf16Pair {
  uint32_t v;
};
struct __attribute__((packed, aligned(4))) F32Pair {
  float a, b;
};

// (m, l) and the accumulators of a workgroup's waves, GH heads each, as they meet in LDS.
template <int WAVES, int GH, int D>
struct WaveStates {
  __attribute__((aligned(16))) float acc[WAVES][GH][D];
  float2 ml[WAVES][GH];
};

// E elements of a head over its splits, and l, relative to the largest m: added four at a time, those past the last being the last again.  Up to
// most_arrivals splits are always added like this, whoever does it, so that a result does not depend on how its splits come together.
template <int E>
__device__ __forceinline__ void add_splits(int s, int splits, const float2 (&ml)[4], const float (&v)[4][E], float& m, float& l,
                                           float (&o)[E]) {
  float mm = m;
#pragma unroll
  for (int j = 0; j < 4; ++j) mm = fmaxf(mm, ml[j].x);
  const float ms = mm == -__builtin_inff() ? 0.f : mm;
  const float old = __builtin_amdgcn_exp2f(m - ms);
  l *= old;
#pragma unroll
  for (int e = 0; e < E; ++e) o[e] *= old;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const bool real = s + j < splits;  // what is no split adds nothing, an infinity of the last one included (0 * inf)
    const float w = __builtin_amdgcn_exp2f(ml[j].x - ms);
    l = fmaf(real ? ml[j].y : 0.f, real ? w : 0.f, l);
#pragma unroll
    for (int e = 0; e < E; ++e) o[e] = fmaf(real ? v[j][e] : 0.f, real ? w : 0.f, o[e]);
  }
  m = mm;
}

// All of them: read(split, ml, v) gets a split's (m, l) and elements.  The next four are on their way while four are added.
template <int E, typename Read>
__device__ __forceinline__ void merge_splits(int splits, float (&result)[E], Read read) {
  float m = -__builtin_inff(), l = 0.f, o[E] = {};
  float2 ml[4];
  float v[4][E];
#pragma unroll
  for (int j = 0; j < 4; ++j) read(j < splits ? j : splits - 1, ml[j], v[j]);
  for (int s = 0;;) {
    const int next = s + 4;
    float2 ml_next[4];
    float v_next[4][E];
    if (next < splits) {
#pragma unroll
      for (int j = 0; j < 4; ++j) read(next + j < splits ? next + j : splits - 1, ml_next[j], v_next[j]);
    }
    add_splits(s, splits, ml, v, m, l, o);
    if (next >= splits) break;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      ml[j] = ml_next[j];
#pragma unroll
      for (int e = 0; e < E; ++e) v[j][e] = v_next[j][e];
    }
    s = next;
  }
#pragma unroll
  for (int e = 0; e < E; ++e) result[e] = l > 0.f ? o[e] / l : 0.f;
}

// How the splits of a row come together: by a launch of its own, or by the last of them to arrive.
enum { kMergeLaunch, kCounted, kTagged };

// ---- splits merged by the last of them to arrive ---------------------------------------------------------------
// No merge launch behind it then.  Every wave of a workgroup stores its part of the split's record, waits until that is where all compute
// dies see it, and makes its arrival known; one that finds all others there reads the records back and writes the output, in the order
// of the splits, whoever it is.  Records are stored and loaded as relaxed atomics at agent scope (write-through, past the first-level
// cache), so that nothing rests on which compute die a workgroup is on.
//
// There is nowhere to keep arrivals from one call to the next (a workspace may hold anything), so they are made known in the output
// itself, at the beginning of what a wave will write there:
//   - kCounted: its first word is a count.  It has to be zero when the launch begins: only the call that knows the next launch's output
//     can provide for that, the one for all layers of a step, whose launch for a layer clears the words of the next layer's output.
//   - kTagged: its first words are a tag for each split, a number that no other launch of the process has (a counter in the host layer
//     makes them: the one thing that a call leaves behind).  A wave stores its own, waits
//     until everyone sees that too, and then looks at all of them: the last to arrive finds every one, and where others do as well
//     they write the same.  What lay in the output before is no tag of this launch; a graph that is replayed has the same tag each
//     time, but the output, by then written, lies over it.  (Of a launch from another process with the same tag nothing is in memory.)
//
// Bound: a chain of round trips, cycles (2.4 GHz) from a clock in the kernel: records stored 530 (the wait is for all that the wave has
// outstanding, the placeholder loads behind its last tile included: loads and stores count alike), counted 960 (tags: one more round trip,
// some 500), read back 720, merged 570; a merge launch costs 1.9 us.  16 layers of 64 rows x 1024 tokens of D = 64 in four splits 2056 /
// 1812 us for 16 steps, 32 layers of 32 rows x 4096 of D = 128 in eight 8295 / 8090; one layer of 64 rows x 2048 of D = 64 in four,
// called by itself, 16 steps 191 / 152 (out of a graph 9.9 / 9.4 us a call: the launch costs the host more than the GPU).
// Where it pays (merge launch / tagged / counted, us a layer out of a graph, D = 128 unless said):
//   - up to eight or twelve splits, merged four at a time one after the other: 16 rows x 2048 in two 14.5 / 13.9 / 13.7, four 10.7 / 10.2
//     / 9.9, six 10.1 / 9.9 / 9.6, seven 10.3 / 9.9 / 9.7, eight 8.7 / 8.6 / 8.3 (D = 64 7.2 / 7.2 / 6.7), ten 8.9 / 9.3 / 8.9, twelve 8.5 /
//     9.0 / 8.5, fifteen 8.8 / 9.7 / 9.2; 20 rows x 2048 in twelve 9.7 / 9.8 / 9.2; with eight query heads of D = 64, 32 rows x 2048 in eight
//     9.3 / 9.2 / 8.7, 8 x 4096 in ten 10.8 / 11.1 / 10.9.  Eight are tagged in workgroups of four waves and pieces of less than 256 KiB, as no slower, for the
//     host's sake: larger ones, which it does not wait for, take 14.5 / 14.7 (fp32 15.4 / 15.6);
//   - one part of a row a wave: with two (four waves, more than four query heads) 32 rows x 2048 in eight 11.9 / 12.7 counted;
//   - workgroups that are all there from the beginning, two a compute unit (one with more than eight splits: 32 rows x 4096 in eight 15.5 /
//     15.1 counted, ten 17.9 / 18.0, twelve 16.0 / 16.7): 128 rows x 2048 of fp32 in four 43.9 / 43.8 tagged; of 640 and
//     more, those that wait for memory at their ends keep others out (160 rows x 4096 in four 62.3 / 65.5, 264 x 2048 52.9 / 54.4 counted).
template <int GH, int D, int WAVES>
constexpr bool one_part_a_wave = GH * (D / 2) <= WAVES * kWave;

__device__ __forceinline__ void store_for_all(float* to, float a, float b) {
  __hip_atomic_store(reinterpret_cast<uint64_t*>(to), __builtin_bit_cast(uint64_t, make_float2(a, b)), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 load_of_all(const float* from) {
  return __builtin_bit_cast(float2, __hip_atomic_load(reinterpret_cast<const uint64_t*>(from), __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT));
}

template <typename T>
__device__ __forceinline__ void store_pair(void* out, int64_t pair, float a, float b) {
  if constexpr (sizeof(T) == 4) {
    static_cast<F32Pair*>(out)[pair] = F32Pair{a, b};
  } else {
    static_cast<Bf16Pair*>(out)[pair].v = (uint32_t)f32_to_bf16(a) | ((uint32_t)f32_to_bf16(b) << 16);
  }
}
// `pair`: the first of a wave's part of a row
template <typename T>
__device__ __forceinline__ uint32_t* arrival_count(void* out, int64_t pair) {
  return reinterpret_cast<uint32_t*>(static_cast<char*>(out) + pair * (2 * (int64_t)sizeof(T)));
}

// (m, l) and two elements of a head over the waves of a workgroup
struct WavesMerged {
  float m, l, o0, o1;
};
template <int WAVES, int GH, int D>
__device__ __forceinline__ WavesMerged over_waves(const WaveStates<WAVES, GH, D>& sm, int h, int d) {
  float2 ml[WAVES], part[WAVES];
#pragma unroll
  for (int w = 0; w < WAVES; ++w) {
    ml[w] = sm.ml[w][h];
    part[w] = *reinterpret_cast<const float2*>(&sm.acc[w][h][d]);
  }
  __builtin_amdgcn_sched_barrier(0);  // all are asked for before the first is used
  WavesMerged r{-__builtin_inff(), 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < WAVES; ++w) r.m = fmaxf(r.m, ml[w].x);
  const float ms = r.m == -__builtin_inff() ? 0.f : r.m;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) {
    const float f = __builtin_amdgcn_exp2f(ml[w].x - ms);
    r.l = fmaf(ml[w].y, f, r.l);
    r.o0 = fmaf(part[w].x, f, r.o0);
    r.o1 = fmaf(part[w].y, f, r.o1);
  }
  return r;
}

// The end of a workgroup: its waves' states merged into the normalised output, or with several splits into the record of this
// one (accumulators, m, l).
template <typename T, int WAVES, int GH, int D>
__device__ __forceinline__ void merge_waves(const WaveStates<WAVES, GH, D>& sm, const DecodeParams& p, int row, int split,
                                            int splits, int g_real) {
  for (int idx = (int)threadIdx.x; idx < g_real * (D / 2); idx += WAVES * kWave) {
    const int h = idx / (D / 2), d = idx % (D / 2) * 2;
    const WavesMerged r = over_waves(sm, h, d);
    const int64_t head = (int64_t)row * g_real + h;  // s * Hq + query head
    if (splits == 1) {
      store_pair<T>(p.out, (head * D + d) / 2, r.l > 0.f ? r.o0 / r.l : 0.f, r.l > 0.f ? r.o1 / r.l : 0.f);
    } else {
      float* record = p.partials + (((int64_t)row * splits + split) * g_real + h) * (D + 2);
      *reinterpret_cast<float2*>(record + d) = make_float2(r.o0, r.o1);
      if (d == 0) *reinterpret_cast<float2*>(record + D) = make_float2(r.m, r.l);
    }
  }
}

// The same where the splits are counted or tagged (every wave has one part of the row: 64 pairs of elements).
template <typename T, bool TAGGED, int WAVES, int GH, int D>
__device__ __forceinline__ void merge_arrived(const WaveStates<WAVES, GH, D>& sm, const DecodeParams& p, int row, int split, int splits,
                                              int g_real) {
  static_assert(one_part_a_wave<GH, D, WAVES>, "one part of a row a wave");
  static_assert(kMostArrivals <= kWave / 2 && kMostArrivals * 8 <= kWave * (int)sizeof(T), "a tag a lane, in the output of half a wave");
  const int pairs = g_real * (D / 2), idx = (int)threadIdx.x, lane = lane_id();
  if (idx >= pairs) return;
  const int h = idx / (D / 2), d = idx % (D / 2) * 2;
  const int record = g_real * (D + 2);  // floats of a split
  const WavesMerged r = over_waves(sm, h, d);
  float* const base = p.partials + (int64_t)row * splits * record;
  float* const to = base + split * record + h * (D + 2);
  store_for_all(to + d, r.o0, r.o1);
  if (d == 0) store_for_all(to + D, r.m, r.l);
  const int64_t pair0 = (int64_t)row * pairs;
  const uint32_t ml_at = (uint32_t)(h * (D + 2) + D), o_at = (uint32_t)(h * (D + 2) + d);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the records are where everyone sees them (and the placeholder loads are back)
  bool last;
  if constexpr (TAGGED) {
    uint64_t* const tags = reinterpret_cast<uint64_t*>(arrival_count<T>(p.out, pair0 + (idx - lane)));
    if (lane == 0) __hip_atomic_store(tags + split, p.tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // and so is the tag, before the others' are looked at
    uint64_t seen = p.tag;
    if (lane < splits) seen = __hip_atomic_load(tags + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last = __builtin_amdgcn_ballot_w64(seen != p.tag) == 0;
  } else {
    uint32_t before = 0;
    if (lane == 0) before = __hip_atomic_fetch_add(arrival_count<T>(p.out, pair0 + idx), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last = __builtin_amdgcn_readfirstlane((int)before) == splits - 1;
  }
  if (last) {
    asm volatile("" ::: "memory");  // (the loads below do not move up)
    float o[2];
    merge_splits(splits, o, [&](int s, float2& ml, float (&v)[2]) {
      const float* of = base + s * record;
      ml = load_of_all(of + ml_at);
      const float2 pair = load_of_all(of + o_at);
      v[0] = pair.x, v[1] = pair.y;
    });
    store_pair<T>(p.out, pair0 + idx, o[0], o[1]);
  }
  if (p.next_out != nullptr && split == 0 && lane == 0) *arrival_count<T>(p.next_out, pair0 + idx) = 0u;
}

// The page that a new token goes to, and the bookkeeping of one that has to be linked for it (by lane 0): the page freed by
// the eviction just before, else the next spare.
__device__ __forceinline__ int link_page(const DecodeParams& p, int32_t* bt, int jb, int64_t table_row, int freed, int used,
                                         int lane) {
  int page = freed;
  if (page < 0) {
    page = used < p.n_spare ? p.spare[table_row * p.n_spare + used] : -1;
    if (lane == 0) p.spare_used[table_row] = used + 1;
  } else if (lane == 0) {
    p.freed_phys[table_row] = -1;
  }
  if (lane == 0) bt[jb] = page;
  return page;
}

}  // namespace pe
