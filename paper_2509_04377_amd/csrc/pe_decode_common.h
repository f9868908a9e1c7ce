// What the attention kernels share: their arguments, and the end of a workgroup.
//
// Small launches are bound by the chain of dependent steps before the first K/V load and behind the last one, not by traffic.
// What shortened it, measured together on an MI355X (microseconds a launch, before / after; splits include the merge launch):
// page lookups first and without a division in front of them (pe_place.h), K and V next, queries and the remaining arguments
// behind them; tiles counted without a division; no wait for the placeholder loads behind a wave's last tile; reductions over
// lane rows on the vector units, wave states read from LDS at once.  bfloat16, 64 rows of D = 64 x 1024 8.3 / 8.0, 32 rows of
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
                                     a.spare, a.spare_used, a.seq_lens_out}};
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
                      a->new_v, a->freed_phys, a->spare,       a->spare_used, a->seq_lens_out};
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

// The end of a workgroup: its waves' states merged into the normalised output, or with several splits into the record of this
// one (accumulators, m, l).
template <typename T, int WAVES, int GH, int D>
__device__ __forceinline__ void merge_waves(const WaveStates<WAVES, GH, D>& sm, const DecodeParams& p, int row, int split,
                                            int splits, int g_real) {
  for (int idx = (int)threadIdx.x; idx < g_real * (D / 2); idx += WAVES * kWave) {
    const int h = idx / (D / 2), d = idx % (D / 2) * 2;
    float2 ml[WAVES], part[WAVES];
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      ml[w] = sm.ml[w][h];
      part[w] = *reinterpret_cast<const float2*>(&sm.acc[w][h][d]);
    }
    __builtin_amdgcn_sched_barrier(0);  // all are asked for before the first is used
    float mm = -__builtin_inff();
#pragma unroll
    for (int w = 0; w < WAVES; ++w) mm = fmaxf(mm, ml[w].x);
    const float ms = mm == -__builtin_inff() ? 0.f : mm;
    float ll = 0.f, o0 = 0.f, o1 = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      const float f = __builtin_amdgcn_exp2f(ml[w].x - ms);
      ll = fmaf(ml[w].y, f, ll);
      o0 = fmaf(part[w].x, f, o0);
      o1 = fmaf(part[w].y, f, o1);
    }
    const int64_t head = (int64_t)row * g_real + h;  // s * Hq + query head
    if (splits == 1) {
      const float r0 = ll > 0.f ? o0 / ll : 0.f, r1 = ll > 0.f ? o1 / ll : 0.f;
      const int64_t pair = (head * D + d) / 2;
      if constexpr (sizeof(T) == 4) {
        static_cast<F32Pair*>(p.out)[pair] = F32Pair{r0, r1};
      } else {
        static_cast<Bf16Pair*>(p.out)[pair].v = (uint32_t)f32_to_bf16(r0) | ((uint32_t)f32_to_bf16(r1) << 16);
      }
    } else {
      float* record = p.partials + (((int64_t)row * splits + split) * g_real + h) * (D + 2);
      *reinterpret_cast<float2*>(record + d) = make_float2(o0, o1);
      if (d == 0) *reinterpret_cast<float2*>(record + D) = make_float2(mm, ll);
    }
  }
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
