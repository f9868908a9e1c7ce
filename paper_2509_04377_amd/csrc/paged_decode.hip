// Paged decode attention (Eq. 1 for one new query per sequence; Alg. 3 "PagedAttention(Q,K,V)") on the vector units, the merge
// of the splits, and the choice of the kernel (on the matrix cores: paged_decode_bf16.hip).
//
// fp32 caches (the fp32 matrix instructions have no higher rate), and bfloat16 ones of one query head per KV head with short
// rows, where the other kernel's longer way from the loads to the output shows and its products stay idle.  A workgroup owns one
// split of one (sequence, KV head) row: every splits-th group of four consecutive tiles of the row's tokens.  Each of
// its four waves walks tiles with a two-deep register pipeline.  Inside a tile every lane holds 16 bytes of two K rows
// and two V rows (consecutive lanes = consecutive addresses, so each wave-load is 1 KiB of one page, found through the
// block table with scalar loads).
//
//   QK:  each lane multiplies its K slice with the matching slice of all G query heads that share this
//        KV head; the partial dots are reduced over the lanes of a token row with a reduce-scatter over
//        heads, so that afterwards each lane owns the logit of ONE (token, head) pair;
//   softmax: online, state (m, l) kept per lane for its head and its own stream of tokens
//        (base-2 exponentials; the scale carries log2 e);
//   PV:  the lane's probability is broadcast inside its group of lanes and multiplies the V slice
//        into per-head fp32 accumulators.
//
// At the end the (wave, token-stream) partial states are merged through LDS; with one split the
// workgroup writes the normalised output, otherwise it writes (acc, m, l) partials that
// paged_decode_reduce_kernel merges.
//
// The FUSED variant also performs the harness append of the same decode iteration: the new token's K/V
// rows are taken from registers as one extra token of the row (they are not read back from the pool),
// the last split's workgroup links a new page if the tail page is full and stores the rows into the
// pool, and the new lengths go to a second array (the caller swaps the two), so no workgroup can see a
// length that another one has already bumped.
//
// The SHARED variant reads the head-shared cache layout: one table row per sequence and pages of
// [B][Hk][D], so the token rows of this workgroup's head are Hk rows apart (a wave-load is then TPL runs
// of one row each instead of one contiguous KiB).  Everything after the loads is the same.
#include "pe_decode_common.h"

namespace pe {
namespace {

constexpr float kNegInf = -__builtin_inff();

constexpr int next_pow2(int x) { return x <= 1 ? 1 : 2 * next_pow2((x + 1) / 2); }

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;

// The 16 bytes of one query head that face a lane's 16-byte K slice.
template <typename T>
struct QSlice;
template <>
struct QSlice<float> {
  float v[4];
  __device__ __forceinline__ void load(const float* p) {
    const uint4 r = *reinterpret_cast<const uint4*>(p);
    v[0] = __uint_as_float(r.x);
    v[1] = __uint_as_float(r.y);
    v[2] = __uint_as_float(r.z);
    v[3] = __uint_as_float(r.w);
  }
  __device__ __forceinline__ float dot(const uint4& k) const {
    float a = __uint_as_float(k.x) * v[0];
    a = fmaf(__uint_as_float(k.y), v[1], a);
    a = fmaf(__uint_as_float(k.z), v[2], a);
    a = fmaf(__uint_as_float(k.w), v[3], a);
    return a;
  }
};

template <>
struct QSlice<bf16_t> {
  uint32_t v[4];  // 8 bf16, packed as in memory
  __device__ __forceinline__ void load(const bf16_t* p) {
    const uint4 r = *reinterpret_cast<const uint4*>(p);
    v[0] = r.x;
    v[1] = r.y;
    v[2] = r.z;
    v[3] = r.w;
  }
  static __device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), c, false);
  }
  __device__ __forceinline__ float dot(const uint4& k) const {
    return dot2(k.w, v[3], dot2(k.z, v[2], dot2(k.y, v[1], dot2(k.x, v[0], 0.f))));
  }
};

template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}

// Slot i of lane l carries head (i ^ c(l)), c(l) = bit_reverse(l & (GP-1)).  A stage with partner
// l ^ M keeps the lower half of the slots and adds the partner's upper half, which carries the same
// heads.  After log2(GP) stages slot 0 is the dot product of head c(l) summed over GP lanes.
template <int N, int M>
__device__ __forceinline__ float head_scatter(float (&v)[N]) {
  if constexpr (N == 1) {
    return v[0];
  } else {
    float w[N / 2];
#pragma unroll
    for (int i = 0; i < N / 2; ++i) w[i] = v[i] + lane_xor_f32<M>(v[i + N / 2]);
    return head_scatter<N / 2, M * 2>(w);
  }
}

// Sum over the remaining lane bits FROM .. LPR/2 of a token row (every lane gets the total).
template <int FROM, int LPR>
__device__ __forceinline__ float row_all_reduce(float v) {
  if constexpr (FROM >= LPR) {
    return v;
  } else if constexpr (FROM == 4 && LPR >= 16) {
    v += dpp_f32<0x124>(v);  // row_ror:4
    v += dpp_f32<0x128>(v);  // row_ror:8 -> total over the four quads of the 16-lane row
    return row_all_reduce<16, LPR>(v);
  } else if constexpr (FROM == 8 && LPR >= 16) {
    v += dpp_f32<0x128>(v);  // row_ror:8 is lane ^ 8 inside a 16-lane row
    return row_all_reduce<16, LPR>(v);
  } else {
    v += lane_xor_f32<FROM>(v);
    return row_all_reduce<FROM * 2, LPR>(v);
  }
}

// Over the lanes of a wave that hold the same slice of a token row (every lane gets the total).
template <int LPR>
__device__ __forceinline__ float streams_sum(float v) {
  if constexpr (LPR == 8) v += dpp_f32<0x128>(v);  // row_ror:8
  if constexpr (LPR == 32) return halves_sum(v);
  return rows_sum(v);
}
template <int LPR>
__device__ __forceinline__ float streams_max(float v) {
  if constexpr (LPR == 8) v = fmaxf(v, dpp_f32<0x128>(v));
  if constexpr (LPR == 32) return halves_max(v);
  return rows_max(v);
}

// The same sums of all elements of a slice, dealt out: a wave's rows of lanes (LPR = 32: its halves) are left with one part of the
// slice each, consecutive elements.  Two operands a swap: a slice of four over four rows takes three swaps and adds, every lane with
// every total eight of each, which cost fp32 rows that are many and short more than a merge of all streams through LDS (eight query
// heads a KV head of D = 64, 552 rows of 64 tokens: through LDS 7.7 us, every total in every lane 8.05, this 6.8; 100 sequences x 8
// heads 9.4 / 9.7 / 8.4).
template <int LPR, int EPL>
struct StreamParts {
  static constexpr int kRows = LPR == 32 ? 2 : 4, kLanes = kWave / kRows, kPart = EPL / kRows;
  static __device__ __forceinline__ void sum(const float (&v)[EPL], float (&part)[kPart]) {
    float w[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) w[e] = LPR == 8 ? v[e] + dpp_f32<0x128>(v[e]) : v[e];  // row_ror:8
#pragma unroll
    for (int i = 0; i < kPart; ++i) {
      if constexpr (kRows == 2) {
        part[i] = halves_sum(w[i], w[kPart + i]);
      } else {
        part[i] = halves_sum(pairs_sum(w[i], w[kPart + i]), pairs_sum(w[2 * kPart + i], w[3 * kPart + i]));
      }
    }
  }
};

// acc[h][:] *= alpha of head h, which lives on lane position bit_reverse(h) of each GP-lane group.
template <int G, int GP, int EPL, int H = 0>
__device__ __forceinline__ void rescale_acc(float (&acc)[G][EPL], float alpha) {
  if constexpr (H < G) {
    const float a = group_bcast_f32<GP, bit_reverse<ilog2(GP)>(H)>(alpha);
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[H][e] *= a;
    rescale_acc<G, GP, EPL, H + 1>(acc, alpha);
  }
}

// acc[h][:] += prob of head h (broadcast as above) * v[:].
template <int G, int GP, int EPL, int H = 0>
__device__ __forceinline__ void accumulate_pv(float (&acc)[G][EPL], float prob, const float (&v)[EPL]) {
  if constexpr (H < G) {
    const float ph = group_bcast_f32<GP, bit_reverse<ilog2(GP)>(H)>(prob);
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[H][e] = fmaf(ph, v[e], acc[H][e]);
    accumulate_pv<G, GP, EPL, H + 1>(acc, prob, v);
  }
}

// Four or eight waves, two register buffers, two wave-loads of K and of V per tile (4 KiB per tile, 8 KiB per wave in flight
// while it waits): the stream runs fastest at about 8 MiB in flight over the chip.
constexpr int kDepth = 2, kLoads = 2;

template <typename T, int D, int G>
struct Tile {
  using Geo = RowGeom<T, D>;
  static constexpr int EPL = Geo::kPerVec;
  static constexpr int LPR = Geo::kLanesPerRow;
  static constexpr int TPL = Geo::kTokensPerLoad;
  static constexpr int NLT = kLoads;  // wave-loads of K (and of V) per tile
  static constexpr int TT = NLT * TPL;  // tokens per tile
  static constexpr int GP = next_pow2(G);
  static_assert(GP <= LPR && GP <= 8, "query group too large");

  static_assert(TT <= 16, "a tile lies in one page");

  // Table entry of the page of tile `tile` (scalar load).  The index is clamped to the table row; nothing here depends on the
  // row length, so that the first lookup can be issued before the length has arrived.
  static __device__ __forceinline__ int lookup(int tile, const int32_t* bt, int max_blocks, int log2_block) {
    int pi = (tile * TT) >> log2_block;
    pi = pi < max_blocks ? pi : max_blocks - 1;
    return __builtin_amdgcn_readfirstlane(bt[pi]);
  }

  // Issue the 2*NLT wave-loads of the tile whose first row lies at 16-byte vector `base`; its page was looked up one step
  // earlier (the table access is off the critical path of the loads).  `lane_off` is the lane's place inside a wave-load.
  static __device__ __forceinline__ void issue(uint4 (&kb)[NLT], uint4 (&vb)[NLT], int64_t base, const T* k_pool,
                                               const T* v_pool, int lane_off, int row_vecs) {
#pragma unroll
    for (int i = 0; i < NLT; ++i) {
      const int64_t vec = base + i * TPL * row_vecs + lane_off;
      kb[i] = load_vec_stream(k_pool, vec);
      vb[i] = load_vec_stream(v_pool, vec);
    }
  }

  // Consume NL wave-loads whose first token is tok0: logits, online softmax update, PV accumulation.
  template <int NL>
  static __device__ __forceinline__ void compute(uint4 (&kb)[NL], uint4 (&vb)[NL], int tok0, int len, int grp,
                                                 float scale_log2e, const QSlice<T> (&qs)[GP], float& m_run,
                                                 float& l_run, float (&acc)[G][EPL]) {
    float x[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      float sd[GP];
#pragma unroll
      for (int j = 0; j < GP; ++j) sd[j] = qs[j].dot(kb[i]);
      float r = head_scatter<GP, 1>(sd);
      r = row_all_reduce<GP, LPR>(r);
      x[i] = r * scale_log2e;
    }
    if (tok0 + NL * TPL > len) {  // the tile reaches past the row: mask logits, keep junk V out of the sum
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const bool ok = tok0 + i * TPL + grp < len;
        x[i] = ok ? x[i] : kNegInf;
        if (!ok) vb[i] = make_uint4(0u, 0u, 0u, 0u);
      }
    }
    float m_new = m_run;
#pragma unroll
    for (int i = 0; i < NL; ++i) m_new = fmaxf(m_new, x[i]);
    const float m_safe = m_new == kNegInf ? 0.f : m_new;
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_safe);
    float pr[NL];
    float psum = 0.f;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      pr[i] = __builtin_amdgcn_exp2f(x[i] - m_safe);
      psum += pr[i];
    }
    l_run = fmaf(l_run, alpha, psum);
    const bool changed = m_new != m_run;
    m_run = m_new;
    if (__builtin_amdgcn_ballot_w64(changed) != 0ull) rescale_acc<G, GP, EPL>(acc, alpha);
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      float ve[EPL];
#pragma unroll
      for (int e = 0; e < EPL; ++e) ve[e] = vec_elem<T>(vb[i], e);
      accumulate_pv<G, GP, EPL>(acc, pr[i], ve);
    }
  }
};

template <typename T, int D, int G, int WAVES, bool FUSED, bool SHARED, int ARRIVALS = kMergeLaunch>
__global__ __launch_bounds__(WAVES * kWave) void paged_decode_kernel(
    const int32_t* seq_lens, const int32_t* block_table, const void* q, const void* k_pool_p, const void* v_pool_p,
    const int num_kv_heads, const int max_blocks, const uint32_t inv_heads, const uint32_t shape, const DecodeParams) {
  static_assert(!(FUSED && SHARED), "the fused append is per-head only");
  using TL = Tile<T, D, G>;
  constexpr int DEPTH = kDepth;
  constexpr int EPL = TL::EPL, LPR = TL::LPR, NLT = TL::NLT, TT = TL::TT, GP = TL::GP;
  constexpr int GBITS = ilog2(GP);

  __shared__ WaveStates<WAVES, GP, D> sm;

  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int u = lane % LPR;    // which 16-byte slice of the token row
  const int grp = lane / LPR;  // which token row of a wave-load
  const int c_lane = bit_reverse<GBITS>(lane & (GP - 1));

  const int log2_block = shape_log2_block(shape), g_real = shape_group(shape), splits = shape_splits(shape);
  const int num_q_heads = num_kv_heads * g_real;
  const Place at = decode_place(shape, num_kv_heads, inv_heads);
  const int row = at.row, split = at.split, s = at.seq, hk = at.head;
  // SHARED: one table row per sequence; a page holds [B][Hk][D], so consecutive tokens of this head are
  // Hk rows apart and a lane's offset inside a wave-load carries the head
  const int32_t* bt = block_table + (int64_t)(SHARED ? s : row) * max_blocks;

  // ---- prologue: page lookups and the length first, then K and V, and everything else behind them ----
  // The row's tiles are dealt out round-robin: tile t belongs to split (t / WAVES) % splits, wave t % WAVES.  A
  // wave's first tile is therefore the same whatever the row length, and the lookup of its page travels
  // together with the length itself instead of waiting for it (one dependent round trip to memory less).
  const int stride = splits * WAVES;
  const int first = split * WAVES + wave;
  int phys[DEPTH];
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) phys[d] = TL::lookup(first + d * stride, bt, max_blocks, log2_block);
  const int len_pool = seq_lens[s];  // tokens that are read from the pool
  __builtin_amdgcn_sched_barrier(0);

  const int row_vecs = SHARED ? LPR * num_kv_heads : LPR;
  const int lane_vec = SHARED ? (grp * num_kv_heads + hk) * LPR + u : lane;
  const T* k_pool = static_cast<const T*>(k_pool_p);
  const T* v_pool = static_cast<const T*>(v_pool_p);
  const int ntiles = (len_pool + TT - 1) >> ilog2(TT);
  // Loads are issued unconditionally, past the row's end all lanes fetch the pool's first 16 bytes: the order of outstanding
  // loads is known at compile time, so that waiting for the oldest tile leaves the younger ones in flight.
  const auto issue = [&](uint4(&kb)[NLT], uint4(&vb)[NLT], int tile, int ph) {
    // (an unused entry, -1, is replaced by page 0: its tokens are masked, so any address inside the pool will do)
    const int64_t there = (((int64_t)(ph < 0 ? 0 : ph) << log2_block) + ((tile * TT) & ((1 << log2_block) - 1))) * row_vecs;
    const bool in = tile < ntiles;
    TL::issue(kb, vb, in ? there : 0, k_pool, v_pool, in ? lane_vec : 0, in ? row_vecs : 0);
  };
  uint4 kb[DEPTH][NLT], vb[DEPTH][NLT];
#pragma unroll
  for (int d = 0; d < DEPTH - 1; ++d) issue(kb[d], vb[d], first + d * stride, phys[d]);
  __builtin_amdgcn_sched_barrier(0);
  // query slices: slot i holds head (i ^ c_lane) of this KV head's group (heads past the group: head 0 again, never written)
  QSlice<T> qs[GP];
#pragma unroll
  for (int i = 0; i < GP; ++i) {
    const int head = i ^ c_lane;
    const int head_ld = head < g_real ? head : 0;
    qs[i].load(static_cast<const T*>(q) + ((int64_t)s * num_q_heads + hk * g_real + head_ld) * D + u * EPL);
  }
  const DecodeParams p = decode_params(phys[0] ^ ntiles);
  uint4 nk[1], nv[1];  // FUSED: the new token's K/V rows, held by the first lane group of every wave
  if constexpr (FUSED) {
    const int64_t vec = (int64_t)row * LPR + u;
    nk[0] = load_vec(p.new_k, vec);
    nv[0] = load_vec(p.new_v, vec);
  }
  // FUSED: requests for what the append needs, issued now and used at the end
  const bool appender = FUSED && split == splits - 1 && wave == WAVES - 1;  // wave-uniform
  const int jb = len_pool >> log2_block;
  int ap_freed = -1, ap_used = 0, ap_page = -1;
  if constexpr (FUSED) {
    if (appender) {
      ap_freed = p.freed_phys[row];
      ap_used = p.spare_used[row];
      ap_page = bt[jb < 0 ? 0 : jb < max_blocks ? jb : max_blocks - 1];
    }
  }

  float m_run = kNegInf;  // running max of head c_lane over this lane's stream of tokens
  float l_run = 0.f;
  float acc[G][EPL];
#pragma unroll
  for (int h = 0; h < G; ++h)
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[h][e] = 0.f;

  // This wave's tiles are first, first + stride, ... < ntiles.  DEPTH register buffers: while a tile is consumed, the next
  // DEPTH - 1 are in flight.
  int ph_next = phys[DEPTH - 1];
  for (int tile0 = first; tile0 < ntiles; tile0 += DEPTH * stride) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      const int tile = tile0 + d * stride, ahead = tile + (DEPTH - 1) * stride;
      issue(kb[(d + DEPTH - 1) % DEPTH], vb[(d + DEPTH - 1) % DEPTH], ahead, ph_next);
      ph_next = TL::lookup(ahead + stride, bt, max_blocks, log2_block);
      if (tile < ntiles)
        TL::template compute<NLT>(kb[d], vb[d], tile * TT, len_pool, grp, p.scale_log2e, qs, m_run, l_run, acc);
    }
  }

  if constexpr (FUSED) {  // the new token is token number len_pool of the row: wave 0 of the last split attends to it
    if (split == splits - 1 && wave == 0)
      TL::template compute<1>(nk, nv, len_pool, len_pool + (grp == 0 ? 1 : 0), 0, p.scale_log2e, qs, m_run, l_run, acc);
  }

  // ---- merge: the token streams of a wave (lanes that hold the same slice) in registers, then the waves through LDS -----
  const float m_wave = streams_max<LPR>(m_run);
  const float f = __builtin_amdgcn_exp2f(m_run - (m_wave == kNegInf ? 0.f : m_wave));
  const float l_wave = streams_sum<LPR>(l_run * f);
  rescale_acc<G, GP, EPL>(acc, f);
  int me = (int)threadIdx.x;  // the lane's place is worked out again: registers kept for it up to here would cost workgroups in flight
  asm("" : "+v"(me));
  me &= kWave - 1;
  if (me < GP) sm.ml[wave][bit_reverse<GBITS>(me)] = make_float2(m_wave, l_wave);
  using Parts = StreamParts<LPR, EPL>;
#pragma unroll
  for (int h = 0; h < G; ++h) {
    float part[Parts::kPart];
    Parts::sum(acc[h], part);
    float* dst = &sm.acc[wave][h][me % LPR * EPL + me / Parts::kLanes * Parts::kPart];
    if (LPR >= 16 || (me & 8) == 0) {
      if constexpr (Parts::kPart == 2) {
        *reinterpret_cast<float2*>(dst) = make_float2(part[0], part[1]);
      } else {
        static_assert(Parts::kPart == 1, "elements of a row of lanes");
        *dst = part[0];
      }
    }
  }
  __syncthreads();
  if constexpr (ARRIVALS != kMergeLaunch)
    merge_arrived<T, ARRIVALS == kTagged>(sm, p, row, split, splits, g_real);
  else
    merge_waves<T>(sm, p, row, split, splits, g_real);

  // FUSED: the first lane group of the last split's last wave stores the new token into the pool, linking a new page first when
  // the tail page is full.  Last of all, so that nothing of this launch waits for a store.
  if constexpr (FUSED) {
    if (appender) {
      const int slot = len_pool & ((1 << log2_block) - 1);
      if (len_pool >= 0 && jb < max_blocks) {  // a length outside the table row is a caller error: touch nothing
        const int page = slot == 0 ? link_page(p, const_cast<int32_t*>(bt), jb, row, ap_freed, ap_used, lane) : ap_page;
        if (page >= 0 && grp == 0) {
          const int64_t vec = (((int64_t)page << log2_block) + slot) * LPR + u;
          reinterpret_cast<uint4*>(const_cast<void*>(k_pool_p))[vec] = nk[0];
          reinterpret_cast<uint4*>(const_cast<void*>(v_pool_p))[vec] = nv[0];
        }
      }
      if (hk == 0 && lane == 0) p.seq_lens_out[s] = len_pool + 1;
    }
  }
  // The placeholder loads behind a wave's last tile are still on their way during the merge; their registers are in use until
  // here, so that nothing there waits for them but the arrival of splits that are counted or tagged (merge_arrived).
#pragma unroll
  for (int d = 0; d < DEPTH; ++d)
#pragma unroll
    for (int i = 0; i < NLT; ++i) {
      asm volatile("" : : "v"(kb[d][i].x), "v"(kb[d][i].y), "v"(kb[d][i].z), "v"(kb[d][i].w));
      asm volatile("" : : "v"(vb[d][i].x), "v"(vb[d][i].y), "v"(vb[d][i].z), "v"(vb[d][i].w));
    }
}

// Merge the split partials of one (sequence, query head), D / 64 elements a lane: by one wave where their number is one that may be
// counted, in the order that has there; more are shared by four waves and more than 32 by eight, whose states meet in LDS (attention and
// merge out of a HIP graph, one wave / four / eight, us: 24 heads of D = 64 in 19 splits 8.7 / 7.3 / 7.6, 64 of D = 128 in 16 8.5 / 7.9 / 8.1, 32
// in 32 9.6 / 8.1 / 8.1, 32 of D = 64 in 36 12.7 / 10.2 / 9.9, four of D = 128 in 64 14.8 / 9.5 / 8.8; nine to twelve, one wave with all records
// asked for at once / four, attention out of calls, 25 rows of D = 128 x 4096 in ten 12.44 / 12.66, 21 in twelve 11.18 / 11.39, 28 x 2048 in nine
// 8.86 / 8.99, fp32, 24 x 2500 of D = 64 in ten 8.46 / 8.43; up to eight no difference).  What a launch of it costs besides is the launch and one round trip to the records, which lie together for a row
// ([row][split][head]: with the heads of all rows under each split 0.4 us more for 32 rows of D = 128 in eight splits, 1.1 us for 16 rows
// in 16).  The grid: the query heads of a row side by side, one row a grid row; with kMergeXcd, wherever the attention kernel keeps a row
// on one XCD, eight rows a grid row, so that a row's records are read on the XCD that wrote them (append, attention and merge out of a HIP
// graph, side by side / so, one wave each: D = 128, four query heads a KV head, 8 rows x 4096 8.8 / 8.0 us, 16 x 5280 12.4 / 11.4, 32 x
// 4096 14.6 / 13.95, 32 x 8192 24.3 / 23.9, 264 x 4096 94.2 / 93.8; D = 64 7.7 / 6.9, 9.3 / 8.4, 9.5 / 9.0, 13.9 / 13.6, 51.5 / 51.2; one
// query head: the same order); kMergeLinear: more rows than a grid has, divided.
enum { kMergeLinear, kMergeRows, kMergeXcd };
template <typename T, int D, bool CLEAR, int WAVES>
__global__ __launch_bounds__(WAVES * kWave) void paged_decode_reduce_kernel(const float* __restrict__ partials, void* __restrict__ out,
                                                                            int g_real, int splits, int order, void* next_out) {
  constexpr int E = D / kWave;
  const int x = (int)blockIdx.x, y = (int)blockIdx.y;
  const int row = order == kMergeLinear ? x / g_real : order == kMergeXcd ? y * 8 + (x & 7) : y;
  const int h = order == kMergeLinear ? x - row * g_real : order == kMergeXcd ? x >> 3 : x;
  const int wave = WAVES == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int d = (int)(threadIdx.x % kWave) * E;
  const float* base = partials + ((int64_t)row * splits * g_real + h) * (D + 2);
  const int64_t stride = (int64_t)g_real * (D + 2);
  const auto read = [&](int split, float2& ml, float (&v)[E]) {
    const float* record = base + split * stride;
    ml = *reinterpret_cast<const float2*>(record + D);
    if constexpr (E == 2) {
      const float2 pair = *reinterpret_cast<const float2*>(record + d);
      v[0] = pair.x, v[1] = pair.y;
    } else {
      v[0] = record[d];
    }
  };
  float o[E] = {};
  if constexpr (WAVES == 1) {
    // all on their way before the first is used
    constexpr int kFours = kMostArrivals / 4;
    static_assert(kMostArrivals % 4 == 0, "fours");
    float2 ml[kFours][4];
    float v[kFours][4][E];
    float m = kNegInf, l = 0.f;
#pragma unroll
    for (int i = 0; i < kFours; ++i)
      if (i == 0 || 4 * i < splits) {
#pragma unroll
        for (int j = 0; j < 4; ++j) read(4 * i + j < splits ? 4 * i + j : splits - 1, ml[i][j], v[i][j]);
      }
#pragma unroll
    for (int i = 0; i < kFours; ++i)
      if (i == 0 || 4 * i < splits) add_splits(4 * i, splits, ml[i], v[i], m, l, o);
#pragma unroll
    for (int e = 0; e < E; ++e) o[e] = l > 0.f ? o[e] / l : 0.f;
  } else {
    // online: all loads are independent of the running state, so they overlap
    float mm = kNegInf, l = 0.f;
    const auto add = [&](const float2& ml, const float (&v)[E]) {
      const float m_new = fmaxf(mm, ml.x);
      // all splits so far empty (m_new = -inf): reference 0, else -inf - -inf = NaN
      const float ms = m_new == kNegInf ? 0.f : m_new;
      const float w_old = __builtin_amdgcn_exp2f(mm - ms), w_new = __builtin_amdgcn_exp2f(ml.x - ms);
      l = fmaf(l, w_old, ml.y * w_new);
#pragma unroll
      for (int e = 0; e < E; ++e) o[e] = fmaf(o[e], w_old, v[e] * w_new);
      mm = m_new;
    };
#pragma unroll 4
    for (int split = wave; split < splits; split += WAVES) {
      float2 ml;
      float v[E];
      read(split, ml, v);
      add(ml, v);
    }
    __shared__ float sm[WAVES][D + 2];
    if (wave > 0) {
#pragma unroll
      for (int e = 0; e < E; ++e) sm[wave][d + e] = o[e];
      if (d == 0) sm[wave][D] = mm, sm[wave][D + 1] = l;
    }
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int w = 1; w < WAVES; ++w) {
      float v[E];
#pragma unroll
      for (int e = 0; e < E; ++e) v[e] = sm[w][d + e];
      add(make_float2(sm[w][D], sm[w][D + 1]), v);
    }
#pragma unroll
    for (int e = 0; e < E; ++e) o[e] = l > 0.f ? o[e] / l : 0.f;
  }
  const int64_t off = ((int64_t)row * g_real + h) * D + d;
  // (the counts of the launch behind this one: one for every 128 elements of a row)
  if (CLEAR && (h * D + d) % (2 * kWave) == 0) *arrival_count<T>(next_out, off / 2) = 0u;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    if constexpr (sizeof(T) == 4)
      static_cast<float*>(out)[off + e] = o[e];
    else
      static_cast<uint16_t*>(out)[off + e] = f32_to_bf16(o[e]);
  }
}

template <typename T, int D, int G, int WAVES>
hipError_t launch_waves(const DecodeArgs& a, hipStream_t stream) {
  DecodeKernelArgs k;
  dim3 blocks;
  if (!decode_kernel_args(a, &k, &blocks)) return hipErrorInvalidValue;
  const dim3 threads(WAVES * kWave);
  if (a.shared && a.new_k != nullptr) return hipErrorInvalidValue;
  if (a.counted || a.tagged) {
    if constexpr (one_part_a_wave<next_pow2(G), D, WAVES>)
      return launch_decode(a.counted             ? paged_decode_kernel<T, D, G, WAVES, true, false, kCounted>
                           : a.new_k != nullptr ? paged_decode_kernel<T, D, G, WAVES, true, false, kTagged>
                                                : paged_decode_kernel<T, D, G, WAVES, false, false, kTagged>, blocks, threads, stream, k);
    return hipErrorInvalidValue;
  }
  const auto kernel = a.shared             ? paged_decode_kernel<T, D, G, WAVES, false, true>
                      : a.new_k != nullptr ? paged_decode_kernel<T, D, G, WAVES, true, false>
                                           : paged_decode_kernel<T, D, G, WAVES, false, false>;
  return launch_decode(kernel, blocks, threads, stream, k);
}
template <typename T, int D, int G>
hipError_t launch_one(const DecodeArgs& a, hipStream_t stream) {
  return a.waves == 8 ? launch_waves<T, D, G, 8>(a, stream) : launch_waves<T, D, G, 4>(a, stream);
}

template <int D>
hipError_t launch_group(const DecodeArgs& a, hipStream_t stream) {
  switch (a.num_q_heads / a.num_kv_heads) {
    case 1: return launch_one<float, D, 1>(a, stream);
    case 2: return launch_one<float, D, 2>(a, stream);
    case 3: return launch_one<float, D, 3>(a, stream);
    case 4: return launch_one<float, D, 4>(a, stream);
    case 5: case 6: case 7: case 8: return launch_one<float, D, 8>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

template <typename T, int D>
void launch_reduce(const DecodeArgs& a, hipStream_t stream) {
  const int64_t rows = (int64_t)a.num_seqs * a.num_kv_heads;
  const int g = a.num_q_heads / a.num_kv_heads;
  const bool xcd = a.xcd_map && rows % 8 == 0;
  const int64_t grid_rows = xcd ? rows / 8 : rows;
  const int order = grid_rows > 65535 ? kMergeLinear : xcd ? kMergeXcd : kMergeRows;
  const dim3 blocks = order == kMergeLinear ? dim3((unsigned)(rows * g)) : dim3((unsigned)(xcd ? 8 * g : g), (unsigned)grid_rows);
  const bool clear = a.next_out != nullptr;
  const int waves = a.splits > 32 ? 8 : a.splits > most_arrivals(g) ? 4 : 1;
  // (counts are cleared for no more splits than one wave merges)
  const auto kernel = waves == 8   ? paged_decode_reduce_kernel<T, D, false, 8>
                      : waves == 4 ? paged_decode_reduce_kernel<T, D, false, 4>
                      : clear      ? paged_decode_reduce_kernel<T, D, true, 1>
                                   : paged_decode_reduce_kernel<T, D, false, 1>;
  hipLaunchKernelGGL(kernel, blocks, dim3(waves * kWave), 0, stream, a.partials, a.out, g, a.splits, order, a.next_out);
}

}  // namespace

size_t decode_partials_bytes(int num_seqs, int num_q_heads, int head_dim, int splits) {
  if (splits <= 1) return 0;
  return (size_t)num_seqs * num_q_heads * splits * (head_dim + 2) * sizeof(float);
}

hipError_t launch_paged_decode(const DecodeArgs& a, hipStream_t stream) {
  if (a.head_dim != 64 && a.head_dim != 128) return hipErrorInvalidValue;
  const bool d64 = a.head_dim == 64;
  hipError_t e;
  if (!a.is_bf16)
    e = d64 ? launch_group<64>(a, stream) : launch_group<128>(a, stream);
  else if (a.vector)
    e = d64 ? launch_one<bf16_t, 64, 1>(a, stream) : launch_one<bf16_t, 128, 1>(a, stream);
  else
    e = launch_paged_decode_bf16(a, stream);
  if (e != hipSuccess || a.splits == 1 || a.counted || a.tagged) return e;
  if (a.is_bf16)
    d64 ? launch_reduce<bf16_t, 64>(a, stream) : launch_reduce<bf16_t, 128>(a, stream);
  else
    d64 ? launch_reduce<float, 64>(a, stream) : launch_reduce<float, 128>(a, stream);
  return hipGetLastError();
}

}  // namespace pe
