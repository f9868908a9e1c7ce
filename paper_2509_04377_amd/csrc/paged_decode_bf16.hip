// Paged decode attention for bfloat16 caches (Eq. 1 for one new query per sequence; Alg. 3 "PagedAttention(Q,K,V)"):
// QK and PV on the matrix cores.
//
// A workgroup owns one split of one (sequence, KV head) row: the row's 16-token tiles are dealt out round-robin, tile
// t to split (t / WAVES) % splits, wave t % WAVES, so a wave's first tile does not depend on the row length.  K and V
// go from memory to registers and from there into the matrix instructions; nothing is staged in LDS (every element
// is used by one wave only).  Both operands are read the way they lie in memory, 16 bytes a lane and 64 or more
// consecutive bytes for four neighbouring lanes; the index maps below make the products come out right.
//
// Lane l = 16*g + m, m = 4*q + r (the roles of q and r: row block and class).  LPR = D/8 lanes cover a token row,
// TPL = 64/LPR token rows make a wave-load, a tile is NL = 16/TPL wave-loads of K and of V.
//
//   QK (16x16x32; A = K, B = queries).  For one wave-load lane l holds 16-byte slice 4*b + r of a token, b being the
//   64-byte block of the row: D = 128: token q, block g; D = 64: token 2*q + g/2, block g%2.  A row m of A thus holds
//   every fourth slice of its token(s) (class r) and the products run over the blocks.  Column n = 4*h + c of B holds
//   the class-c slices of query head h, so C[m][n] is the part of <k, q_h> in class c where c == r and meaningless
//   elsewhere; the logit is the sum of the four meaningful entries, which sit in the four lanes of a quad (one register
//   each): a select and two quad-permuted adds.  D = 64: a row of A carries two tokens (g/2); two products with the
//   other token's blocks zeroed in B tell them apart.  Afterwards lane l holds, for head n/4 = m/4 (the same in the
//   four lanes of a quad), the logits of tokens TPL*i + NT*g + t of the tile, i < NL, t < NT: NL*NT = 4 values.
//
//   PV (16x16x16; A = V transposed, B = probabilities).  Lane l holds slice l % LPR of token TPL*i + l/LPR of V, so
//   element e of the slices of the NL wave-loads, brought together with byte permutes, is a column of A whose
//   contraction index is exactly the token order in which the lane holds its probabilities: the logits' registers
//   are the B operand as they stand.  (D = 64: row m of A holds tokens of parity m/8 only; the other parity's
//   places are zero, and the two halves are added at the end.)  Probabilities keep their 32 bits: the four lanes of
//   a quad hold the same value, and each turns one term of its exact decomposition into three bfloat16 terms (the
//   fourth a zero) into the operand, so the columns of C are partial sums that are added once, at the end of the row.
//
// Softmax: online, base 2, one reference value m per head and wave.  The reference is set kGrow above the largest logit
// and moves again only when a logit exceeds it (the result does not depend on the reference), so that the rescaling of
// the accumulators, and the exchange between the lane groups, are rare.  No probability exceeds 1: the accumulators
// overflow no earlier than the sums that define the result do (a reference that lags behind, with probabilities of up to
// 2^kGrow, lost finite results from |V| = 2^125 on).
//
// At the end the quads' columns are added, the four waves' (m, l, acc) merged through LDS behind one barrier, and the
// normalised output (or, with more than one split, the partial record) is written.
//
// FUSED also performs the harness append of the same decode iteration: the wave that owns the tile of the new token
// puts the token's K/V rows into its registers in place of what it loaded, links a new page first when the tail page
// is full, and stores the rows into the pool behind its last tile (a store in flight would turn every wait for a load
// into a full wait); the new lengths go to a second array (the caller swaps the two), so no workgroup can see a
// length that another one has already bumped.
//
// SHARED reads the head-shared cache layout: one table row per sequence and pages of [B][Hk][D], so the token rows of
// this workgroup's head are Hk rows apart.  (FUSED there took the place of an append launch in front of the attention:
// 32 sequences x 8 heads x 2048 tokens 45.7 us a layer in two launches, 43.6 in one; 8 x 4 x 2304 13.9 and 11.1.)
#include "pe_decode_common.h"

namespace pe {
namespace {

constexpr float kNegInf = -__builtin_inff();
constexpr float kGrow = 3.f;   // how far above the largest logit (log2) the reference is set
constexpr int kTile = 16;      // tokens per tile

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) short s16x4_t;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

template <int CTRL>
__device__ __forceinline__ float quad_perm_add(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
// Sum over the four lanes of a quad, in every lane.
__device__ __forceinline__ float quad_sum(float v) { return quad_perm_add<0x4E>(quad_perm_add<0xB1>(v)); }

// Element c (0..3) of a vector, c per lane: b0 = c & 1, b1 = c & 2.
__device__ __forceinline__ float pick4(const f32x4_t& v, bool b0, bool b1) {
  const float lo = b0 ? v[1] : v[0];
  const float hi = b0 ? v[3] : v[2];
  return b1 ? hi : lo;
}

// One wave's view of a tile.  HG: groups of four query heads (G <= 4: 1, G <= 8: 2).
template <int D, int HG>
struct Tile {
  static constexpr int LPR = D / 8;
  static constexpr int TPL = kWave / LPR;
  static constexpr int NL = kTile / TPL;
  static constexpr int NT = 4 / NL;  // tokens that a row of A carries (1 or 2)

  const u32x4_t* k_pool;
  const u32x4_t* v_pool;
  int row_vecs;        // 16-byte vectors between consecutive tokens of this head
  int k_off, v_off;    // this lane's offset inside a wave-load of K and of V
  int k_tok, v_tok;    // and the token of the wave-load it belongs to
  int g;
  bool b0, b1;         // bits of the class c = lane & 3
  uint32_t term1, term2, term3;     // all ones in the upper half for classes >= 1, 2, 3
  uint32_t sel_even, sel_odd;       // D = 64: byte selectors that put an element into its parity's place

  __device__ __forceinline__ void issue(u32x4_t (&buf)[NL], const u32x4_t* pool, int64_t base, int off) const {
#pragma unroll
    for (int i = 0; i < NL; ++i) buf[i] = __builtin_nontemporal_load(pool + base + i * TPL * row_vecs + off);
  }

  // Token (inside the tile) of logit j of this lane.
  __device__ __forceinline__ int token_of(int j) const { return TPL * (j / NT) + NT * g + j % NT; }

  __device__ __forceinline__ void logits(const u32x4_t (&kb)[NL], const bf16x8_t (&qop)[HG][NT], float scale,
                                         float (&x)[HG][4]) const {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
#pragma unroll
      for (int hg = 0; hg < HG; ++hg) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
          const f32x4_t c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kb[i]), qop[hg][t], zero,
                                                                    0, 0, 0);
          x[hg][i * NT + t] = quad_sum(pick4(c, b0, b1)) * scale;
        }
      }
    }
  }

  // The same in two steps, with room for something between them: the products, and the logits from them.
  __device__ __forceinline__ void products(const u32x4_t (&kb)[NL], const bf16x8_t (&qop)[HG][NT], f32x4_t (&c)[NL][HG][NT]) const {
#pragma unroll
    for (int i = 0; i < NL; ++i)
#pragma unroll
      for (int hg = 0; hg < HG; ++hg)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
          c[i][hg][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kb[i]), qop[hg][t], zero, 0, 0, 0);
        }
  }
  __device__ __forceinline__ void logits_of(const f32x4_t (&c)[NL][HG][NT], float scale, float (&x)[HG][4]) const {
#pragma unroll
    for (int i = 0; i < NL; ++i)
#pragma unroll
      for (int hg = 0; hg < HG; ++hg)
#pragma unroll
        for (int t = 0; t < NT; ++t) x[hg][i * NT + t] = quad_sum(pick4(c[i][hg][t], b0, b1)) * scale;
  }

  // Move the reference m_run of a head group above the logits of this tile, where one of them exceeds it.  m_ref is the
  // same, but finite before the first logit (-inf - -inf is no number).
  static __device__ __forceinline__ void regrow(float mx, float& m_run, float& m_ref, float& l_run, f32x4_t (&acc)[8]) {
    mx = rows_max(mx);
    const float m_new = mx > m_run ? mx + kGrow : m_run;
    const float ref = m_new == kNegInf ? 0.f : m_new;
    const float alpha = __builtin_amdgcn_exp2f(m_run - ref);
    l_run *= alpha;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] *= alpha;
    m_run = m_new;
    m_ref = ref;
  }

  // Probabilities of this lane's four tokens, their sum, and the operand of PV.
  __device__ __forceinline__ s16x4_t probs(const float (&x)[4], float m_ref, float& l_run) const {
    uint32_t t[4];
    float sum = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float p = __builtin_amdgcn_exp2f(x[j] - m_ref);
      sum += p;
      // the exact terms of p = t1 + t2 + t3: what is left after class-many truncations to bfloat16
      p -= __uint_as_float(__float_as_uint(p) & term1);
      p -= __uint_as_float(__float_as_uint(p) & term2);
      p -= __uint_as_float(__float_as_uint(p) & term3);
      t[j] = __float_as_uint(p);
    }
    l_run += sum;
    const u32x2_t packed = {__builtin_amdgcn_perm(t[1], t[0], 0x07060302u), __builtin_amdgcn_perm(t[3], t[2], 0x07060302u)};
    return __builtin_bit_cast(s16x4_t, packed);
  }

  // Element e of the tile's V slices as an operand (contraction over the tile's tokens).
  __device__ __forceinline__ s16x4_t v_operand(const u32x4_t (&vb)[NL], int e) const {
    u32x2_t a;
    if constexpr (D == 128) {
      const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
      a[0] = __builtin_amdgcn_perm(vb[1][e >> 1], vb[0][e >> 1], sel);
      a[1] = __builtin_amdgcn_perm(vb[3][e >> 1], vb[2][e >> 1], sel);
    } else {
      const uint32_t sel = (e & 1) ? sel_odd : sel_even;
      a[0] = __builtin_amdgcn_perm(0u, vb[0][e >> 1], sel);
      a[1] = __builtin_amdgcn_perm(0u, vb[1][e >> 1], sel);
    }
    return __builtin_bit_cast(s16x4_t, a);
  }

  __device__ __forceinline__ void accumulate(const u32x4_t (&vb)[NL], const s16x4_t (&pop)[HG], f32x4_t (&acc)[HG][8]) const {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const s16x4_t a = v_operand(vb, e);
#pragma unroll
      for (int hg = 0; hg < HG; ++hg) acc[hg][e] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, pop[hg], acc[hg][e], 0, 0, 0);
    }
  }
};

// Table entry of the page of tile `tile` of a row (scalar load).  The index is clamped to the row; nothing here depends on
// the row length.
__device__ __forceinline__ int lookup(const int32_t* bt, int tile, int max_blocks, int log2_block) {
  int pi = (tile * kTile) >> log2_block;
  pi = pi < max_blocks ? pi : max_blocks - 1;
  return __builtin_amdgcn_readfirstlane(bt[pi]);
}

template <int D, int HG, int WAVES, int DEPTH, bool FUSED, bool SHARED, int ARRIVALS = kMergeLaunch>
// (the 2 asks for two waves per SIMD at least, i.e. at most 256 registers: the compiler then keeps the accumulators in
// vector registers instead of moving them to and from accumulation registers in every step.  The 3, at most 168: head-shared,
// appending, with D = 64 and more than four query heads it would take 170, and 176 rows x 2000 23.9 us instead of 21.6 (192 ragged
// rows of up to 8192 take 56.3 with three waves, 53.7 with two); the per-head form stays at two: there 832 rows x 3680 take 130 us,
// with three 145)
__global__ __launch_bounds__(WAVES * kWave, D == 64 && HG == 2 && DEPTH == 1 && FUSED && SHARED ? 3 : 2)
void paged_decode_bf16_kernel(
    const int32_t* seq_lens, const int32_t* block_table, const void* q, const void* k_pool, const void* v_pool,
    const int num_kv_heads, const int max_blocks, const uint32_t inv_heads, const uint32_t shape, const DecodeParams) {
  using TL = Tile<D, HG>;
  constexpr int LPR = TL::LPR, TPL = TL::TPL, NL = TL::NL, NT = TL::NT;
  constexpr int GH = 4 * HG;  // heads computed; g_real of them exist
  // The next K goes out between the products and the logits where that is what a tile waits for: one tile in flight, short wave
  // loads, twice the arithmetic (512 rows of up to 4000 tokens of D = 64, eight query heads 59.8 us behind the logits, 57.6 so; 384 x
  // 1024 19.9 / 19.4).  It takes registers that the other forms do not have.
  constexpr bool kEarlyK = D == 64 && HG == 2 && DEPTH == 1 && !FUSED && !SHARED;

  __shared__ WaveStates<WAVES, GH, D> sm;

  const int log2_block = shape_log2_block(shape), g_real = shape_group(shape), splits = shape_splits(shape);
  const int num_q_heads = num_kv_heads * g_real;
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int g = lane >> 4, m = lane & 15, c = lane & 3;

  const Place at = decode_place(shape, num_kv_heads, inv_heads);
  const int row = at.row, split = at.split, s = at.seq, hk = at.head;
  const int table_row = SHARED ? s : row;
  const int32_t* bt = block_table + (int64_t)table_row * max_blocks;

  // ---- prologue: everything that does not depend on the row length is requested first --------------
  const int stride = splits * WAVES;
  const int first = split * WAVES + wave;
  int phys[DEPTH + 1];
#pragma unroll
  for (int d = 0; d <= DEPTH; ++d) phys[d] = lookup(bt, first + d * stride, max_blocks, log2_block);
  const int len_pool = seq_lens[s];                                // tokens that are read from the pool
  const int len = FUSED ? len_pool + 1 : len_pool;  // tokens attended to
  __builtin_amdgcn_sched_barrier(0);  // (what follows, some sixty instructions, runs while they travel)

  TL tl;
  tl.k_pool = static_cast<const u32x4_t*>(k_pool);
  tl.v_pool = static_cast<const u32x4_t*>(v_pool);
  tl.row_vecs = SHARED ? LPR * num_kv_heads : LPR;
  tl.g = g;
  tl.b0 = (c & 1) != 0;
  tl.b1 = (c & 2) != 0;
  tl.term1 = c >= 1 ? 0xffff0000u : 0u;
  tl.term2 = c >= 2 ? 0xffff0000u : 0u;
  tl.term3 = c >= 3 ? 0xffff0000u : 0u;
  const bool tp = m >= 8;  // D = 64: token parity of this lane's V rows
  tl.sel_even = tp ? 0x01000c0cu : 0x0c0c0100u;
  tl.sel_odd = tp ? 0x03020c0cu : 0x0c0c0302u;
  const int block = D == 128 ? g : (g & 1);
  const int k_slice = 4 * block + c;
  const int v_slice = lane % LPR;
  tl.k_tok = D == 128 ? (m >> 2) : 2 * (m >> 2) + (g >> 1);
  tl.v_tok = lane / LPR;
  tl.k_off = tl.k_tok * tl.row_vecs + (SHARED ? hk * LPR : 0) + k_slice;
  tl.v_off = tl.v_tok * tl.row_vecs + (SHARED ? hk * LPR : 0) + v_slice;

  const int ntiles = (len + kTile - 1) >> ilog2(kTile);
  const int block_mask = (1 << log2_block) - 1;

  // This wave's tiles are first, first + stride, ... < ntiles.  DEPTH tiles are in flight: as soon as the K (V) registers of
  // a tile have been used, the K (V) loads of the tile DEPTH further on go out into them.  Loads are issued
  // unconditionally, past the end all lanes fetch the same 16 bytes: the order of outstanding loads is known at
  // compile time, so that waiting for the oldest leaves the younger ones in flight.
  // (an unused entry, -1, is replaced by page 0: its tokens are masked, so any address inside the pool will do)
  const auto base_of = [&](int tile, int ph) {
    return (((int64_t)(ph < 0 ? 0 : ph) << log2_block) + ((tile * kTile) & block_mask)) * tl.row_vecs;
  };
  DecodeParams p;
  u32x4_t nk = {0u, 0u, 0u, 0u}, nv = {0u, 0u, 0u, 0u};  // FUSED: the new token's K/V rows
  int ap_freed = -1, ap_used = 0;
  int ap_page = -1;  // the tail page, where it is not full
  bool owner = len_pool < 0 && first == 0;  // FUSED: this wave has the new token's tile (or the length is no length)
  float m_run[HG], m_ref[HG], l_run[HG];
  f32x4_t acc[HG][8];
#pragma unroll
  for (int hg = 0; hg < HG; ++hg) {
    m_run[hg] = kNegInf;
    m_ref[hg] = 0.f;
    l_run[hg] = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[hg][e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }
  u32x4_t kb[DEPTH][NL], vb[DEPTH][NL];
  if (__builtin_expect(first < ntiles, 1)) {
    u32x4_t q_raw[HG];
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      const bool more = first + d * stride < ntiles;
      const int64_t there = base_of(first + d * stride, phys[d]), base = more ? there : 0;
      tl.issue(kb[d], tl.k_pool, base, more ? tl.k_off : 0);
      if (d == 0) {
        // queries, needed together with the first K: column n = 4*h + c of the operand holds the class-c slices of head h
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int hg = 0; hg < HG; ++hg) {
          const int h = 4 * hg + (m >> 2);
          const int64_t head = (int64_t)s * num_q_heads + hk * g_real + (h < g_real ? h : 0);
          q_raw[hg] = static_cast<const u32x4_t*>(q)[head * LPR + k_slice];
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      tl.issue(vb[d], tl.v_pool, base, more ? tl.v_off : 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    p = decode_params(phys[0]);
    if constexpr (FUSED) {
      nk = static_cast<const u32x4_t*>(p.new_k)[(int64_t)row * LPR + k_slice];
      nv = static_cast<const u32x4_t*>(p.new_v)[(int64_t)row * LPR + v_slice];
      ap_freed = p.freed_phys[table_row];
      ap_used = p.spare_used[table_row];
      const int jb = len_pool >> log2_block;
      ap_page = bt[jb < 0 ? 0 : jb < max_blocks ? jb : max_blocks - 1];
    }
    bf16x8_t qop[HG][NT];
#pragma unroll
    for (int hg = 0; hg < HG; ++hg) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const u32x4_t zero = {0u, 0u, 0u, 0u};
        const bool in = 4 * hg + (m >> 2) < g_real && (NT == 1 || (g >> 1) == t);
        qop[hg][t] = __builtin_bit_cast(bf16x8_t, in ? q_raw[hg] : zero);
      }
    }
    int ph_next = phys[DEPTH];
    for (int tile0 = first; tile0 < ntiles; tile0 += DEPTH * stride) {
#pragma unroll
      for (int d = 0; d < DEPTH; ++d) {
        const int tile = tile0 + d * stride;   // past the end (an odd last one): every token is masked
        const int tok0 = tile * kTile;
        const bool tail = tok0 + kTile > len_pool;
        if (tail) {
          owner = owner || tok0 <= len_pool;
#pragma unroll
          for (int w = 0; w < NL; ++w) {
            if constexpr (FUSED) {  // the new token takes its place among the loaded ones
              if (tok0 + TPL * w + tl.k_tok == len_pool) kb[d][w] = nk;
              if (tok0 + TPL * w + tl.v_tok == len_pool) vb[d][w] = nv;
            }
            if constexpr (NT > 1) {  // junk K must not meet the zeros of its neighbour's operand (0 * NaN)
              if (tok0 + TPL * w + tl.k_tok >= len) kb[d][w] = u32x4_t{0u, 0u, 0u, 0u};
            }
          }
        }
        float x[HG][4];
        f32x4_t qk[NL][HG][NT];
        if constexpr (kEarlyK) {
          tl.products(kb[d], qop, qk);
        } else {
          tl.logits(kb[d], qop, p.scale_log2e, x);
        }
        const int ahead = tile + DEPTH * stride;
        const bool more = ahead < ntiles;
        const int64_t there = base_of(ahead, ph_next), base = more ? there : 0;
        ph_next = lookup(bt, ahead + stride, max_blocks, log2_block);
        tl.issue(kb[d], tl.k_pool, base, more ? tl.k_off : 0);
        if constexpr (kEarlyK) tl.logits_of(qk, p.scale_log2e, x);
        if (tail) {  // mask logits past the row's end, keep junk V out of the sum
#pragma unroll
          for (int hg = 0; hg < HG; ++hg)
#pragma unroll
            for (int j = 0; j < 4; ++j) x[hg][j] = tok0 + tl.token_of(j) < len ? x[hg][j] : kNegInf;
#pragma unroll
          for (int w = 0; w < NL; ++w)
            if (tok0 + TPL * w + tl.v_tok >= len) vb[d][w] = u32x4_t{0u, 0u, 0u, 0u};
        }
        float mx[HG];
        bool grow = false;
#pragma unroll
        for (int hg = 0; hg < HG; ++hg) {
          mx[hg] = fmaxf(fmaxf(x[hg][0], x[hg][1]), fmaxf(x[hg][2], x[hg][3]));
          grow = grow || mx[hg] > m_run[hg];
        }
        if (__builtin_amdgcn_ballot_w64(grow) != 0ull) {
#pragma unroll
          for (int hg = 0; hg < HG; ++hg) TL::regrow(mx[hg], m_run[hg], m_ref[hg], l_run[hg], acc[hg]);
        }
        s16x4_t pop[HG];
#pragma unroll
        for (int hg = 0; hg < HG; ++hg) pop[hg] = tl.probs(x[hg], m_ref[hg], l_run[hg]);
        tl.accumulate(vb[d], pop, acc);
        tl.issue(vb[d], tl.v_pool, base, more ? tl.v_off : 0);
      }
    }
  } else {
    p = decode_params(ntiles);
  }

  // ---- merge: columns of a quad, lane groups, then the waves through LDS -------------------------------
#pragma unroll
  for (int hg = 0; hg < HG; ++hg) {
    const float l = rows_sum(l_run[hg]);
    const int h = 4 * hg + (m >> 2);
    if (g == 0 && c == 0) {
      sm.ml[wave][h] = make_float2(m_run[hg], l);
    }
    // lane (g, 4*h + c) keeps row 4*g + c of C: elements 8*slice .. 8*slice + 7 of head h
    float o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      f32x4_t a = acc[hg][e];
#pragma unroll
      for (int r = 0; r < 4; ++r) a[r] = quad_sum(a[r]);
      o[e] = pick4(a, tl.b0, tl.b1);
      if constexpr (D == 64) o[e] = halves_sum(o[e]);  // the two token parities
    }
    if (D == 128 || g < 2) {
      float4* dst = reinterpret_cast<float4*>(&sm.acc[wave][h][(4 * g + c) * 8]);
      dst[0] = make_float4(o[0], o[1], o[2], o[3]);
      dst[1] = make_float4(o[4], o[5], o[6], o[7]);
    }
  }
  __syncthreads();
  if constexpr (ARRIVALS != kMergeLaunch)
    merge_arrived<bf16_t, ARRIVALS == kTagged>(sm, p, row, split, splits, g_real);
  else
    merge_waves<bf16_t>(sm, p, row, split, splits, g_real);

  if constexpr (FUSED) {
    // the wave whose tile holds the new token stores it into the pool; when the tail page is full it links a new page
    // first.  Last of all, so that nothing of this launch waits for a store.
    if (owner) {
      const int B = 1 << log2_block;
      const int slot = len_pool & (B - 1);
      const int jb = len_pool >> log2_block;
      if (len_pool >= 0 && jb < max_blocks) {  // a length outside the table row is a caller error: touch nothing
        // head-shared: a page that has to be linked first is head 0's to link and to fill for all heads, so that no
        // workgroup has to learn from another one which page it is
        const bool link = slot == 0;
        int page = ap_page;
        if (link) {
          page = ap_freed;
          if (!SHARED || hk == 0) page = link_page(p, const_cast<int32_t*>(bt), jb, table_row, ap_freed, ap_used, lane);
        }
        u32x4_t* k_to = static_cast<u32x4_t*>(const_cast<void*>(k_pool));
        u32x4_t* v_to = static_cast<u32x4_t*>(const_cast<void*>(v_pool));
        if (SHARED && link) {
          if (hk == 0 && page >= 0) {
            const int64_t to = ((int64_t)page << log2_block) * tl.row_vecs, from = (int64_t)s * tl.row_vecs;
            for (int i = lane; i < tl.row_vecs; i += kWave) {
              k_to[to + i] = static_cast<const u32x4_t*>(p.new_k)[from + i];
              v_to[to + i] = static_cast<const u32x4_t*>(p.new_v)[from + i];
            }
          }
        } else if (page >= 0) {
          const int64_t base = (((int64_t)page << log2_block) + slot) * tl.row_vecs + (SHARED ? hk * LPR : 0);
          // the lanes of the first token row of a wave-load hold the whole row between them
          if (tl.k_tok == 0) k_to[base + k_slice] = nk;
          if (tl.v_tok == 0) v_to[base + v_slice] = nv;
        }
      }
      if (hk == 0 && lane == 0) p.seq_lens_out[s] = len_pool + 1;
    }
  }
  // The loads behind a wave's last tiles are still on their way while the rows are merged.  Their registers are not to be given
  // to anything before (whatever is written to a register waits for the load into it): they are in use until here.  (The arrival of splits
  // that are counted or tagged waits for them all the same: merge_arrived.)
  if (first < ntiles) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d)
#pragma unroll
      for (int i = 0; i < NL; ++i) asm volatile("" : : "v"(kb[d][i]), "v"(vb[d][i]));
  }
}

// (the forms that the head-shared layout never takes, and that are never counted or tagged, are not built for it)
template <int D, int HG, int WAVES, int DEPTH>
hipError_t launch_one(const DecodeArgs& a, hipStream_t stream) {
  constexpr bool kShared = DEPTH == 1 || (WAVES == 4 && DEPTH == 2);
  if (a.shared && !kShared) return hipErrorInvalidValue;
  DecodeKernelArgs k;
  dim3 blocks;
  if (!decode_kernel_args(a, &k, &blocks)) return hipErrorInvalidValue;
  const dim3 threads(WAVES * kWave);
  const bool fused = a.new_k != nullptr;
  if (a.counted || a.tagged) {
    if constexpr (kShared && one_part_a_wave<4 * HG, D, WAVES>)
      return launch_decode(a.counted ? (a.shared ? paged_decode_bf16_kernel<D, HG, WAVES, DEPTH, true, true, kCounted>
                                                 : paged_decode_bf16_kernel<D, HG, WAVES, DEPTH, true, false, kCounted>)
                           : a.shared ? (fused ? paged_decode_bf16_kernel<D, HG, WAVES, DEPTH, true, true, kTagged>
                                               : paged_decode_bf16_kernel<D, HG, WAVES, DEPTH, false, true, kTagged>)
                                      : (fused ? paged_decode_bf16_kernel<D, HG, WAVES, DEPTH, true, false, kTagged>
                                               : paged_decode_bf16_kernel<D, HG, WAVES, DEPTH, false, false, kTagged>),
                           blocks, threads, stream, k);
    return hipErrorInvalidValue;
  }
  const auto kernel = a.shared ? (fused ? paged_decode_bf16_kernel<D, HG, WAVES, DEPTH, true, kShared>
                                        : paged_decode_bf16_kernel<D, HG, WAVES, DEPTH, false, kShared>)
                               : (fused ? paged_decode_bf16_kernel<D, HG, WAVES, DEPTH, true, false>
                                        : paged_decode_bf16_kernel<D, HG, WAVES, DEPTH, false, false>);
  return launch_decode(kernel, blocks, threads, stream, k);
}

// The workgroup forms that the rule in front of the launch chooses from, and one (4 x 3) for tuning.  Three and four tiles in flight were no faster than
// two (256 rows x 2048 tokens of D = 128 42.1 / 42.5 / 42.6 us, 128 rows x 1024 14.4 / 15.5 / 15.2).  The same rows through the
// vector units (dot products, a cross-lane reduction per token, broadcast probabilities) took 43.7 us (256 x 2048, 4 query
// heads per KV head) and 59.8 (8 heads; now 42.6).
template <int D>
hipError_t launch_shape(const DecodeArgs& a, hipStream_t stream) {
  const bool wide = a.num_q_heads / a.num_kv_heads > 4;
  if constexpr (D == 128) {
    if (a.waves == 8 && a.depth == 1) return wide ? launch_one<D, 2, 8, 1>(a, stream) : hipErrorInvalidValue;
    if (a.waves == 8) return wide ? launch_one<D, 2, 8, 2>(a, stream) : launch_one<D, 1, 8, 2>(a, stream);
    if (a.depth == 3) return wide ? hipErrorInvalidValue : launch_one<D, 1, 4, 3>(a, stream);
  }
  if (a.depth == 1) return wide ? launch_one<D, 2, 4, 1>(a, stream) : launch_one<D, 1, 4, 1>(a, stream);
  return wide ? launch_one<D, 2, 4, 2>(a, stream) : launch_one<D, 1, 4, 2>(a, stream);
}

}  // namespace

hipError_t launch_paged_decode_bf16(const DecodeArgs& a, hipStream_t stream) {
  if (a.head_dim == 64) return launch_shape<64>(a, stream);
  if (a.head_dim == 128) return launch_shape<128>(a, stream);
  return hipErrorInvalidValue;
}

}  // namespace pe
