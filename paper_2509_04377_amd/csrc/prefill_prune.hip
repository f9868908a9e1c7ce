// Prefill token pruning (Alg. 2, the steps after the prompt's attention): score every prompt token,
// evict the E = max(0, L - C) tokens that come first under (score ascending, index ascending), and
// write the survivors, order kept, into the row's pages.
//
// Three kernels on one stream, or two:
//   1. token_scores:  sweep of the packed K/V prompt; S_i = ||V_i||/||K_i|| in fp64, rounded once to
//                     fp32, stored per KV head as a contiguous run  scores[hk][token].
//   2. select:        per row, on the fp32 bit patterns (scores are >= +0, so they order like unsigned integers): a
//                     histogram, then the few scores of one bin settled bit by bit, give the E-th smallest score T and
//                     the number q of tokens equal to T that must go; then, per chunk of 1024 tokens of the row, how
//                     many scores are > T and how many == T (none counted, and q = the largest number, where all go).
//   3. gather:        per row and chunk, an index-ordered scan turns those counts into the destination
//                     of every kept token; token rows are then copied with 16-byte lane accesses.
//   2 + 3. select_gather, where that is faster (prune_log2_parts): every workgroup of a row selects by itself, and copies its
//                     share of what is kept.
// A token is kept iff score > T, or score == T and at least q equal-score tokens precede it.
//
// Head-shared mode (one decision per sequence, pages [B][Hk][D]): a token's score is the mean of its heads' scores (head
// order, fp64, one rounding), taken by the sweep itself where none of its workgroups ends inside a token, else by a
// kernel behind it.  The selection is made on that one score row, the copy head by head with its result.
#include "pe_device.h"
#include "pe_launch.h"
#include "pe_norms.h"
#include "pe_place.h"

namespace pe {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr int kChunk = 1024;  // tokens per chunk in the count pass and in the gather
constexpr int kSweepLoads = 4;  // token sweep: wave-loads of K (and of V) per step
constexpr int kSweepIters = 2;  // and steps per wave (4 and 8: the same on 2 GB of prompt, 5 us slower on 1 GB: longer tail)

__host__ __device__ inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct Workspace {
  float* scores;  // [Hk][total_tokens]; shared mode: one more row, the mean over heads
  uint32_t* sel;  // [rows][2]: threshold bits T, tie quota q
  int32_t* before;  // [Hk][chunk_slots][2]: (#score > T, #score == T) in the earlier chunks of the row
  int64_t chunk_slots;
};

__host__ inline int64_t chunk_slots_for(int64_t total_tokens, int num_seqs) {
  return total_tokens / kChunk + num_seqs + 1;
}

__host__ inline Workspace carve(void* base, int num_seqs, int num_kv_heads, int64_t total_tokens, bool shared) {
  Workspace w;
  char* p = static_cast<char*>(base);
  w.scores = reinterpret_cast<float*>(p);
  p += align256(sizeof(float) * (size_t)(num_kv_heads + (shared ? 1 : 0)) * (size_t)total_tokens);
  w.sel = reinterpret_cast<uint32_t*>(p);
  p += align256(sizeof(uint32_t) * 2 * (size_t)num_seqs * num_kv_heads);
  w.before = reinterpret_cast<int32_t*>(p);
  w.chunk_slots = chunk_slots_for(total_tokens, num_seqs);
  return w;
}

// Chunk slot of (sequence s, local chunk c): sequences never overlap because
// floor((a+b)/n) + 1 >= floor(a/n) + ceil(b/n).
__device__ __forceinline__ int64_t chunk_slot(int cu_s, int s, int c) { return (int64_t)(cu_s / kChunk) + s + c; }

// ---- 1. token scores -------------------------------------------------------------------------------
// The packed prompt is a flat array of (token, head) rows of D elements.  A wave-load covers TPL rows;
// a wave handles kIters groups of NL wave-loads for K and for V, software-pipelined.
// STREAM: K and V with the non-temporal hint.  Without it a prompt stays in the Infinity Cache for the gather, and one that
// was written a moment ago is found there; one that is too large for that is read more slowly (see the rule at the launch).
template <typename T, int D, bool STREAM>
__global__ __launch_bounds__(kThreads) void token_scores_kernel(const T* __restrict__ k_in,
                                                                const T* __restrict__ v_in,
                                                                float* __restrict__ scores, int64_t total_rows,
                                                                int64_t total_tokens, int num_kv_heads, int head_mean) {
  using G = RowGeom<T, D>;
  constexpr int LPR = G::kLanesPerRow;
  constexpr int TPL = G::kTokensPerLoad;
  constexpr int NL = kSweepLoads;
  constexpr int kRowsPerStep = NL * TPL;
  constexpr int kIters = kSweepIters;
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int grp = lane / LPR;
  constexpr int kRowsPerWave = kIters * kRowsPerStep;
  constexpr int kRowsPerGroup = kWaves * kRowsPerWave;
  __shared__ float sm_score[kRowsPerGroup];  // the workgroup's scores in row order, stored head by head at the end
  const int64_t group_row0 = (int64_t)blockIdx.x * kRowsPerGroup;
  const int64_t row0 = group_row0 + (int64_t)wave * kRowsPerWave;

  uint4 kb[2][NL], vb[2][NL];
  // loads are unconditional: a row past the end is read from the last row instead (its result is never
  // stored), so the compiler keeps the order of outstanding loads and the next group stays in flight
  const int64_t last_row = total_rows - 1;
  const int u = lane % LPR;
  auto issue = [&](int buf, int64_t base_row) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int64_t r = base_row + i * TPL + grp;
      const int64_t vec = (r < last_row ? r : last_row) * LPR + u;
      kb[buf][i] = STREAM ? load_vec_stream(k_in, vec) : load_vec(k_in, vec);
      vb[buf][i] = STREAM ? load_vec_stream(v_in, vec) : load_vec(v_in, vec);
    }
  };
  issue(0, row0);
#pragma unroll
  for (int it = 0; it < kIters; ++it) {
    const int64_t base_row = row0 + (int64_t)it * kRowsPerStep;
    if (it + 1 < kIters) issue((it + 1) & 1, base_row + kRowsPerStep);
    if (base_row >= total_rows) break;
    const int buf = it & 1;
    double part[2 * NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      part[i] = sumsq_vec<T>(kb[buf][i], 0.0);
      part[NL + i] = sumsq_vec<T>(vb[buf][i], 0.0);
    }
    const double ratio = token_ratio_from_partials<NL, LPR>(part, lane);
    // the lane at position 2*k of its row group (k < NL) stores the row of wave-load bit_reverse(k)
    const int uu = u;
    if ((uu & 1) == 0 && uu < 2 * NL) {
      const int i = bit_reverse<ilog2(NL)>(uu >> 1);
      const int64_t r = base_row + i * TPL + grp;
      if (r < total_rows) sm_score[(int)(r - group_row0)] = (float)ratio;
    }
  }
  // The group's rows are (token, head) pairs in token-major order; the score array is head-major.  Written
  // head by head, the tokens of one head are consecutive floats (a full 128-byte line for 32 tokens).
  __syncthreads();
  const int64_t group_end = group_row0 + kRowsPerGroup < total_rows ? group_row0 + kRowsPerGroup : total_rows;
  if (group_row0 >= group_end) return;
  const int64_t tok_lo = group_row0 / num_kv_heads;
  const int ntok = (int)((group_end - 1) / num_kv_heads - tok_lo) + 1;
  if (head_mean) {  // the heads of a token lie in one workgroup: as head_mean_kernel does it
    if ((int)threadIdx.x < ntok) {
      const float* of = &sm_score[(int)threadIdx.x * num_kv_heads];
      double sum = 0.0;
      for (int h = 0; h < num_kv_heads; ++h) sum += (double)of[h];
      __hip_atomic_store(&scores[tok_lo + threadIdx.x], (float)(sum / (double)num_kv_heads), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    }
    return;
  }
  for (int p = (int)threadIdx.x; p < ntok * num_kv_heads; p += kThreads) {
    const int h = p / ntok;
    const int64_t tok = tok_lo + (p - h * ntok);
    const int64_t r = tok * num_kv_heads + h;
    // written through to memory, where the selection's workgroups find them whichever L2 they have: lines left in the L2s are
    // written back when the kernel ends (whole prunes, plain / non-temporal / this: 2.1 GB of prompt 493 / 464 / 465 us,
    // 0.6 GB ragged 139 / 142 / 137, 1.1 GB of four prompts 222 / 221 / 215)
    if (r >= group_row0 && r < group_end)
      __hip_atomic_store(&scores[(int64_t)h * total_tokens + tok], sm_score[(int)(r - group_row0)], __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
  }
}

// ---- 1b. head-shared mode: mean over heads of the fp32 token scores (where a sweep workgroup ends inside a token) ---
__global__ __launch_bounds__(kThreads) void head_mean_kernel(const float* __restrict__ scores,
                                                             float* __restrict__ mean_out, int64_t total_tokens,
                                                             int num_kv_heads) {
  const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (t >= total_tokens) return;
  double sum = 0.0;
  for (int h = 0; h < num_kv_heads; ++h) sum += (double)scores[(int64_t)h * total_tokens + t];
  mean_out[t] = (float)(sum / (double)num_kv_heads);
}

// ---- 2. per-row select + per-chunk counts ------------------------------------------------------------
// One workgroup of 1024 threads per row finds the threshold on the row's fp32 bit patterns, which order like unsigned integers.
// A histogram of 4096 equal bins is laid over the range of a sample (one score a thread, without zeros and infinities where the
// threshold is likely none; what lies outside falls into the first or the last bin), so that few scores share a bin whatever their
// magnitude and spread.
// The bin that holds rank k is found with a workgroup-wide scan; a row of some ten thousand ordinary scores leaves some ten
// candidates in it.  They are collected in LDS, and one wave settles the remaining bits of the threshold, bit by bit, with ballots over
// the candidates in its registers: no barriers in between.  More than 256 candidates go through further digits of up to 12
// bits, with a histogram each, between the least and the largest of them; more than LDS holds (e.g. scores of few distinct values)
// are looked for in the whole row again, for their range and for each digit.  A bin of one number, as with equal scores, is done.
// A row is worked on by one compute unit, and one compute unit pulls about 45 GB/s from L2 however many loads it keeps
// in flight: that, not the histogram atomics, bounds the reading of a long row.  So up to 65536 scores of it are read once and
// held, 32768 in registers (32 a thread: 64 would leave too few for the rest) and as many in LDS, and every pass works from
// there; only what a row has beyond is read from memory in each pass.
// What bounds a long row is the vector issue of its one compute unit, 0.43 us per operation on each of 65536 scores: so equal scores
// are counted only where some of them stay, a wave's scores are consecutive, candidates are looked for four at a time, and the last
// vector of a row is filled up with numbers that rank behind all scores, instead of every element of every vector having a predicate
// (which took 221 scalar registers in lanes of vector registers, now 78; prunes of 4 x 65536 tokens 209.3 / 207.8 us).
// Zeros and infinities are kept out of the range (as part of it they spread the bins: 4 x 131072 tokens 458 us a prune, now 451).
// The ways that ordinary scores don't take are kept out of the straight line (8 x 4096 tokens, 8 heads of D = 64, 26.7 us a prune
// with them in it, 26.2 without, in three launches).
constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / kWave;
constexpr int kSelBins = 4096;
constexpr int kSelDigit = ilog2(kSelBins);
constexpr int kSelUnroll = 4;   // 16-byte loads in flight per thread beyond the held scores
constexpr int kSelCand = 2048;  // candidates kept in LDS after the first digit
constexpr int kSelFew = 256;    // candidates that a wave settles in its registers
constexpr int kSelMaxVecs = 8;
constexpr uint32_t kInfBits = 0x7f800000u;
constexpr int kSelMaxHeldChunks = 2 * kSelMaxVecs * 4;

struct __attribute__((packed, aligned(4))) Unaligned4 {  // 16 bytes at any 4-byte boundary, in one load
  uint32_t v[4];
};

// The scores of a row as its workgroup holds them, n * 256 consecutive ones a wave (so that a chunk of 1024 is counted by as few
// waves as possible): score 256*j + 4*lane + e of a wave is element e of vector j of a lane, the first NV vectors in registers, the
// next LV in LDS (a thread reads back only what it has written).  n, at most NV + LV, follows from the row itself, so that all waves
// share a row that is much shorter than the longest of its call (prunes of 127 prompts of 4096 tokens beside one of 40000, 8 heads
// of D = 64: 383 us with NV + LV for every row, now 353; of 63 of 1500 beside it 146 and 136).
template <int NV, int LV>
struct RowScores {
  static constexpr int kHeld = 4 * (NV + LV) * kSelThreads;
  static constexpr int kVector = 4 * kWave;  // scores of a vector of a wave
  const uint32_t* bits;
  uint4* lds;
  int L, tid;
  int n, wave0, end;  // vectors of a wave; first score of this wave, and where its scores end
  Unaligned4 reg[NV];

  __device__ __forceinline__ void deal(int wave) {
    constexpr int kRound = kSelWaves * kVector;
    n = 1;
    if constexpr (NV + LV > 1) n = L >= kHeld ? NV + LV : (L + kRound - 1) / kRound;
    wave0 = wave * n * kVector;
    end = wave0 + n * kVector < L ? wave0 + n * kVector : L;
  }
  __device__ __forceinline__ int index(int j) const { return wave0 + j * kVector + 4 * (tid & (kWave - 1)); }

  __device__ __forceinline__ Unaligned4 request(int j) const {  // past the end the row's last four again
    const int i = j < n ? index(j) : L;
    const int last = L >= 4 ? L - 4 : 0;
    return L >= 4 ? *reinterpret_cast<const Unaligned4*>(bits + (i < last ? i : last)) : Unaligned4{{0u, 0u, 0u, 0u}};
  }
  // Past the row's end the largest number: it ranks behind every score of the row, so that whole vectors can be looked at.
  __device__ __forceinline__ void mend(int j, Unaligned4& r) const {
    const int i = index(j);
    if (i + 4 > L) {
#pragma unroll
      for (int e = 0; e < 4; ++e) r.v[e] = i + e < L ? bits[i + e] : ~0u;
    }
  }
  __device__ __forceinline__ void load() {
#pragma unroll
    for (int j = 0; j < NV; ++j) reg[j] = request(j);  // unconditional, so that all are in flight
    constexpr int kStep = 4;
#pragma unroll
    for (int j0 = 0; j0 < LV; j0 += kStep) {
      if (NV + j0 >= n) break;
      Unaligned4 r[kStep];
#pragma unroll
      for (int j = 0; j < kStep; ++j) r[j] = request(NV + j0 + j);
#pragma unroll
      for (int j = 0; j < kStep; ++j) {
        mend(NV + j0 + j, r[j]);
        lds[(j0 + j) * kSelThreads + tid] = make_uint4(r[j].v[0], r[j].v[1], r[j].v[2], r[j].v[3]);
      }
    }
#pragma unroll
    for (int j = 0; j < NV; ++j) mend(j, reg[j]);
  }

  __device__ __forceinline__ Unaligned4 in_lds(int j) const {
    const uint4 r = lds[(j - NV) * kSelThreads + tid];
    return Unaligned4{{r.x, r.y, r.z, r.w}};
  }
  // Every score of the row: four(vector) for the held ones, and what fills the last vector, ...
  template <typename F4, typename F1>
  __device__ __forceinline__ void visit(F4 four, F1 one) const {
#pragma unroll
    for (int j = 0; j < NV; ++j)
      if (wave0 + j * kVector < end) four(reg[j]);  // the same for all lanes
#pragma unroll 1
    for (int j = NV; wave0 + j * kVector < end; ++j) four(in_lds(j));
    // ... four(vector) or one(score) for the rest, from memory: 16 bytes a load, past the end the row's last four again
    constexpr int kUnroll = LV > 0 ? kSelUnroll : 1;  // a smaller holding covers every row of its call
    for (int i0 = kHeld + 4 * tid; i0 < L; i0 += kUnroll * 4 * kSelThreads) {
      Unaligned4 r[kUnroll];
#pragma unroll
      for (int k = 0; k < kUnroll; ++k) {
        const int i = i0 + k * 4 * kSelThreads;
        r[k] = *reinterpret_cast<const Unaligned4*>(bits + (i < L - 4 ? i : L - 4));
      }
#pragma unroll
      for (int k = 0; k < kUnroll; ++k) {
        const int i = i0 + k * 4 * kSelThreads;
        if (i + 4 <= L) {
          four(r[k]);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (L - 4 + e >= i) one(r[k].v[e]);
        }
      }
    }
  }
};

// Largest value of a wave's lanes.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  const auto step = [&v](uint32_t o) { v = v > o ? v : o; };
  step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111 /* row_shr:1 */, 0xf, 0xf, false));
  step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112 /* row_shr:2 */, 0xf, 0xf, false));
  step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114 /* row_shr:4 */, 0xf, 0xf, false));
  step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118 /* row_shr:8 */, 0xf, 0xf, false));
  step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142 /* row_bcast:15 */, 0xa, 0xf, false));
  step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143 /* row_bcast:31 */, 0xc, 0xf, false));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, kWave - 1);
}

// The highest bit in which two numbers differ (-1: none), and what they share above it.
__device__ __forceinline__ int top_bit(uint32_t lo, uint32_t hi) { return lo == hi ? -1 : 31 - __builtin_clz(lo ^ hi); }
__device__ __forceinline__ uint32_t above(uint32_t v, int bit) { return bit < 31 ? v >> (bit + 1) << (bit + 1) : 0u; }

// The value of rank k among n <= 64 * R candidates between lo and hi, bit by bit; k becomes the rank among those equal to it,
// `same` their number.  One wave.
template <int R>
__device__ __forceinline__ uint32_t settle(const uint32_t* cand, uint32_t n, uint32_t lo, uint32_t hi, uint32_t& k, uint32_t& same,
                                            int lane) {
  int bit = top_bit(lo, hi);
  uint32_t T = above(lo, bit);
  uint32_t x[R];
  uint64_t left[R];  // lanes whose candidate agrees with the bits settled so far
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool is = (uint32_t)(r * kWave + lane) < n;
    x[r] = is ? cand[r * kWave + lane] : 0u;
    left[r] = __builtin_amdgcn_ballot_w64(is);
  }
  for (; bit >= 0; --bit) {
    uint64_t ones[R];
    uint32_t zeros = 0u;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      ones[r] = __builtin_amdgcn_ballot_w64((x[r] >> bit & 1u) != 0u);
      zeros += (uint32_t)__popcll(left[r] & ~ones[r]);
    }
    const bool up = k >= zeros;
    k -= up ? zeros : 0u;
    T |= up ? 1u << bit : 0u;
#pragma unroll
    for (int r = 0; r < R; ++r) left[r] &= up ? ones[r] : ~ones[r];
  }
  same = 0u;
#pragma unroll
  for (int r = 0; r < R; ++r) same += (uint32_t)__popcll(left[r]);
  return T;
}

constexpr int kAllGo = 0x7fffffff;

// What the selection of a row keeps in LDS besides the held scores.
struct SelectLds {
  __attribute__((aligned(16))) uint32_t hist[kSelBins];
  uint32_t cand[kSelCand];
  __attribute__((aligned(16))) uint32_t wave_tot[kSelWaves];
  uint2 wave_range[kSelWaves];
  uint32_t bin, k, in_bin, ncand;
};

// Of a row's scores, held in rs: the threshold, and how many tokens (in index order) with that score go.
struct Threshold {
  uint32_t T;  // bit pattern of the E-th smallest score
  int q;       // that many of those equal to it go; the largest number where all do
};
template <int NV, int LV>
__device__ __forceinline__ Threshold select_threshold(const RowScores<NV, LV>& rs, SelectLds& sm, int E, int keep, int wave, int lane) {
  const int L = rs.L, tid = rs.tid;
  constexpr int kBinsPerThread = kSelBins / kSelThreads;
  static_assert(kBinsPerThread == 4, "a thread reads its bins as one vector");
  const auto clear_hist = [&] { reinterpret_cast<uint4*>(sm.hist)[tid] = make_uint4(0u, 0u, 0u, 0u); };
  // The bin of the histogram that rank k falls into (sm.bin), the rank inside it (sm.k) and what it holds (sm.in_bin).
  const auto find_bin = [&](uint32_t k) {
    const uint4 c4 = reinterpret_cast<const uint4*>(sm.hist)[tid];
    const uint32_t c[kBinsPerThread] = {c4.x, c4.y, c4.z, c4.w};
    const uint32_t tot = c[0] + c[1] + c[2] + c[3];
    const uint32_t incl = wave_prefix_sum_u32(tot);
    if (lane == kWave - 1) sm.wave_tot[wave] = incl;
    __syncthreads();
    uint32_t first = incl - tot;  // elements in lower bins
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) first += w < wave ? sm.wave_tot[w] : 0u;
    if (k >= first && k < first + tot) {  // exactly one thread
#pragma unroll
      for (int j = 0; j < kBinsPerThread; ++j) {
        if (k >= first && k < first + c[j]) {
          sm.bin = (uint32_t)(tid * kBinsPerThread + j);
          sm.k = k - first;
          sm.in_bin = c[j];
        }
        first += c[j];
      }
    }
    __syncthreads();
  };

  // The least and the largest of all threads' (lo, hi); nothing (lo > hi) counts as the largest, or the least, number.
  const auto publish_range = [&](uint32_t lo, uint32_t hi) {
    const uint2 r = make_uint2(wave_max_u32(~lo), wave_max_u32(hi));
    if (lane == 0) sm.wave_range[wave] = r;
  };
  const auto read_range = [&](uint32_t& lo, uint32_t& hi) {  // behind a barrier
    const uint2 r = sm.wave_range[lane % kSelWaves];
    lo = ~wave_max_u32(r.x);
    hi = wave_max_u32(r.y);
  };

  clear_hist();
  if (tid == 0) sm.ncand = 0u;
  {
    const uint32_t b = rs.reg[0].v[0];
    bool in = rs.index(0) < L;
    const bool extreme = in && b - 1u >= kInfBits - 1u;  // zero, or infinity
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(extreme) != 0ull, 0)) {   // they count where more of them were sampled than are to go, or to stay
      const uint32_t zeros = (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(extreme && b == 0u));
      const uint32_t infs = (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(extreme && b != 0u));
      const uint32_t share = (uint32_t)L / kWave;  // scores that one of a wave's sample stands for
      in = in && (!extreme || (b == 0u ? zeros * share > (uint32_t)E : infs * share > (uint32_t)keep));
    }
    publish_range(in ? b : 0xffffffffu, in ? b : 0u);
  }
  __syncthreads();
  // E == 0, nothing to evict: T = +0.0, q = 0 keeps every token (scores are >= +0)
  uint32_t T = 0u, k = (uint32_t)(E > 0 ? E - 1 : 0);  // k: 0-based rank of the threshold among the remaining ones
  if (E > 0) {
    uint32_t low, top;
    read_range(low, top);
    const int shift0 = top_bit(top - low, 0u) < kSelDigit ? 0 : top_bit(top - low, 0u) + 1 - kSelDigit;
    low -= low < 1u << shift0 ? low : 1u << shift0;  // the first bin: all below the sample, and its least begins the second
    const auto count_one = [&](uint32_t b) {
      const uint32_t up = __builtin_elementwise_sub_sat(b, low) >> shift0;
      atomicAdd(&sm.hist[up < (uint32_t)kSelBins - 1u ? up : (uint32_t)kSelBins - 1u], 1u);
    };
    rs.visit([&](const Unaligned4& r) {
#pragma unroll
      for (int e = 0; e < 4; ++e) count_one(r.v[e]);
    }, count_one);
    __syncthreads();
    find_bin(k);
    const uint32_t bin = sm.bin;
    uint32_t n = sm.in_bin;
    k = sm.k;
    uint32_t lo = bin == 0u ? 0u : low + (bin << shift0);
    uint32_t hi = bin == (uint32_t)kSelBins - 1u ? 0xffffffffu : low + ((bin + 1u) << shift0) - 1u;
    const uint32_t span = hi - lo;
    if (__builtin_expect(span == 0u, 0)) n = (uint32_t)kSelCand + 1u;  // one number, as with equal scores: it is the threshold, nothing to collect
    if (__builtin_expect(n <= (uint32_t)kSelCand, 1)) {  // collect the bin's scores (their order does not matter: only values are counted)
      const auto keep_one = [&](uint32_t b) {
        if (b - lo <= span) sm.cand[atomicAdd(&sm.ncand, 1u)] = b;
      };
      rs.visit([&](const Unaligned4& r) {
        const uint32_t d0 = r.v[0] - lo, d1 = r.v[1] - lo, d2 = r.v[2] - lo, d3 = r.v[3] - lo;
        const uint32_t d01 = d0 < d1 ? d0 : d1, d23 = d2 < d3 ? d2 : d3;
        if (__builtin_amdgcn_ballot_w64((d01 < d23 ? d01 : d23) <= span) != 0ull) {  // false for most vectors
          const uint32_t d[4] = {d0, d1, d2, d3};
          uint64_t who[4];
          uint32_t all = 0u, at = 0u;
#pragma unroll
          for (int e = 0; e < 4; ++e) all += (uint32_t)__popcll(who[e] = __builtin_amdgcn_ballot_w64(d[e] <= span));
          if (lane == 0) at = atomicAdd(&sm.ncand, all);
          at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (d[e] <= span)
              sm.cand[at + __builtin_amdgcn_mbcnt_hi((uint32_t)(who[e] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)who[e], 0u))] = r.v[e];
            at += (uint32_t)__popcll(who[e]);
          }
        }
      }, keep_one);
      __syncthreads();
    }
    if (__builtin_expect(n <= (uint32_t)kSelFew, 1)) {
      if (wave == 0) {  // (all sixteen at once would be in one another's way)
        uint32_t same;
        T = n <= (uint32_t)kWave ? settle<1>(sm.cand, n, lo, hi, k, same, lane)
                                 : settle<kSelFew / kWave>(sm.cand, n, lo, hi, k, same, lane);
        if (lane == 0) {
          sm.bin = T;
          sm.k = k;
          sm.in_bin = same;
        }
      }
      __syncthreads();
      T = sm.bin;
      k = sm.k;
    } else {
      if (span != 0u) {
        uint32_t mn = 0xffffffffu, mx = 0u;
        const auto widen = [&](uint32_t b) {
          const bool in = b - lo <= span;
          mn = in && b < mn ? b : mn;
          mx = in && b > mx ? b : mx;
        };
        if (n <= (uint32_t)kSelCand) {
          for (uint32_t i = (uint32_t)tid; i < n; i += kSelThreads) widen(sm.cand[i]);
        } else {
          rs.visit([&](const Unaligned4& r) {
#pragma unroll
            for (int e = 0; e < 4; ++e) widen(r.v[e]);
          }, widen);
        }
        publish_range(mn, mx);
        __syncthreads();
        read_range(lo, hi);
      }
      int bits = top_bit(lo, hi) + 1;  // not settled yet
      T = above(lo, bits - 1);
#pragma unroll 1
      while (bits > 0) {
        const int shift = bits > kSelDigit ? bits - kSelDigit : 0;
        const uint32_t digit = (1u << (bits - shift)) - 1u, settled = bits < 32 ? ~0u << bits : 0u;
        clear_hist();
        __syncthreads();
        const auto count = [&](uint32_t b) {
          if (b - lo <= hi - lo && ((b ^ T) & settled) == 0u) atomicAdd(&sm.hist[(b >> shift) & digit], 1u);
        };
        if (n <= (uint32_t)kSelCand) {
          for (uint32_t i = (uint32_t)tid; i < n; i += kSelThreads) count(sm.cand[i]);
        } else {
          rs.visit([&](const Unaligned4& r) {
#pragma unroll
            for (int e = 0; e < 4; ++e) count(r.v[e]);
          }, count);
        }
        __syncthreads();
        find_bin(k);
        T |= sm.bin << shift;
        k = sm.k;
        bits = shift;
      }
    }
  }
  // The first k + 1 tokens (index order) with score == T go.  Where that is all there are, as almost always, nobody has to count
  // them: q = the largest number, none before any token.
  return {T, E == 0 ? 0 : k + 1u == sm.in_bin ? kAllGo : (int)k + 1};
}

// The selection by itself: the threshold, and, per chunk of 1024 tokens, how many scores before it are > T and == T (the gather turns
// these into destinations).  Two workgroups a compute unit (eight waves per SIMD, 64 registers) as long as the row leaves the
// registers for it: more rows than compute units then still run at once.
template <int NV, int LV>
__global__ __launch_bounds__(kSelThreads, NV <= 4 ? 8 : 4) void select_kernel(const float* __restrict__ scores,
                                                             const int32_t* __restrict__ cu_seqlens,
                                                             uint32_t* __restrict__ sel, int32_t* __restrict__ before,
                                                             int32_t* __restrict__ seq_lens_out,
                                                             int32_t* __restrict__ kept_idx_out, int64_t total_tokens,
                                                             int64_t chunk_slots, int num_kv_heads, int budget) {
  using Row = RowScores<NV, LV>;
  constexpr int kHeldChunks = Row::kHeld / kChunk;
  static_assert(kHeldChunks <= kSelMaxHeldChunks, "chunk counters");
  __shared__ SelectLds sm;
  uint32_t* const hist = sm.hist;  // at the end, counts of chunks beyond the held ones
  __shared__ uint4 held_lds[LV > 0 ? LV * kSelThreads : 1];
  __shared__ uint32_t held_count[kSelMaxHeldChunks];
  const int row = (int)blockIdx.x;
  const int s = row / num_kv_heads, h = row % num_kv_heads;
  const int t0 = cu_seqlens[s];
  const int L = cu_seqlens[s + 1] - t0;
  const int keep = L < budget ? L : budget;
  const int E = L - keep;
  const int tid = (int)threadIdx.x;
  const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  Row rs;
  rs.bits = reinterpret_cast<const uint32_t*>(scores) + (int64_t)h * total_tokens + t0;
  rs.lds = held_lds;
  rs.L = L;
  rs.tid = tid;
  rs.deal(wave);
  rs.load();

  if (h == 0 && tid == 0) seq_lens_out[s] = keep;
  if (kept_idx_out != nullptr)
    for (int i = keep + tid; i < budget; i += kSelThreads) kept_idx_out[(int64_t)row * budget + i] = -1;

  if (tid < kSelMaxHeldChunks) held_count[tid] = 0u;  // (barriers come before they are used)
  const Threshold at = select_threshold(rs, sm, E, keep, wave, lane);
  const uint32_t T = at.T;
  const bool all_go = at.q == kAllGo;
  if (tid == 0) {
    sel[2 * row] = T;  // threshold score (bit pattern)
    sel[2 * row + 1] = (uint32_t)at.q;
  }

  // Scores > T (lower half) and == T (upper half) per chunk, then how many there are before each chunk of the row.
  const int nchunks = (L + kChunk - 1) / kChunk;
  int32_t* brow = before + ((int64_t)h * chunk_slots + chunk_slot(t0, s, 0)) * 2;
  constexpr int kVectorsPerChunk = kChunk / Row::kVector;
  uint32_t n = 0u;  // of this lane, of the chunk at hand
  const auto count_vector = [&](int j, const Unaligned4& r) {
    const int left = rs.wave0 + (j + 1) * Row::kVector <= rs.end ? 4 : rs.end - rs.index(j);
#pragma unroll
    for (int e = 0; e < 4; ++e) n += e < left && r.v[e] > T ? 1u : 0u;
    if (!all_go) {
#pragma unroll
      for (int e = 0; e < 4; ++e) n += e < left && r.v[e] == T ? 0x10000u : 0u;
    }
    const int v = rs.wave0 / Row::kVector + j;  // number of the vector in the row
    if (v % kVectorsPerChunk == kVectorsPerChunk - 1 || j == rs.n - 1) {
      n = wave_prefix_sum_u32(n);
      if (lane == kWave - 1) atomicAdd(&held_count[v / kVectorsPerChunk], n);
      n = 0u;
    }
  };
#pragma unroll
  for (int j = 0; j < NV; ++j)
    if (j < rs.n) count_vector(j, rs.reg[j]);
#pragma unroll 1
  for (int j = NV; j < rs.n; ++j) count_vector(j, rs.in_lds(j));
  int gt_total = 0, eq_total = 0;  // of the pieces done
  for (int c0 = 0; c0 < nchunks; c0 += kSelBins) {
    const int nc = nchunks - c0 < kSelBins ? nchunks - c0 : kSelBins;
    // beyond them, one wave per chunk: 16 tokens per lane, all loads issued before the first compare
    for (int cc = (c0 == 0 ? kHeldChunks : 0) + wave; cc < nc; cc += kSelWaves) {
      constexpr int kPerLane = kChunk / kWave;
      const int i0 = (c0 + cc) * kChunk + lane;
      uint32_t b[kPerLane], n = 0u;
#pragma unroll
      for (int j = 0; j < kPerLane; ++j) b[j] = rs.bits[i0 + j * kWave < L ? i0 + j * kWave : L - 1];
#pragma unroll
      for (int j = 0; j < kPerLane; ++j)
        n += i0 + j * kWave < L ? (b[j] > T ? 1u : 0u) + (!all_go && b[j] == T ? 0x10000u : 0u) : 0u;
      n = wave_prefix_sum_u32(n);
      if (lane == kWave - 1) hist[cc] = n;
    }
    __syncthreads();
    if (wave == 0) {
      for (int cc = 0; cc < nc; cc += kWave) {
        const uint32_t n = cc + lane >= nc ? 0u : c0 + cc + lane < kHeldChunks ? held_count[cc + lane] : hist[cc + lane];
        const int gt = (int)wave_prefix_sum_u32(n & 0xffffu), eq = (int)wave_prefix_sum_u32(n >> 16);
        if (cc + lane < nc) {
          const int2 v = make_int2(gt_total + gt - (int)(n & 0xffffu), eq_total + eq - (int)(n >> 16));
          *reinterpret_cast<int2*>(brow + 2 * (c0 + cc + lane)) = v;
        }
        gt_total += __builtin_amdgcn_readlane(gt, kWave - 1);
        eq_total += __builtin_amdgcn_readlane(eq, kWave - 1);
      }
    }
    __syncthreads();
  }
}

// The smallest holding that covers rows of max_seqlen tokens (or the largest there is): a larger one than needed costs loads,
// branches and, beyond 16 scores a thread, the second workgroup of a compute unit.
using SelectKernel = void (*)(const float*, const int32_t*, uint32_t*, int32_t*, int32_t*, int32_t*, int64_t, int64_t, int, int);
SelectKernel select_kernel_for(int max_seqlen) {
  const int vecs = (max_seqlen + 4 * kSelThreads - 1) / (4 * kSelThreads);
  if (vecs <= 1) return select_kernel<1, 0>;
  if (vecs <= 2) return select_kernel<2, 0>;
  if (vecs <= 4) return select_kernel<4, 0>;
  if (vecs <= kSelMaxVecs) return select_kernel<kSelMaxVecs, 0>;
  return select_kernel<kSelMaxVecs, kSelMaxVecs>;
}

// ---- 3. gather ----------------------------------------------------------------------------------------
// One workgroup per (row, chunk) copies the kept token rows of one head, with 512 threads: a chunk that is kept whole, as of short rows
// beside a long one, is a long way for 256 (whole prunes, 256 / 512 / 1024 threads, us: fp32, 39 of D = 128 of up to 1459 tokens 74.7 /
// 54.1 / 54.4, one of 9802 beside eleven of 980, 1280 kept 67.7 / 49.9 / 50.0).  Where less than a thirty-second of the average row is
// kept they have little to copy, and it takes 256 (256 / 512: 14 of up to 14652 of D = 64, 224 kept 72.4 / 73.8, 448 kept 74.8 / 74.9, 912 79.2 /
// 79.2; 4 x 40960 of D = 128, 640 kept 124.8 / 126.4, 1280 127.8 / 128.0, 20480 263.5 / 262.1; 2 x 40960, four heads of D = 64, 1280 kept 30.6 /
// 30.4).  SHARED: the heads of a sequence share its selection and its
// table row, their token rows lie num_kv_heads apart in the pages (whole records by one workgroup were a division per
// 16 bytes and an eighth of the workgroups: 16 prompts of 2048 to 8192 tokens, 8 heads, 1024 kept 204 us a prune, now 98; 8 x 4096 of
// D = 64 54.8, now 31.1).
template <int VEC_PER_ROW, bool SHARED, int THREADS>
__global__ __launch_bounds__(THREADS) void gather_kernel(const uint4* __restrict__ k_in, const uint4* __restrict__ v_in,
                                                         const float* __restrict__ scores,
                                                         const int32_t* __restrict__ cu_seqlens,
                                                         const uint32_t* __restrict__ sel,
                                                         const int32_t* __restrict__ before,
                                                         const int32_t* __restrict__ block_table,
                                                         uint4* __restrict__ k_pool, uint4* __restrict__ v_pool,
                                                         int32_t* __restrict__ kept_idx_out, int64_t total_tokens,
                                                         int64_t chunk_slots, int num_kv_heads, int rows,
                                                         int log2_block, int max_blocks, int budget, int row0,
                                                         int chunk0) {
  constexpr int kTokPerThread = kChunk / THREADS;
  __shared__ uint32_t wave_sum[THREADS / kWave];
  __shared__ int32_t src_tok[kChunk];  // kept tokens of this chunk, in order: in-sequence index
  __shared__ int n_kept_sh;
  // Rows fastest: the first chunks of a ragged batch, which short sequences keep most of, spread over all XCDs (workgroup
  // number % 8).  Chunks fastest put the first chunks of all sequences on one: 47 us instead of 30 for 16 sequences of
  // 2048 to 16384 tokens, 8 heads, 1024 kept of each (134 MB moved; the other prompts below did not change).
  const int row = row0 + (int)(blockIdx.x % (unsigned)rows);
  const int chunk = chunk0 + (int)(blockIdx.x / (unsigned)rows);
  const int s = row / num_kv_heads, h = row % num_kv_heads;
  const int sel_row = SHARED ? s : row, sel_h = SHARED ? 0 : h;  // whose scores decide
  const int t0 = cu_seqlens[s];
  const int L = cu_seqlens[s + 1] - t0;
  if (chunk * kChunk >= L) return;
  const int tid = (int)threadIdx.x;
  const int lane = lane_id();
  const int wave = tid / kWave;
  const uint32_t T = sel[2 * sel_row];
  const int q = (int)sel[2 * sel_row + 1];

  // counts over all earlier chunks of this row
  const int2 earlier = reinterpret_cast<const int2*>(before)[(int64_t)sel_h * chunk_slots + chunk_slot(t0, s, chunk)];
  const int gt_before = earlier.x, eq_before = earlier.y;

  // this thread's kTokPerThread consecutive tokens
  const uint32_t* bits = reinterpret_cast<const uint32_t*>(scores) + (int64_t)sel_h * total_tokens + t0;
  const int i0 = chunk * kChunk + tid * kTokPerThread;
  uint32_t b[kTokPerThread];
  int n_gt = 0, n_eq = 0;
#pragma unroll
  for (int j = 0; j < kTokPerThread; ++j) {
    b[j] = (i0 + j < L) ? bits[i0 + j] : 0u;
    const bool in = i0 + j < L;
    n_gt += in && b[j] > T;
    n_eq += in && b[j] == T;
  }
  // exclusive scan of (n_gt, n_eq) over the threads, in thread (= index) order; each fits 16 bits
  const uint32_t n_both = (uint32_t)n_gt | ((uint32_t)n_eq << 16);
  const uint32_t inc = wave_prefix_sum_u32(n_both);
  if (lane == kWave - 1) wave_sum[wave] = inc;
  __syncthreads();
  uint32_t ex = inc - n_both;
#pragma unroll
  for (int w = 0; w < THREADS / kWave; ++w) ex += w < wave ? wave_sum[w] : 0u;
  int ex_gt = (int)(ex & 0xffffu) + gt_before, ex_eq = (int)(ex >> 16) + eq_before;
  // kept tokens before this chunk's start: the chunk's kept tokens take consecutive positions from here
  const int kept_before_chunk = gt_before + (eq_before > q ? eq_before - q : 0);
#pragma unroll
  for (int j = 0; j < kTokPerThread; ++j) {
    const bool in = i0 + j < L;
    const bool is_gt = in && b[j] > T;
    const bool is_eq = in && b[j] == T;
    const bool kept = is_gt || (is_eq && ex_eq >= q);
    if (kept) {
      const int pos = ex_gt + (ex_eq > q ? ex_eq - q : 0);  // kept tokens before this one in the row
      src_tok[pos - kept_before_chunk] = i0 + j;
    }
    ex_gt += is_gt;
    ex_eq += is_eq;
  }
  if (tid == THREADS - 1) n_kept_sh = ex_gt + (ex_eq > q ? ex_eq - q : 0) - kept_before_chunk;
  __syncthreads();
  const int n_kept = n_kept_sh;

  if (kept_idx_out != nullptr && (!SHARED || h == 0))  // consecutive positions: whole lines
    for (int e = tid; e < n_kept; e += THREADS) kept_idx_out[(int64_t)sel_row * budget + kept_before_chunk + e] = src_tok[e];

  // copy the kept rows: VEC_PER_ROW lanes per token row, K and V (two or four rows of a thread in flight, or the pages looked up
  // beforehand: no faster)
  const int32_t* bt = block_table + (int64_t)sel_row * max_blocks;
  const int block_mask = (1 << log2_block) - 1;
  constexpr int kRowsPerPass = THREADS / VEC_PER_ROW;
  const int u = tid % VEC_PER_ROW, r = tid / VEC_PER_ROW;
  for (int e = r; e < n_kept; e += kRowsPerPass) {
    const int pos = kept_before_chunk + e;
    const int64_t src = ((int64_t)(t0 + src_tok[e]) * num_kv_heads + h) * VEC_PER_ROW + u;
    const int64_t slot = ((int64_t)bt[pos >> log2_block] << log2_block) + (pos & block_mask);
    const int64_t dst = (SHARED ? slot * num_kv_heads + h : slot) * VEC_PER_ROW + u;
    k_pool[dst] = k_in[src];
    v_pool[dst] = v_in[src];
  }
}

// ---- 2 + 3 in one launch ---------------------------------------------------------------------------------
// The workgroups of a row all find its threshold, each by itself, and each copies its share of the positions of the kept tokens (equal
// shares, whatever the row's length).  What that saves is a launch between the two and the second reading and counting of the scores;
// what it costs nothing, as long as every workgroup has a compute unit for itself, is that a row is selected several times.
// Bound: the chain of launches and barriers for short prompts, memory for long ones.  Measured on an MI355X, two kernels / so, whole
// prunes, us: 1 x 1000 tokens, 8 heads of D = 128, 15.0 / 10.2; 1 x 8000 20.7 / 16.8; 4 x 4096 28.6 / 22.8; 8 x 4096 of D = 64 26.1 /
// 23.0; 16 of 2048 to 16384 128.8 / 125.3; 32 x 16384 467 / 466, each of a model's layers into its own pool 442 / 437; fp32, 8 x 8192
// 112.4 / 110.2; head-shared, 8 of 2048 to 8192 57.3 / 49.3; 2 of 20000 to 32768 60.5 / 60.4.  Longer rows, which one compute unit
// holds in LDS too, lose (4 x 65536 210.4 / 213.8): there they stay two kernels.
// (Not faster: two or four rows of a thread in flight in the copy, and K and V read or written with the non-temporal hint: prunes into
// the same pools again and again win up to 2 %, those of layers that go each into their own lose up to 4.)
// Two workgroups a compute unit (eight waves per SIMD, 64 registers) as long as the row leaves the registers for it: more rows
// than compute units then still run at once.
template <int NV, int VEC_PER_ROW, bool SHARED>
__global__ __launch_bounds__(kSelThreads, NV <= 4 ? 8 : 4) void select_gather_kernel(
    const uint4* __restrict__ k_in, const uint4* __restrict__ v_in, const float* __restrict__ scores,
    const int32_t* __restrict__ cu_seqlens, const int32_t* __restrict__ block_table, uint4* __restrict__ k_pool,
    uint4* __restrict__ v_pool, int32_t* __restrict__ seq_lens_out, int32_t* __restrict__ kept_idx_out, int64_t total_tokens,
    int log2_block, int max_blocks, int budget, int log2_parts, int seq0) {
  using Row = RowScores<NV, 0>;
  __shared__ SelectLds sm;
  uint32_t* const list = sm.hist;  // tokens of the positions at hand, once the threshold is known
  constexpr int kList = kSelBins;
  // (head, sequence, part): the parts of a row lie side by side on one XCD where the number of rows is a multiple of eight
  const int h = (int)blockIdx.x, heads = (int)gridDim.x, s = seq0 + (int)blockIdx.y, part = (int)blockIdx.z;
  const int sel_row = SHARED ? s : s * heads + h, sel_h = SHARED ? 0 : h;
  const int t0 = cu_seqlens[s];
  const int L = cu_seqlens[s + 1] - t0;
  const int keep = L < budget ? L : budget;
  const int E = L - keep;
  const int tid = (int)threadIdx.x;
  const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const bool reports = !SHARED || h == 0;
  if (part == 0) {
    if (h == 0 && tid == 0) seq_lens_out[s] = keep;
    if (kept_idx_out != nullptr && reports)
      for (int i = keep + tid; i < budget; i += kSelThreads) kept_idx_out[(int64_t)sel_row * budget + i] = -1;
  }
  constexpr int kRowsPerPass = kSelThreads / VEC_PER_ROW;
  const int share = (((keep + (1 << log2_parts) - 1) >> log2_parts) + kRowsPerPass - 1) & ~(kRowsPerPass - 1);  // whole passes of the copy
  const int lo = part * share, hi = lo + share < keep ? lo + share : keep;
  // (a row longer than the caller has said is pruned like any other as long as it is held here and its table row holds it, else its
  // pages are left alone)
  if (lo >= hi || L > Row::kHeld || (keep - 1) >> log2_block >= max_blocks) return;

  const int32_t* bt = block_table + (int64_t)sel_row * max_blocks;
  const int block_mask = (1 << log2_block) - 1;
  const int u = tid % VEC_PER_ROW, r = tid / VEC_PER_ROW;
  const auto copy = [&](int p0, int m, auto token_of) {
    for (int e = r; e < m; e += kRowsPerPass) {
      const int pos = p0 + e;
      const int64_t src = ((int64_t)(t0 + token_of(e)) * heads + h) * VEC_PER_ROW + u;
      const int64_t slot = ((int64_t)bt[pos >> log2_block] << log2_block) + (pos & block_mask);
      const int64_t dst = (SHARED ? slot * heads + h : slot) * VEC_PER_ROW + u;
      k_pool[dst] = k_in[src];
      v_pool[dst] = v_in[src];
    }
    if (kept_idx_out != nullptr && reports)
      for (int e = tid; e < m; e += kSelThreads) kept_idx_out[(int64_t)sel_row * budget + p0 + e] = token_of(e);
  };
  if (E == 0) {
    copy(lo, hi - lo, [&](int e) { return lo + e; });
    return;
  }

  Row rs;
  rs.bits = reinterpret_cast<const uint32_t*>(scores) + (int64_t)sel_h * total_tokens + t0;
  rs.lds = nullptr;
  rs.L = L;
  rs.tid = tid;
  rs.deal(wave);
  rs.load();
  const Threshold at = select_threshold(rs, sm, E, keep, wave, lane);

  // How many of a vector's scores are > T (lower half) and == T (upper half) in this lane, the latter where some of those stay.
  // (What fills the last vector behind the row's end comes behind every token that is kept.)
  const auto count4 = [&](const Unaligned4& v, bool ties) {
    uint32_t n = 0u;
#pragma unroll
    for (int e = 0; e < 4; ++e) n += v.v[e] > at.T ? 1u : 0u;
    if (ties) {
#pragma unroll
      for (int e = 0; e < 4; ++e) n += v.v[e] == at.T ? 0x10000u : 0u;
    }
    return n;
  };
  const bool ties = at.q != kAllGo;
  uint32_t n = 0u;
#pragma unroll
  for (int j = 0; j < NV; ++j)
    if (j < rs.n) n += count4(rs.reg[j], ties);
  n = wave_prefix_sum_u32(n);
  if (lane == kWave - 1) sm.wave_tot[wave] = n;
  const uint32_t mine = (uint32_t)__builtin_amdgcn_readlane((int)n, kWave - 1);
  __syncthreads();
  int gt0 = 0, eq0 = 0;  // in the waves before this one
#pragma unroll
  for (int w = 0; w < kSelWaves; ++w) {
    const uint32_t t = sm.wave_tot[w];
    gt0 += w < wave ? (int)(t & 0xffffu) : 0;
    eq0 += w < wave ? (int)(t >> 16) : 0;
  }
  const auto kept_before = [&](int gt, int eq) { return gt + (eq > at.q ? eq - at.q : 0); };
  const int mine0 = kept_before(gt0, eq0), mine1 = kept_before(gt0 + (int)(mine & 0xffffu), eq0 + (int)(mine >> 16));
  for (int p0 = lo; p0 < hi; p0 += kList) {
    const int p1 = p0 + kList < hi ? p0 + kList : hi;
    if (p0 > lo) __syncthreads();  // the list has been read
    if (mine0 < p1 && mine1 > p0) {
      int gt = gt0, eq = eq0;
      const auto place4 = [&](int j, const Unaligned4& v) {
        const uint32_t c = count4(v, ties);
        const uint32_t inc = wave_prefix_sum_u32(c), ex = inc - c;
        int g = gt + (int)(ex & 0xffffu), q = eq + (int)(ex >> 16);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool is_gt = v.v[e] > at.T, is_eq = ties && v.v[e] == at.T;
          const int pos = kept_before(g, q);
          if ((is_gt || (is_eq && q >= at.q)) && pos >= p0 && pos < p1) list[pos - p0] = (uint32_t)(rs.index(j) + e);
          g += is_gt;
          q += is_eq;
        }
        const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)inc, kWave - 1);
        gt += (int)(all & 0xffffu);
        eq += (int)(all >> 16);
      };
#pragma unroll
      for (int j = 0; j < NV; ++j)
        if (j < rs.n) place4(j, rs.reg[j]);
    }
    __syncthreads();
    copy(p0, p1 - p0, [&](int e) { return (int)list[e]; });
  }
}

// The smallest holding again.
template <int VPR, bool SHARED>
auto select_gather_kernel_for(int max_seqlen) {
  const int vecs = (max_seqlen + 4 * kSelThreads - 1) / (4 * kSelThreads);
  return vecs <= 1   ? select_gather_kernel<1, VPR, SHARED>
         : vecs <= 2 ? select_gather_kernel<2, VPR, SHARED>
         : vecs <= 4 ? select_gather_kernel<4, VPR, SHARED>
                     : select_gather_kernel<kSelMaxVecs, VPR, SHARED>;
}

template <typename T, int D>
hipError_t launch(const PruneArgs& a, hipStream_t stream) {
  using G = RowGeom<T, D>;
  const Workspace w = carve(a.workspace, a.num_seqs, a.num_kv_heads, a.total_tokens, a.shared);
  const int64_t total_rows = a.total_tokens * a.num_kv_heads;
  // Head-shared: where no sweep workgroup ends inside a token it averages the heads itself; their scores are then not written (16
  // prompts of 2048 to 8192 tokens, 8 heads 99 us a prune, now 94, 32 x 16384 465 and 434).
  constexpr int rows_per_group = kWaves * kSweepIters * kSweepLoads * G::kTokensPerLoad;
  static_assert(rows_per_group <= kThreads, "one thread a token averages its heads");
  const bool mean_in_sweep = a.shared && rows_per_group % a.num_kv_heads == 0;
  float* mean = w.scores + (size_t)a.num_kv_heads * (size_t)a.total_tokens;
  hipError_t e;
  const int64_t row_bytes = 2 * (int64_t)a.num_kv_heads * D * (int64_t)sizeof(T);  // K and V of a token
  if (total_rows > 0) {
    const int64_t grid = (total_rows + rows_per_group - 1) / rows_per_group;
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    // Prompts of up to 96 MiB are swept without the hint: they then lie in the Infinity Cache (256 MB) when the gather comes, and
    // what the model has just written, as in a prefill, is found there.  The line is where that costs nothing out of memory either
    // as long as a quarter of the prompt or more is kept.  Whole prunes of some 4500 tokens a prompt, 8 heads, with / without the hint
    // (256, 1024 or 2048 tokens kept; D = 64, fp32 and the head-shared layout cross at the same sizes), us:
    //   bf16, D = 128    K and V written right before                   out of memory
    //    34 MB           23.8 / 22.2   32.8 / 27.9   42.8 / 34.1        21.4 / 21.8   30.5 / 28.1   41.8 / 34.7
    //    84 MB           32.3 / 29.1   41.8 / 35.0   54.7 / 42.5        29.5 / 31.4   41.6 / 39.6   55.9 / 47.9
    //   100 MB           34.7 / 31.5   42.4 / 36.2   53.0 / 42.7        31.5 / 34.0   41.4 / 40.9   53.9 / 48.4
    //   134 MB           39.4 / 37.5   50.4 / 43.7   63.4 / 52.6        37.3 / 40.3   48.8 / 51.1   64.3 / 64.3
    //   200 MB           53.1 / 48.4   65.8 / 57.7   82.7 / 80.2        49.3 / 54.9   64.0 / 71.9   85.1 / 97.4
    const bool streamed = a.total_tokens * row_bytes > (int64_t)96 << 20;
    const auto sweep = streamed ? token_scores_kernel<T, D, true> : token_scores_kernel<T, D, false>;
    hipLaunchKernelGGL(sweep, dim3((unsigned)grid), dim3(kThreads), 0, stream, (const T*)a.k_in, (const T*)a.v_in,
                       mean_in_sweep ? mean : w.scores, total_rows, a.total_tokens, a.num_kv_heads, mean_in_sweep ? 1 : 0);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  // what kernel 2 sees: per-head rows, or (shared) one row per sequence whose scores are the head means
  const int heads = a.shared ? 1 : a.num_kv_heads;
  const float* sel_scores = w.scores;
  if (a.shared) {
    if (a.total_tokens > 0 && !mean_in_sweep) {
      const int64_t grid = (a.total_tokens + kThreads - 1) / kThreads;
      hipLaunchKernelGGL(head_mean_kernel, dim3((unsigned)grid), dim3(kThreads), 0, stream, w.scores, mean,
                         a.total_tokens, a.num_kv_heads);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    sel_scores = mean;
  }
  const int rows = a.num_seqs * heads, chunks_per_row = (a.max_seqlen + kChunk - 1) / kChunk;
  if ((int64_t)rows * (chunks_per_row > 4 ? chunks_per_row : 4) >= (1LL << 32) / kThreads) return hipErrorInvalidValue;
  constexpr int VPR = G::kLanesPerRow;
  constexpr int kMostGroups = 1 << 22;  // of a launch: 2^32 threads
  static_assert(4 * kSelMaxVecs * kSelThreads == 32768 && kChunk == 1024 && kSelThreads == 1024, "as prune_log2_parts has it");
  const int log2_parts = prune_log2_parts(a.num_seqs, a.num_kv_heads, a.total_tokens, a.max_seqlen, a.budget, 4 * D * (int)sizeof(T),
                                          a.compute_units);
  if (log2_parts >= 0 && a.num_kv_heads < kMostGroups) {
    const auto kernel = a.shared ? select_gather_kernel_for<VPR, true>(a.max_seqlen) : select_gather_kernel_for<VPR, false>(a.max_seqlen);
    const int room = (kMostGroups - 1) / a.num_kv_heads, seqs = room < 65535 ? room : 65535;  // of a launch
    for (int s0 = 0; s0 < a.num_seqs; s0 += seqs) {
      const int ns = a.num_seqs - s0 < seqs ? a.num_seqs - s0 : seqs;
      hipLaunchKernelGGL(kernel, dim3((unsigned)a.num_kv_heads, (unsigned)ns, 1u << log2_parts), dim3(kSelThreads), 0, stream,
                         (const uint4*)a.k_in, (const uint4*)a.v_in, sel_scores, a.cu_seqlens, a.block_table, (uint4*)a.k_pool,
                         (uint4*)a.v_pool, a.seq_lens_out, a.kept_idx_out, a.total_tokens, ilog2(a.block_size), a.max_blocks,
                         a.budget, log2_parts, s0);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return e;
  }
  hipLaunchKernelGGL(select_kernel_for(a.max_seqlen), dim3((unsigned)rows), dim3(kSelThreads), 0, stream, sel_scores, a.cu_seqlens,
                     w.sel, w.before, a.seq_lens_out, a.kept_idx_out, a.total_tokens, w.chunk_slots, heads, a.budget);
  if ((e = hipGetLastError()) != hipSuccess || chunks_per_row == 0) return e;
  // Plain stores for what is kept.  With the non-temporal hint prunes of 32 x 16384 tokens that go into the same pools again and
  // again take 454 us instead of 467, but those of a model's layers, one after the other and each into its own pool, 475 instead of
  // 457 (four prompts of 65536 229 and 223, 3B prompts 141 and 137, the head-shared layout 455 and 436).
  const bool little = (int64_t)a.budget * 32 < a.total_tokens / a.num_seqs;
  const int threads = little ? 256 : 512;
  const auto gather = little ? (a.shared ? gather_kernel<VPR, true, 256> : gather_kernel<VPR, false, 256>)
                             : (a.shared ? gather_kernel<VPR, true, 512> : gather_kernel<VPR, false, 512>);
  e = hipErrorInvalidValue;  // (one launch, but where a batch has more (head, chunk) pairs than 2^32 threads)
  launch_pieces(a.num_seqs, a.num_kv_heads, chunks_per_row, threads, [&](int s0, int ns, int c0, int nc) {
    const int copied = ns * a.num_kv_heads;  // (row, head) pairs that this launch copies
    hipLaunchKernelGGL(gather, dim3((unsigned)copied * (unsigned)nc), dim3(threads), 0, stream, (const uint4*)a.k_in,
                       (const uint4*)a.v_in, sel_scores, a.cu_seqlens, w.sel, w.before, a.block_table, (uint4*)a.k_pool,
                       (uint4*)a.v_pool, a.kept_idx_out, a.total_tokens, w.chunk_slots, a.num_kv_heads, copied,
                       ilog2(a.block_size), a.max_blocks, a.budget, s0 * a.num_kv_heads, c0);
    return (e = hipGetLastError()) == hipSuccess;
  });
  return e;
}

}  // namespace

size_t prune_workspace_bytes(int num_seqs, int num_kv_heads, int64_t total_tokens, bool shared) {
  return align256(sizeof(float) * (size_t)(num_kv_heads + (shared ? 1 : 0)) * (size_t)total_tokens) +
         align256(sizeof(uint32_t) * 2 * (size_t)num_seqs * num_kv_heads) +
         align256(sizeof(int32_t) * 2 * (size_t)num_kv_heads * (size_t)chunk_slots_for(total_tokens, num_seqs));
}

hipError_t launch_prefill_prune(const PruneArgs& a, hipStream_t stream) {
  if (a.is_bf16) {
    if (a.head_dim == 64) return launch<bf16_t, 64>(a, stream);
    if (a.head_dim == 128) return launch<bf16_t, 128>(a, stream);
  } else {
    if (a.head_dim == 64) return launch<float, 64>(a, stream);
    if (a.head_dim == 128) return launch<float, 128>(a, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace pe
