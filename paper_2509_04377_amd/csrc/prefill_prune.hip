// Prefill token pruning (Alg. 2, the steps after the prompt's attention): score every prompt token,
// evict the E = max(0, L - C) tokens that come first under (score ascending, index ascending), and
// write the survivors, order kept, into the row's pages.
//
// Three kernels on one stream:
//   1. token_scores:  sweep of the packed K/V prompt; S_i = ||V_i||/||K_i|| in fp64, rounded once to
//                     fp32, stored per KV head as a contiguous run  scores[hk][token].
//   2. select:        per row, radix select (digits of 12, 10 and 10 bits, most significant first) on the
//                     fp32 bit patterns (scores are >= +0, so they order like unsigned integers) for the
//                     E-th smallest score T and the number q of tokens equal to T that must go; then, per
//                     chunk of 1024 tokens of the row, how many scores are > T and how many == T.
//   3. gather:        per row and chunk, an index-ordered scan turns those counts into the destination
//                     of every kept token; token rows are then copied with 16-byte lane accesses.
// A token is kept iff score > T, or score == T and at least q equal-score tokens precede it.
//
// Head-shared mode (one decision per sequence, pages [B][Hk][D]): after kernel 1 the per-head scores are
// averaged over the heads (head order, fp64, one rounding) into one more score row, and kernels 2-3 run on
// that row with the whole (token, all heads) record as the unit that is copied.
#include "pe_device.h"
#include "pe_launch.h"
#include "pe_norms.h"

namespace pe {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr int kChunk = 1024;  // tokens per chunk in the count pass and in the gather (4 per gather thread)
constexpr int kTokPerThread = kChunk / kThreads;
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
                                                                int64_t total_tokens, int num_kv_heads) {
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

// ---- 1b. head-shared mode: mean over heads of the fp32 token scores -----------------------------------
__global__ __launch_bounds__(kThreads) void head_mean_kernel(const float* __restrict__ scores,
                                                             float* __restrict__ mean_out, int64_t total_tokens,
                                                             int num_kv_heads) {
  const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (t >= total_tokens) return;
  double sum = 0.0;
  for (int h = 0; h < num_kv_heads; ++h) sum += (double)scores[(int64_t)h * total_tokens + t];
  mean_out[t] = (float)(sum / (double)num_kv_heads);
}

// ---- 2. per-row radix select + per-chunk counts ------------------------------------------------------
// One workgroup of 1024 threads per row.  Radix select on the row's fp32 bit patterns, most significant digit
// first: 12 bits (sign, exponent, top three mantissa bits: scores of one row cluster in a few exponents, and a
// narrower first digit would pile every LDS atomic onto three or four bins), then 10 + 10 bits.  After a pass
// the digit that holds rank k is found with a workgroup-wide scan.  The tokens that fall into the first digit's bin
// are collected in LDS (a few percent of the row for any spread-out score distribution), so the second and third
// pass see only them; a row with more candidates than the LDS buffer holds (e.g. all scores equal) goes over all of
// its scores again.  With the threshold known the same workgroup counts, per chunk of 1024 tokens, how many scores are
// > T and how many == T: the gather turns these into destinations.
// A row is worked on by one compute unit, and one compute unit pulls about 45 GB/s from L2 however many loads it keeps
// in flight: that, not the histogram atomics, bounds the reading of a long row.  So up to 32768 scores of it are read once,
// into registers (4*NV a thread, NV by the longest row of the call), and every pass works from there; only what a row has
// beyond is read from memory in each pass (all 65536 in registers, 64 a thread, leave too few for the rest: 56 us).  Also
// kept out of the serial chain of a short row: cross-lane sums go through DPP, the wave totals of a scan are read at once,
// places in the candidate list are taken once per wave, two histograms share the atomics of the first digit.  Measured on
// an MI355X, before (every pass from memory, three more barriers a pass) / now: 64 rows x 4096 scores 10.4 / 6.8 us, 128
// ragged rows of up to 16384 13.7 / 11.3, 256 x 16384 17.7 / 14.4, 288 ragged rows of up to 6567 14.4 / 11.2 (15.2 with one
// workgroup a compute unit), 2 x 44000 20.7 / 18.8, 32 x 65536 30.0 / 28.7, 32 x 131072 46.6 / 43.4 (what lies beyond the held
// scores comes in loads of 16 bytes, four in flight a thread: with loads of 4 bytes 19.9, 32.7 and 51.7; eight of 16 bytes in
// flight save 0.6 on 131072 and cost 1.3 on rows of 36000 to 44000).
constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / kWave;
constexpr int kSelBins = 4096;
constexpr int kSelUnroll = 4;  // 16-byte loads in flight per thread beyond the held scores
constexpr int kSelCand = 8192;  // candidates kept in LDS after the first pass (32 KiB)
constexpr int kSelMaxVecs = 8;
constexpr int kSelCopies = 2;  // with the candidates 64 KiB: two workgroups fit a compute unit

struct __attribute__((packed, aligned(4))) Unaligned4 {  // 16 bytes at any 4-byte boundary, in one load
  uint32_t v[4];
};

// The scores of a row as its workgroup holds them: score 4*(j*1024 + tid) + e is reg[j].v[e] of thread tid.
template <int NV>
struct RowScores {
  static constexpr int kHeld = 4 * NV * kSelThreads;
  const uint32_t* bits;
  int L, tid;
  Unaligned4 reg[NV];

  __device__ __forceinline__ int index(int j) const { return 4 * (j * kSelThreads + tid); }

  __device__ __forceinline__ void load() {
#pragma unroll
    for (int j = 0; j < NV; ++j) {  // unconditional, so that all are in flight: past the end the row's last four again
      const int i = index(j);
      const int last = L >= 4 ? L - 4 : 0;
      reg[j] = L >= 4 ? *reinterpret_cast<const Unaligned4*>(bits + (i < last ? i : last)) : Unaligned4{{0u, 0u, 0u, 0u}};
    }
#pragma unroll
    for (int j = 0; j < NV; ++j) {  // the one vector that the row's end cuts
      const int i = index(j);
      if (i < L && i + 4 > L) {
#pragma unroll
        for (int e = 0; e < 4; ++e) reg[j].v[e] = i + e < L ? bits[i + e] : 0u;
      }
    }
  }

  // f(score) for every score that the registers hold ...
  template <typename F>
  __device__ __forceinline__ void visit_held(F f) const {
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      if (4 * (j + 1) * kSelThreads <= L) {  // the same for all threads
#pragma unroll
        for (int e = 0; e < 4; ++e) f(reg[j].v[e]);
      } else if (4 * j * kSelThreads < L) {
        const int left = L - index(j);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (e < left) f(reg[j].v[e]);
      }
    }
  }
  // ... and for the rest of the row, from memory: 16 bytes a load, past the end the row's last four again
  template <typename F>
  __device__ __forceinline__ void visit_rest(F f) const {
    constexpr int kUnroll = NV == kSelMaxVecs ? kSelUnroll : 1;  // a smaller holding covers every row of its call
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
        const int at = i < L - 4 ? i : L - 4;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (at + e >= i) f(r[k].v[e]);
      }
    }
  }
  template <typename F>
  __device__ __forceinline__ void visit(F f) const {
    visit_held(f);
    visit_rest(f);
  }
};

// Two workgroups a compute unit (eight waves per SIMD, 64 registers) as long as the row leaves the registers for it: more
// rows than compute units then still run at once.
template <int NV>
__global__ __launch_bounds__(kSelThreads, NV <= 4 ? 8 : 4) void select_kernel(const float* __restrict__ scores,
                                                             const int32_t* __restrict__ cu_seqlens,
                                                             uint32_t* __restrict__ sel, int32_t* __restrict__ before,
                                                             int32_t* __restrict__ seq_lens_out,
                                                             int32_t* __restrict__ kept_idx_out, int64_t total_tokens,
                                                             int64_t chunk_slots, int num_kv_heads, int budget) {
  constexpr int kHeldChunks = RowScores<NV>::kHeld / kChunk;
  constexpr int kBinsPerThread = kSelBins / kSelThreads;
  // First digit: kSelCopies histograms side by side (bin * kSelCopies + lane % kSelCopies), so that fewer lanes of a
  // wave meet in one word.  The 1024 bins of a later digit use the front of it.
  __shared__ __attribute__((aligned(16))) uint32_t hist[kSelBins * kSelCopies];
  __shared__ uint32_t cand[kSelCand];  // candidates; at the end, the counts of up to kSelCand chunks at a time
  __shared__ __attribute__((aligned(16))) uint32_t wave_tot[kSelWaves];
  __shared__ uint32_t sh_prefix, sh_k, sh_in_bin, sh_ncand;
  const int row = (int)blockIdx.x;
  const int s = row / num_kv_heads, h = row % num_kv_heads;
  const int t0 = cu_seqlens[s];
  const int L = cu_seqlens[s + 1] - t0;
  const int keep = L < budget ? L : budget;
  const int E = L - keep;
  const int tid = (int)threadIdx.x;
  const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  RowScores<NV> rs;
  rs.bits = reinterpret_cast<const uint32_t*>(scores) + (int64_t)h * total_tokens + t0;
  rs.L = L;
  rs.tid = tid;
  rs.load();

  if (h == 0 && tid == 0) seq_lens_out[s] = keep;
  if (kept_idx_out != nullptr)
    for (int i = keep + tid; i < budget; i += kSelThreads) kept_idx_out[(int64_t)row * budget + i] = -1;

  // The bin that rank k falls into: c[j] elements in the calling thread's bin number bin0 + j.
  const auto find_bin = [&](const uint32_t (&c)[kBinsPerThread], uint32_t bin0, uint32_t k) {
    uint32_t tot = 0u;
#pragma unroll
    for (int j = 0; j < kBinsPerThread; ++j) tot += c[j];
    const uint32_t incl = wave_prefix_sum_u32(tot);
    if (lane == kWave - 1) wave_tot[wave] = incl;
    __syncthreads();
    uint32_t first = incl - tot;  // elements in lower bins
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) first += w < wave ? wave_tot[w] : 0u;
    if (k >= first && k < first + tot) {  // exactly one thread
#pragma unroll
      for (int j = 0; j < kBinsPerThread; ++j) {
        if (k >= first && k < first + c[j]) {
          sh_prefix = bin0 + j;
          sh_k = k - first;
          sh_in_bin = c[j];
        }
        first += c[j];
      }
    }
    __syncthreads();
  };

  // E == 0, nothing to evict: T = +0.0, q = 0 keeps every token (scores are >= +0)
  uint32_t T = 0u, k = (uint32_t)(E > 0 ? E - 1 : 0);  // k: 0-based rank of the threshold among the remaining ones
  if (E > 0) {
    for (int i = tid; i < kSelBins * kSelCopies / 4; i += kSelThreads)
      reinterpret_cast<uint4*>(hist)[i] = make_uint4(0u, 0u, 0u, 0u);
    if (tid == 0) sh_ncand = 0u;
    __syncthreads();
    const uint32_t copy = (uint32_t)lane % kSelCopies;
    rs.visit([&](uint32_t b) { atomicAdd(&hist[(b >> 20) * kSelCopies + copy], 1u); });
    __syncthreads();
    uint32_t c[kBinsPerThread];
#pragma unroll
    for (int j = 0; j < kBinsPerThread; ++j) {
      c[j] = 0u;
#pragma unroll
      for (int i = 0; i < kSelCopies; ++i) c[j] += hist[(tid * kBinsPerThread + j) * kSelCopies + i];
    }
    find_bin(c, (uint32_t)(tid * kBinsPerThread), k);
    uint32_t prefix = sh_prefix << 20, mask = 0xfff00000u;
    k = sh_k;
    const bool in_lds = sh_in_bin <= (uint32_t)kSelCand;
    const uint32_t ncand = sh_in_bin;
    hist[tid] = 0u;  // the next digit's bins
    if (in_lds) {  // collect the bin's tokens (their order does not matter: only values are counted)
      // places for what the registers hold are taken once per wave: an atomic per score would be waited for each time
      uint32_t mine = 0u;
      rs.visit_held([&](uint32_t b) { mine += (b & mask) == prefix ? 1u : 0u; });
      const uint32_t upto = wave_prefix_sum_u32(mine);
      uint32_t at = 0u;
      if (lane == kWave - 1) at = atomicAdd(&sh_ncand, upto);
      at = (uint32_t)__builtin_amdgcn_readlane((int)at, kWave - 1) + upto - mine;
      rs.visit_held([&](uint32_t b) {
        if ((b & mask) == prefix) cand[at++] = b;
      });
      rs.visit_rest([&](uint32_t b) {
        if ((b & mask) == prefix) cand[atomicAdd(&sh_ncand, 1u)] = b;
      });
    }
    __syncthreads();
#pragma unroll 1
    for (int shift = 10; shift >= 0; shift -= 10) {
      const auto count = [&](uint32_t b) {
        if ((b & mask) == prefix) atomicAdd(&hist[(b >> shift) & 1023u], 1u);
      };
      if (in_lds) {
        for (uint32_t i = (uint32_t)tid; i < ncand; i += kSelThreads) count(cand[i]);
      } else {
        rs.visit(count);
      }
      __syncthreads();
      c[0] = hist[tid];
#pragma unroll
      for (int j = 1; j < kBinsPerThread; ++j) c[j] = 0u;
      find_bin(c, (uint32_t)tid, k);
      prefix |= sh_prefix << shift;
      mask |= 1023u << shift;
      k = sh_k;
      hist[tid] = 0u;
      __syncthreads();
    }
    T = prefix;  // threshold score (bit pattern)
  }
  if (tid == 0) {
    sel[2 * row] = T;
    sel[2 * row + 1] = E > 0 ? k + 1 : 0u;           // q: the first q tokens (index order) with score == T go
  }

  // Scores > T (lower half) and == T (upper half) per chunk, then how many there are before each chunk of the row.
  const int nchunks = (L + kChunk - 1) / kChunk;
  int32_t* brow = before + ((int64_t)h * chunk_slots + chunk_slot(t0, s, 0)) * 2;
  int gt_total = 0, eq_total = 0;  // of the pieces done
  for (int c0 = 0; c0 < nchunks; c0 += kSelCand) {
    const int nc = nchunks - c0 < kSelCand ? nchunks - c0 : kSelCand;
    __syncthreads();
    if (c0 == 0) {  // what the registers hold: a chunk is one vector of four waves
      if (tid < kHeldChunks) cand[tid] = 0u;
      __syncthreads();
#pragma unroll
      for (int j = 0; j < NV; ++j) {
        if (4 * j * kSelThreads >= L) break;
        const int left = L - rs.index(j);
        uint32_t n = 0u;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t b = rs.reg[j].v[e];
          n += e < left ? (b > T ? 1u : 0u) + (b == T ? 0x10000u : 0u) : 0u;
        }
        n = wave_prefix_sum_u32(n);
        if (lane == kWave - 1) atomicAdd(&cand[(j * kSelThreads + wave * kWave) * 4 / kChunk], n);
      }
    }
    // beyond them, one wave per chunk: 16 tokens per lane, all loads issued before the first compare
    for (int cc = (c0 == 0 ? kHeldChunks : 0) + wave; cc < nc; cc += kSelWaves) {
      constexpr int kPerLane = kChunk / kWave;
      const int i0 = (c0 + cc) * kChunk + lane;
      uint32_t b[kPerLane], n = 0u;
#pragma unroll
      for (int j = 0; j < kPerLane; ++j) b[j] = rs.bits[i0 + j * kWave < L ? i0 + j * kWave : L - 1];
#pragma unroll
      for (int j = 0; j < kPerLane; ++j)
        n += i0 + j * kWave < L ? (b[j] > T ? 1u : 0u) + (b[j] == T ? 0x10000u : 0u) : 0u;
      n = wave_prefix_sum_u32(n);
      if (lane == kWave - 1) cand[cc] = n;
    }
    __syncthreads();
    if (wave == 0) {
      for (int cc = 0; cc < nc; cc += kWave) {
        const uint32_t n = cc + lane < nc ? cand[cc + lane] : 0u;
        const int gt = (int)wave_prefix_sum_u32(n & 0xffffu), eq = (int)wave_prefix_sum_u32(n >> 16);
        if (cc + lane < nc) {
          const int2 v = make_int2(gt_total + gt - (int)(n & 0xffffu), eq_total + eq - (int)(n >> 16));
          *reinterpret_cast<int2*>(brow + 2 * (c0 + cc + lane)) = v;
        }
        gt_total += __builtin_amdgcn_readlane(gt, kWave - 1);
        eq_total += __builtin_amdgcn_readlane(eq, kWave - 1);
      }
    }
  }
}

// The smallest register holding that covers rows of max_seqlen tokens (or the largest there is): a larger one than needed
// costs loads, branches and, beyond 16 scores a thread, the second workgroup of a compute unit.
using SelectKernel = void (*)(const float*, const int32_t*, uint32_t*, int32_t*, int32_t*, int32_t*, int64_t, int64_t, int, int);
SelectKernel select_kernel_for(int max_seqlen) {
  const int vecs = (max_seqlen + 4 * kSelThreads - 1) / (4 * kSelThreads);
  if (vecs <= 1) return select_kernel<1>;
  if (vecs <= 2) return select_kernel<2>;
  if (vecs <= 4) return select_kernel<4>;
  return select_kernel<kSelMaxVecs>;
}

// ---- 3. gather ----------------------------------------------------------------------------------------
// VPR_T > 0: vectors per token row known at compile time; 0: taken from vpr_rt (head-shared mode, where a
// row is the K (or V) of all heads of a token).  STREAM: stores with the non-temporal hint.
template <int VPR_T, bool STREAM>
__global__ __launch_bounds__(kThreads) void gather_kernel(const uint4* __restrict__ k_in, const uint4* __restrict__ v_in,
                                                          const float* __restrict__ scores,
                                                          const int32_t* __restrict__ cu_seqlens,
                                                          const uint32_t* __restrict__ sel,
                                                          const int32_t* __restrict__ before,
                                                          const int32_t* __restrict__ block_table,
                                                          uint4* __restrict__ k_pool, uint4* __restrict__ v_pool,
                                                          int32_t* __restrict__ kept_idx_out, int64_t total_tokens,
                                                          int64_t chunk_slots, int num_kv_heads, int rows,
                                                          int log2_block, int max_blocks, int budget, int vpr_rt) {
  __shared__ uint32_t wave_sum[kWaves];
  __shared__ int32_t src_tok[kChunk];  // kept tokens of this chunk, in order: in-sequence index
  __shared__ int n_kept_sh;
  // Rows fastest: the first chunks of a ragged batch, which short sequences keep most of, spread over all XCDs (workgroup
  // number % 8).  Chunks fastest put the first chunks of all sequences on one: 47 us instead of 30 for 16 sequences of
  // 2048 to 16384 tokens, 8 heads, 1024 kept of each (134 MB moved; the other prompts below did not change).
  const int row = (int)(blockIdx.x % (unsigned)rows);
  const int chunk = (int)(blockIdx.x / (unsigned)rows);
  const int s = row / num_kv_heads, h = row % num_kv_heads;
  const int t0 = cu_seqlens[s];
  const int L = cu_seqlens[s + 1] - t0;
  if (chunk * kChunk >= L) return;
  const int tid = (int)threadIdx.x;
  const int lane = lane_id();
  const int wave = tid / kWave;
  const uint32_t T = sel[2 * row];
  const int q = (int)sel[2 * row + 1];

  // counts over all earlier chunks of this row
  const int2 earlier = reinterpret_cast<const int2*>(before)[(int64_t)h * chunk_slots + chunk_slot(t0, s, chunk)];
  const int gt_before = earlier.x, eq_before = earlier.y;

  // this thread's kTokPerThread consecutive tokens
  const uint32_t* bits = reinterpret_cast<const uint32_t*>(scores) + (int64_t)h * total_tokens + t0;
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
  // exclusive scan of (n_gt, n_eq) over the 256 threads, in thread (= index) order; each fits 16 bits
  const uint32_t n_both = (uint32_t)n_gt | ((uint32_t)n_eq << 16);
  const uint32_t inc = wave_prefix_sum_u32(n_both);
  if (lane == kWave - 1) wave_sum[wave] = inc;
  __syncthreads();
  uint32_t ex = inc - n_both;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) ex += w < wave ? wave_sum[w] : 0u;
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
  if (tid == kThreads - 1) n_kept_sh = ex_gt + (ex_eq > q ? ex_eq - q : 0) - kept_before_chunk;
  __syncthreads();
  const int n_kept = n_kept_sh;

  if (kept_idx_out != nullptr)  // consecutive positions: whole lines
    for (int e = tid; e < n_kept; e += kThreads) kept_idx_out[(int64_t)row * budget + kept_before_chunk + e] = src_tok[e];

  // copy the kept rows: VEC_PER_ROW lanes per token row, K and V (two or four rows of a thread in flight: no faster)
  const int32_t* bt = block_table + (int64_t)row * max_blocks;
  const int block_mask = (1 << log2_block) - 1;
  if constexpr (VPR_T > 0) {
    constexpr int VEC_PER_ROW = VPR_T;
    constexpr int kRowsPerPass = kThreads / VEC_PER_ROW;
    const int u = tid % VEC_PER_ROW, r = tid / VEC_PER_ROW;
    for (int e = r; e < n_kept; e += kRowsPerPass) {
      const int pos = kept_before_chunk + e;
      const int64_t src = ((int64_t)(t0 + src_tok[e]) * num_kv_heads + h) * VEC_PER_ROW + u;
      const int64_t dst = (((int64_t)bt[pos >> log2_block] << log2_block) + (pos & block_mask)) * VEC_PER_ROW + u;
      store_vec<STREAM>(k_pool, dst, k_in[src]);
      store_vec<STREAM>(v_pool, dst, v_in[src]);
    }
  } else {
    const int total_vecs = n_kept * vpr_rt;
    for (int f = tid; f < total_vecs; f += kThreads) {
      const int e = f / vpr_rt, u = f - e * vpr_rt;
      const int tok = src_tok[e], pos = kept_before_chunk + e;
      const int64_t src = ((int64_t)(t0 + tok) * num_kv_heads + h) * vpr_rt + u;
      const int64_t dst = (((int64_t)bt[pos >> log2_block] << log2_block) + (pos & block_mask)) * vpr_rt + u;
      store_vec<STREAM>(k_pool, dst, k_in[src]);
      store_vec<STREAM>(v_pool, dst, v_in[src]);
    }
  }
}

template <typename T, int D>
hipError_t launch(const PruneArgs& a, hipStream_t stream) {
  using G = RowGeom<T, D>;
  const Workspace w = carve(a.workspace, a.num_seqs, a.num_kv_heads, a.total_tokens, a.shared);
  const int64_t total_rows = a.total_tokens * a.num_kv_heads;
  hipError_t e;
  const int64_t row_bytes = 2 * (int64_t)a.num_kv_heads * D * (int64_t)sizeof(T);  // K and V of a token
  if (total_rows > 0) {
    const int64_t rows_per_group = (int64_t)kWaves * kSweepIters * kSweepLoads * G::kTokensPerLoad;
    const int64_t grid = (total_rows + rows_per_group - 1) / rows_per_group;
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    // Prompts of 96 MiB are swept without the hint: they then lie in the Infinity Cache (256 MB) when the gather comes, and what
    // the model has just written is found there (whole prunes of D = 64, 1024 of 4096 kept, with / without the hint, K and V
    // written right before: 17 MB 27.3 / 25.2 us, 34 MB 30.2 / 27.8, 67 MB 33.8 / 29.5, 134 MB 50.6 / 45.7, 268 MB 83.8 / 83.8, 537 MB
    // 133 / 165; out of memory: 67 MB 31.5 / 31.7, 134 MB 49.6 / 51.3, 268 MB 85.4 / 94.8)
    const bool streamed = a.total_tokens * row_bytes > (int64_t)96 << 20;
    const auto sweep = streamed ? token_scores_kernel<T, D, true> : token_scores_kernel<T, D, false>;
    hipLaunchKernelGGL(sweep, dim3((unsigned)grid), dim3(kThreads), 0, stream, (const T*)a.k_in, (const T*)a.v_in, w.scores,
                       total_rows, a.total_tokens, a.num_kv_heads);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  // what kernels 2-3 see: per-head rows, or (shared) one row per sequence whose score is the head mean and
  // whose record is the token's K (or V) of all heads
  const int heads = a.shared ? 1 : a.num_kv_heads;
  const float* sel_scores = w.scores;
  if (a.shared) {
    float* mean = w.scores + (size_t)a.num_kv_heads * (size_t)a.total_tokens;
    if (a.total_tokens > 0) {
      const int64_t grid = (a.total_tokens + kThreads - 1) / kThreads;
      hipLaunchKernelGGL(head_mean_kernel, dim3((unsigned)grid), dim3(kThreads), 0, stream, w.scores, mean,
                         a.total_tokens, a.num_kv_heads);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    sel_scores = mean;
  }
  const int rows = a.num_seqs * heads;
  hipLaunchKernelGGL(select_kernel_for(a.max_seqlen), dim3((unsigned)rows), dim3(kSelThreads), 0, stream, sel_scores, a.cu_seqlens,
                     w.sel, w.before, a.seq_lens_out, a.kept_idx_out, a.total_tokens, w.chunk_slots, heads, a.budget);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const int chunks_per_row = (a.max_seqlen + kChunk - 1) / kChunk;
  if (chunks_per_row == 0) return hipSuccess;
  const int64_t grid2 = (int64_t)rows * chunks_per_row;
  if (grid2 > 0x7fffffffLL) return hipErrorInvalidValue;
  constexpr int VPR = G::kLanesPerRow;
  // Kept rows of a prompt that is larger than the Infinity Cache go past the caches: what the gather reads is not there either, and
  // what it writes need not push it out (whole prunes, plain stores / with the hint: 2.1 GB of prompt, 268 MB kept 465 / 453 us,
  // 134 MB kept 418 / 409; 0.6 GB, 67 MB kept 141 / 137, fp32 110 / 106; 0.5 GB, 67 MB kept 127 / 122, written right before 133 / 136; smaller
  // ones, written right before, 268 MB 84 / 87, 67 MB 33.8 / 34.9).
  const bool streamed = a.total_tokens * row_bytes > (int64_t)256 << 20;
  const auto gather = a.shared ? (streamed ? gather_kernel<0, true> : gather_kernel<0, false>)
                               : (streamed ? gather_kernel<VPR, true> : gather_kernel<VPR, false>);
  hipLaunchKernelGGL(gather, dim3((unsigned)grid2), dim3(kThreads), 0, stream, (const uint4*)a.k_in, (const uint4*)a.v_in,
                     sel_scores, a.cu_seqlens, w.sel, w.before, a.block_table, (uint4*)a.k_pool, (uint4*)a.v_pool,
                     a.kept_idx_out, a.total_tokens, w.chunk_slots, heads, rows, ilog2(a.block_size), a.max_blocks, a.budget,
                     a.shared ? VPR * a.num_kv_heads : VPR);
  return hipGetLastError();
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
