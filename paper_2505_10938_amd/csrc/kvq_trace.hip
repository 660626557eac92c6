// Outlier-token competition as kernels of its own: one group per launch (one workgroup of 4 wavefronts
// per unit), or the groups of a whole prompt (all at once).
#include "kvq_common.h"
#include "kvq_trace_core.h"

#include <cmath>
#include <type_traits>

namespace kvq {

namespace {

// All loads of the first phase (state, stored scores, the group's K rows) go out together; the
// rows that move (evicted -> auxiliary pool, new -> pool) are loaded together in a second phase.
template <int G>
__global__ void __launch_bounds__(trace_core::kWorkers) trace_kernel(
    Dims d, int32_t group_index, const __half* __restrict__ k_group, const __half* __restrict__ v_group,
    int64_t unit_stride, __half* pool_k, __half* pool_v, int32_t* pool_idx, double* pool_score, int32_t* pool_count,
    int32_t* aux_count, int32_t* frozen, uint8_t* __restrict__ selected) {
  const int tid = threadIdx.x;
  const int ul = blockIdx.x;
  const int64_t u = d.unit0 + ul;
  uint8_t* sel = selected + (int64_t)ul * G;
  if (d.N == 0) {                                      // no pool: nothing is ever selected
    if (tid < G) sel[tid] = 0;
    return;
  }
  const __half* gk = k_group + (int64_t)ul * unit_stride;
  const __half* gv = v_group + (int64_t)ul * unit_stride;
  const trace_core::UnitPool p =
      trace_core::unit_pool(d, u, pool_k, pool_v, pool_idx, pool_score, pool_count, aux_count, frozen);
  trace_core::Loaded<G> in;
  trace_core::load<G>(in, d, p, gk, tid);
  trace_core::compete<G>(in, d, group_index, p, gk, gv, sel, nullptr, tid);
}

// ---- the competitions of a whole prompt -----------------------------------------------------------
// The state that the group-by-group competitions leave can be computed for all groups at once: a token is
// selected if fewer than N tokens of its own and the earlier groups have a smaller key (score, index); the
// pool is the N smallest of the selected tokens; with S_i tokens selected up to group i, S_i - min(N, (i+1)G)
// have fallen out, and the first group where that exceeds A is where tracing stops.  None of it depends on
// the order of insertion, and only selected tokens can displace one, so that counting needs few of them.
//
// prompt_compete_kernel, one workgroup per unit, does all of it, T tokens (one per thread) at a time: scores, a first
// look by the segment's own bounds or the pool's largest key, then a count among the few tokens left; the Key rows of
// the next T tokens are in flight meanwhile, and nothing is read any more once tracing has stopped.  With as many
// units as compute units the read of the Keys bounds it; one workgroup alone reads about 1024 tokens in 10 us.
// Few units and a long prompt: prompt_candidates_kernel, one workgroup per unit and segment of 1024 tokens, computes
// the scores and flags the tokens that may be selected, judged by the segment alone (for N = 8 and random scores about
// 50 of 1024); prompt_compete_kernel then gathers the flagged ones.  It reads all Keys, however early tracing stops.
//
// Us of a prompt's whole call (G = 32, N = 8, 2-bit; the quantization, 89 us per 256 x 4096 tokens, included), three sets of rows
// in turn, by segments / one workgroup per unit:
//   8 units x 8192 tokens; 32 x 8192, A = 32     29 /  66;  50 /  87
//   128 x 4096, A = 32; A = 16                   82 /  88;  81 /  78
//   256 x 4096, A = 32; A = 16                  159 / 150; 158 / 143
//   128 x 8192; 192 x 8192, A = 32              157 / 164; 242 / 219
//   64 x 16384, A = 32; A = 16                  163 / 226; 163 / 158
//   1024 x 4096, A = 32; A = 16                 758 / 703; 710 / 565   (T = 512)
//   1024 x 1120, A = 32                         239 / 201              (T = 512)

constexpr int kSegment = 1024;                         // tokens of a workgroup of prompt_candidates_kernel
constexpr int kRound = 128;                            // tokens ranked at a time: at least a whole group

typedef unsigned long long u64;

// A first look that is cheap and lets few entries through that will not be selected: an entry must be among
// the N smallest of any prefix of the entries that ends with its group or before.  The N-th smallest score
// of the first 32, 64, 128 and 256 entries is found by bisection over coarse scores (fp32 rounded, the first
// 8 bits of the significand: the order is kept, only some neighbours become equal), one wavefront each.
// What takes the time is the ballots, 16 ns each.  Few members: the N-th smallest of the lanes' own smallest entries serves as
// well, N entries are no larger, and seldom does one lane have two of the N (N = 8: a bound by 6 % too many entries).
// 64 / 16 ballots, the whole call: a prompt of 8191 tokens that joins, 8 kv heads, 4 layers, 51.8 / 50.6 us; 32 units of 8192 tokens 54.5 / 53.2; 24 of 1500 31.9 / 31.2.
// (Short prompts of few units, 4 .. 32 units of 200 .. 500 tokens: 0.4 .. 0.5 us of 11 .. 15 less with few members; with N = 32, which
// gains nothing by the second way and by the order of rows below, 0.1 .. 0.2 more.)
constexpr int kPrefixes = 4;
constexpr int kCoarseBits = 16;
constexpr int kFewMembers = 16;
template <class Score>
__device__ __forceinline__ uint32_t coarse_score(Score score) {
  return score < (Score)8388608.0 ? __float_as_uint((float)score) >> (31 - kCoarseBits) : (1u << kCoarseBits) - 1u;
}
__device__ __forceinline__ void prefix_bounds(const uint32_t* coarse, int n, int N, uint32_t* bound, int wave, int lane) {
  if (wave >= kPrefixes) return;
  constexpr int kWords = (32 << (kPrefixes - 1)) / 64;
  const int p = min(32 << wave, n);
  uint32_t v[kWords], t = 0;
#pragma unroll
  for (int k = 0; k < kWords; ++k) v[k] = k * 64 + lane < p ? coarse[k * 64 + lane] : ~0u;
  auto bisect = [&](auto words_c) {                      // the N-th smallest of the first `words` of each lane
    constexpr int words = decltype(words_c)::value;
#pragma unroll
    for (int b = kCoarseBits - 1; b >= 0; --b) {
      int at_most = 0;
#pragma unroll
      for (int k = 0; k < words; ++k) at_most += __popcll(__ballot(v[k] <= (t | ((1u << b) - 1u))));
      t |= at_most < N ? 1u << b : 0u;
    }
  };
  if (N <= kFewMembers) {
#pragma unroll
    for (int k = 1; k < kWords; ++k) v[0] = min(v[0], v[k]);
    bisect(std::integral_constant<int, 1>{});
  } else {
    bisect(std::integral_constant<int, kWords>{});
  }
  if (lane == 0) bound[wave] = t;                      // (fewer than N entries: the largest value there is)
}

// The order of the competition, (score, token index) ascending, as one integer.  A score is a multiple of
// 2^-24 below 2^23: added to 2^28 it leaves score * 2^24 in the significand (47 bits).  Below it stands the
// place among the entries that compete (ascending by token index), and 0 for a member of the pool, which is
// older than all of them.  Sums that are no such number (infinities, NaN: not supported) rank last.
constexpr int kPlaceBits = 11;
constexpr u64 kPlaceMask = (1ull << kPlaceBits) - 1ull;
__device__ __forceinline__ u64 competition_key(double score, int place) {
  const u64 fixed = score < 8388608.0 ? (u64)__double_as_longlong(score + 268435456.0) & ((1ull << 52) - 1ull)
                                      : (1ull << 47) - 1ull;
  return (fixed << kPlaceBits) | (u64)place;
}
template <int T>
struct CompeteLds {
  u64 key[T];                                          // the entries competing, ascending by token index
  int32_t idx[T];
  uint32_t coarse[T];                                  // their scores, coarsely
  uint32_t bound[kPrefixes];
  u64 mask[8 * T / 64];                                // marked entries, 64 per word
  u64 r_key[kRound];                                   // the round's
  int32_t r_idx[kRound];
  uint32_t r_less[kRound];                             // smaller keys: up to the entry's group, and << 16 in all
  u64 p_key[2][64];                                    // the pool, ascending; two buffers taken in turn
  uint32_t p_less[64];
  uint8_t r_sel[kRound];
  int32_t cut_group, cut_rank, cut_at;
};

// Ranks of marked entries: `before(w)` = marked entries in the words ahead of word w.  Every wavefront
// computes the sums for itself (two words per lane), no barrier.
struct MaskRanks {
  int ex0, ex1, total;                                 // ahead of words 2 lane, 2 lane + 1; in all
  __device__ __forceinline__ MaskRanks(const u64* mask, int n_words, int lane) {
    const int c0 = 2 * lane < n_words ? __popcll(mask[2 * lane]) : 0;
    const int c1 = 2 * lane + 1 < n_words ? __popcll(mask[2 * lane + 1]) : 0;
    const int incl = wave_scan(c0 + c1);
    ex0 = incl - c0 - c1;
    ex1 = incl - c1;
    total = __builtin_amdgcn_readlane(incl, 63);
  }
  __device__ __forceinline__ int before(int w) const {  // (uniform w)
    return (w & 1) ? __builtin_amdgcn_readlane(ex1, w >> 1) : __builtin_amdgcn_readlane(ex0, w >> 1);
  }
};

// Sums over a team of 16 lanes of ROWS (16 or 8) values per lane: lane `sub` returns the sum over the team of
// s(sub * ROWS / 16).  Where the lanes of a team held the same sum of one row after the other and the first of them
// put it away, a row took 12 instructions to add up and 25 under a mask of four lanes; this way 16 rows take 15
// exchanges of 7 and are put away by all lanes at once.  The sums are exact, in any order.  s is asked for the rows in
// the order of first_to_last.  (With the competition's loads issued as the rows are used up, 256 units x 4096 tokens,
// the whole call 180.7 -> 177.4 us; 32 units x 8191, with candidates, 59.5 -> 57.7.)
constexpr int first_to_last(int rows, int i) {            // i with its bits in reverse
  int q = 0;
  for (int b = 1; b < rows; b *= 2) q = 2 * q + ((i / b) & 1);
  return q;
}
template <int ROWS, int BIT = 0, class S>
__device__ __forceinline__ auto team_sums(int sub, const S& s, int q = 0) {
  if constexpr (BIT == 4) {
    return s(q);
  } else {
    const auto a = team_sums<ROWS, BIT + 1>(sub, s, q);
    if constexpr (ROWS == 8 && BIT == 0) {
      return a + row_partner<BIT>(a);
    } else {
      const auto b = team_sums<ROWS, BIT + 1>(sub, s, q + (1 << BIT) * ROWS / 16);
      const bool upper = (sub >> BIT) & 1;              // (the partner's bit is the other way)
      return (upper ? b : a) + row_partner<BIT>(upper ? a : b);
    }
  }
}

// About the sum of eight magnitudes, in fp32: one instruction each, where the exact sum in fp64 takes three.
__device__ __forceinline__ float about_abs_sum8(uint4 w) {
  float a = 0.0f, b = 0.0f;
  auto add = [&](uint32_t x) {
    asm("v_fma_mix_f32 %0, |%1|, 1.0, %0 op_sel_hi:[1,0,0]" : "+v"(a) : "v"(x));
    asm("v_fma_mix_f32 %0, |%1|, 1.0, %0 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(b) : "v"(x));
  };
  add(w.x), add(w.y), add(w.z), add(w.w);
  return a + b;
}

// L1 scores of the Key rows row(0) .. row(n - 1), the sums of `sum8` of their eighths, handed to put(e, score) by one lane
// each: 16 lanes per row, kInFlight (8 or 16) rows of a team of lanes in flight.
template <int kInFlight, class Sum8, class Row, class Put>
__device__ __forceinline__ void score_rows(int n, int tid, Sum8 sum8, Row row, Put put) {
  constexpr int kTeams = kSegment / 16;
  const int team = tid >> 4, sub = tid & 15;
  // (a whole segment: 64 rows next to each other per wavefront, four at a time, as in prompt_compete_kernel)
  const int first = n == kSegment ? (team >> 2) * 64 + (team & 3) : team, step = n == kSegment ? 4 : kTeams;
  for (int i0 = 0; i0 * kTeams < n; i0 += kInFlight) {
    uint4 w[kInFlight];
#pragma unroll
    for (int i = 0; i < kInFlight; ++i) {
      const int q = first_to_last(kInFlight, i);
      w[q] = *(const uint4*)(row(min(first + (i0 + q) * step, n - 1)) + sub * 8);
    }
    const auto sc = team_sums<kInFlight>(sub, [&](int q) { return sum8(w[q]); });
    const int e = first + (i0 + sub * kInFlight / 16) * step;
    if ((kInFlight == 16 || !(sub & 1)) && e < n) put(e, sc);
  }
}

// One round: ranks the next entries (from entry `pos` on, of the n in LDS) and updates the pool (P members in
// buffer `cur`, which changes).  Entry j of the round, j < the result, is L.r_idx[j] and was selected if
// L.r_sel[j].  `pos` becomes the first entry not looked at.  `may`: entry `tid` passed the first look.  Four
// barriers, the last one at the end.
template <int G, int T>
__device__ __forceinline__ int compete_round(CompeteLds<T>& L, int n, bool may, int& pos, int N, int& P, int& cur, int tid) {
  constexpr int kGroupShift = G == 32 ? 5 : G == 64 ? 6 : 7;
  constexpr int kWaves = T / 64;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const u64 max_key = L.p_key[cur][N - 1];             // (counts only where P == N)
  const u64 key = L.key[tid];
  const int ix = L.idx[tid];
  const u64 m = __ballot(may && tid >= pos && tid < n && (P < N || key < max_key));
  if (lane == 0) L.mask[wave] = m;
  if (tid < kRound) L.r_less[tid] = 0;
  if (tid < 64) L.p_less[tid] = 0;
  __syncthreads();
  const MaskRanks ranks(L.mask, T / 64, lane);
  const bool marked = (m >> lane) & 1ull;
  const int rank = ranks.before(wave) + __popcll(m & ((1ull << lane) - 1ull));
  int nr = ranks.total, next = n;
  if (nr == 0) {                                       // uniform: nothing can enter the pool any more
    __syncthreads();                                   // (the marks have been read by all)
    pos = n;
    return 0;
  }
  if (nr > kRound) {                                   // uniform: only the groups that are in whole
    if (tid == 0) L.cut_rank = L.cut_at = T;
    if (marked && rank == kRound) L.cut_group = ix >> kGroupShift;
    __syncthreads();
    if (marked && (ix >> kGroupShift) >= L.cut_group) {
      atomicMin(&L.cut_rank, rank);
      atomicMin(&L.cut_at, tid);
    }
    __syncthreads();
    nr = min(L.cut_rank, kRound);
    next = L.cut_at;
  }
  if (marked && rank < nr) {
    L.r_key[rank] = key;
    L.r_idx[rank] = ix;
  }
  __syncthreads();
  // A lane counts for entries lane, 64 + lane and for member lane; the wavefronts share what is counted.
  const u64 none = ~0ull;
  const u64 kp = lane < P ? L.p_key[cur][lane] : none;
  const u64 k0 = lane < nr ? L.r_key[lane] : none, k1 = 64 + lane < nr ? L.r_key[64 + lane] : none;
  const int end0 = L.r_idx[lane] | (G - 1), end1 = L.r_idx[64 + lane] | (G - 1);
  uint32_t c0 = 0, c1 = 0, cp = 0;
#pragma unroll
  for (int i = 0; i < kRound / kWaves; ++i) {
    const int j = i * kWaves + wave;
    if (j < nr) {
      const u64 jk = L.r_key[j];
      const int jx = L.r_idx[j];
      c0 += jk < k0 ? (jx <= end0 ? 0x10001u : 0x10000u) : 0u;
      c1 += jk < k1 ? (jx <= end1 ? 0x10001u : 0x10000u) : 0u;
      cp += jk < kp ? 1u : 0u;
    }
  }
  for (int p = wave; p < P; p += kWaves) {
    const u64 pk = L.p_key[cur][p];
    c0 += pk < k0 ? 0x10001u : 0u;
    c1 += pk < k1 ? 0x10001u : 0u;
  }
  if (lane < nr) atomicAdd(&L.r_less[lane], c0);
  if (64 + lane < nr) atomicAdd(&L.r_less[64 + lane], c1);
  if (lane < P) atomicAdd(&L.p_less[lane], cp);
  __syncthreads();
  if (tid < nr) {
    const int own = (int)(L.r_less[tid] & 0xFFFFu), all = (int)(L.r_less[tid] >> 16);
    L.r_sel[tid] = own < N ? 1 : 0;
    if (all < N) L.p_key[cur ^ 1][all] = L.r_key[tid] & ~kPlaceMask;
  } else if (tid >= kRound && tid < kRound + P) {
    const int p = tid - kRound, to = p + (int)L.p_less[p];
    if (to < N) L.p_key[cur ^ 1][to] = L.p_key[cur][p];
  }
  __syncthreads();
  P = min(N, P + nr);
  cur ^= 1;
  pos = next;
  return nr;
}

// Is entry e, token idx (n entries, `at(p)` = token of entry p), among those that the first look lets through?
// `margin`: coarse scores by which the bounds are too low at worst.
template <int G, class At>
__device__ __forceinline__ bool may_be_selected(const uint32_t* coarse, const uint32_t* bound, int n, int e, int idx, At at,
                                                uint32_t margin = 0) {
  uint32_t b = (1u << kCoarseBits) - 1u;
#pragma unroll
  for (int i = 0; i < kPrefixes; ++i)
    if ((32 << i) <= n && at((32 << i) - 1) <= (idx | (G - 1))) b = bound[i];   // (bounds fall with the prefix)
  return coarse[e] <= b + margin;
}

// grid (units, segments, layers).  Requires N > 0.  The scores are sums in fp32: at most 127 roundings, 2^-17 of the sum,
// so that a coarse score is one off at most, the bounds too, and what is at or below a bound by exact scores is at or
// below it by two more.
// Sixteen rows of a team in flight, so that a workgroup makes one trip to memory; in 64 registers, so that two workgroups fit
// a compute unit.  Whole calls, G = 32, N = 8, three sets of rows in turn, exact sums with eight rows / fp32 sums with eight /
// with sixteen in 67 registers / in 64: joining prompts of 8000 tokens, 8 kv heads, one layer 30.8 / 28.4 / 28.3 / 28.2 us, of
// 3000, 4 kv heads, 4 layers 30.8 / 28.7 / 28.5 / 28.6, of 8191, 8 kv heads, 8 layers (512 workgroups) 87.5 / 87.1 / 87.2 / 86.1;
// 384 workgroups (96 units x 4096 tokens, 48 x 8192) 66.7 / 66.2 / 67.2 / 65.7 and 68.4 / 67.7 / 68.7 / 67.3; 512 (64 x 8192)
// 83.8 / 83.3 / 84.2 / 82.8; 1024 (64 x 16384) 164.7 / 163.7 / 166.1 / 164.1.
template <int G, int LAYERS>
__global__ void __launch_bounds__(kSegment) __attribute__((amdgpu_waves_per_eu(8))) prompt_candidates_kernel(
    Dims d, int32_t n_tok, int64_t unit_stride, uint8_t* __restrict__ selected, LayerRows<LAYERS> src) {
  __shared__ uint32_t coarse[kSegment];
  __shared__ uint32_t bound[kPrefixes];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ul = blockIdx.x, t0 = blockIdx.y * kSegment, layer = LAYERS > 1 ? blockIdx.z : 0;
  const int n = min(kSegment, n_tok - t0);
  const __half* rows = src.k[layer] + (int64_t)ul * unit_stride + (int64_t)t0 * kHeadDim;
  score_rows<16>(n, tid, about_abs_sum8, [&](int e) { return rows + e * kHeadDim; },
                 [&](int e, float sc) { coarse[e] = coarse_score(sc); });
  __syncthreads();
  prefix_bounds(coarse, n, d.N, bound, wave, lane);
  __syncthreads();
  // (segments begin with a group: token numbers inside the segment number its groups as well)
  if (tid < n)
    selected[((int64_t)layer * d.units_per_layer + ul) * n_tok + t0 + tid] =
        may_be_selected<G>(coarse, bound, n, tid, tid, [](int p) { return p; }, 2u) ? 1 : 0;
}

// grid (units, 1, layers).  FLAGGED: the tokens that can be selected are flagged in `selected`, else all of them are looked at, T
// at a time, the Key rows of the next T in flight meanwhile: each row is asked for when the one before it in its
// registers has been added up, so that memory is not idle during the sums.  Pools are taken to be empty on entry (a
// prompt starts a sequence) and are not read.
template <int G, int T, bool FLAGGED, int LAYERS>
__global__ void __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(4))) prompt_compete_kernel(
    Dims d, int32_t n_tok, int64_t unit_stride, __half* pool_k, __half* pool_v, int32_t* pool_idx, double* pool_score,
    int32_t* pool_count, int32_t* aux_count, int32_t* frozen, uint8_t* __restrict__ selected, LayerRows<LAYERS> src) {
  constexpr int kGroupShift = G == 32 ? 5 : G == 64 ? 6 : 7;
  constexpr int kListed = 64 + 64 + kRound;            // at most N + A selected tokens before the last round
  constexpr int kWaves = T / 64;
  __shared__ CompeteLds<T> L;
  __shared__ u64 s_key[kListed];                       // every token selected so far, ascending by index
  __shared__ int32_t s_idx[kListed];
  __shared__ int32_t s_out[kListed];                   // the group at which it falls out (none: kStays)
  __shared__ int32_t slot_idx[128];                    // token of each pool and auxiliary slot
  constexpr int32_t kStays = 0x7FFFFFFF;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ul = blockIdx.x, layer = LAYERS > 1 ? blockIdx.z : 0;
  const int64_t u = d.unit0 + (int64_t)layer * d.layer_units + ul;
  uint8_t* sel = selected + ((int64_t)layer * d.units_per_layer + ul) * n_tok;
  const int N = d.N, A = d.A;
  if (N == 0) {                                        // no pool: nothing is ever selected
    for (int i = tid; i < n_tok; i += T) sel[i] = 0;
    return;
  }
  const __half* __restrict__ kr = src.k[layer] + (int64_t)ul * unit_stride;
  const __half* __restrict__ vr = src.v[layer] + (int64_t)ul * unit_stride;
  const u64 below = (1ull << lane) - 1ull;
  int P = 0, cur = 0, S = 0;                           // pool members, pool buffer, selected tokens
  bool stopped = false;
  int t0 = 0;                                          // tokens before t0 have been looked at
  // Key rows of tokens t .., sixteen per team of 16 lanes
  constexpr int kTeams = T / 16, kRows = 16, kFewRows = 8;
  const int team = tid >> 4, sub = tid & 15;
  uint4 w[kRows];
  // Row q of a team is token first + q * step of those.  Of a whole 1024 a wavefront has 64 next to each other, 16 KB that
  // it asks for 1 KB at a time, where the teams' rows taken in turn had every wavefront jump by 16 KB from load to load
  // (whole call, 256 units x 4096 tokens 158.5 -> 154.9 us, x 8192 292.7 -> 290.2; with T = 512 it cost 0.5 %).
  constexpr bool kNextToEachOther = T == 1024;
  int first = team, step = kTeams;
  auto place = [&](int t) {
    const bool whole = kNextToEachOther && n_tok - t >= T;
    first = whole ? (team >> 2) * 64 + (team & 3) : team;
    step = whole ? 4 : kTeams;
  };
  auto load_row = [&](int t, int q) {
    w[q] = *(const uint4*)(kr + (int64_t)min(t + first + q * step, n_tok - 1) * kHeadDim + sub * 8);
  };
  auto load_rows = [&](int t) {
    place(t);
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
      const int q = first_to_last(kRows, i);
      if (n_tok - t >= T || t + q * kTeams < n_tok) load_row(t, q);      // uniform
    }
  };
  auto put_score = [&](int e, double sc) {
    L.key[e] = competition_key(sc, e + 1);
    L.coarse[e] = coarse_score(sc);
  };
  if constexpr (!FLAGGED) load_rows(0);
  while (t0 < n_tok && !stopped) {
    int n, next;                                       // entries that compete now, first token of the next ones
    if constexpr (FLAGGED) {
      // ---- the next candidates, at most T (whole groups), and their scores
      constexpr int kPer = 8;
      const int here = min(kPer * T, n_tok - t0);
      u64 m[kPer];
      uint8_t f[kPer];
#pragma unroll
      for (int k = 0; k < kPer; ++k) {
        const int t = k * T + tid;
        f[k] = sel[t0 + min(t, here - 1)];
      }
#pragma unroll
      for (int k = 0; k < kPer; ++k) {
        const int t = k * T + tid;
        m[k] = __ballot(t < here && f[k]);
        if (lane == 0) L.mask[k * kWaves + wave] = m[k];
      }
      __syncthreads();
      const MaskRanks ranks(L.mask, kPer * T / 64, lane);
      auto rank_of = [&](int k) -> int {
        return ((m[k] >> lane) & 1ull) ? ranks.before(k * kWaves + wave) + __popcll(m[k] & below) : kPer * T;
      };
      // A group never competes in parts: t0 is always the first token of a group (a window holds whole groups, and
      // where a window is cut short, it ends, and the next one begins, with a whole group, flagged or not).
      n = ranks.total;
      next = t0 + here;
      if (n > T) {                                // uniform: only the groups that are in whole
#pragma unroll
        for (int k = 0; k < kPer; ++k)
          if (rank_of(k) == T) L.cut_group = (t0 + k * T + tid) >> kGroupShift;
        __syncthreads();
        next = __builtin_amdgcn_readfirstlane(L.cut_group) << kGroupShift;
        const int w = (next - t0) >> 6, bit = (next - t0) & 63;
        n = ranks.before(w) + __popcll(L.mask[w] & ((1ull << bit) - 1ull));
      }
#pragma unroll
      for (int k = 0; k < kPer; ++k) {
        const int t = k * T + tid, r = rank_of(k);
        if (r < n) {
          L.idx[r] = t0 + t;
          sel[t0 + t] = 0;                               // the selected ones are flagged again at the end
        }
      }
      __syncthreads();
      score_rows<8>(n, tid, trace_core::abs_sum8, [&](int e) { return kr + (int64_t)L.idx[e] * kHeadDim; }, put_score);
    } else {
      n = min(T, n_tok - t0);
      next = t0 + n;
      const int e = first + sub * step;
      double sc;
      if (next < n_tok) {                              // uniform: n = T, and a row's place is taken by one of the next T
        place(next);
        sc = team_sums<kRows>(sub, [&](int q) {
          const double s = trace_core::abs_sum8(w[q]);
          load_row(next, q);
          return s;
        });
      } else if (n > kFewRows * kTeams) {
        sc = team_sums<kRows>(sub, [&](int q) { return q * kTeams < n ? trace_core::abs_sum8(w[q]) : 0.0; });
      } else {
        // At most eight rows per team (short prompts, and the end of others): each for itself, kept by the lane that
        // puts it away.  Folding sixteen of which eight or more are missing takes longer: whole call, all folded / so,
        // 8 units of 64 tokens 12.2 / 11.6 us, of 160 13.1 / 12.5; 128 units of 352 22.4 / 22.1; of 512, 24.0 / 24.1.
        // (Up to twelve rows this way the compiler put all of them into scratch memory.)
        sc = 0.0;
#pragma unroll
        for (int q = 0; q < kFewRows; ++q) {
          if (q * kTeams >= n) break;                  // uniform
          const double s = trace_core::team_sum_f64(trace_core::abs_sum8(w[q]));
          if (sub == q) sc = s;
        }
      }
      if (e < n) put_score(e, sc);
      if (tid < n) {
        L.idx[tid] = t0 + tid;
        sel[t0 + tid] = 0;                             // the selected ones are flagged at the end
      }
    }
    __syncthreads();
    bool may = true;
    if (FLAGGED || P < N) {                            // (once the pool is full its largest key lets fewer through)
      prefix_bounds(L.coarse, n, N, L.bound, wave, lane);
      __syncthreads();
      may = may_be_selected<G>(L.coarse, L.bound, n, tid, L.idx[tid], [&](int p) { return L.idx[p]; });
    }
    // ---- select among them
    int pos = 0;
    while (pos < n && !stopped) {
      const int nr = compete_round<G, T>(L, n, may, pos, N, P, cur, tid);
      // The round's selected tokens join the list.  With token k of the list (from 0), min(N, tokens so far)
      // of k + 1 are in the pool; the others have fallen out and must fit in the auxiliary pool.
      // (every wavefront works this out for itself: lane = entries lane, 64 + lane of the round)
      const bool c0 = lane < nr && L.r_sel[lane], c1 = 64 + lane < nr && L.r_sel[64 + lane];
      const int i0 = L.r_idx[lane], i1 = L.r_idx[64 + lane];
      const u64 b0 = __ballot(c0), b1 = __ballot(c1);
      const int k0 = S + __popcll(b0 & below), k1 = S + __popcll(b0) + __popcll(b1 & below);
      const u64 o0 = __ballot(c0 && k0 + 1 - min(N, (i0 | (G - 1)) + 1) > A);
      const u64 o1 = __ballot(c1 && k1 + 1 - min(N, (i1 | (G - 1)) + 1) > A);
      u64 t0m = b0, t1m = b1;
      if (o0 | o1) {                                   // uniform: tracing stops at the first group that overflows
        const int first = o0 ? __builtin_amdgcn_readlane(i0, __ffsll((long long)o0) - 1)
                             : __builtin_amdgcn_readlane(i1, __ffsll((long long)o1) - 1);
        const int start = first & ~(G - 1);
        t0m = __ballot(c0 && i0 < start);
        t1m = __ballot(c1 && i1 < start);
        stopped = true;
      }
      if (wave == 0 && c0) {
        s_key[k0] = (L.r_key[lane] & ~kPlaceMask) | (u64)k0;
        s_idx[k0] = i0;
      }
      if (wave == 1 && c1) {
        s_key[k1] = (L.r_key[64 + lane] & ~kPlaceMask) | (u64)k1;
        s_idx[k1] = i1;
      }
      S += __popcll(t0m) + __popcll(t1m);
    }
    t0 = next;
  }
  for (int t = t0 + tid; t < n_tok; t += T) sel[t] = 0;   // after the stop nothing is selected
  __syncthreads();
  // ---- the S selected tokens (at most N + A): pool, ascending by key, or auxiliary pool, in the order they
  // fall out (by group; inside a group the largest key first).  One wavefront per token, lane = the others.
  u64 os[2];
  int oi[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int e = 64 * h + lane;
    os[h] = e < S ? s_key[e] : ~0ull;
    oi[h] = e < S ? s_idx[e] : 0;
  }
  for (int e = wave; e < S; e += kWaves) {
    const u64 es = s_key[e];
    const int ei = s_idx[e];
    const u64 b0 = __ballot(os[0] < es), b1 = __ballot(os[1] < es);
    const int rank = __popcll(b0) + __popcll(b1);
    int out = kStays;
    if (rank >= N) {                                   // the N-th smaller key, in token order, displaces it
      const u64 n0 = __ballot(((b0 >> lane) & 1ull) && __popcll(b0 & below) == N - 1);
      const u64 n1 = __ballot(((b1 >> lane) & 1ull) && __popcll(b0) + __popcll(b1 & below) == N - 1);
      out = (n0 ? __builtin_amdgcn_readlane(oi[0], __ffsll((long long)n0) - 1)
                : __builtin_amdgcn_readlane(oi[1], __ffsll((long long)n1) - 1)) >> kGroupShift;
    } else if (lane == 0) {
      slot_idx[rank] = ei;
    }
    if (lane == 0) {
      s_out[e] = out;
      sel[ei] = 1;
    }
  }
  __syncthreads();
  const int in_pool = min(N, S), aux_n = S - in_pool;
  if (aux_n > 0) {
    const int out0 = lane < S ? s_out[lane] : kStays, out1 = 64 + lane < S ? s_out[64 + lane] : kStays;
    for (int e = wave; e < S; e += kWaves) {
      const int out = s_out[e];
      if (out == kStays) continue;
      const u64 es = s_key[e];
      const u64 b0 = __ballot(out0 != kStays && (out0 < out || (out0 == out && es < os[0])));
      const u64 b1 = __ballot(out1 != kStays && (out1 < out || (out1 == out && es < os[1])));
      if (lane == 0) slot_idx[in_pool + __popcll(b0) + __popcll(b1)] = s_idx[e];
    }
    __syncthreads();
  }
  // the unit's state, and the members' rows bit for bit from the prompt: 16 lanes per row
  const int64_t slot0 = u * d.pool_slots;
  if (tid == 0) {
    pool_count[u] = in_pool;
    aux_count[u] = aux_n;
    frozen[u] = stopped ? 1 : 0;
  }
  for (int j = tid >> 4; j < S; j += T / 16) {
    const int idx = slot_idx[j];
    const int64_t slot = slot0 + (j < in_pool ? j : N + (j - in_pool));
    const uint4 kw = *(const uint4*)(kr + (int64_t)idx * kHeadDim + sub * 8);
    const uint4 vw = *(const uint4*)(vr + (int64_t)idx * kHeadDim + sub * 8);
    const double sc = trace_core::team_sum_f64(trace_core::abs_sum8(kw));
    if (sub == 0) {
      pool_idx[slot] = idx;
      pool_score[slot] = sc;
    }
    *(uint4*)(pool_k + slot * kHeadDim + sub * 8) = kw;
    *(uint4*)(pool_v + slot * kHeadDim + sub * 8) = vw;
  }
}

// Do the segments of a prompt go to workgroups of their own (if there are several)?  By segments a call's Keys take
// 10 us per 250 units and segment plus about 20 us for two launches one after the other, by unit 10 us per segment and
// about 12: `early` is the number of segments at which the two are even.  (These were the times when the line was drawn.  One
// workgroup per unit has gained more since: whole call, A = 32, by segments / by unit, 4096 tokens: 128 units 82 / 88 us, 160
// 99 / 100, 192 117 / 116, 256 159 / 150; 8192: 128 157 / 164, 160 201 / 192, 192 242 / 219; 16384: 192 525 / 471.  From 160 units on
// the line lies too far towards the segments, by up to a tenth of the call.)
// By unit it is as well if tracing has stopped by then in all units, to be expected with a small auxiliary pool: were
// the scores independent, group i would displace N / i tokens on average, about Poisson, E = N ln(groups, or tokens / N)
// in all; Chernoff's bound on at most A of them, for all units, is held against e^-2.  (If that is wrong for the
// prompt at hand one workgroup per unit reads all of it after all, or the segments read what they need not.)
bool by_segments(const Dims& d, int32_t units, int32_t n_tok) {
  if (d.N == 0 || n_tok <= kSegment) return false;
  const double segments = (double)n_tok / kSegment, early = 0.75 + units * segments / 250.0;
  if (early >= segments) return false;
  const double groups = early * kSegment / (d.G > d.N ? d.G : d.N), e = d.N * std::log(groups > 1.0 ? groups : 1.0);
  if (e <= d.A) return true;
  const double log_p = d.A - e + (d.A > 0 ? d.A * std::log(e / d.A) : 0.0);
  return log_p + std::log((double)units) >= -2.0;
}

}  // namespace

hipError_t launch_prefill_trace(const Dims& d, int32_t n_groups, const PromptRows& rows,
                                const kvq_pool& pool, uint8_t* selected, hipStream_t s) {
  const int32_t n_tok = n_groups * d.G, units = d.units_per_layer * rows.layers;
  auto compete = [&](auto kern, int threads, const auto& at) {
    hipLaunchKernelGGL(kern, dim3(d.units_per_layer, 1, rows.layers), dim3(threads), 0, s, d, n_tok, rows.unit_stride,
                       (__half*)pool.pool_k, (__half*)pool.pool_v, pool.pool_idx, pool.pool_score, pool.pool_count,
                       pool.aux_count, pool.frozen, selected, at);
  };
  // Threads of a workgroup: 1024 where every unit can have a compute unit to itself; with more units 512, so that two
  // workgroups fit one, and 256 for prompts no longer than that.  1024 units x 300 tokens, T = 1024 / 512 / 256: 92 /
  // 70 / 64 us; x 600: 138 / 120 / 121.
  auto of_layers = [&](auto group, auto count) {
    constexpr int G = decltype(group)::value, L = decltype(count)::value;
    const LayerRows<L> at = layer_rows<L>(rows);
    if (by_segments(d, units, n_tok)) {
      hipLaunchKernelGGL((prompt_candidates_kernel<G, L>),
                         dim3(d.units_per_layer, (n_tok + kSegment - 1) / kSegment, rows.layers), dim3(kSegment), 0, s,
                         d, n_tok, rows.unit_stride, selected, at);
      compete(prompt_compete_kernel<G, 1024, true, L>, 1024, at);
    } else if (units > 2 * kComputeUnits && n_tok <= 256) {
      compete(prompt_compete_kernel<G, 256, false, L>, 256, at);
    } else if (units > kComputeUnits) {
      compete(prompt_compete_kernel<G, 512, false, L>, 512, at);
    } else {
      compete(prompt_compete_kernel<G, 1024, false, L>, 1024, at);
    }
  };
  auto go = [&](auto group) {
    if (rows.layers == 1) of_layers(group, std::integral_constant<int, 1>{});
    else of_layers(group, std::integral_constant<int, kPromptLayers>{});
  };
  switch (d.G) {
    case 32: go(std::integral_constant<int, 32>{}); break;
    case 64: go(std::integral_constant<int, 64>{}); break;
    default: go(std::integral_constant<int, 128>{}); break;
  }
  return hipGetLastError();
}

// Empty pools for the units of the launch (a new sequence in a slot that held another).  grid (units, layers).
__global__ void reset_pools_kernel(Dims d, int32_t* pool_count, int32_t* aux_count, int32_t* frozen) {
  const int ul = blockIdx.x * blockDim.x + threadIdx.x;
  if (ul >= d.units_per_layer) return;
  const int64_t u = d.unit0 + (int64_t)blockIdx.y * d.layer_units + ul;
  pool_count[u] = 0;
  aux_count[u] = 0;
  frozen[u] = 0;
}
hipError_t launch_reset_pools(const Dims& d, int32_t layers, const kvq_pool& pool, hipStream_t s) {
  hipLaunchKernelGGL(reset_pools_kernel, dim3((d.units_per_layer + 63) / 64, layers), dim3(64), 0, s, d,
                     pool.pool_count, pool.aux_count, pool.frozen);
  return hipGetLastError();
}

hipError_t launch_trace(const Dims& d, int32_t group_index, const __half* k_group, const __half* v_group,
                        int64_t unit_stride, const kvq_pool& pool, uint8_t* selected, hipStream_t s) {
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(d.units_per_layer), dim3(trace_core::kWorkers), 0, s, d, group_index, k_group,
                       v_group, unit_stride, (__half*)pool.pool_k, (__half*)pool.pool_v, pool.pool_idx,
                       pool.pool_score, pool.pool_count, pool.aux_count, pool.frozen, selected);
  };
  switch (d.G) {
    case 32: go(trace_kernel<32>); break;
    case 64: go(trace_kernel<64>); break;
    default: go(trace_kernel<128>); break;
  }
  return hipGetLastError();
}

}  // namespace kvq
