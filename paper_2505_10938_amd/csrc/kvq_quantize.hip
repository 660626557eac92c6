// Residual append and group quantization (mean replacement, Eq. 2 per group, packing), and the
// fused group step (append + outlier competition + quantization in one launch).
#include "kvq_common.h"
#include "kvq_trace_core.h"

#include <type_traits>

// The integer code decisions must not depend on how the compiler fuses multiplies and adds.
#pragma clang fp contract(off)

namespace kvq {

namespace {

// ---- residual append: one row of 128 fp16 per unit, K and V -----------------------------------
__global__ void __launch_bounds__(128) append_kernel(Dims d, const __half* __restrict__ k_new,
                                                     const __half* __restrict__ v_new, __half* __restrict__ k_res,
                                                     __half* __restrict__ v_res, int32_t row) {
  const int ul = blockIdx.x;                       // unit inside the layer
  const int64_t u = d.unit0 + ul;
  const int tid = threadIdx.x;                     // 64 threads for K, 64 for V, 4 bytes each
  const int which = tid >> 6, lane = tid & 63;
  const uint32_t* src = (const uint32_t*)((which ? v_new : k_new) + (int64_t)ul * kHeadDim);
  uint32_t* dst = (uint32_t*)((which ? v_res : k_res) + (u * d.res_rows + row) * kHeadDim);
  dst[lane] = src[lane];
}

// ---- Eq. 2 for one value against its group's (min, step) -------------------------------------
// step is the fp16-rounded step as float; code = number of thresholds (k + 1/2) * step reached
// by fl32(x - mn).  The products are exact in fp32, so the decision is IEEE-reproducible.
__device__ inline uint32_t quant_code(float x, float mn, float step, int levels) {
  if (step == 0.0f) return 0u;
  const float t = x - mn;
  uint32_t code = 0;
  for (int k = 0; k < levels; ++k) {
    const float thr = ((float)k + 0.5f) * step;
    code += (t >= thr) ? 1u : 0u;
  }
  return code;
}

// The same decision as quant_code, as a binary search: code k is reached when fl32(x - mn) >= (2k - 1) * h
// with h = step / 2 (exact products again: 2k - 1 has 5 bits, h 11).  Returns 2 * code as a float.  A group
// whose step is zero passes h = +infinity: no threshold is reached, the code is 0.
template <int BITS>
__device__ __forceinline__ float quant_code_twice(float x, float mn, float h) {
  const float t = x - mn;
  float acc = 0.0f;
#pragma unroll
  for (int l = BITS - 1; l >= 0; --l) {
    const float c = (float)(2 << l);
    const float w = acc + (c - 1.0f);
    acc = (t >= w * h) ? acc + c : acc;
  }
  return acc;
}
__device__ __forceinline__ float half_step_of(__half st) {
  const float s = __half2float(st);
  return s == 0.0f ? __uint_as_float(0x7F800000u) : 0.5f * s;
}
// 2 * code (as returned above) put at bit position p of a packed word (a compile-time position of the
// first field of a word; bits beyond 31 wrap around)
template <int BITS>
__device__ __forceinline__ uint32_t place_twice(float acc, int p) {
  const uint32_t b = (uint32_t)acc;
  return (b << (p - 1)) | (p + BITS > 32 ? b >> (33 - p) : 0u);
}

// fp16 step from a group's min and max: fl32(fl32(max - min) * c_b) rounded to nearest even.
__device__ inline __half step_of(float mn, float mx, int bits) {
  const float c = bits == 2 ? __uint_as_float(0x3EAAAAABu) : __uint_as_float(0x3D888889u);  // 1/3, 1/15
  const float d = mx - mn;
  float s32 = d * c;
  // Keep the fp32 product as its own rounding step: without this the compiler merges the
  // multiply and the fp16 conversion into one instruction with a single rounding.
  asm volatile("" : "+v"(s32));
  return __float2half_rn(s32);
}

constexpr int kRowB = 272;   // LDS row: 128 fp16 + 16 bytes of padding (spreads rows over the banks)

__device__ inline float half_at(const unsigned char* p) { return __half2float(*(const __half*)p); }
__device__ inline float lo_half(uint32_t w) { return __half2float(__ushort_as_half((unsigned short)(w & 0xFFFFu))); }
__device__ inline float hi_half(uint32_t w) { return __half2float(__ushort_as_half((unsigned short)(w >> 16))); }

constexpr int kQuantThreads = 1024;
// From this many groups in one launch on, prompt_quantize_kernel takes them (1024 threads keep a group of 128 tokens longest,
// and one workgroup of them fills half a compute unit).  Us of calls recorded in a graph, three sets of rows in turn,
// quantize_kernel / prompt_quantize_kernel; 2-bit, then 4-bit codes:
//   prompt without a pool   G = 32, 128 groups 6.7 / 5.7, 6.9 / 6.3   256 7.0 / 5.8, 7.2 / 6.5    512 9.0 / 7.2, 9.5 / 8.6    768 11.8 / 8.6, 12.4 / 10.0
//                           G = 64,  32 groups 7.8 / 5.9, 8.2 / 6.5   512 12.9 / 9.3, 14.0 / 11.0
//                           G = 128,  8 groups 10.8 / 6.5, 11.7 / 7.7 256 14.1 / 9.4, 15.3 / 11.0
//   with a pool, N = 8      G = 32, 256 groups 17.5 / 16.5, 17.7 / 17.2;  G = 64, 32 14.3 / 12.0, 14.7 / 12.8;  G = 128, 8 17.4 / 12.4, 18.3 / 13.6
//   kvq_quantize_group      G = 32, 256 units 5.0 / 4.0, 5.2 / 4.5;  G = 64, 32 5.8 / 3.9, 6.1 / 4.5;  G = 128, one 8.5 / 4.4, 9.5 / 5.4
// Its code is 29 .. 37 KB, the other's 5 .. 6.  With a decode step, products and elementwise kernels ahead of each call, so
// that neither finds its code in the instruction cache, a group of 128 tokens still gains 4 us and one of 64 tokens 1 .. 2.  With
// G = 32 the two are even at 256 groups (ten shapes, N = 0 and 8: 2-bit 0.5 us faster in the mean, -0.9 .. 1.3, 4-bit 0.3 slower,
// -1.6 .. 0.8); from 320 on it is ahead there too (4-bit 0.3 .. 1.1 us, from 640 on 2 .. 3).
constexpr int64_t prompt_groups(int G) { return G == 32 ? 256 : G == 64 ? 32 : 1; }

// Minimum and maximum over groups of `n` adjacent lanes (n = 4, 8 or 16).
__device__ inline void team_minmax(float& mn, float& mx, int n) {
  mn = fminf(mn, row_partner<0>(mn));
  mx = fmaxf(mx, row_partner<0>(mx));
  mn = fminf(mn, row_partner<1>(mn));
  mx = fmaxf(mx, row_partner<1>(mx));
  if (n > 4) {
    mn = fminf(mn, row_partner<2>(mn));
    mx = fmaxf(mx, row_partner<2>(mx));
  }
  if (n > 8) {
    mn = fminf(mn, row_partner<3>(mn));
    mx = fmaxf(mx, row_partner<3>(mx));
  }
}

// LDS of the quantization: the whole group (G x 128, K and V) and its meta.
template <int G>
struct QuantLds {
  unsigned char* sk;     // [G] rows of kRowB bytes
  unsigned char* sv;     // [G] rows
  float2* skm;           // [128] K meta: {zero, step / 2 (+infinity for a zero step)}
  float2* svm;           // [vgroups][G] V meta, the same pair
  uint8_t* ssel;         // [G] selected flags
  __device__ QuantLds(unsigned char* smem, int vgroups) {
    sk = smem;
    sv = sk + G * kRowB;
    skm = (float2*)(sv + G * kRowB);
    svm = skm + kHeadDim;
    ssel = (uint8_t*)(svm + G * vgroups);
  }
};
template <int G>
size_t quant_lds_bytes(int vgroups) { return (size_t)2 * G * kRowB + kHeadDim * 8 + (size_t)G * vgroups * 8 + G; }

// The group's rows, 16 bytes per thread: K rows first, then V rows.  (Of a vector type of the compiler's: HIP's uint4 is
// a structure, which it copies as memory.  Where nothing says that the rows are not written to meanwhile, quantize_kernel
// put such copies into scratch memory with G = 64 and 128, each behind a wait for its load.  A prompt's whole call with
// structures / vectors, 16 units: G = 64, 300 tokens 15.8 / 14.6 us, 3000 37.3 / 33.8; G = 128, 700 24.6 / 20.9.)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
template <int G>
struct GroupRows {
  static constexpr int kLoads = 2 * G * 16 / kQuantThreads;   // 1, 2 or 4
  u32x4 rw[kLoads];
};
template <int G>
__device__ __forceinline__ void rows_issue(GroupRows<G>& r, const __half* gk, const __half* gv, int tid) {
#pragma unroll
  for (int q = 0; q < GroupRows<G>::kLoads; ++q) {
    const int e = q * kQuantThreads + tid;
    const int kv = e / (G * 16), rem = e % (G * 16);
    r.rw[q] = *(const u32x4*)((kv ? gv : gk) + (rem >> 4) * kHeadDim + (rem & 15) * 8);
  }
}
template <int G>
__device__ __forceinline__ void rows_to_lds(const GroupRows<G>& r, const QuantLds<G>& L, int tid) {
#pragma unroll
  for (int q = 0; q < GroupRows<G>::kLoads; ++q) {
    const int e = q * kQuantThreads + tid;
    const int kv = e / (G * 16), rem = e % (G * 16);
    *(u32x4*)((kv ? L.sv : L.sk) + (rem >> 4) * kRowB + (rem & 15) * 16) = r.rw[q];
  }
}

// Quantization of the group held in LDS (rows stored, not yet synchronized): mean replacement of
// the rows flagged (`flag` = this thread's token, threads below G), meta, codes, mask words.
// Every thread of the 1024-thread workgroup calls it.  (u, group_index) say where the group is stored
// (place_of_group): the unit and the group's index, or, in a paged cache, the plane and the page.
template <int BITS, int G>
__device__ __forceinline__ void quantize_body(const Dims& d, int64_t u, int32_t group_index, const QuantLds<G>& L,
                                              uint8_t flag, uint8_t* __restrict__ k_codes,
                                              uint32_t* __restrict__ k_meta, uint8_t* __restrict__ v_codes,
                                              uint32_t* __restrict__ v_meta, uint32_t* __restrict__ mask, int tid) {
  unsigned char* sk = L.sk;
  unsigned char* sv = L.sv;
  float2* skm = L.skm;
  float2* svm = L.svm;
  uint8_t* ssel = L.ssel;
  const int gv_shift = 31 - __clz(d.Gv);             // Gv is a power of two
  if (tid < G) ssel[tid] = flag;
  const int any = __syncthreads_or(flag);

  // mean replacement: per-channel mean of the original rows of all G tokens, exact fp64 sum,
  // scaled by the power of two 1/G, rounded to fp32 then fp16.
  if (any) {
    // four adjacent lanes per (matrix, channel), each summing every fourth token (the adds are exact,
    // so the split changes nothing), then each replacing the flagged ones among its own tokens
    const int part = tid & 3, c = (tid >> 2) & 127;
    unsigned char* rows = (tid < 512) ? sk : sv;
    double sum = 0.0;
#pragma unroll 8
    for (int t = part; t < G; t += 4) sum += (double)half_at(rows + t * kRowB + 2 * c);
    sum += row_partner<0>(sum);
    sum += row_partner<1>(sum);
    const float m32 = (float)(sum / (double)G);
    const __half m16 = __float2half_rn(m32);
    for (int t = part; t < G; t += 4)
      if (ssel[t]) *(__half*)(rows + t * kRowB + 2 * c) = m16;
    __syncthreads();
  }

  // K meta: 8 adjacent lanes share a channel, each taking every 8th token.
  {
    const int c = tid >> 3, part = tid & 7;
    float mn = half_at(sk + part * kRowB + 2 * c), mx = mn;
#pragma unroll
    for (int t = part + 8; t < G; t += 8) {
      const float x = half_at(sk + t * kRowB + 2 * c);
      mn = fminf(mn, x);
      mx = fmaxf(mx, x);
    }
    team_minmax(mn, mx, 8);
    mn += 0.0f;                                        // a zero minimum is stored as +0 (-0 + +0 = +0)
    if (part == 0) {
      const __half st = step_of(mn, mx, BITS);
      skm[c] = make_float2(mn, half_step_of(st));      // (mn is an fp16 value)
      // global layout of a group's Key meta: fp16 step[128], then fp16 zero[128]
      __half* gm = (__half*)(k_meta + (u * d.groups_per_unit + group_index) * kHeadDim);
      gm[c] = st;
      gm[kHeadDim + c] = __float2half_rn(mn);
    }
  }
  // V meta: Gv / 8 adjacent lanes share a (token, channel group), 8 channels each.
  if (!d.keys_only) {
    const int lanes = d.Gv >> 3;                       // 4, 8 or 16
#pragma unroll 1
    for (int e = tid; e < G * 16; e += kQuantThreads) {
      const int t = e >> 4, c8 = e & 15;               // 8 channels from 8 * c8 on
      const uint4 w = *(const uint4*)(sv + t * kRowB + c8 * 16);
      const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
      float mn = lo_half(ww[0]), mx = mn;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float x0 = lo_half(ww[k]), x1 = hi_half(ww[k]);
        mn = fminf(mn, fminf(x0, x1));
        mx = fmaxf(mx, fmaxf(x0, x1));
      }
      team_minmax(mn, mx, lanes);
      mn += 0.0f;                                      // a zero minimum is stored as +0
      if ((c8 & (lanes - 1)) == 0) {
        const int j = (c8 * 8) >> gv_shift;
        const __half st = step_of(mn, mx, BITS);
        svm[j * G + t] = make_float2(mn, half_step_of(st));
        // global layout of a 32-token block's Value meta (NV = value groups per token):
        // fp16 step[16 token pairs][NV][2], then fp16 zero[16 token pairs][NV][2]
        const int64_t tok = (int64_t)group_index * G + t;
        const int tb = (int)(tok & 31);
        __half* gm = (__half*)(v_meta + (u * d.blocks_per_unit + (tok >> 5)) * 32 * d.vgroups);
        gm[((tb >> 1) * d.vgroups + j) * 2 + (tb & 1)] = st;
        gm[32 * d.vgroups + ((tb >> 1) * d.vgroups + j) * 2 + (tb & 1)] = __float2half_rn(mn);
      }
    }
  }
  __syncthreads();

  // codes: one field (8 codes) of one packed u32 word of K or V per thread step.  Word w of lane l
  // of block blk holds 4/BITS fields; with two fields per word, adjacent lanes hold them.
  constexpr int kWordsPerBlock = 128 * BITS;          // 512*BITS bytes / 4
  constexpr int kFieldsPerWord = 4 / BITS;            // 2 (2-bit) or 1 (4-bit)
  constexpr int nblk = G / kBlockTokens;
  constexpr int kItems = 2 * nblk * kWordsPerBlock * kFieldsPerWord;   // a multiple of 1024
  const int first_block = group_index * nblk;
  const int n_items = d.keys_only ? kItems / 2 : kItems;          // Key words first, then Value words
#pragma unroll 1
  for (int e = tid; e < n_items; e += kQuantThreads) {
    const int kv = e / (kItems / 2);
    const int wf = e % (kItems / 2);
    const int i = wf / kFieldsPerWord, ff = wf % kFieldsPerWord;
    const int blk = i / kWordsPerBlock;
    const int wi = i - blk * kWordsPerBlock;
    // invert word_byte(): byte = 4*wi
    int lane, f0;
    if (BITS == 2) {
      lane = wi >> 2;
      f0 = (wi & 3) * 2;
    } else {
      const int half = wi >> 8;                        // 256 words per 1 KiB half
      lane = (wi & 255) >> 2;
      f0 = half * 4 + (wi & 3);
    }
    const int r = lane >> 4, mn_ = lane & 15;
    const int f = f0 + ff;
    // the word as if the field were the first of its word; the second field of a 2-bit word sits 8 bits up
    uint32_t word = 0;
    float2 ms[8];
    float val[8];
    if (kv == 0) {  // Key: lane = 16 r + m, field = 4 th + cb: 8 consecutive channels of one token
      const int t = 16 * (f >> 2) + mn_;
      const int c0 = 32 * (f & 3) + 8 * r;
      const uint4 xv = *(const uint4*)(sk + (blk * kBlockTokens + t) * kRowB + 2 * c0);
      const uint32_t xs[4] = {xv.x, xv.y, xv.z, xv.w};
#pragma unroll
      for (int x = 0; x < 8; x += 2) {
        const float4 m2 = *(const float4*)(skm + c0 + x);
        ms[x] = make_float2(m2.x, m2.y);
        ms[x + 1] = make_float2(m2.z, m2.w);
      }
#pragma unroll
      for (int x = 0; x < 8; ++x) val[x] = (x & 1) ? hi_half(xs[x >> 1]) : lo_half(xs[x >> 1]);
    } else {        // Value: lane = 16 r + n, field = ct: one channel of 8 consecutive tokens
      const int c = 16 * f + mn_;
      const int t0 = blk * kBlockTokens + 8 * r;
      const float2* pm = svm + (c >> gv_shift) * G + t0;
#pragma unroll
      for (int x = 0; x < 8; x += 2) {
        const float4 m2 = *(const float4*)(pm + x);
        ms[x] = make_float2(m2.x, m2.y);
        ms[x + 1] = make_float2(m2.z, m2.w);
      }
#pragma unroll
      for (int x = 0; x < 8; ++x) val[x] = half_at(sv + (t0 + x) * kRowB + 2 * c);
    }
#pragma unroll
    for (int x = 0; x < 8; ++x)
      word |= place_twice<BITS>(quant_code_twice<BITS>(val[x], ms[x].x, ms[x].y), code_bit(BITS, 0, x));
    if (ff) word = (word << 8) | (word >> 24);
    if (kFieldsPerWord == 2) word |= row_partner_u32<0>(word);      // the word's other field (the adjacent lane)
    if (ff == 0) {
      const int64_t boff = (u * d.blocks_per_unit + first_block + blk) * (int64_t)d.block_bytes;
      ((uint32_t*)((kv ? v_codes : k_codes) + boff))[wi] = word;
    }
  }

  // mask words
  if (tid < nblk) {
    uint32_t w = 0;
    for (int t = 0; t < 32; ++t) w |= (ssel[tid * 32 + t] ? 1u : 0u) << t;
    mask[u * d.blocks_per_unit + first_block + tid] = w;
  }
}

// One workgroup of 16 wavefronts per unit.  Every global load of the kernel is issued before the
// first wait, so a launch costs one trip to memory; the work after it is spread over all 1024
// threads because nothing else hides latency.  LDS: 2 * G * 272 bytes (<= 68 KB) + meta.
template <int BITS, int G, int LAYERS>
__global__ void __launch_bounds__(kQuantThreads) quantize_kernel(
    Dims d, int32_t group_index, int64_t unit_stride, const uint8_t* __restrict__ selected, int64_t selected_unit_stride,
    uint8_t* __restrict__ k_codes, uint32_t* __restrict__ k_meta, uint8_t* __restrict__ v_codes,
    uint32_t* __restrict__ v_meta, uint32_t* __restrict__ mask, int32_t n_groups, int32_t tail_n,
    __half* __restrict__ k_res, __half* __restrict__ v_res, LayerRows<LAYERS> rows) {
  // grid (units, groups + tail blocks, layers): workgroup (ul, gy) with gy < n_groups quantizes the G rows from row
  // gy * G of the unit's rows as group group_index + gy; its flags are
  // selected[(layer * units + ul) * selected_unit_stride + gy * G ..].  The workgroups behind them copy the tail_n
  // rows that follow the last group into ring rows 0 .. of the unit (a whole prompt: the rows that stay in full
  // precision), 16 bytes of K and of V per thread.
  extern __shared__ __align__(16) unsigned char smem[];
  const QuantLds<G> L(smem, d.vgroups);
  const int tid = threadIdx.x;
  const int ul = blockIdx.x, gy = blockIdx.y, layer = LAYERS > 1 ? blockIdx.z : 0;
  const __half* __restrict__ k_rows = rows.k[layer];
  const __half* __restrict__ v_rows = rows.v[layer];
  if (gy >= n_groups) {
    const int i = (gy - n_groups) * kQuantThreads + tid;
    if (i < tail_n * 16) {
      const int64_t src = (int64_t)ul * unit_stride + (int64_t)n_groups * G * kHeadDim;
      const int64_t dst = (d.unit0 + (int64_t)layer * d.layer_units + ul) * d.res_rows * kHeadDim;
      ((uint4*)(k_res + dst))[i] = ((const uint4*)(k_rows + src))[i];
      ((uint4*)(v_res + dst))[i] = ((const uint4*)(v_rows + src))[i];
    }
    return;
  }
  GroupRows<G> group;
  const int64_t row0 = (int64_t)ul * unit_stride + (int64_t)gy * G * kHeadDim;
  rows_issue<G>(group, k_rows + row0, v_rows + row0, tid);
  const int64_t sel0 = ((int64_t)layer * d.units_per_layer + ul) * selected_unit_stride + (int64_t)gy * G;
  uint8_t flag = 0;
  if (tid < G && selected) flag = selected[sel0 + tid];
  const GroupPlace at = place_of_group(d, ul, group_index + gy, layer);
  rows_to_lds<G>(group, L, tid);
  quantize_body<BITS, G>(d, at.row, at.slot, L, flag, k_codes, k_meta, v_codes, v_meta, mask, tid);
}

// ---- many groups per launch (a prompt): one workgroup per group, two wavefronts per block of 32 tokens ----
// The kernel above spreads one group over 1024 threads because a decode step waits for it.  A prompt has
// thousands of groups, and what counts is the instructions spent per group.  Here one wavefront quantizes a block's
// Keys and one its Values, each with a lane-to-element mapping in which the packed words fall out of the lanes that
// computed the codes:
//   Keys:   a lane owns one channel pair for all tokens, so minimum and maximum over the tokens are packed
//           fp16 operations inside the lane (exact: they only select).  It gathers its codes of 8 (2-bit) or
//           4 (4-bit) tokens in one register; the 8 (4) lanes that share a packed word trade fields of it, 3 (2)
//           exchanges after which each has the word of one of the tokens.
//   Values: a lane has 8 channels of 8 tokens.  Minimum and maximum per (token, channel group) are folded over
//           a quad on the packed pair {min, -max} so that each of its lanes ends up with two tokens, whose step, zero
//           and thresholds it works out for the quad.  Codes become words by trades between lanes and between
//           registers, and a lane stores 16 bytes.
// No row goes through LDS, and each is read once: the blocks of a longer group exchange minimum, maximum and, where a
// token is flagged, sums.  What bounds it: the rows and codes on their way (256 units x 4096 tokens, 2-bit: 653 MB in
// 89 us, 7.3 TB/s, the Keys in part from the memory-side cache).  When every code was decided by fp32 comparisons, gathered by
// an OR over the lanes token by token and the Values turned through LDS, it was the instructions, 1900 per block where
// there are now about 1050; when one wavefront took the blocks of a group one after the other, a second read of the Keys.
// Whole calls, three sets of rows in turn, before all that / with the blocks one after the other / now (accesses past the
// caches included): G = 32 183 / 161 / 156 us, 4-bit 231 / 175 / 177; G = 64 188 / 167 / 155; G = 128 217 / 213 / 160, 4-bit 248 /
// 226 / 187.  A joining prompt of 8191 tokens, 8 kv heads, 4 layers: G = 32 59 / 52 / 51, G = 128 79 / 74 / 55.
// Results are those of quantize_body bit for bit (same roundings in the same order; minimum, maximum and
// the exact fp64 sums do not depend on the order they are taken in).
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ h2 as_h2(uint32_t w) { return __builtin_bit_cast(h2, w); }
__device__ __forceinline__ uint32_t as_u32(h2 v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ uint32_t rotl32(uint32_t w, int n) { return __builtin_amdgcn_alignbit(w, w, (32 - n) & 31); }
__device__ __forceinline__ uint32_t half_bits(float x) { return (uint32_t)__half_as_ushort(__float2half_rn(x)); }
__device__ __forceinline__ uint32_t mean_half_bits(double sum, int G) { return half_bits((float)(sum / (double)G)); }
// Is one of the two an infinity or a NaN?  (In integers: the compiler took a comparison with infinity for one that is true
// of a NaN.)
__device__ __forceinline__ uint32_t not_finite(h2 v) {
  return ((as_u32(v) & 0x7C007C00u) + 0x04000400u) & 0x80008000u;
}

// A load that is the last one, and a store that nothing soon reads: with ONCE they leave what the caches hold alone.
template <bool ONCE, class T>
__device__ __forceinline__ T last_load(const T* p) {
  if constexpr (ONCE) return __builtin_nontemporal_load(p);
  else return *p;
}
template <bool ONCE, class T>
__device__ __forceinline__ void put_away(T v, T* p) {
  if constexpr (ONCE) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// 2-bit codes are decided two at a time, in packed fp16: code k is reached where fl32(x - mn) >= (2k - 1) h, which a
// value of larger x reaches too, so that x >= T_k decides it, T_k being the smallest fp16 value that reaches it; and the
// sign of the fp16 difference x - T_k is that decision, whatever the rounding (a difference of unequal numbers never
// rounds to zero).  Kept is -T_k, a zero with the sign +: equal numbers, zeros of either sign among them, give +0.
// T_k: fl32(v) >= t for t of at most 14 bits is v >= t - u / 2, u the distance to the number below t (a tie rounds to t,
// whose last bit is 0), and v >= t - u / 4 at a power of two: in both cases the fp64 number 2^28 units below t.  mn + that
// is exact in fp64 (a group whose extremes differ has a step of at least 2^-14 of |mn|); rounded up to fp32 and then
// to fp16 it is the smallest fp16 number that is no less.  A step of zero has h = +infinity, and T_k = +infinity.
// Finite rows only: where a minimum or maximum is not finite, codes2 compares as the other kernels do.
struct Thresholds2 {
  h2 neg[3];                                           // -T_1 .. -T_3 of two groups
};
__device__ __forceinline__ Thresholds2 thresholds2(float mn0, float h0, float mn1, float h1) {
  double b[6];
  const double m[2] = {(double)mn0, (double)mn1}, h[2] = {(double)h0, (double)h1};
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    const unsigned long long t = (unsigned long long)__double_as_longlong((double)(2 * (i >> 1) + 1) * h[i & 1]);
    b[i] = m[i & 1] + __longlong_as_double((long long)(t - (1ull << 28)));
  }
  float f[6];                                          // fp16 in the low half
  asm("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 4), 5\n\t"          // round up
      "v_cvt_f32_f64 %0, %6\n\tv_cvt_f32_f64 %1, %7\n\tv_cvt_f32_f64 %2, %8\n\t"
      "v_cvt_f32_f64 %3, %9\n\tv_cvt_f32_f64 %4, %10\n\tv_cvt_f32_f64 %5, %11\n\t"
      "v_cvt_f16_f32 %0, %0\n\tv_cvt_f16_f32 %1, %1\n\tv_cvt_f16_f32 %2, %2\n\t"
      "v_cvt_f16_f32 %3, %3\n\tv_cvt_f16_f32 %4, %4\n\tv_cvt_f16_f32 %5, %5\n\t"
      "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 4), 0"
      : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3]), "=&v"(f[4]), "=&v"(f[5])
      : "v"(b[0]), "v"(b[1]), "v"(b[2]), "v"(b[3]), "v"(b[4]), "v"(b[5]));
  Thresholds2 r;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const uint32_t lo = __float_as_uint(f[2 * k]), hi = __float_as_uint(f[2 * k + 1]);
    r.neg[k] = h2{(_Float16)0.0f, (_Float16)0.0f} - as_h2(__builtin_amdgcn_perm(hi, lo, 0x05040100u));
  }
  return r;
}
// The bits of two codes (a pair of fp16 values) as the sign bits of two halves each.
struct Bits2 {
  uint32_t low, not_high;
};
__device__ __forceinline__ Bits2 bits2(uint32_t d1, uint32_t d2, uint32_t d3) {     // sign set: T_k not reached
  return {(~d1 & d2) | ~d3, d2};
}
__device__ __forceinline__ Bits2 codes2(uint32_t x, h2 n1, h2 n2, h2 n3) {
  return bits2(as_u32(as_h2(x) + n1), as_u32(as_h2(x) + n2), as_u32(as_h2(x) + n3));
}
__device__ __forceinline__ Bits2 codes2_compared(uint32_t x, float mn0, float h0, float mn1, float h1) {
  const float a = lo_half(x) - mn0, b = hi_half(x) - mn1;
  auto below = [&](float k) { return (a >= k * h0 ? 0u : 0x8000u) | (b >= k * h1 ? 0u : 0x80000000u); };
  return bits2(below(1.0f), below(3.0f), below(5.0f));
}
// Two pairs of codes into pair i (0 .. 3) of each byte of a register of sixteen 2-bit codes: the low halves' codes of p
// and q go to bytes 0 and 1, the high halves' to 2 and 3 (SWAPPED: 0 and 2, 1 and 3).  One byte permutation, which can
// replicate sign bits, serves four codes.
template <bool SWAPPED>
__device__ __forceinline__ void gather2(uint32_t& acc, const Bits2& p, const Bits2& q, int i) {
  constexpr uint32_t sel = SWAPPED ? 0x0B0A0908u : 0x0B090A08u;
  const uint32_t low = __builtin_amdgcn_perm(q.low, p.low, sel), not_high = __builtin_amdgcn_perm(q.not_high, p.not_high, sel);
  acc |= low & (0x01010101u << (2 * i));
  acc |= ~not_high & (0x02020202u << (2 * i));
}
// 4-bit codes: k is the number of thresholds (2k - 1) h that t = fl32(x - mn) reaches, at most 15, that is t / step + 1/2
// rounded down.  The product with the reciprocal is off by less than 2^-17 (t is at most 23 steps, where a step is the
// smallest number there is), so that with 2^-16 more it is k or k + 1 rounded down; one exact threshold tells which.
// A step of zero is taken with a reciprocal of zero: no threshold is reached.  Finite rows only, as above.
struct Scale4 {
  float mn, inv, step;
};
__device__ __forceinline__ Scale4 scale4(float mn, __half st) {
  const float s = __half2float(st);
  return {mn, s == 0.0f ? 0.0f : 1.0f / s, s};
}
__device__ __forceinline__ uint32_t code4(float t, const Scale4& q) {
  uint32_t k = (uint32_t)__builtin_fmaf(t, q.inv, 0.5f + 0x1p-16f);
  k = k < 15u ? k : 15u;
  return k - (t < __builtin_fmaf((float)k, q.step, -0.5f * q.step) ? 1u : 0u);
}
__device__ __forceinline__ float low_less(uint32_t x, float mn) {       // fl32(low half - mn)
  float t;
  asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel_hi:[1,0,0]" : "=v"(t) : "v"(x), "v"(mn));
  return t;
}
__device__ __forceinline__ float high_less(uint32_t x, float mn) {
  float t;
  asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(t) : "v"(x), "v"(mn));
  return t;
}
__device__ __forceinline__ uint32_t code4_compared(float x, float mn, float h) { return (uint32_t)quant_code_twice<4>(x, mn, h) >> 1; }
// The four rows of 16 lanes trade registers: row i gets register i of all rows, row k's as its register k.
__device__ __forceinline__ void trade_rows(uint32_t& a0, uint32_t& a1, uint32_t& a2, uint32_t& a3) {
  auto s = __builtin_amdgcn_permlane32_swap(a0, a2, false, false);
  a0 = s[0], a2 = s[1];
  s = __builtin_amdgcn_permlane32_swap(a1, a3, false, false);
  a1 = s[0], a3 = s[1];
  s = __builtin_amdgcn_permlane16_swap(a0, a1, false, false);
  a0 = s[0], a1 = s[1];
  s = __builtin_amdgcn_permlane16_swap(a2, a3, false, false);
  a2 = s[0], a3 = s[1];
}
// Two registers: those fields (`zeros` and as many next to each, `by` bits up) that a has second against those that b has first.
__device__ __forceinline__ void trade_fields(uint32_t& a, uint32_t& b, uint32_t zeros, int by) {
  const uint32_t x = (a & zeros) | ((b << by) & ~zeros);
  b = ((a >> by) & zeros) | (b & ~zeros);
  a = x;
}
// A register of sixteen 2-bit codes per lane, numbered 0 .. 15: what a lane keeps are the codes whose bit BIT of that number is
// its own (`upper`), and in the place of the others it takes those that the partner lane has for it.  (4-bit codes: two numbers each.)
template <int BIT>
__device__ __forceinline__ uint32_t trade2(uint32_t own, uint32_t partner, bool upper) {
  constexpr uint32_t zeros = BIT == 0 ? 0x33333333u : BIT == 1 ? 0x0F0F0F0Fu : 0x00FF00FFu;
  constexpr int by = 2 << BIT;
  const uint32_t keep = upper ? ~zeros : zeros;
  const uint32_t turned = __builtin_amdgcn_alignbit(partner, partner, upper ? by : 32 - by);
  return (own & keep) | (turned & ~keep);
}
// Lanes of a row of 16, by banks of four: bank BANK's get `v` from BY lanes below (modulo 16), the others keep `old`.
template <int BANK, int BY>
__device__ __forceinline__ uint32_t from_bank(uint32_t old, uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, 0x120 + BY /* row_ror */, 0xf, 1 << BANK, false);
}
// Lanes of a quad: each gets lane S's.
template <int S>
__device__ __forceinline__ uint32_t of_quad_lane(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, S * 0x55, 0xf, 0xf, false);
}

template <int BITS, int G, int LAYERS, bool ONCE>
__global__ void __launch_bounds__(4 * G) __attribute__((amdgpu_waves_per_eu(4, 8))) prompt_quantize_kernel(
    Dims d, int32_t group_index, int64_t unit_stride, const uint8_t* __restrict__ selected, int64_t selected_unit_stride,
    uint8_t* __restrict__ k_codes, uint32_t* __restrict__ k_meta, uint8_t* __restrict__ v_codes,
    uint32_t* __restrict__ v_meta, uint32_t* __restrict__ mask, int32_t n_groups, int32_t tail_n,
    __half* __restrict__ k_res, __half* __restrict__ v_res, int32_t last_first, LayerRows<LAYERS> rows) {
  // grid (units, groups + tail blocks, layers), as quantize_kernel's.  Wavefronts 0 .. nblk - 1 have the Keys of a block of 32
  // tokens each, the others the Values.
  constexpr int nblk = G / kBlockTokens, kThreads = 128 * nblk;
  // what the blocks of a longer group tell each other: minimum and maximum of the Keys, sums of Keys and Values (for means)
  __shared__ uint2 s_extremes[nblk][64];
  __shared__ __align__(16) double s_sums[nblk > 1 ? 2 : 1][nblk > 1 ? nblk : 1][kHeadDim];
  const int tid = threadIdx.x;
  const int ul = blockIdx.x, by = blockIdx.y, layer = LAYERS > 1 ? blockIdx.z : 0;
  const __half* __restrict__ k_rows = rows.k[layer];
  const __half* __restrict__ v_rows = rows.v[layer];
  const int gy = last_first && by < n_groups ? n_groups - 1 - by : by;
  if (gy >= n_groups) {
    const int i = (gy - n_groups) * kThreads + tid;
    if (i < tail_n * 16) {
      const int64_t src = (int64_t)ul * unit_stride + (int64_t)n_groups * G * kHeadDim;
      const int64_t dst = (d.unit0 + (int64_t)layer * d.layer_units + ul) * d.res_rows * kHeadDim;
      ((uint4*)(k_res + dst))[i] = ((const uint4*)(k_rows + src))[i];
      ((uint4*)(v_res + dst))[i] = ((const uint4*)(v_rows + src))[i];
    }
    return;
  }
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int blk = nblk == 1 ? 0 : wave & (nblk - 1);
  const int64_t row0 = (int64_t)ul * unit_stride + (int64_t)gy * G * kHeadDim;
  const int64_t sel0 = ((int64_t)layer * d.units_per_layer + ul) * selected_unit_stride + (int64_t)gy * G;
  const GroupPlace at = place_of_group(d, ul, group_index + gy, layer);
  const int64_t block0 = at.row * d.blocks_per_unit + (int64_t)at.slot * nblk;   // the group's first packed block
  // The flags of the group's tokens, as bit masks (uniform).  The rows are asked for while they come.
  constexpr int kSelWords = (G + 63) / 64;
  unsigned long long sel[kSelWords];
  uint8_t flags[kSelWords];
#pragma unroll
  for (int w = 0; w < kSelWords; ++w) flags[w] = selected && 64 * w + lane < G ? selected[sel0 + 64 * w + lane] : (uint8_t)0;
  auto any_flag = [&]() -> bool {
    bool any = false;
#pragma unroll
    for (int w = 0; w < kSelWords; ++w) {
      sel[w] = __ballot(flags[w] != 0);
      any |= sel[w] != 0;
    }
    return any;
  };
  auto is_sel = [&](int t) -> bool { return (sel[kSelWords == 1 ? 0 : t >> 6] >> (t & 63)) & 1ull; };

  auto exchange = [&]() {                              // of the blocks of a longer group: one barrier per wavefront
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  };

  if (wave < nblk) {
    // ---- Keys ------------------------------------------------------------------------------------------
    int cp, r, hi = 0, p = 0, cb = 0, v = lane & 3;    // cp: the lane's channel pair (channels 2 cp, 2 cp + 1)
    if (BITS == 2) {
      hi = lane >> 5, r = (lane >> 3) & 3, p = (lane >> 2) & 1;
      v ^= p ? 3 : 0;                                  // (so that the mirror lane inside 8 has the other p and the same v)
      cp = 16 * (2 * hi + p) + 4 * r + v;
    } else {
      cp = lane, cb = lane >> 4, r = (lane >> 2) & 3;
    }
    const uint32_t* kr = (const uint32_t*)(k_rows + row0) + cp;        // token t: kr[64 t]
    uint32_t y[32];
#pragma unroll
    for (int t = 0; t < 32; ++t) y[t] = last_load<ONCE>(kr + (blk * 32 + t) * 64);
    auto keys = [&](auto any_c) {
      constexpr bool ANY = decltype(any_c)::value;     // some token of the group is flagged (uniform)
      double s0 = 0.0, s1 = 0.0;
      h2 mn = {(_Float16)__builtin_inff(), (_Float16)__builtin_inff()};
      h2 mx = {(_Float16)(-__builtin_inff()), (_Float16)(-__builtin_inff())};
      // (a NaN among the rows is found out by its being the result; where it is passed over comes below)
      auto lower = [](h2 a, h2 b) { return __builtin_elementwise_minimum(a, b); };
      auto upper = [](h2 a, h2 b) { return __builtin_elementwise_maximum(a, b); };
#pragma unroll
      for (int t = 0; t < 32; ++t) {
        const h2 x = as_h2(y[t]);
        if (ANY) {
          const bool s = is_sel(blk * 32 + t);
          mn = s ? mn : lower(mn, x);
          mx = s ? mx : upper(mx, x);
        } else {
          mn = lower(mn, x);
          mx = upper(mx, x);
        }
      }
      if (ANY) {                                       // the exact sums of ALL rows as they came (two chains of
#pragma unroll                                         // dependent additions: few conversions in flight at a time)
        for (int t = 0; t < 32; ++t) {
          uint32_t x = y[t];
          asm volatile("" : "+v"(x), "+v"(s0), "+v"(s1));
          s0 += (double)lo_half(x);
          s1 += (double)hi_half(x);
        }
      }
      if constexpr (nblk > 1) {
        s_extremes[blk][lane] = make_uint2(as_u32(mn), as_u32(mx));
        if (ANY) {
          s_sums[0][blk][lane] = s0;
          s_sums[0][blk][64 + lane] = s1;
        }
        exchange();
        if (ANY) s0 = s1 = 0.0;
#pragma unroll
        for (int k = 0; k < nblk; ++k) {
          const uint2 e = s_extremes[k][lane];
          mn = lower(mn, as_h2(e.x));
          mx = upper(mx, as_h2(e.y));
          if (ANY) {
            s0 += s_sums[0][k][lane];
            s1 += s_sums[0][k][64 + lane];
          }
        }
      }
      uint32_t mean = 0;
      if (ANY) {
        mean = mean_half_bits(s0, G) | (mean_half_bits(s1, G) << 16);
        mn = lower(mn, as_h2(mean));
        mx = upper(mx, as_h2(mean));
      }
      auto row = [&](int t) -> uint32_t { return ANY && is_sel(t) ? mean : kr[t * 64]; };
      const bool finite = __ballot(not_finite(mn) | not_finite(mx)) == 0;
      if (!finite) {                                   // (uniform; such rows are not supported, and nothing here is made to be fast)
        mn = mx = as_h2(row(0));                       // (from a row on, not from infinity: all NaN gives NaN)
#pragma unroll 1
        for (int t = 1; t < G; ++t) {
          const h2 x = as_h2(row(t));
          mn = __builtin_elementwise_min(mn, x);
          mx = __builtin_elementwise_max(mx, x);
        }
      }
      const float mn0 = (float)mn[0] + 0.0f, mn1 = (float)mn[1] + 0.0f;   // a zero minimum is stored as +0
      const __half st0 = step_of(mn0, (float)mx[0], BITS), st1 = step_of(mn1, (float)mx[1], BITS);
      const float h0 = half_step_of(st0), h1 = half_step_of(st1);
      if (blk == 0) {
        uint32_t* gm = k_meta + (at.row * d.groups_per_unit + at.slot) * kHeadDim;   // fp16 step[128], then zero[128]
        gm[cp] = (uint32_t)__half_as_ushort(st0) | ((uint32_t)__half_as_ushort(st1) << 16);
        gm[64 + cp] = half_bits(mn0) | (half_bits(mn1) << 16);
      }
      Thresholds2 th = {};
      Scale4 sc0 = {}, sc1 = {};
      if (BITS == 2) th = thresholds2(mn0, h0, mn1, h1);
      else sc0 = scale4(mn0, st0), sc1 = scale4(mn1, st1);
      // The packed word of token 8 b + 4 p + v from the codes of tokens 8 b .. 8 b + 7 (2-bit), of token 4 b + v from those of
      // tokens 4 b .. 4 b + 3 (4-bit): code(t) of the channel pair
      auto word_of = [&](auto code) {
        if constexpr (BITS == 4) {
          uint32_t acc = 0;                            // code 4 * channel of the pair + token
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const uint2 c = code(i);
            acc |= (c.x << (4 * i)) | (c.y << (16 + 4 * i));
          }
          acc = trade2<1>(acc, row_partner_u32<0>(acc), v & 1);
          acc = trade2<2>(acc, row_partner_u32<1>(acc), v & 2);
          return rotl32(acc, 2);
        } else {
          uint32_t acc = 0;                            // code 8 * channel of the pair + token
#pragma unroll
          for (int i = 0; i < 4; ++i) gather2<false>(acc, code(i), code(4 + i), i);
          acc = trade2<0>(acc, row_partner_u32<0>(acc), v & 1);
          acc = trade2<1>(acc, row_partner_u32<1>(acc), v & 2);
          acc = trade2<2>(acc, row_partner_u32<2>(acc), p);
          return rotl32(acc, 2);
        }
      };
      uint8_t* kb = k_codes + (block0 + blk) * (int64_t)d.block_bytes;
      if (ANY) {                                     // the flagged rows become the mean row
#pragma unroll
        for (int t = 0; t < 32; ++t) y[t] = is_sel(blk * 32 + t) ? mean : y[t];
      }
      if constexpr (BITS == 2) {
        if (finite) {                                // uniform
          uint32_t word[4];
#pragma unroll
          for (int b = 0; b < 4; ++b) {
            word[b] = word_of([&](int t) { return codes2(y[8 * b + t], th.neg[0], th.neg[1], th.neg[2]); });
          }
          // the two words of a token and half (tokens 0 .. 15, 16 .. 31) to one lane
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
            const auto sw = __builtin_amdgcn_permlane32_swap(word[b], word[2 + b], false, false);
            put_away<ONCE>(u32x2{sw[0], sw[1]}, (u32x2*)(kb + 16 * (16 * r + 8 * b + 4 * p + v) + 8 * hi));
          }
        } else {
#pragma unroll 1
          for (int b = 0; b < 4; ++b) {
            const uint32_t w = word_of([&](int t) { return codes2_compared(row(blk * 32 + 8 * b + t), mn0, h0, mn1, h1); });
            *(uint32_t*)(kb + 16 * (16 * r + 8 * (b & 1) + 4 * p + v) + 4 * (2 * (b >> 1) + hi)) = w;
          }
        }
      } else {
        if (finite) {                                // uniform
#pragma unroll
          for (int th16 = 0; th16 < 2; ++th16) {     // tokens 0 .. 15, 16 .. 31
            uint32_t word[4];
#pragma unroll
            for (int b = 0; b < 4; ++b)
              word[b] = word_of([&](int t) {
                const uint32_t x = y[16 * th16 + 4 * b + t];
                return make_uint2(code4(low_less(x, sc0.mn), sc0), code4(high_less(x, sc1.mn), sc1));
              });
            // row i of lanes gets the words of tokens 4 i + v, all four of a token
            trade_rows(word[0], word[1], word[2], word[3]);
            put_away<ONCE>(u32x4{word[0], word[1], word[2], word[3]},
                           (u32x4*)(kb + 1024 * th16 + 16 * (16 * r + 4 * cb + v)));
          }
        } else {
#pragma unroll 1
          for (int b = 0; b < 8; ++b) {
            const uint32_t w = word_of([&](int t) {
              const uint32_t x = row(blk * 32 + 4 * b + t);
              return make_uint2(code4_compared(lo_half(x), mn0, h0), code4_compared(hi_half(x), mn1, h1));
            });
            *(uint32_t*)(kb + 1024 * (b >> 2) + 16 * (16 * r + 4 * (b & 3) + v) + 4 * cb) = w;
          }
        }
      }
      if (lane == 0) {
        const uint32_t mw = (uint32_t)(sel[kSelWords == 1 ? 0 : (blk * 32) >> 6] >> ((blk * 32) & 63));
        mask[block0 + blk] = mw;
      }
    };
    if (any_flag()) keys(std::true_type{});
    else keys(std::false_type{});
    return;
  }

  // ---- Values ----------------------------------------------------------------------------------------------
  const int gv_shift = 31 - __clz(d.Gv);
  const int lanes = d.Gv >> 3;                          // lanes per (token, channel group) in the first mapping
  const int NV = d.vgroups;
  const int t4 = lane >> 4, c16 = lane & 15;            // the lane's channels are 8 c16 .. + 7, its tokens 8 r + 2 t4 + s
  const __half* vr = v_rows + row0 + 8 * c16;
  u32x4 w[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {                         // row i = 2 r + s: the lane's tokens come in pairs, as steps and zeros are stored
    w[i] = last_load<ONCE>((const u32x4*)(vr + (blk * 32 + 8 * (i >> 1) + 2 * t4 + (i & 1)) * kHeadDim));
  }
  auto values = [&](auto any_c) {
    constexpr bool ANY = decltype(any_c)::value;
    uint32_t mean4[4] = {0u, 0u, 0u, 0u};
    if (ANY) {                                          // per-channel means of the group's Value rows, exact
#pragma unroll
      for (int k = 0; k < 4; ++k) {                     // (a channel pair at a time: few registers)
        double a = 0.0, b = 0.0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          uint32_t x = w[i][k];
          asm volatile("" : "+v"(x), "+v"(a), "+v"(b));
          a += (double)lo_half(x);
          b += (double)hi_half(x);
        }
        a += __shfl_xor(a, 16);
        b += __shfl_xor(b, 16);
        a += __shfl_xor(a, 32);
        b += __shfl_xor(b, 32);
        if constexpr (nblk == 1) mean4[k] = mean_half_bits(a, G) | (mean_half_bits(b, G) << 16);
        else if (t4 == 0) *(double2*)&s_sums[1][blk][8 * c16 + 2 * k] = make_double2(a, b);
      }
      if constexpr (nblk > 1) {
        exchange();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          double a = 0.0, b = 0.0;
#pragma unroll
          for (int i = 0; i < nblk; ++i) {
            const double2 part = *(const double2*)&s_sums[1][i][8 * c16 + 2 * k];
            a += part.x;
            b += part.y;
          }
          mean4[k] = mean_half_bits(a, G) | (mean_half_bits(b, G) << 16);
        }
      }
    } else if (nblk > 1) {
      __builtin_amdgcn_s_barrier();                     // (the Keys' exchange, of which the Values need nothing)
    }
    if (ANY) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int T = blk * 32 + 8 * (i >> 1) + 2 * t4 + (i & 1);
        if ((sel[kSelWords == 1 ? 0 : T >> 6] >> (T & 63)) & 1ull)
          w[i] = u32x4{mean4[0], mean4[1], mean4[2], mean4[3]};
      }
    }
    // {minimum, -maximum} of the rows in each channel group: lane `own` of a quad gets those of r = own, s = 0, 1.
    // (A NaN is found out by its being the result; where it is passed over comes below.)
    const int own = lane & 3;
    auto channels = [](u32x4 x, auto lower, auto upper) {   // of one row's eight
      const h2 a = lower(lower(as_h2(x.x), as_h2(x.y)), lower(as_h2(x.z), as_h2(x.w)));
      const h2 b = upper(upper(as_h2(x.x), as_h2(x.y)), upper(as_h2(x.z), as_h2(x.w)));
      const uint32_t nb = as_u32(b) ^ 0x80008000u;          // the halves against each other: {a0, -b0} and {a1, -b1}
      return as_u32(lower(as_h2(__builtin_amdgcn_perm(nb, as_u32(a), 0x05040100u)),
                          as_h2(__builtin_amdgcn_perm(nb, as_u32(a), 0x07060302u))));
    };
    auto quads = [&](uint32_t x, auto lower) {              // of the quads of a channel group
      if (lanes > 4) {                             // uniform; the lane with the same place in the next quad
        const uint32_t mirror = row_partner_u32<2>(x);
        x = as_u32(lower(as_h2(x), as_h2((uint32_t)__builtin_amdgcn_mov_dpp((int)mirror, 0x1B, 0xf, 0xf, false))));
      }
      if (lanes > 8) x = as_u32(lower(as_h2(x), as_h2((uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x128 /* row_ror:8 */, 0xf, 0xf, false))));
      return x;
    };
    h2 pair[2];
    {
      auto lower = [](h2 a, h2 b) { return __builtin_elementwise_minimum(a, b); };
      auto upper = [](h2 a, h2 b) { return __builtin_elementwise_maximum(a, b); };
      uint32_t pr[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) pr[i] = channels(w[i], lower, upper);
      auto fold = [&](uint32_t a, uint32_t b, bool up, auto bit_c) {   // lanes with the bit keep b, the others a
        return as_u32(lower(as_h2(up ? b : a), as_h2(row_partner_u32<decltype(bit_c)::value>(up ? a : b))));
      };
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const uint32_t r01 = fold(pr[s], pr[2 + s], own & 1, std::integral_constant<int, 0>{});
        const uint32_t r23 = fold(pr[4 + s], pr[6 + s], own & 1, std::integral_constant<int, 0>{});
        pair[s] = as_h2(quads(fold(r01, r23, own & 2, std::integral_constant<int, 1>{}), lower));
      }
    }
    auto row = [&](int r, int s) -> u32x4 {
      const int t = 8 * r + 2 * t4 + s, T = blk * 32 + t;
      if (ANY && ((sel[kSelWords == 1 ? 0 : T >> 6] >> (T & 63)) & 1ull)) return u32x4{mean4[0], mean4[1], mean4[2], mean4[3]};
      return *(const u32x4*)(vr + T * kHeadDim);
    };
    const bool finite = __ballot(not_finite(pair[0]) | not_finite(pair[1])) == 0;
    if (!finite) {
      auto lower = [](h2 a, h2 b) { return __builtin_elementwise_min(a, b); };
      auto upper = [](h2 a, h2 b) { return __builtin_elementwise_max(a, b); };
#pragma unroll 1
      for (int i = 0; i < 8; ++i) {
        uint32_t x = channels(row(i >> 1, i & 1), lower, upper);
        x = as_u32(lower(as_h2(x), as_h2(row_partner_u32<0>(x))));
        x = as_u32(lower(as_h2(x), as_h2(row_partner_u32<1>(x))));
        x = quads(x, lower);
        pair[0] = (i >> 1) == own && !(i & 1) ? as_h2(x) : pair[0];
        pair[1] = (i >> 1) == own && (i & 1) ? as_h2(x) : pair[1];
      }
    }
    const float mn0 = (float)pair[0][0] + 0.0f, mn1 = (float)pair[1][0] + 0.0f;   // a zero minimum is stored as +0
    const __half st0 = step_of(mn0, -(float)pair[0][1], BITS), st1 = step_of(mn1, -(float)pair[1][1], BITS);
    const float h0 = half_step_of(st0), h1 = half_step_of(st1);
    if ((c16 & (lanes - 1)) < 4) {                 // fp16 step[16 token pairs][NV][2], then fp16 zero[16 token pairs][NV][2]
      uint32_t* gm = v_meta + (block0 + blk) * 32 * NV + (4 * own + t4) * NV + ((8 * c16) >> gv_shift);
      gm[0] = (uint32_t)__half_as_ushort(st0) | ((uint32_t)__half_as_ushort(st1) << 16);
      gm[16 * NV] = half_bits(mn0) | (half_bits(mn1) << 16);
    }
    uint8_t* vb = v_codes + (block0 + blk) * (int64_t)d.block_bytes;
    if constexpr (BITS == 4) {
      uint32_t acc[4][2] = {};                       // r, half of the lane's channels: code 4 s + channel of the four
      if (finite) {                                  // uniform
        const Scale4 q0 = scale4(mn0, st0), q1 = scale4(mn1, st1);
        auto codes = [&](auto r_c) {
          constexpr int R = decltype(r_c)::value;
          auto of_lane = [](float x) { return __uint_as_float(of_quad_lane<R>(__float_as_uint(x))); };
          const Scale4 q[2] = {{of_lane(q0.mn), of_lane(q0.inv), of_lane(q0.step)}, {of_lane(q1.mn), of_lane(q1.inv), of_lane(q1.step)}};
#pragma unroll
          for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const uint32_t x = w[2 * R + s][i];
              const int at = 16 * s + 8 * (i & 1);
              acc[R][i >> 1] |= (code4(low_less(x, q[s].mn), q[s]) << at) | (code4(high_less(x, q[s].mn), q[s]) << (at + 4));
            }
        };
        codes(std::integral_constant<int, 0>{});
        codes(std::integral_constant<int, 1>{});
        codes(std::integral_constant<int, 2>{});
        codes(std::integral_constant<int, 3>{});
      } else {
#pragma unroll 1
        for (int i = 0; i < 8; ++i) {
          const int r = i >> 1, s = i & 1, from = (lane & ~3) | r;
          const float m = __shfl(s ? mn1 : mn0, from), h = __shfl(s ? h1 : h0, from);
          const u32x4 x = row(r, s);
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            const uint32_t c = code4_compared(k & 1 ? hi_half(x[k >> 1]) : lo_half(x[k >> 1]), m, h) << (16 * s + 4 * (k & 3));
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[b][k >> 2] |= b == r ? c : 0u;
          }
        }
      }
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        uint32_t x0 = acc[0][a], x1 = acc[1][a], x2 = acc[2][a], x3 = acc[3][a];
        trade_rows(x0, x1, x2, x3);                  // row t4 gets r = t4, register i the tokens that row i had
        // registers against channels: register i the codes of channel 4 a + i, numbered 4 s + t4: a word, but for its turn
        trade_fields(x0, x1, 0x0F0F0F0Fu, 4);
        trade_fields(x2, x3, 0x0F0F0F0Fu, 4);
        trade_fields(x0, x2, 0x00FF00FFu, 8);
        trade_fields(x1, x3, 0x00FF00FFu, 8);
        // Registers against bits 1 and 2 of the lane, which with bit 3 number the field: a lane gets the four words of
        // its 16 bytes.
        const bool up = lane & 2;
        auto swap1 = [&](uint32_t& p, uint32_t& q) {
          const uint32_t got = row_partner_u32<1>(up ? p : q);
          p = up ? got : p;
          q = up ? q : got;
        };
        swap1(x0, x1);
        swap1(x2, x3);
        auto swap2 = [&](uint32_t& p, uint32_t& q) {
          const uint32_t was = p;
          p = from_bank<3, 4>(from_bank<1, 4>(p, q), q);
          q = from_bank<2, 12>(from_bank<0, 12>(q, was), was);
        };
        swap2(x0, x2);
        swap2(x1, x3);
        put_away<ONCE>(u32x4{rotl32(x0, 2), rotl32(x1, 2), rotl32(x2, 2), rotl32(x3, 2)},
                       (u32x4*)(vb + 1024 * (c16 >> 3) + 16 * (16 * t4 + 8 * (lane & 1) + 4 * a + ((lane >> 1) & 3))));
      }
    } else {
      const Thresholds2 th = thresholds2(mn0, h0, mn1, h1);
      uint32_t acc[4] = {0, 0, 0, 0};                // r: code 8 s + 4 (channel & 1) + channel pair of the lane's four
      if (finite) {                                  // uniform
        auto codes = [&](auto r_c) {
          constexpr int R = decltype(r_c)::value;
          h2 n[3];
#pragma unroll
          for (int k = 0; k < 3; ++k) n[k] = as_h2(of_quad_lane<R>(as_u32(th.neg[k])));
#pragma unroll
          for (int i = 0; i < 4; ++i)
            gather2<true>(acc[R], codes2(w[2 * R][i], h2{n[0][0], n[0][0]}, h2{n[1][0], n[1][0]}, h2{n[2][0], n[2][0]}),
                          codes2(w[2 * R + 1][i], h2{n[0][1], n[0][1]}, h2{n[1][1], n[1][1]}, h2{n[2][1], n[2][1]}), i);
        };
        codes(std::integral_constant<int, 0>{});
        codes(std::integral_constant<int, 1>{});
        codes(std::integral_constant<int, 2>{});
        codes(std::integral_constant<int, 3>{});
      } else {
#pragma unroll 1
        for (int r = 0; r < 4; ++r) {
          const int from = (lane & ~3) | r;
          const float m0 = __shfl(mn0, from), m1 = __shfl(mn1, from), g0 = __shfl(h0, from), g1 = __shfl(h1, from);
          const u32x4 x0 = row(r, 0), x1 = row(r, 1);
          uint32_t a = 0;
#pragma unroll
          for (int i = 0; i < 4; ++i)
            gather2<true>(a, codes2_compared(x0[i], m0, g0, m0, g0), codes2_compared(x1[i], m1, g1, m1, g1), i);
#pragma unroll
          for (int k = 0; k < 4; ++k) acc[k] = k == r ? a : acc[k];
        }
      }
      // row t4 of 16 lanes gets r = t4, register i the tokens that row i had
      trade_rows(acc[0], acc[1], acc[2], acc[3]);
      // registers against channel pairs: register i the codes of pair i, numbered 8 s + 4 (channel & 1) + t4
      trade_fields(acc[0], acc[1], 0x33333333u, 2);
      trade_fields(acc[2], acc[3], 0x33333333u, 2);
      trade_fields(acc[0], acc[2], 0x0F0F0F0Fu, 4);
      trade_fields(acc[1], acc[3], 0x0F0F0F0Fu, 4);
      // Bit 1 of the lane, which tells channels c and c + 16 apart, against the parity of the channel: a word of both.
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] = rotl32(trade2<2>(acc[i], row_partner_u32<1>(acc[i]), lane & 2), 2);
      // Registers against the lanes' banks of four, so that a lane has the four words of its 16 bytes: bank b passes its
      // register k to bank k, register b.
      u32x4 words = {acc[0], acc[1], acc[2], acc[3]};
      words[0] = from_bank<1, 4>(words[0], acc[1]), words[0] = from_bank<2, 8>(words[0], acc[2]), words[0] = from_bank<3, 12>(words[0], acc[3]);
      words[1] = from_bank<0, 12>(words[1], acc[0]), words[1] = from_bank<2, 4>(words[1], acc[2]), words[1] = from_bank<3, 8>(words[1], acc[3]);
      words[2] = from_bank<0, 8>(words[2], acc[0]), words[2] = from_bank<1, 12>(words[2], acc[1]), words[2] = from_bank<3, 4>(words[2], acc[3]);
      words[3] = from_bank<0, 4>(words[3], acc[0]), words[3] = from_bank<1, 8>(words[3], acc[1]), words[3] = from_bank<2, 12>(words[3], acc[2]);
      // lane: row r = t4, bank k = channel pair, bit 1 the parity of the channel, bit 0 the channel's bit 3
      put_away<ONCE>(words, (u32x4*)(vb + 16 * (16 * t4 + 8 * (lane & 1) + 2 * (c16 >> 2) + ((lane >> 1) & 1))));
    }
  };
  if (any_flag()) values(std::true_type{});
  else values(std::false_type{});
}

// The n rows of every unit into ring rows 0 .. n - 1 (16 bytes per thread).  grid (units, blocks, layers).
template <int LAYERS>
__global__ void __launch_bounds__(256) tail_copy_kernel(Dims d, int64_t unit_stride, int32_t n, __half* __restrict__ k_res,
                                                        __half* __restrict__ v_res, LayerRows<LAYERS> rows) {
  const int ul = blockIdx.x, layer = LAYERS > 1 ? blockIdx.z : 0;
  const int64_t u = d.unit0 + (int64_t)layer * d.layer_units + ul;
  const uint4* sk = (const uint4*)(rows.k[layer] + (int64_t)ul * unit_stride);
  const uint4* sv = (const uint4*)(rows.v[layer] + (int64_t)ul * unit_stride);
  uint4* dk = (uint4*)(k_res + u * d.res_rows * kHeadDim);
  uint4* dv = (uint4*)(v_res + u * d.res_rows * kHeadDim);
  for (int i = blockIdx.y * 256 + threadIdx.x; i < n * 16; i += gridDim.y * 256) {
    dk[i] = sk[i];
    dv[i] = sv[i];
  }
}

// The whole group step of one unit in one launch: append the new token's row to the ring, run the
// outlier competition on the oldest G rows, quantize them.  The ring must be full after the
// append (R + G rows), its oldest G rows starting at ring row `group_row0`.
template <int BITS, int G>
__global__ void __launch_bounds__(kQuantThreads) group_step_kernel(
    Dims d, int32_t group_index, const __half* __restrict__ k_new, const __half* __restrict__ v_new, __half* k_res,
    __half* v_res, int32_t append_row, int32_t group_row0, const int32_t* __restrict__ seq, __half* pool_k,
    __half* pool_v, int32_t* pool_idx,
    double* pool_score, int32_t* pool_count, int32_t* aux_count, int32_t* frozen, uint8_t* selected,
    uint8_t* __restrict__ k_codes, uint32_t* __restrict__ k_meta, uint8_t* __restrict__ v_codes,
    uint32_t* __restrict__ v_meta, uint32_t* __restrict__ mask) {
  extern __shared__ __align__(16) unsigned char smem[];
  const QuantLds<G> L(smem, d.vgroups);
  const int tid = threadIdx.x;
  const int ul = blockIdx.x;
  const int64_t u = d.unit0 + ul;
  __half* kring = k_res + u * d.res_rows * kHeadDim;
  __half* vring = v_res + u * d.res_rows * kHeadDim;
  bool close_group = true;
  if (seq) {
    // A batch of sequences of different lengths: the unit's sequence says where its new row goes
    // and whether its ring is full with it.  A sequence that is inactive, or whose state does not
    // fit the buffers, is left alone; all of this is uniform over the workgroup.
    const int4 own = *(const int4*)(seq + 4 * (ul / d.kv_heads));
    const int nq = own.x, rs = own.y, nr = own.z;
    if (!own.w || nq < 0 || rs < 0 || rs >= d.res_rows || nr < 0 || nr >= d.res_rows) return;
    append_row = rs + nr;
    append_row -= append_row >= d.res_rows ? d.res_rows : 0;
    group_row0 = rs;
    group_index = nq / G;
    close_group = nr + 1 == d.R + G && rs % G == 0 && nq % G == 0 && nq + G <= d.max_seq;
  }
  if (tid < 128) {                                   // the new row: 64 threads for K, 64 for V, 4 bytes each
    const int which = tid >> 6, lane = tid & 63;
    const uint32_t* src = (const uint32_t*)((which ? v_new : k_new) + (int64_t)ul * kHeadDim);
    ((uint32_t*)((which ? vring : kring) + append_row * kHeadDim))[lane] = src[lane];
  }
  if (!close_group) return;
  const GroupPlace at = place_of_group(d, ul, group_index);        // where the group's codes and meta go
  if (append_row >= group_row0 && append_row < group_row0 + G) {   // R = 0: the new token closes the group
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  }
  const __half* gk = kring + group_row0 * kHeadDim;
  const __half* gv = vring + group_row0 * kHeadDim;
  GroupRows<G> rows;
  rows_issue<G>(rows, gk, gv, tid);
  uint8_t* sel = selected ? selected + (int64_t)ul * G : nullptr;
  if (d.N > 0) {
    const trace_core::UnitPool p =
        trace_core::unit_pool(d, u, pool_k, pool_v, pool_idx, pool_score, pool_count, aux_count, frozen);
    trace_core::Loaded<G> in;
    const bool ahead = d.N <= trace_core::kPoolRowsAhead;
    trace_core::load<G>(in, d, p, gk, tid, ahead);
    rows_to_lds<G>(rows, L, tid);
    trace_core::compete<G>(in, d, group_index, p, gk, gv, sel, L.ssel, tid, L.sk, L.sv, kRowB, ahead);
  } else {
    rows_to_lds<G>(rows, L, tid);
    if (tid < G) {
      L.ssel[tid] = 0;
      if (sel) sel[tid] = 0;
    }
  }
  __syncthreads();                                   // the flags are in LDS
  const uint8_t flag = tid < G ? L.ssel[tid] : (uint8_t)0;
  quantize_body<BITS, G>(d, at.row, at.slot, L, flag, k_codes, k_meta, v_codes, v_meta, mask, tid);
}

template <int BITS, int G, int LAYERS>
hipError_t launch_quantize_one(const Dims& d, int32_t group_index, int32_t n_groups, const PromptRows& rows,
                               const uint8_t* selected, int64_t selected_unit_stride,
                               const kvq_qcache& qc, int32_t tail_n, __half* k_res, __half* v_res, hipStream_t s) {
  // many groups (a prompt): the kernel that spends the fewest instructions per group; few: the one that is
  // done with a group soonest
  const int64_t groups = (int64_t)d.units_per_layer * rows.layers * n_groups;
  const bool many = groups >= prompt_groups(G) && !d.keys_only;
  const int threads = many ? 4 * G : kQuantThreads;
  const dim3 grid(d.units_per_layer, n_groups + (tail_n * 16 + threads - 1) / threads, rows.layers);
  auto go = [&](auto kern, size_t smem, auto... more) {
    hipLaunchKernelGGL(kern, grid, dim3(threads), smem, s, d, group_index, rows.unit_stride, selected,
                       selected_unit_stride, (uint8_t*)qc.k_codes, (uint32_t*)qc.k_meta, (uint8_t*)qc.v_codes,
                       (uint32_t*)qc.v_meta, (uint32_t*)qc.mask, n_groups, tail_n, k_res, v_res, more...,
                       layer_rows<LAYERS>(rows));
    return hipGetLastError();
  };
  // Two rules on the Keys' size.  (Times of the whole call, MB of 2^20 bytes; the memory-side cache holds 256.)
  // Where the competition has just read more Keys than the cache keeps besides everything else, the last groups come
  // first: their Keys are still there.  First to last / last to first, three sets of rows in turn, G = 32 2-bit, 4-bit, G = 128
  // 2-bit: 128 units x 4096 tokens (128 MB) 82.8 / 81.9 us, 96.2 / 94.9, 92.4 / 90.4; 256 x 4096 150.4 / 149.3, 173.9 / 171.2,
  // 170.4 / 167.6; 256 x 8192 286.0 / 285.0, 316.2 / 312.5, 324.0 / 321.6; 512 x 4096 319.4 / 317.7, 344.5 / 348.9, 340.5 / 340.2.
  // ONCE keeps rows that are not needed again, and the codes, from displacing the rest.  It pays where the rows have to
  // come from memory, and costs where the next call would have found the same rows in the same place in the cache (which
  // a prompt does not do).  Whole calls, three sets of rows in turn, without / with, G = 32 (64 and 128 alike):
  //   Keys   12 MB, 128 units   24, 128       36, 256       64, 32        100, 128      200, 128    400, 256    1100 MB, 512 units
  //   2-bit  26.4 / 26.1 us     31.7 / 32.2   41.2 / 38.9   60.4 / 54.7   83.4 / 77.1   153 / 134   275 / 238   745 / 688
  //   4-bit  29.0 / 28.9        35.5 / 35.6   45.5 / 44.1   67.3 / 62.4   92.7 / 88.3   166 / 150   304 / 263   794 / 732
  // With one set of rows, read again and again, it costs 2 .. 4 % from 32 to 100 MB, and gives 5 .. 13 % from 200 MB on.  Without
  // a pool, three sets that the cache holds together (32 MB): 18.5 / 20.9.  Rows that a copy has just written (the copies are
  // in the times), 128 units, without / with:
  //   Keys              32 MB         48           64              96              128             192
  //   G = 32, 2-bit     54.4 / 54.5   78.4 / 74.2  105.4 / 104.8   150.5 / 153.4   198.9 / 191.9   297.8 / 280.8
  //   G = 32, 4-bit     58.7 / 59.2   87.5 / 82.0  111.3 / 113.0   159.3 / 162.2   211.0 / 204.8   362.1 / 349.7
  //   G = 64, 2-bit     55.6 / 55.7   77.9 / 75.8  104.5 / 105.4   150.9 / 154.9   231.6 / 227.3   347.6 / 332.3
  //   G = 128, 2-bit    56.7 / 56.5   80.5 / 79.1  109.6 / 110.2   155.1 / 157.1   237.6 / 232.7   353.5 / 341.8
  //   no pool, G = 32   41.2 / 40.9   55.5 / 55.0  81.9 / 79.3     122.5 / 121.4   166.3 / 155.7   253.7 / 239.8
  // So it costs up to 4 us of about 75 there around 96 MB, where rows that are not so new gain 6, and gives on either side.
  const int64_t key_bytes = groups * G * (2 * kHeadDim);
  const int32_t last_first = key_bytes >= (1ll << 27);
  const bool once = key_bytes >= (1ll << 25);
  if (many && once) return go(prompt_quantize_kernel<BITS, G, LAYERS, true>, 0, last_first);
  if (many) return go(prompt_quantize_kernel<BITS, G, LAYERS, false>, 0, last_first);
  const size_t smem = quant_lds_bytes<G>(d.vgroups);
  if (smem > 48 * 1024) {  // more than the default limit of dynamic LDS per workgroup
    hipError_t e = hipFuncSetAttribute((const void*)quantize_kernel<BITS, G, LAYERS>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)smem);
    if (e != hipSuccess) return e;
  }
  return go(quantize_kernel<BITS, G, LAYERS>, smem);
}

}  // namespace

hipError_t launch_append(const Dims& d, const __half* k_new, const __half* v_new, __half* k_res, __half* v_res,
                         int32_t row, hipStream_t s) {
  hipLaunchKernelGGL(append_kernel, dim3(d.units_per_layer), dim3(128), 0, s, d, k_new, v_new, k_res, v_res, row);
  return hipGetLastError();
}

namespace {

template <int BITS, int G>
hipError_t launch_group_step_one(const Dims& d, int32_t group_index, const __half* k_new, const __half* v_new,
                                 __half* k_res, __half* v_res, int32_t append_row, int32_t group_row0,
                                 const int32_t* seq, const kvq_pool& pool, uint8_t* selected, const kvq_qcache& qc,
                                 hipStream_t s) {
  const size_t smem = quant_lds_bytes<G>(d.vgroups);
  if (smem > 48 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)group_step_kernel<BITS, G>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((group_step_kernel<BITS, G>), dim3(d.units_per_layer), dim3(kQuantThreads), smem, s, d,
                     group_index, k_new, v_new, k_res, v_res, append_row, group_row0, seq, (__half*)pool.pool_k,
                     (__half*)pool.pool_v, pool.pool_idx, pool.pool_score, pool.pool_count, pool.aux_count,
                     pool.frozen, selected, (uint8_t*)qc.k_codes, (uint32_t*)qc.k_meta, (uint8_t*)qc.v_codes,
                     (uint32_t*)qc.v_meta, (uint32_t*)qc.mask);
  return hipGetLastError();
}

template <int BITS>
hipError_t launch_group_step_bits(const Dims& d, int32_t group_index, const __half* k_new, const __half* v_new,
                                  __half* k_res, __half* v_res, int32_t append_row, int32_t group_row0,
                                  const int32_t* seq, const kvq_pool& pool, uint8_t* selected, const kvq_qcache& qc,
                                  hipStream_t s) {
  switch (d.G) {
    case 32: return launch_group_step_one<BITS, 32>(d, group_index, k_new, v_new, k_res, v_res, append_row, group_row0, seq, pool, selected, qc, s);
    case 64: return launch_group_step_one<BITS, 64>(d, group_index, k_new, v_new, k_res, v_res, append_row, group_row0, seq, pool, selected, qc, s);
    default: return launch_group_step_one<BITS, 128>(d, group_index, k_new, v_new, k_res, v_res, append_row, group_row0, seq, pool, selected, qc, s);
  }
}

}  // namespace

// ---- per-step Value quantization ---------------------------------------------------------------
// One workgroup of 128 threads (thread = channel) per unit; the tokens of the call one after the
// other.  Per token: minimum and maximum of each group of Gv channels, step and zero, codes (Eq. 2,
// the same device functions as the group quantization), the dequantized row back into the ring, the
// steps and zeros to their places in the block's meta, and the token's 2 or 4 bits of 64 or 128
// packed words replaced (the words also hold the block's other tokens of the same 8).
template <int BITS>
__global__ void __launch_bounds__(128) value_tokens_kernel(Dims d, int32_t first_token, int32_t count,
                                                           __half* __restrict__ v_res, int32_t ring_row,
                                                           uint8_t* __restrict__ v_codes,
                                                           uint32_t* __restrict__ v_meta) {
  constexpr int kLevels = (1 << BITS) - 1;
  constexpr int kWords = 32 * BITS;                     // packed words that hold one token's codes
  __shared__ float s_mn[2], s_mx[2];
  __shared__ uint32_t s_words[kWords];
  const int ul = blockIdx.x;
  const int64_t u = d.unit0 + ul;
  const int c = threadIdx.x;                            // channel
  const int gv_shift = 31 - __clz(d.Gv);
  const int nblk_shift = d.bpg_shift;                   // blocks per Key group
  __half* ring = v_res + u * d.res_rows * kHeadDim;
  for (int i = 0; i < count; ++i) {
    const int tok = first_token + i;
    int row = ring_row + i;
    row -= row >= d.res_rows ? d.res_rows : 0;
    const float x = __half2float(ring[row * kHeadDim + c]);
    float mn = x, mx = x;
    const int team = d.Gv < 64 ? d.Gv : 64;
    for (int off = 1; off < team; off <<= 1) {
      mn = fminf(mn, __shfl_xor(mn, off));
      mx = fmaxf(mx, __shfl_xor(mx, off));
    }
    if (d.Gv == 128) {                                  // the group spans both wavefronts
      if ((c & 63) == 0) {
        s_mn[c >> 6] = mn;
        s_mx[c >> 6] = mx;
      }
      __syncthreads();
      mn = fminf(s_mn[0], s_mn[1]);
      mx = fmaxf(s_mx[0], s_mx[1]);
    }
    mn += 0.0f;                                         // a zero minimum is stored as +0
    const __half st = step_of(mn, mx, BITS);
    const float stf = __half2float(st);
    const uint32_t code = quant_code(x, mn, stf, kLevels);
    const float prod = (float)code * stf;               // exact
    ring[row * kHeadDim + c] = __float2half_rn(mn + prod);
    // where the token's block is stored
    const GroupPlace at = place_of_group(d, ul, tok / d.G);
    const int64_t blk = at.row * d.blocks_per_unit + ((int64_t)at.slot << nblk_shift) + ((tok % d.G) >> 5);
    const int tb = tok & 31;
    if ((c & (d.Gv - 1)) == 0) {
      const int j = c >> gv_shift;
      __half* gm = (__half*)(v_meta + blk * 32 * d.vgroups);
      gm[((tb >> 1) * d.vgroups + j) * 2 + (tb & 1)] = st;
      gm[32 * d.vgroups + ((tb >> 1) * d.vgroups + j) * 2 + (tb & 1)] = __float2half_rn(mn);
    }
    // codes: channel c = 16 f + n of token tb = 8 r + xx lives in lane 16 r + n, field f, code xx
    const int n = c & 15, f = c >> 4, xx = tb & 7, r = tb >> 3;
    const int slot = BITS == 2 ? n * 4 + (f >> 1) : (f >> 2) * 64 + n * 4 + (f & 3);
    __syncthreads();                                    // the previous token's words have been used
    if (c < kWords) s_words[c] = 0;
    __syncthreads();
    atomicOr(&s_words[slot], place_code(code, code_bit(BITS, f, xx)));
    __syncthreads();
    if (c < kWords) {
      const int half = BITS == 2 ? 0 : c >> 6, nn = (c & 63) >> 2, w = c & 3;
      const uint32_t clear = BITS == 2 ? (place_code(3u, code_bit(2, 0, xx)) | place_code(3u, code_bit(2, 1, xx)))
                                       : place_code(15u, code_bit(4, 0, xx));
      uint32_t* gw = (uint32_t*)(v_codes + blk * d.block_bytes + 1024 * half + 16 * (16 * r + nn) + 4 * w);
      *gw = (*gw & ~clear) | s_words[c];
    }
  }
}

hipError_t launch_value_tokens(const Dims& d, int32_t first_token, int32_t count, __half* v_res, int32_t ring_row,
                               const kvq_qcache& qc, hipStream_t s) {
  if (d.bits == 2)
    hipLaunchKernelGGL(value_tokens_kernel<2>, dim3(d.units_per_layer), dim3(128), 0, s, d, first_token, count, v_res,
                       ring_row, (uint8_t*)qc.v_codes, (uint32_t*)qc.v_meta);
  else
    hipLaunchKernelGGL(value_tokens_kernel<4>, dim3(d.units_per_layer), dim3(128), 0, s, d, first_token, count, v_res,
                       ring_row, (uint8_t*)qc.v_codes, (uint32_t*)qc.v_meta);
  return hipGetLastError();
}

// The state of every active sequence after one token has been appended to it (and its oldest group
// quantized if that filled its ring): the rule group_step_kernel applies, applied to the array.
__global__ void seq_advance_kernel(Dims d, int32_t* seq) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= d.batch) return;
  int4 own = *(const int4*)(seq + 4 * b);
  if (!own.w || own.x < 0 || own.y < 0 || own.y >= d.res_rows || own.z < 0 || own.z >= d.res_rows) return;
  const bool close_group =
      own.z + 1 == d.R + d.G && own.y % d.G == 0 && own.x % d.G == 0 && own.x + d.G <= d.max_seq;
  own.z += 1;
  if (close_group) {
    own.x += d.G;
    own.z -= d.G;
    own.y += d.G;
    own.y -= own.y >= d.res_rows ? d.res_rows : 0;
  }
  *(int4*)(seq + 4 * b) = own;
}

// A launch plan for the decode attention of sequences of different lengths: `entries` workgroups per kv
// head are dealt to the sequences by the work each has (mini-chunks of quantized tokens, groups of
// full-precision rows at half a mini-chunk each), every sequence at least one; a sequence's workgroups
// share its mini-chunks equally.  The share m of one workgroup is the smallest for which the sequences'
// workgroups, ceil(work / m) each, are at most `entries` in all (found by bisection: that count does not
// grow with m).  One workgroup, one thread per sequence.  What bounds it is the bisection, one sum over the
// sequences per step: up to 64 sequences are one wavefront's, which needs neither LDS nor barriers for it
// (32 sequences of 128 .. 8192 tokens: 6.6 -> 4.6 us).
template <bool ONE_WAVE>
__global__ void __launch_bounds__(1024) seq_plan_kernel(Dims d, const int32_t* __restrict__ seq, int32_t max_nq,
                                                         int32_t max_nres, int32_t entries, int32_t* __restrict__ plan) {
  __shared__ int s_acc;
  __shared__ int s_wave[16];
  const int b = threadIdx.x;
  const bool live = b < d.batch;
  int nq = 0, rs = 0, nr = 0, w = 0, mc = 0;
  if (live) {
    const int4 own = *(const int4*)(seq + 4 * b);
    nq = min(max(own.x, 0), max_nq) & ~(kBlockTokens - 1);
    rs = (own.y >= 0 && own.y < d.res_rows) ? own.y & ~15 : 0;
    nr = min(max(own.z, 0), max_nres);
    mc = (nq + kMiniChunk - 1) / kMiniChunk;
    w = 2 * mc + ((nr + kFpGroupRows - 1) / kFpGroupRows) + ((d.pool_slots + kFpGroupRows - 1) / kFpGroupRows);
  }
  auto block_sum = [&](int v) {
    if (ONE_WAVE) return __builtin_amdgcn_readlane(wave_scan(v), 63);
    if (threadIdx.x == 0) s_acc = 0;
    __syncthreads();
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if ((threadIdx.x & 63) == 0) atomicAdd(&s_acc, v);
    __syncthreads();
    const int r = s_acc;
    __syncthreads();
    return r;
  };
  auto block_max = [&](int v) {
    for (int off = 32; off > 0; off >>= 1) v = max(v, __shfl_xor(v, off));
    if (ONE_WAVE) return __builtin_amdgcn_readfirstlane(v);
    if (threadIdx.x == 0) s_acc = 0;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) atomicMax(&s_acc, v);
    __syncthreads();
    const int r = s_acc;
    __syncthreads();
    return r;
  };
  auto splits_for = [&](int m) { return live ? min(max((w + m - 1) / m, 1), max(mc, 1)) : 0; };
  int lo = 1, hi = max(block_max(w), 1);                // at m = hi every sequence has one workgroup: entries >= batch
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (block_sum(splits_for(mid)) <= entries) hi = mid;
    else lo = mid + 1;
  }
  const int sp = splits_for(lo);
  // exclusive prefix of the sequences' workgroup counts
  const int incl = wave_scan(sp);
  int before = 0;
  if (!ONE_WAVE) {
    if ((threadIdx.x & 63) == 63) s_wave[threadIdx.x >> 6] = incl;
    __syncthreads();
    for (int k = 0; k < (int)(threadIdx.x >> 6); ++k) before += s_wave[k];
  }
  const int first = before + incl - sp;
  if (threadIdx.x == blockDim.x - 1) plan[0] = min(first + sp, entries);
  if (live) {
    const int per = (mc + sp - 1) / sp;                  // mini-chunks per workgroup of this sequence
    for (int k = 0; k < sp && first + k < entries; ++k) {
      int4* e = (int4*)(plan + 8 + 8 * (first + k));
      e[0] = make_int4(b, k, sp, min(k * per, mc));
      e[1] = make_int4(nq, rs, nr, min((k + 1) * per, mc));
    }
  }
}

hipError_t launch_seq_plan(const Dims& d, const int32_t* seq, int32_t max_n_quant, int32_t max_n_res, int32_t entries,
                           int32_t* plan, hipStream_t s) {
  if (d.batch <= 64)
    hipLaunchKernelGGL(seq_plan_kernel<true>, dim3(1), dim3(64), 0, s, d, seq, max_n_quant, max_n_res, entries, plan);
  else
    hipLaunchKernelGGL(seq_plan_kernel<false>, dim3(1), dim3(1024), 0, s, d, seq, max_n_quant, max_n_res, entries, plan);
  return hipGetLastError();
}

hipError_t launch_seq_advance(const Dims& d, int32_t* seq, hipStream_t s) {
  hipLaunchKernelGGL(seq_advance_kernel, dim3((d.batch + 255) / 256), dim3(256), 0, s, d, seq);
  return hipGetLastError();
}

hipError_t launch_group_step(const Dims& d, int32_t group_index, const __half* k_new, const __half* v_new,
                             __half* k_res, __half* v_res, int32_t append_row, int32_t group_row0,
                             const int32_t* seq, const kvq_pool& pool, uint8_t* selected, const kvq_qcache& qc,
                             hipStream_t s) {
  return d.bits == 2 ? launch_group_step_bits<2>(d, group_index, k_new, v_new, k_res, v_res, append_row, group_row0, seq, pool, selected, qc, s)
                     : launch_group_step_bits<4>(d, group_index, k_new, v_new, k_res, v_res, append_row, group_row0, seq, pool, selected, qc, s);
}

// The entry of a sequence in the array of states, {n_quant, 0, n_res, active}.  A launch of its own, behind those that
// write what the entry speaks of: a launch on another stream that finds the sequence active finds its rows and codes
// too.  (Written by a workgroup of the quantization it is seen while others are still at work, and ahead of their loads
// it cost each of them a test.  With it a prompt of 8191 tokens, 8 kv heads, 4 layers takes 60.4 us, 59.0 without.)
__global__ void seq_entry_kernel(int4* at, int4 state) { *at = state; }
hipError_t launch_seq_entry(int32_t* at, int32_t n_quant, int32_t n_res, int32_t active, hipStream_t s) {
  hipLaunchKernelGGL(seq_entry_kernel, dim3(1), dim3(1), 0, s, (int4*)at, make_int4(n_quant, 0, n_res, active));
  return hipGetLastError();
}

hipError_t launch_quantize(const Dims& d, int32_t group_index, int32_t n_groups, const PromptRows& rows,
                           const uint8_t* selected, int64_t selected_unit_stride, const kvq_qcache& qc, hipStream_t s,
                           int32_t tail_n, __half* k_res, __half* v_res) {
  auto go = [&](auto bits, auto group) {
    constexpr int BITS = decltype(bits)::value, G = decltype(group)::value;
    const auto one = rows.layers == 1 ? launch_quantize_one<BITS, G, 1> : launch_quantize_one<BITS, G, kPromptLayers>;
    return one(d, group_index, n_groups, rows, selected, selected_unit_stride, qc, tail_n, k_res, v_res, s);
  };
  auto of_bits = [&](auto bits) {
    switch (d.G) {
      case 32: return go(bits, std::integral_constant<int, 32>{});
      case 64: return go(bits, std::integral_constant<int, 64>{});
      default: return go(bits, std::integral_constant<int, 128>{});
    }
  };
  return d.bits == 2 ? of_bits(std::integral_constant<int, 2>{}) : of_bits(std::integral_constant<int, 4>{});
}

hipError_t launch_tail_copy(const Dims& d, const PromptRows& rows, int32_t n, __half* k_res,
                            __half* v_res, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int by = (n * 16 + 255) / 256;
  auto go = [&](auto kern, const auto& at) {
    hipLaunchKernelGGL(kern, dim3(d.units_per_layer, by > 16 ? 16 : by, rows.layers), dim3(256), 0, s, d,
                       rows.unit_stride, n, k_res, v_res, at);
    return hipGetLastError();
  };
  return rows.layers == 1 ? go(tail_copy_kernel<1>, layer_rows<1>(rows))
                          : go(tail_copy_kernel<kPromptLayers>, rows.at);
}

}  // namespace kvq
