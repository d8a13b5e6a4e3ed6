// Next-token draw (eq. auto-regressive, section 3) fused with the per-row
// state update of the generation loop.
//
// The draw is an exact integer inverse CDF so that it is a function of the
// logits alone:  m = max l;  z_i = (l_i - m) * (1/T);  p_i = exp_sr(z_i);
// w_i = trunc(p_i * 2^32) (uint64);  W = sum w_i;  x = word 0 of
// Philox4x32-10((step, cand, 0, 0), seed);  t = floor(x W / 2^32);
// token = min{i : w_0 + ... + w_i > t}.  Integer sums make the result
// independent of the reduction order.  A row without positive weight (all
// logits -inf or NaN) yields token 0.
//
// exp_sr: Cody-Waite range reduction (Cody & Waite, Software Manual for the
// Elementary Functions, 1980) with n = rint(z log2 e), r = z - n ln2_hi -
// n ln2_lo, then the degree-7 Taylor polynomial of e^r by Horner's rule and
// a scaling by 2^n.  Each step is a separately rounded float32 operation
// (this file is built with contraction off); inputs below -24 give 0.
#include "common.h"
#include "kernels.h"
#include "philox.h"

#pragma clang fp contract(off)

namespace sr {

// trunc(exp_sr((l - m) / T) * 2^32) as a saturating 32-bit word: 2^32 itself
// (exp_sr = 1) comes back as 0xFFFFFFFF, which no smaller float truncates to.
// The same rounded steps in fewer instructions:
//  - n = rint(z log2 e) by adding 1.5 * 2^23 + 32 (an even offset, so ties
//    round alike); the low bits of the sum are n + 32, added to the exponent
//    of the polynomial, which is the exact scaling by 2^n 2^32;
//  - arguments below -24, -inf and NaN are clamped to -25, where the weight
//    truncates to 0 like that of every argument below -22.2.
__device__ __forceinline__ uint32_t weight32(float l, float m, float inv_t) {
  const float kLog2e = __uint_as_float(0x3FB8AA3Bu);
  const float kLn2Hi = __uint_as_float(0x3F317200u);
  const float kLn2Lo = __uint_as_float(0x35BFBE8Eu);
  const float c2 = 0.5f, c3 = __uint_as_float(0x3E2AAAABu), c4 = __uint_as_float(0x3D2AAAABu),
              c5 = __uint_as_float(0x3C088889u), c6 = __uint_as_float(0x3AB60B61u),
              c7 = __uint_as_float(0x39500D01u);
  const float kRound = 12582912.0f + 32.0f;
  const float z = fmaxf(__fmul_rn(__fsub_rn(l, m), inv_t), -25.0f);
  const float t = __fadd_rn(__fmul_rn(z, kLog2e), kRound);
  const float n = __fsub_rn(t, kRound);
  float r = __fsub_rn(z, __fmul_rn(n, kLn2Hi));
  r = __fsub_rn(r, __fmul_rn(n, kLn2Lo));
  float p = c7;
  p = __fadd_rn(__fmul_rn(p, r), c6);
  p = __fadd_rn(__fmul_rn(p, r), c5);
  p = __fadd_rn(__fmul_rn(p, r), c4);
  p = __fadd_rn(__fmul_rn(p, r), c3);
  p = __fadd_rn(__fmul_rn(p, r), c2);
  p = __fadd_rn(__fmul_rn(p, r), 1.0f);
  p = __fadd_rn(__fmul_rn(p, r), 1.0f);
  const float x = __uint_as_float(__float_as_uint(p) + (__float_as_uint(t) << 23));
  uint32_t w;
  asm("v_cvt_u32_f32 %0, %1" : "=v"(w) : "v"(x));
  return w;
}

__device__ __forceinline__ uint64_t weight_of(float l, float m, float inv_t) {
  const uint32_t w = weight32(l, m, inv_t);
  return (uint64_t)w + (w == 0xFFFFFFFFu ? 1u : 0u);
}

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int o) {
  uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
  lo = __shfl_xor(lo, o, 64);
  hi = __shfl_xor(hi, o, 64);
  return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t shfl_up_u64(uint64_t v, int o) {
  uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
  lo = __shfl_up(lo, o, 64);
  hi = __shfl_up(hi, o, 64);
  return ((uint64_t)hi << 32) | lo;
}

constexpr int kSampleThreads = 1024;
constexpr int kSampleWaves = kSampleThreads / 64;
constexpr int kMaxSegments = 128;                 // two per lane of the searching wave

// 4 Q entries per lane of a segment of 256 Q entries, a group of G float4s
// (or 4 G floats) at a time: with 16-byte aligned rows lane l takes float4
// 64 g + l of the segment, else entries 64 e + l.  Past the end: -inf.
template <int G>
__device__ __forceinline__ void load_group(const float* __restrict__ lg, int base, int vocab, bool vec, int lane,
                                           float (&v)[4 * G]) {
  if (vec && base + 256 * G <= vocab) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const float4 a = *reinterpret_cast<const float4*>(lg + base + 256 * g + 4 * lane);
      v[4 * g] = a.x; v[4 * g + 1] = a.y; v[4 * g + 2] = a.z; v[4 * g + 3] = a.w;
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4 * G; ++e) {
      const int i = base + 64 * e + lane;
      v[e] = i < vocab ? lg[i] : -INFINITY;
    }
  }
}

// One work-group per row.  Pass 1: the maximum (greedy: its first index).
// Pass 2: exact integer weights, summed per segment of 256 Q entries; a wave
// takes every 16th segment, its lanes accumulate over the whole segment and
// are summed once.  Then wave 0 alone scans the segment sums, finds the
// segment holding the drawn point, in it the lane (4 Q consecutive entries)
// and among those the entry.  All sums are exact 64-bit integers, so the
// drawn token does not depend on the grouping.
//
// Memory bound where the rows in flight exceed the last-level cache (512
// rows of 128256 entries: both passes from HBM, 97 -> 92 us at 5.7 TB/s);
// the weight is ~28 float operations (no packed or fused forms: every step
// is rounded), 47 us of that.  Q = 8 where the row gives every wave a
// segment, else Q = 2 to spread short rows over the waves.
template <int Q, bool GREEDY>
__global__ void __launch_bounds__(kSampleThreads, 8)
sample_kernel(const float* __restrict__ logits, int64_t row_stride, int vocab,
              const int32_t* __restrict__ cand, int step, float inv_t, uint2 key,
              int32_t* __restrict__ next_tok, int32_t* __restrict__ done, int32_t* __restrict__ len,
              int32_t* __restrict__ store, int store_ld, int eos_id) {
  constexpr int G = Q < 4 ? Q : 4;             // float4s of a group
  constexpr int SEG = 256 * Q, GRP = 256 * G;  // entries
  __shared__ uint64_t segsum[kMaxSegments];
  __shared__ float red_v[kSampleWaves];
  __shared__ int red_i[kSampleWaves];

  const int r = blockIdx.x;
  if (done && done[r]) return;  // uniform per block
  const float* lg = logits + (int64_t)r * row_stride;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool vec = (reinterpret_cast<uintptr_t>(lg) & 15) == 0;
  const int ngrp = (vocab + GRP - 1) / GRP;

  // pass 1: groups dealt to the waves, the next one loaded before the
  // current one is compared
  float m = -INFINITY;
  int am = 0x7FFFFFFF;
  {
    float cur[4 * G], nxt[4 * G];
    load_group<G>(lg, wave * GRP, vocab, vec, lane, cur);
    for (int g = wave; g < ngrp; g += kSampleWaves) {
      load_group<G>(lg, (g + kSampleWaves) * GRP, vocab, vec, lane, nxt);
      if constexpr (GREEDY) {
        const bool v4 = vec && (g + 1) * GRP <= vocab;
#pragma unroll
        for (int e = 0; e < 4 * G; ++e)
          if (cur[e] > m) {
            m = cur[e];
            am = g * GRP + (v4 ? 256 * (e >> 2) + 4 * lane + (e & 3) : 64 * e + lane);
          }
      } else {
#pragma unroll
        for (int e = 0; e < 4 * G; ++e) m = fmaxf(m, cur[e]);
      }
#pragma unroll
      for (int e = 0; e < 4 * G; ++e) cur[e] = nxt[e];
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float ov = __shfl_xor(m, o, 64);
    if constexpr (GREEDY) {
      const int oi = __shfl_xor(am, o, 64);
      if (ov > m || (ov == m && oi < am)) { m = ov; am = oi; }
    } else {
      m = fmaxf(m, ov);
    }
  }
  if (lane == 0) {
    red_v[wave] = m;
    if constexpr (GREEDY) red_i[wave] = am;
  }
  __syncthreads();
  m = red_v[0];
  if constexpr (GREEDY) am = red_i[0];
#pragma unroll
  for (int w = 1; w < kSampleWaves; ++w) {
    if constexpr (GREEDY) {
      if (red_v[w] > m || (red_v[w] == m && red_i[w] < am)) { m = red_v[w]; am = red_i[w]; }
    } else {
      m = fmaxf(m, red_v[w]);
    }
  }

  int token = 0;
  if constexpr (GREEDY) {
    if (wave != 0) return;
    token = am < vocab ? am : 0;
  } else {
    // pass 2: segment sums
    const int nseg = (vocab + SEG - 1) / SEG;
    {
      float cur[4 * G], nxt[4 * G];
      load_group<G>(lg, wave * SEG, vocab, vec, lane, cur);
      for (int seg = wave; seg < nseg; seg += kSampleWaves) {
        uint64_t w = 0;
#pragma unroll
        for (int h = 0; h < Q / G; ++h) {
          const int next = h + 1 < Q / G ? seg * SEG + (h + 1) * GRP : (seg + kSampleWaves) * SEG;
          load_group<G>(lg, next, vocab, vec, lane, nxt);
          uint32_t top = 0;
#pragma unroll
          for (int e = 0; e < 4 * G; ++e) {
            const uint32_t u = weight32(cur[e], m, inv_t);  // -inf weighs 0
            w += u;
            top = max(top, u);
          }
          // weights of 2^32 (at least the maximum's own) count one more each;
          // the empty asm keeps this rare second evaluation out of the loop's
          // straight line
          if (__builtin_expect(__any(top == 0xFFFFFFFFu), 0)) {
#pragma unroll
            for (int e = 0; e < 4 * G; ++e) {
              asm volatile("" : "+v"(cur[e]));
              w += weight32(cur[e], m, inv_t) == 0xFFFFFFFFu ? 1u : 0u;
            }
          }
#pragma unroll
          for (int e = 0; e < 4 * G; ++e) cur[e] = nxt[e];
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) w += shfl_xor_u64(w, o);
        if (lane == 0) segsum[seg] = w;
      }
    }
    __syncthreads();
    if (wave != 0) return;
    // scan of the segment sums: lane l owns segments 2 l and 2 l + 1
    const uint64_t s0 = 2 * lane < nseg ? segsum[2 * lane] : 0;
    const uint64_t s1 = 2 * lane + 1 < nseg ? segsum[2 * lane + 1] : 0;
    uint64_t inc = s0 + s1;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint64_t v = shfl_up_u64(inc, o);
      if (lane >= o) inc += v;
    }
    auto from_lane = [](uint64_t v, int src) {
      return ((uint64_t)__shfl((uint32_t)(v >> 32), src, 64) << 32) | __shfl((uint32_t)v, src, 64);
    };
    const uint64_t total = from_lane(inc, 63);
    if (total != 0) {  // (else no distribution: token 0)
      const uint64_t x = philox4x32_10(make_uint4((uint32_t)step, (uint32_t)cand[r], 0u, 0u), key).x;
      const uint64_t t = x * (total >> 32) + ((x * (total & 0xFFFFFFFFull)) >> 32);
      // the first lane, then segment, whose running sum exceeds t (t < total)
      const int hl = (int)__builtin_ctzll(__ballot(inc > t));
      uint64_t base_sum = from_lane(inc - s0 - s1, hl);
      const uint64_t first = from_lane(s0, hl);
      int seg = 2 * hl;
      if (base_sum + first <= t) {
        base_sum += first;
        ++seg;
      }
      // lane l: the 4 Q consecutive entries from 4 Q l of the segment
      const int at = seg * SEG + 4 * Q * lane;
      uint64_t sum = 0;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        float v[4];
        if (vec && at + 4 * q + 4 <= vocab) {
          const float4 a = *reinterpret_cast<const float4*>(lg + at + 4 * q);
          v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = at + 4 * q + e < vocab ? lg[at + 4 * q + e] : -INFINITY;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) sum += weight_of(v[e], m, inv_t);
      }
      uint64_t c = sum;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint64_t v = shfl_up_u64(c, o);
        if (lane >= o) c += v;
      }
      const int hit = (int)__builtin_ctzll(__ballot(base_sum + c > t));
      base_sum += from_lane(c - sum, hit);
      // lane e < 4 Q: entry e of that lane's run
      const int ent = seg * SEG + 4 * Q * hit + lane;
      c = lane < 4 * Q && ent < vocab ? weight_of(lg[ent], m, inv_t) : 0;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint64_t v = shfl_up_u64(c, o);
        if (lane >= o) c += v;
      }
      token = seg * SEG + 4 * Q * hit + (int)__builtin_ctzll(__ballot(base_sum + c > t));
    }
  }
  if (tid == 0) {
    next_tok[r] = token;
    if (store) store[(int64_t)cand[r] * store_ld + step] = token;
    if (len) len[r] = step + 1;
    if (done && token == eos_id) done[r] = 1;
  }
}

void sample(const SampleArgs& a, hipStream_t s) {
  if (a.rows <= 0) return;
  SR_REQUIRE(a.vocab >= 1 && a.vocab <= kMaxSegments * 2048, 3, "vocabulary too large for the sampler");
  const float inv_t = a.temperature == 0.0f ? 1.0f : (float)(1.0 / (double)a.temperature);
  const uint2 key = make_uint2((uint32_t)a.seed, (uint32_t)(a.seed >> 32));
#define SR_SAMPLE(Q, GREEDY)                                                                                       \
  SR_LAUNCH((sample_kernel<Q, GREEDY>), dim3(a.rows), dim3(kSampleThreads), 0, s, a.logits, a.row_stride, a.vocab, \
            a.cand, a.step, inv_t, key, a.next_tok, a.done, a.len, a.store, a.store_ld, a.eos_id)
  // segments of 2048 entries once they give every wave about one, else 512
  const bool longrow = a.vocab > 12 * 2048;
  if (a.temperature == 0.0f) {
    if (longrow) SR_SAMPLE(8, true);
    else SR_SAMPLE(2, true);
  } else {
    if (longrow) SR_SAMPLE(8, false);
    else SR_SAMPLE(2, false);
  }
#undef SR_SAMPLE
  SR_CHECK_LAUNCH();
}

// ---------------------------------------------- probability as the reward
// ln p(tok) = (l_tok - m) - ln sum_i exp(l_i - m), one block per row, sums in
// a fixed order (per thread over a strided range, then the wave butterfly,
// then the waves in order).
__global__ void __launch_bounds__(256)
logprob_kernel(const float* __restrict__ logits, int64_t row_stride, int vocab, const int32_t* __restrict__ cand,
               const int32_t* __restrict__ tok, const int32_t* __restrict__ len, int step,
               float* __restrict__ lp_sum) {
  __shared__ float red[4];
  const int r = blockIdx.x;
  if (len[r] != step + 1) return;  // uniform per block: the row was not sampled at this step
  const float* lg = logits + (int64_t)r * row_stride;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float mv = -INFINITY;
  for (int i = tid; i < vocab; i += 256) mv = fmaxf(mv, lg[i]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mv = fmaxf(mv, __shfl_xor(mv, o, 64));
  if (lane == 0) red[wave] = mv;
  __syncthreads();
  const float m = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  __syncthreads();
  float sum = 0.f;
  for (int i = tid; i < vocab; i += 256) sum += expf(lg[i] - m);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  if (lane == 0) red[wave] = sum;
  __syncthreads();
  if (tid == 0) {
    const float tot = ((red[0] + red[1]) + red[2]) + red[3];
    lp_sum[cand[r]] += (lg[tok[r]] - m) - logf(tot);
  }
}

__global__ void logprob_score_kernel(const float* __restrict__ lp_sum, const int32_t* __restrict__ cand,
                                     const int32_t* __restrict__ len, int rows, float* __restrict__ score) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r < rows) score[r] = len[r] > 0 ? lp_sum[cand[r]] / (float)len[r] : 0.f;
}

void logprob_accumulate(const float* logits, int64_t row_stride, int rows, int vocab, const int32_t* cand,
                        const int32_t* tok, const int32_t* len, int step, float* lp_sum, hipStream_t s) {
  if (rows <= 0) return;
  SR_LAUNCH(logprob_kernel, dim3(rows), dim3(256), 0, s, logits, row_stride, vocab, cand, tok, len, step,
                     lp_sum);
  SR_CHECK_LAUNCH();
}

void logprob_scores(const float* lp_sum, const int32_t* cand, const int32_t* len, int rows, float* score,
                    hipStream_t s) {
  if (rows <= 0) return;
  SR_LAUNCH(logprob_score_kernel, dim3((rows + 255) / 256), dim3(256), 0, s, lp_sum, cand, len, rows,
                     score);
  SR_CHECK_LAUNCH();
}

}  // namespace sr
