// Attention of the decoder.
//
// Decode: every candidate row has one query (the newest token).  Keys are
// the prompt prefix, stored once and shared by all rows, followed by the
// row's own tail.  The query heads of one KV head are the columns of a
// v_mfma_f32_16x16x32_bf16 (S^T = K Q^T, O^T += V^T P^T), so each K/V byte is
// read once per row, and once per group of 16 / G rows for the prefix:
//   decode_group_kernel  (bf16, 64+ rows): a work-group takes a row group;
//                        its waves share the prefix blocks and split the
//                        rows' tails;
//   decode_wave_kernel   (bf16, fewer rows or no prefix): a work-group takes
//                        one (row, KV head), its waves split the keys;
//   decode_attn_kernel   (fp32 and head_dim 32): vector ALU, 16-byte loads,
//                        DPP reductions;
//   prefix_attn_mfma_kernel: the prefix of 16 rows at once, for the
//                        one-query-head-per-KV-head case at 128+ rows.
// Online softmax in base 2; split partials are merged by log-sum-exp.
//
// Prefill (reward-model scoring, prompt): a work-group owns 4 / G blocks (one
// with 8 query heads per KV head) of 32 queries of one row and one KV head
// (MFMA flash attention, bf16 head_dim 64/128), or a block of queries on the vector ALU with K/V staged
// in LDS as fp32.
#include <algorithm>
#include <cfloat>
#include <mutex>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace sr {

constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ float exp2_or_zero(float x) { return x == -INFINITY ? 0.f : exp2f(x); }

// Work-group barrier after this wave's LDS reads and writes complete; vector
// memory loads issued before it stay in flight (__syncthreads would wait for
// them too).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// DPP move within rows of 16 lanes (ctrl: quad_perm 0x00-0xff, row_mirror
// 0x140, row_half_mirror 0x141).
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}

// Sum over aligned groups of LPK lanes; every lane of a group gets the sum.
// Groups of 16 use DPP within the row (xor 1, xor 2, then the mirrored
// quad and half), wider groups cross-lane shuffles.
template <int LPK>
__device__ __forceinline__ float group_sum(float d) {
  if constexpr (LPK == 16) {
    d += dpp_f32<0xB1>(d);   // quad_perm [1,0,3,2]
    d += dpp_f32<0x4E>(d);   // quad_perm [2,3,0,1]
    d += dpp_f32<0x141>(d);  // row_half_mirror
    d += dpp_f32<0x140>(d);  // row_mirror
    return d;
  } else {
#pragma unroll
    for (int o = LPK / 2; o > 0; o >>= 1) d += __shfl_xor(d, o, 64);
    return d;
  }
}

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef short i16x8 __attribute__((ext_vector_type(8)));

// gfx950 LDS transpose read (ds_read_b64_tr_b16).  Every lane names 8 bytes
// (four bf16); within each group of 16 lanes, element e of lane i's result
// is element (i & 3) of the four named by lane 4 e + (i >> 2).
__device__ __forceinline__ i16x4 lds_read_tr16(const bf16_t* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)(p));
}
// LDS byte address of a shared-memory pointer.
__device__ __forceinline__ uint32_t lds_addr(const bf16_t* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const bf16_t*)(p);
}
// Transpose reads at byte offsets LO and HI from each of N LDS addresses,
// complete on return (issue and wait are one block).  Unlike the builtin,
// after which the compiler waits for every copy into LDS still in flight
// (vmcnt 0), they leave the next tile's copies flying.
template <int N, int LO, int HI>
__device__ __forceinline__ void lds_read_tr16_pairs(const uint32_t (&a)[N], i16x4 (&lo)[N], i16x4 (&hi)[N]) {
  static_assert(N == 2 || N == 4, "pairs");
  if constexpr (N == 2) {
    asm volatile(
        "ds_read_b64_tr_b16 %0, %4 offset:%6\n\tds_read_b64_tr_b16 %1, %4 offset:%7\n\t"
        "ds_read_b64_tr_b16 %2, %5 offset:%6\n\tds_read_b64_tr_b16 %3, %5 offset:%7\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(lo[0]), "=&v"(hi[0]), "=&v"(lo[1]), "=&v"(hi[1])
        : "v"(a[0]), "v"(a[1]), "n"(LO), "n"(HI)
        : "memory");
  } else if constexpr (N == 4) {
    asm volatile(
        "ds_read_b64_tr_b16 %0, %8 offset:%12\n\tds_read_b64_tr_b16 %1, %8 offset:%13\n\t"
        "ds_read_b64_tr_b16 %2, %9 offset:%12\n\tds_read_b64_tr_b16 %3, %9 offset:%13\n\t"
        "ds_read_b64_tr_b16 %4, %10 offset:%12\n\tds_read_b64_tr_b16 %5, %10 offset:%13\n\t"
        "ds_read_b64_tr_b16 %6, %11 offset:%12\n\tds_read_b64_tr_b16 %7, %11 offset:%13\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(lo[0]), "=&v"(hi[0]), "=&v"(lo[1]), "=&v"(hi[1]), "=&v"(lo[2]), "=&v"(hi[2]), "=&v"(lo[3]),
          "=&v"(hi[3])
        : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "n"(LO), "n"(HI)
        : "memory");
  }
}

// the value of lane l ^ 32
__device__ __forceinline__ float other_half(float v) {
  const uint32_t u = __float_as_uint(v);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float((threadIdx.x & 32) ? r[0] : r[1]);
}

// two transpose reads as one MFMA operand (the 16-bit words reinterpreted
// as a whole vector)
__device__ __forceinline__ bf16x8 tr16_pair(i16x4 lo, i16x4 hi) {
  const i16x8 w = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, w);
}

template <typename T, int HD, int G>
__global__ void __launch_bounds__(256)
decode_attn_kernel(const float* __restrict__ q, const T* __restrict__ kpre, const T* __restrict__ vpre,
                   int P, const T* __restrict__ ktail, const T* __restrict__ vtail, int cap, int lt,
                   int hq, int hkv, int kps, int splits, float* __restrict__ part,
                   T* __restrict__ out, float qscale) {
  constexpr int EPL = Vec16<T>::N;   // elements per 16-byte load
  constexpr int LPK = HD / EPL;      // lanes per key row
  constexpr int KPW = 64 / LPK;      // keys per wave step
  constexpr int U = 4;               // keys per lane per iteration
  constexpr int NW = 4;              // waves
  // keys [0, P + lt) in splits of kps
  const int split = blockIdx.x, h = blockIdx.y, row = blockIdx.z;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sub = lane % LPK, ks = lane / LPK;
  const int total = P + lt;
  const int k0 = split * kps, k1 = min(total, k0 + kps);

  float qv[G][EPL];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int e = 0; e < EPL; ++e)
      qv[g][e] = q[((int64_t)row * hq + h * G + g) * HD + sub * EPL + e] * qscale;

  float m[G], l[G], acc[G][EPL];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    m[g] = -INFINITY;
    l[g] = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[g][e] = 0.f;
  }
  const T* kt = ktail + ((int64_t)row * hkv + h) * cap * HD;
  const T* vt = vtail + ((int64_t)row * hkv + h) * cap * HD;
  const T* kp = kpre + (int64_t)h * P * HD;
  const T* vp = vpre + (int64_t)h * P * HD;

  // Raw 16-byte loads of the next U keys are issued before the current U
  // keys are consumed (two register sets, unrolled by two).
  constexpr int STEP = NW * KPW * U;
  uint4 rk0[U], rv0[U], rk1[U], rv1[U];
  auto fetch = [&](int base, uint4 (&rk)[U], uint4 (&rv)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = min(base + (u * NW + wave) * KPW + ks, k1 - 1);
      const T* kr = (j < P) ? kp + (int64_t)j * HD : kt + (int64_t)(j - P) * HD;
      const T* vr = (j < P) ? vp + (int64_t)j * HD : vt + (int64_t)(j - P) * HD;
      rk[u] = *reinterpret_cast<const uint4*>(kr + sub * EPL);
      rv[u] = *reinterpret_cast<const uint4*>(vr + sub * EPL);
    }
  };
  auto consume = [&](int base, const uint4 (&rk)[U], const uint4 (&rv)[U]) {
    float s[U][G];
    bool valid[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = base + (u * NW + wave) * KPW + ks;
      valid[u] = j < k1;
      float kf[EPL];
      Vec16<T>::load(reinterpret_cast<const T*>(&rk[u]), kf);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        float d = 0.f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) d = fmaf(qv[g][e], kf[e], d);
        d = group_sum<LPK>(d);
        s[u][g] = valid[u] ? d : -INFINITY;
      }
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      float mt = s[0][g];
#pragma unroll
      for (int u = 1; u < U; ++u) mt = fmaxf(mt, s[u][g]);
      const float mn = fmaxf(m[g], mt);
      if (mn == -INFINITY) continue;
      const float corr = exp2_or_zero(m[g] - mn);
      l[g] *= corr;
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[g][e] *= corr;
      m[g] = mn;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float vf[EPL];
      Vec16<T>::load(reinterpret_cast<const T*>(&rv[u]), vf);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const float p = (m[g] == -INFINITY) ? 0.f : exp2_or_zero(s[u][g] - m[g]);
        l[g] += p;
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[g][e] = fmaf(p, vf[e], acc[g][e]);
      }
    }
  };
  if (k0 < k1) {
    fetch(k0, rk0, rv0);
    for (int base = k0; base < k1; base += 2 * STEP) {
      fetch(base + STEP, rk1, rv1);
      consume(base, rk0, rv0);
      fetch(base + 2 * STEP, rk0, rv0);
      if (base + STEP < k1) consume(base + STEP, rk1, rv1);
    }
  }

  // merge the KPW key slots of a wave (lanes with equal `sub`)
#pragma unroll
  for (int o = LPK; o < 64; o <<= 1) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const float mo = __shfl_xor(m[g], o, 64);
      const float lo = __shfl_xor(l[g], o, 64);
      const float mn = fmaxf(m[g], mo);
      const float c1 = (mn == -INFINITY) ? 0.f : exp2_or_zero(m[g] - mn);
      const float c2 = (mn == -INFINITY) ? 0.f : exp2_or_zero(mo - mn);
      l[g] = l[g] * c1 + lo * c2;
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        const float ao = __shfl_xor(acc[g][e], o, 64);
        acc[g][e] = acc[g][e] * c1 + ao * c2;
      }
      m[g] = mn;
    }
  }
  // merge the waves through LDS
  __shared__ float sm[NW][G], sl[NW][G];
  __shared__ float sacc[NW][G][HD];
  if (ks == 0) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (sub == 0) {
        sm[wave][g] = m[g];
        sl[wave][g] = l[g];
      }
#pragma unroll
      for (int e = 0; e < EPL; ++e) sacc[wave][g][sub * EPL + e] = acc[g][e];
    }
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < G * HD; idx += blockDim.x) {
    const int g = idx / HD, dd = idx % HD;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, sm[w][g]);
    float L = 0.f, A = 0.f;
    if (M != -INFINITY) {
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float c = exp2_or_zero(sm[w][g] - M);
        L += sl[w][g] * c;
        A += sacc[w][g][dd] * c;
      }
    }
    const int qh = h * G + g;
    if (out) {
      out[((int64_t)row * hq + qh) * HD + dd] = from_f32<T>(A / L);
    } else {
      float* p = part + (((int64_t)row * hq + qh) * splits + split) * (HD + 2);
      p[dd] = A;
      if (dd == 0) {
        p[HD] = M;
        p[HD + 1] = L;
      }
    }
  }
}

// ------------------------------------------------ decode (waves split keys)
// Wait until at most N vector-memory operations of this wave are in flight.
template <int N>
__device__ __forceinline__ void vm_wait() {
  if constexpr (N == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  else if constexpr (N == 8) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
  else if constexpr (N == 16) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
  else static_assert(N < 0, "add this wait count");
}

// 16-byte chunk slot of chunk c of key k (k = key index within a 32-key V
// block) in the LDS copy: XOR-swizzled so that the transpose reads of a
// wave (four consecutive keys per lane group, two chunks each) spread over
// the banks.
template <int CPK>
__device__ __forceinline__ int vslot(int k, int c) {
  if constexpr (CPK == 16) return c ^ (((k & 3) << 1) | (((k >> 2) & 1) << 3));
  else return c ^ ((k & 3) << 1);
}

// Sum of split partials: load(offset, x) reads NX values of a split, add(x)
// accumulates them, in split order; the loads of U splits go out together
// (one memory round trip per U splits).
template <int U, int NX, typename T = float, typename Load, typename Add>
__device__ __forceinline__ void sum_splits(int splits, int64_t stride, Load&& load, Add&& add) {
  for (int s0 = 0; s0 < splits; s0 += U) {
    T x[U][NX];
#pragma unroll
    for (int u = 0; u < U; ++u) load(min(s0 + u, splits - 1) * stride, x[u]);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (s0 + u < splits) add(x[u]);
  }
}

// The K rows of keys [k0, k1) (at most 32) as A operand rows: key 16 t + l %
// 16, dims 32 st + 8 (l / 16) .. + 8; keys past the end repeat the last.
template <int HD>
__device__ __forceinline__ void load_k_block(const bf16_t* __restrict__ k, int k0, int k1, uint4 (&kr)[2][HD / 32]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const bf16_t* src = k + (int64_t)min(k0 + 16 * t + (lane & 15), k1 - 1) * HD + 8 * (lane >> 4);
#pragma unroll
    for (int st = 0; st < HD / 32; ++st) kr[t][st] = *reinterpret_cast<const uint4*>(src + 32 * st);
  }
}

// The V rows of the same keys into an LDS buffer of 32 rows, chunks swizzled
// (vslot).  Buffer loads: with global_load_lds in flight (an access of two
// address spaces to the compiler) every use of a loaded register would wait
// for all loads (vmcnt 0), the next block's among them.
template <int HD>
__device__ __forceinline__ void copy_v_block(BufRsrc v, int k0, int k1, bf16_t* dst) {
  constexpr int CPK = HD / 8, KPD = 64 / CPK;   // chunks per key, keys per copy
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < 32 / KPD; ++i) {
    const int kk = i * KPD + lane / CPK;
    const int j = min(kk, k1 - k0 - 1);
    dma16(v, (uint32_t)((j * HD + 8 * vslot<CPK>(kk, lane % CPK)) * 2), k0 * HD * 2, dst + i * 512);
  }
}

// Decode attention over the prefix (unless another pass attends it) and the
// tail for bf16, head_dim 64 or 128, on MFMA, with the keys split between the
// NW waves of a work-group (and between `splits` work-groups per (row, KV
// head)): each wave streams its own contiguous run of bpw 32-key blocks and
// waits on no other wave until the final merge.  Work-group = (split, KV head,
// row); the G query heads of the KV head are the MFMA's 16 columns (columns
// >= G are zero queries whose results are dropped).
//   S^T = K Q^T: the A operand (16 keys x 32 dims) is loaded from memory
//         straight into registers, 16 bytes of one key row per lane.
//   O^T += V^T P^T: a V block is copied memory -> LDS (buffer loads into
//         the wave's own double buffer) and the A operand (16 dims x 32
//         keys) comes from two LDS transpose reads; the key order of the
//         contraction is permuted so that the B operand is the lane's own 8
//         probabilities (keys 4 (l/16) + i and 16 + 4 (l/16) + i).
// The K loads and V copy of the next block are in flight while a block is
// computed.  Online softmax in base 2 (q carries log2 e / sqrt(hd)).  The
// waves' (max, sum, unnormalised output) are merged through LDS; the
// work-group writes the output or, with several splits, its partial slot.
// Fused QKV finalize (the decode step's QKV projection leaves split-K
// partials): q is summed from them and rotated here, and the wave that holds
// the newest key sums, rotates and writes its K and V row before it loads
// that key's block.
template <int HD, int G, int NW>
__global__ void __launch_bounds__(64 * NW)
decode_wave_kernel(const float* __restrict__ q, const bf16_t* __restrict__ kpre, const bf16_t* __restrict__ vpre,
                   int P, bf16_t* ktail, bf16_t* vtail, int cap, int lt, int hq, int hkv, int bpw, int prefix,
                   int splits, float* __restrict__ part, bf16_t* __restrict__ out, float qscale,
                   const float* __restrict__ qpart, int qsplits, int qkv_dim, const float2* __restrict__ rope,
                   float* __restrict__ qout) {
  constexpr int KS = HD / 32;           // k-steps of the score product
  constexpr int DT = HD / 16;           // 16-dim tiles of the output
  constexpr int CPK = HD / 8;           // 16-byte chunks per key row
  constexpr int VB = 32 * HD;           // bf16 elements of a 32-key V block
  constexpr int NDMA = VB * 2 / 1024;   // 1 KB copies per V block
  constexpr int INFLIGHT = 2 * KS + NDMA;  // memory operations of one block
  static_assert(HD == 64 || HD == 128, "head_dim");
  static_assert(G >= 1 && G <= 16, "query heads per KV head");
  __shared__ __attribute__((aligned(1024))) bf16_t lds[NW * 2 * VB];
  const int split = blockIdx.x, h = blockIdx.y, row = blockIdx.z;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int fr = lane & 15, fg = lane >> 4;
  // The keys in 32-key blocks: nbp of the prefix (none when another pass
  // attends it), then the tail's; this wave's are blocks [i0, i1).
  const int nbp = prefix ? (P + 31) >> 5 : 0, nball = nbp + ((lt + 31) >> 5);
  const int i0 = min(nball, (split * NW + wave) * bpw), i1 = min(nball, i0 + bpw);
  const int nb = i1 - i0;
  const bf16_t* kt = ktail + ((int64_t)row * hkv + h) * cap * HD;
  const bf16_t* vt = vtail + ((int64_t)row * hkv + h) * cap * HD;
  const bf16_t* kp = kpre + (int64_t)h * P * HD;
  const bf16_t* vp = vpre + (int64_t)h * P * HD;
  const BufRsrc rvp = buf_rsrc(vp), rvt = buf_rsrc(vt);
  bf16_t* vbuf = lds + wave * 2 * VB;

  auto in_tail = [&](int b) { return i0 + b >= nbp; };
  auto key0 = [&](int b) { return 32 * (i0 + b - (in_tail(b) ? nbp : 0)); };
  auto keyend = [&](int b) { return min(key0(b) + 32, in_tail(b) ? lt : P); };
  auto load_k = [&](int b, uint4 (&kr)[2][KS]) { load_k_block<HD>(in_tail(b) ? kt : kp, key0(b), keyend(b), kr); };
  auto copy_v = [&](int b, int buf) {
    copy_v_block<HD>(in_tail(b) ? rvt : rvp, key0(b), keyend(b), vbuf + buf * VB);
  };

  // The first block's loads go out before anything else unless it holds
  // the newest key, which this wave writes first (fused QKV finalize).
  const bool writer = qpart && nb > 0 && i1 == nball;
  const bool early = nb > 0 && !(writer && nb == 1);
  uint4 ka[2][KS], kb[2][KS];
  if (early) {
    load_k(0, ka);
    copy_v(0, 0);
  }

  // fused QKV finalize: the newest key's K (rotated) and V row
  if (writer) {
    const int64_t qs = (int64_t)gridDim.z * qkv_dim;
    const float* pk = qpart + (int64_t)row * qkv_dim + (hq + h) * HD;
    const float* pv = pk + hkv * HD;
    const int64_t at = (((int64_t)row * hkv + h) * cap + lt - 1) * HD;
    for (int d = lane; d < HD / 2; d += 64) {
      const float2 c = rope[d];
      float k1v = 0.f, k2v = 0.f, v1 = 0.f, v2 = 0.f;
      sum_splits<4, 4>(qsplits, qs, [&](int64_t o, float(&x)[4]) {
        x[0] = pk[o + d];
        x[1] = pk[o + HD / 2 + d];
        x[2] = pv[o + d];
        x[3] = pv[o + HD / 2 + d];
      }, [&](const float(&x)[4]) {
        k1v += x[0]; k2v += x[1]; v1 += x[2]; v2 += x[3];
      });
      ktail[at + d] = f32_to_bf16(k1v * c.x - k2v * c.y);
      ktail[at + HD / 2 + d] = f32_to_bf16(k2v * c.x + k1v * c.y);
      vtail[at + d] = f32_to_bf16(v1);
      vtail[at + HD / 2 + d] = f32_to_bf16(v2);
    }
  }

  // Q^T fragments (B operand): lane holds Q[query fr][32 s + 8 fg .. + 8],
  // scaled, bf16.  Fused: the rotation pairs (d, d + hd/2) are the lane's
  // k-steps s and s + KS/2.
  bf16x8 qf[KS];
  {
    const bool qvalid = fr < G;
    const int qh = h * G + (qvalid ? fr : 0);
    float x[KS][8];
#pragma unroll
    for (int st = 0; st < KS; ++st)
#pragma unroll
      for (int e = 0; e < 8; ++e) x[st][e] = 0.f;
    if (qpart) {
      const int64_t qs = (int64_t)gridDim.z * qkv_dim;
      const float* pq = qpart + (int64_t)row * qkv_dim + qh * HD + 8 * fg;
      if (qvalid)
        sum_splits<HD == 64 ? 4 : 2, 2 * KS, f32x4>(qsplits, qs, [&](int64_t o, f32x4(&v)[2 * KS]) {
#pragma unroll
          for (int i = 0; i < 2 * KS; ++i) v[i] = *reinterpret_cast<const f32x4*>(pq + o + 32 * (i / 2) + 4 * (i % 2));
        }, [&](const f32x4(&v)[2 * KS]) {
#pragma unroll
          for (int i = 0; i < 2 * KS; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) x[i / 2][4 * (i % 2) + e] += v[i][e];
        });
      float* qo = qout && split == 0 && wave == 0 && qvalid ? qout + ((int64_t)row * hq + qh) * HD : nullptr;
#pragma unroll
      for (int st = 0; st < KS / 2; ++st)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int d = 32 * st + 8 * fg + e;
          const float x1 = x[st][e], x2 = x[st + KS / 2][e];
          const float2 c = rope[d];
          x[st][e] = x1 * c.x - x2 * c.y;
          x[st + KS / 2][e] = x2 * c.x + x1 * c.y;
          if (qo) {
            qo[d] = x[st][e];
            qo[HD / 2 + d] = x[st + KS / 2][e];
          }
        }
    } else if (qvalid) {
      const float* qr = q + ((int64_t)row * hq + qh) * HD;
#pragma unroll
      for (int st = 0; st < KS; ++st)
#pragma unroll
        for (int e = 0; e < 8; ++e) x[st][e] = qr[32 * st + 8 * fg + e];
    }
#pragma unroll
    for (int st = 0; st < KS; ++st)
#pragma unroll
      for (int e = 0; e < 8; ++e) qf[st][e] = (__bf16)(qvalid ? x[st][e] * qscale : 0.f);
  }

  f32x4 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  // transpose-read addresses: lane names 4 dims (dt 16 + 4 (fr & 3) ..) of
  // key 4 fg + (fr >> 2), and of the key 16 on
  // (in the first buffer; the second key's row sits 16 rows on, same slots)
  uint32_t vaddr[DT];
  {
    const int kr0 = 4 * fg + (fr >> 2);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
      vaddr[dt] = lds_addr(vbuf + kr0 * HD + 8 * vslot<CPK>(kr0, 2 * dt + ((fr & 3) >> 1)) + 4 * (fr & 1));
  }
  auto compute = [&](int b, const uint4 (&kr)[2][KS], auto bufc) {
    f32x4 st[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      st[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s2 = 0; s2 < KS; ++s2)
        st[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kr[t][s2]), qf[s2], st[t], 0, 0,
                                                        0);
    }
    const int left = keyend(b) - key0(b) - 4 * fg;   // keys of the block from this lane's first
    float sv[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      sv[i] = i < left ? st[0][i] : -INFINITY;
      sv[4 + i] = 16 + i < left ? st[1][i] : -INFINITY;
    }
    float mt = sv[0];
#pragma unroll
    for (int i = 1; i < 8; ++i) mt = fmaxf(mt, sv[i]);
    mt = fmaxf(mt, __shfl_xor(mt, 16, 64));
    mt = fmaxf(mt, __shfl_xor(mt, 32, 64));
    // The accumulators are rescaled only when some column's maximum grows (by
    // exactly 1 elsewhere).  Probabilities are relative to the exact maximum, so
    // the largest, 1, loses nothing in bf16: relative to a maximum up to 2^8
    // stale the output was 3-5 % further off.
    if (__any(mt > m)) {
      const float mn = fmaxf(m, mt);
      const float corr = mn == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m - mn);
      l *= corr;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) o[dt] *= corr;
      m = mn;
    }
    const float mr = m == -INFINITY ? 0.f : m;   // (a column without a key so far)
    bf16x8 pf;
    float ps = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float pv = __builtin_amdgcn_exp2f(sv[i] - mr);
      ps += pv;
      pf[i] = (__bf16)pv;
    }
    l += ps;
    constexpr int BUF = decltype(bufc)::value;
#pragma unroll
    for (int d0 = 0; d0 < DT; d0 += 4) {
      const uint32_t va[4] = {vaddr[d0], vaddr[d0 + 1], vaddr[d0 + 2], vaddr[d0 + 3]};
      i16x4 lo[4], hi[4];
      lds_read_tr16_pairs<4, BUF * VB * 2, (BUF * VB + 16 * HD) * 2>(va, lo, hi);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        o[d0 + i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tr16_pair(lo[i], hi[i]), pf, o[d0 + i], 0, 0, 0);
      }
    }
  };

  // One block ahead: a block's loads are in flight while the one before is
  // computed.  Every fetch in the loop is unconditional, so the compiler's
  // own waits for the K registers count the younger block's loads as in
  // flight instead of draining them.
  const std::integral_constant<int, 0> buf0{};
  const std::integral_constant<int, 1> buf1{};
  auto compute_after = [&](auto left, int b, const uint4 (&kr)[2][KS], auto bufc) {
    __builtin_amdgcn_sched_barrier(0);   // (the fetch before it stays before it)
    vm_wait<decltype(left)::value>();
    compute(b, kr, bufc);
    __builtin_amdgcn_sched_barrier(0);
  };
  const std::integral_constant<int, INFLIGHT> next{};
  if (nb > 0) {
    if (writer) vm_wait<0>();   // the newest key's row is in memory before it is read
    if (!early) {
      load_k(0, ka);
      copy_v(0, 0);
    }
    int b = 0;
    for (; b + 2 < nb; b += 2) {
      load_k(b + 1, kb);
      copy_v(b + 1, 1);
      compute_after(next, b, ka, buf0);
      load_k(b + 2, ka);
      copy_v(b + 2, 0);
      compute_after(next, b + 1, kb, buf1);
    }
    if (b + 1 < nb) {
      load_k(b + 1, kb);
      copy_v(b + 1, 1);
      compute_after(next, b, ka, buf0);
      compute_after(buf0, b + 1, kb, buf1);
    } else {
      compute_after(buf0, b, ka, buf0);
    }
  }

  // merge the waves: per query (max, sum, unnormalised output)
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  __syncthreads();
  float* sm = reinterpret_cast<float*>(lds);  // [NW][G][HD + 2]
  if (fr < G) {
    float* w = sm + (wave * G + fr) * (HD + 2);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int i = 0; i < 4; ++i) w[dt * 16 + 4 * fg + i] = o[dt][i];
    if (fg == 0) {
      w[HD] = m;
      w[HD + 1] = l;
    }
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < G * HD; idx += 64 * NW) {
    const int g = idx / HD, d = idx % HD;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, sm[(w * G + g) * (HD + 2) + HD]);
    float L = 0.f, A = 0.f;
    if (M != -INFINITY) {
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float* ws = sm + (w * G + g) * (HD + 2);
        const float c = exp2_or_zero(ws[HD] - M);
        L += ws[HD + 1] * c;
        A += ws[d] * c;
      }
    }
    const int qh = h * G + g;
    if (splits == 1 && out) {
      out[((int64_t)row * hq + qh) * HD + d] = f32_to_bf16(A / L);
    } else {
      float* pp = part + (((int64_t)row * hq + qh) * splits + split) * (HD + 2);
      pp[d] = A;
      if (d == 0) {
        pp[HD] = M;
        pp[HD + 1] = L;
      }
    }
  }
}

// Decode attention of a group of R = 16 / G rows of one KV head, the shared
// prefix attended once for the whole group (bf16, head_dim 64 or 128, MFMA).
// The 16 MFMA columns are the group's R rows x G query heads, so a prefix
// key block costs the same MFMAs as one row's tail block but serves R rows.
// Work-group = (split, KV head, row group), NW = R WPR waves: wave w takes
// an even share of the prefix blocks (all 16 columns) and one WPR-th of row
// (w mod R)'s tail blocks (the other rows' columns masked), all streamed as
// one run as in decode_wave_kernel (K into registers, V copied to the wave's
// LDS double buffer and read back transposed), with one softmax state per
// column.  The waves' partials are merged per column through LDS; the
// work-group writes the output or, with several splits, its partial slot.
// Fused QKV finalize: the wave holding a row's last tail block writes the
// row's newest K/V first.
template <int HD, int G, int WPR>
__global__ void __launch_bounds__(64 * (16 / G) * WPR)
decode_group_kernel(const float* __restrict__ q, const bf16_t* __restrict__ kpre, const bf16_t* __restrict__ vpre,
                    int P, bf16_t* ktail, bf16_t* vtail, int cap, int lt, int hq, int hkv, int rows, int splits,
                    float* __restrict__ part, bf16_t* __restrict__ out, float qscale, const float* __restrict__ qpart,
                    int qsplits, int qkv_dim, const float2* __restrict__ rope) {
  constexpr int R = 16 / G;             // rows per group
  constexpr int NW = R * WPR;           // waves
  constexpr int KS = HD / 32, DT = HD / 16, CPK = HD / 8;
  constexpr int VB = 32 * HD;
  constexpr int NDMA = VB * 2 / 1024;
  constexpr int INFLIGHT = 2 * KS + NDMA;
  static_assert(HD == 64 || HD == 128, "head_dim");
  static_assert(G == 2 || G == 4 || G == 8, "query heads per KV head");
  static_assert(NW <= 8 && NW * 16 * (HD + 2) * 4 <= NW * 2 * VB * 2, "merge area within the V buffers");
  __shared__ __attribute__((aligned(1024))) bf16_t lds[NW * 2 * VB];
  const int split = blockIdx.x, h = blockIdx.y, grp = blockIdx.z;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int fr = lane & 15, fg = lane >> 4;
  const int rr = wave % R, wpart = wave / R;
  const int row = grp * R + rr;                 // this wave's tail row
  const bool rowvalid = row < rows;
  // blocks: prefix [pb0, pb1) over all splits x waves; tail [tb0, tb1) of the row
  const int nbp = (P + 31) >> 5, nbt = (lt + 31) >> 5;
  const int pi = split * NW + wave, pn = splits * NW;
  const int pb0 = nbp * pi / pn, pb1 = nbp * (pi + 1) / pn;
  const int ti = split * WPR + wpart, tn = splits * WPR;
  const int tb0 = rowvalid ? nbt * ti / tn : 0, tb1 = rowvalid ? nbt * (ti + 1) / tn : 0;
  const bf16_t* kt = ktail + ((int64_t)(rowvalid ? row : 0) * hkv + h) * cap * HD;
  const bf16_t* vt = vtail + ((int64_t)(rowvalid ? row : 0) * hkv + h) * cap * HD;
  const bf16_t* kp = kpre + (int64_t)h * P * HD;
  const bf16_t* vp = vpre + (int64_t)h * P * HD;
  const BufRsrc rvp = buf_rsrc(vp), rvt = buf_rsrc(vt);
  bf16_t* vbuf = lds + wave * 2 * VB;

  // fused QKV finalize: the newest key's K (rotated) and V row of this row
  const bool writer = qpart && rowvalid && lt > 0 && tb1 == nbt && tb1 > tb0;
  if (writer) {
    const int64_t qs = (int64_t)rows * qkv_dim;
    const float* pk = qpart + (int64_t)row * qkv_dim + (hq + h) * HD;
    const float* pv = pk + hkv * HD;
    const int64_t at = (((int64_t)row * hkv + h) * cap + lt - 1) * HD;
    for (int d = lane; d < HD / 2; d += 64) {
      const float2 c = rope[d];
      float k1v = 0.f, k2v = 0.f, v1 = 0.f, v2 = 0.f;
      sum_splits<4, 4>(qsplits, qs, [&](int64_t o, float(&x)[4]) {
        x[0] = pk[o + d];
        x[1] = pk[o + HD / 2 + d];
        x[2] = pv[o + d];
        x[3] = pv[o + HD / 2 + d];
      }, [&](const float(&x)[4]) {
        k1v += x[0]; k2v += x[1]; v1 += x[2]; v2 += x[3];
      });
      ktail[at + d] = f32_to_bf16(k1v * c.x - k2v * c.y);
      ktail[at + HD / 2 + d] = f32_to_bf16(k2v * c.x + k1v * c.y);
      vtail[at + d] = f32_to_bf16(v1);
      vtail[at + HD / 2 + d] = f32_to_bf16(v2);
    }
  }

  // Q^T (B operand): column fr = row grp R + fr / G, query head h G + fr % G
  bf16x8 qf[KS];
  {
    const int qrow = grp * R + fr / G;
    const bool qvalid = qrow < rows;
    const int qr = qvalid ? qrow : 0, qh = h * G + fr % G;
    float x[KS][8];
#pragma unroll
    for (int st = 0; st < KS; ++st)
#pragma unroll
      for (int e = 0; e < 8; ++e) x[st][e] = 0.f;
    if (qpart) {
      const int64_t qs = (int64_t)rows * qkv_dim;
      const float* pq = qpart + (int64_t)qr * qkv_dim + qh * HD + 8 * fg;
      if (qvalid)
        sum_splits<HD == 64 ? 4 : 2, 2 * KS, f32x4>(qsplits, qs, [&](int64_t o, f32x4(&v)[2 * KS]) {
#pragma unroll
          for (int i = 0; i < 2 * KS; ++i) v[i] = *reinterpret_cast<const f32x4*>(pq + o + 32 * (i / 2) + 4 * (i % 2));
        }, [&](const f32x4(&v)[2 * KS]) {
#pragma unroll
          for (int i = 0; i < 2 * KS; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) x[i / 2][4 * (i % 2) + e] += v[i][e];
        });
#pragma unroll
      for (int st = 0; st < KS / 2; ++st)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int d = 32 * st + 8 * fg + e;
          const float x1 = x[st][e], x2 = x[st + KS / 2][e];
          const float2 c = rope[d];
          x[st][e] = x1 * c.x - x2 * c.y;
          x[st + KS / 2][e] = x2 * c.x + x1 * c.y;
        }
    } else if (qvalid) {
      const float* qp = q + ((int64_t)qr * hq + qh) * HD;
#pragma unroll
      for (int st = 0; st < KS; ++st)
#pragma unroll
        for (int e = 0; e < 8; ++e) x[st][e] = qp[32 * st + 8 * fg + e];
    }
#pragma unroll
    for (int st = 0; st < KS; ++st)
#pragma unroll
      for (int e = 0; e < 8; ++e) qf[st][e] = (__bf16)(qvalid ? x[st][e] * qscale : 0.f);
  }

  // transpose-read addresses: lane names 4 dims (dt 16 + 4 (fr & 3) ..) of key
  // 4 fg + (fr >> 2) in the first buffer; the key 16 on has the same slots
  uint32_t vaddr[DT];
  {
    const int kr0 = 4 * fg + (fr >> 2);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
      vaddr[dt] = lds_addr(vbuf + kr0 * HD + 8 * vslot<CPK>(kr0, 2 * dt + ((fr & 3) >> 1)) + 4 * (fr & 1));
  }
  f32x4 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  // A block of a row's tail serves only that row's G columns: the other
  // columns' scores are masked, so prefix and tail blocks share one
  // softmax state per column.
  auto compute = [&](int k0, int k1, bool tail, const uint4 (&kr)[2][KS], auto bufc) {
    f32x4 st[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      st[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s2 = 0; s2 < KS; ++s2)
        st[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kr[t][s2]), qf[s2], st[t], 0, 0,
                                                        0);
    }
    const int jb = k0 + 4 * fg;
    const int kend = tail && fr / G != rr ? k0 : k1;   // masked columns: no key
    float sv[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      sv[i] = jb + i < kend ? st[0][i] : -INFINITY;
      sv[4 + i] = jb + 16 + i < kend ? st[1][i] : -INFINITY;
    }
    float mt = sv[0];
#pragma unroll
    for (int i = 1; i < 8; ++i) mt = fmaxf(mt, sv[i]);
    mt = fmaxf(mt, __shfl_xor(mt, 16, 64));
    mt = fmaxf(mt, __shfl_xor(mt, 32, 64));
    // The accumulators are rescaled only when some column's maximum grows (by
    // exactly 1 elsewhere).  Probabilities are relative to the exact maximum, so
    // the largest, 1, loses nothing in bf16: relative to a maximum up to 2^8
    // stale the output was 3-5 % further off.
    if (__any(mt > m)) {
      const float mn = fmaxf(m, mt);
      const float corr = mn == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m - mn);
      l *= corr;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) o[dt] *= corr;
      m = mn;
    }
    const float mr = m == -INFINITY ? 0.f : m;   // (a column without a key so far)
    bf16x8 pf;
    float ps = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float pv = __builtin_amdgcn_exp2f(sv[i] - mr);
      ps += pv;
      pf[i] = (__bf16)pv;
    }
    l += ps;
    constexpr int BUF = decltype(bufc)::value;
#pragma unroll
    for (int d0 = 0; d0 < DT; d0 += 4) {
      const uint32_t va[4] = {vaddr[d0], vaddr[d0 + 1], vaddr[d0 + 2], vaddr[d0 + 3]};
      i16x4 lo[4], hi[4];
      lds_read_tr16_pairs<4, BUF * VB * 2, (BUF * VB + 16 * HD) * 2>(va, lo, hi);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        o[d0 + i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tr16_pair(lo[i], hi[i]), pf, o[d0 + i], 0, 0, 0);
      }
    }
  };
  // The wave's blocks: its prefix share [pk0, pk1) of (kp, vp), then its
  // share [tk0, tk1) of row rr's tail in (kt, vt); one pipeline over both,
  // the next block's loads in flight while a block is computed.
  const int pk0 = 32 * pb0, pk1 = min(32 * pb1, P);
  const int tk0 = 32 * tb0, tk1 = min(32 * tb1, lt);
  const int np = pk1 > pk0 ? (pk1 - pk0 + 31) >> 5 : 0;
  const int nb = np + (tk1 > tk0 ? (tk1 - tk0 + 31) >> 5 : 0);
  auto key0 = [&](int b) { return b < np ? pk0 + 32 * b : tk0 + 32 * (b - np); };
  auto keyend = [&](int b) { return b < np ? min(pk0 + 32 * b + 32, pk1) : min(tk0 + 32 * (b - np) + 32, tk1); };
  auto fetch = [&](int b, uint4 (&kr)[2][KS], int buf) {
    const bool tail = b >= np;
    load_k_block<HD>(tail ? kt : kp, key0(b), keyend(b), kr);
    copy_v_block<HD>(tail ? rvt : rvp, key0(b), keyend(b), vbuf + buf * VB);
  };
  // (fetches in the loop unconditional, as in decode_wave_kernel)
  const std::integral_constant<int, 0> buf0{};
  const std::integral_constant<int, 1> buf1{};
  const std::integral_constant<int, INFLIGHT> next{};
  auto compute_after = [&](auto left, int b, const uint4 (&kr)[2][KS], auto bufc) {
    __builtin_amdgcn_sched_barrier(0);
    vm_wait<decltype(left)::value>();
    compute(key0(b), keyend(b), b >= np, kr, bufc);
    __builtin_amdgcn_sched_barrier(0);
  };
  if (writer) vm_wait<0>();   // the newest key's row is in memory before it is read
  if (nb > 0) {
    uint4 ka[2][KS], kb[2][KS];
    fetch(0, ka, 0);
    int b = 0;
    for (; b + 2 < nb; b += 2) {
      fetch(b + 1, kb, 1);
      compute_after(next, b, ka, buf0);
      fetch(b + 2, ka, 0);
      compute_after(next, b + 1, kb, buf1);
    }
    if (b + 1 < nb) {
      fetch(b + 1, kb, 1);
      compute_after(next, b, ka, buf0);
      compute_after(buf0, b + 1, kb, buf1);
    } else {
      compute_after(buf0, b, ka, buf0);
    }
  }

  // merge: per column c (row grp R + c / G, head h G + c % G) the partials
  // of all waves (prefix shares, and the tail shares of the row's waves)
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  __syncthreads();
  constexpr int SL = HD + 2;
  float* sp_ = reinterpret_cast<float*>(lds);   // [NW][16][SL]
  {
    float* w = sp_ + (wave * 16 + fr) * SL;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int i = 0; i < 4; ++i) w[dt * 16 + 4 * fg + i] = o[dt][i];
    if (fg == 0) {
      w[HD] = m;
      w[HD + 1] = l;
    }
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < 16 * HD; idx += 64 * NW) {
    const int c = idx / HD, d = idx % HD;
    const int orow = grp * R + c / G, g = c % G;
    if (orow >= rows) continue;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, sp_[(w * 16 + c) * SL + HD]);
    float L = 0.f, A = 0.f;
    if (M != -INFINITY) {
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float* ws = sp_ + (w * 16 + c) * SL;
        const float cf = exp2_or_zero(ws[HD] - M);
        L += ws[HD + 1] * cf;
        A += ws[d] * cf;
      }
    }
    const int qh = h * G + g;
    if (splits == 1) {
      out[((int64_t)orow * hq + qh) * HD + d] = f32_to_bf16(A / L);
    } else {
      float* pp = part + (((int64_t)orow * hq + qh) * splits + split) * (HD + 2);
      pp[d] = A;
      if (d == 0) {
        pp[HD] = M;
        pp[HD + 1] = L;
      }
    }
  }
}

template <typename T, int HD>
__global__ void decode_merge_kernel(const float* __restrict__ part, int splits, T* __restrict__ out) {
  const int rq = blockIdx.x;  // row * hq + qh
  const float* p = part + (int64_t)rq * splits * (HD + 2);
  float M = -INFINITY;
  for (int s = 0; s < splits; ++s) M = fmaxf(M, p[s * (HD + 2) + HD]);
  for (int dd = threadIdx.x; dd < HD; dd += blockDim.x) {
    float L = 0.f, A = 0.f;
    for (int s = 0; s < splits; ++s) {
      const float c = exp2_or_zero(p[s * (HD + 2) + HD] - M);
      L += p[s * (HD + 2) + HD + 1] * c;
      A += p[s * (HD + 2) + dd] * c;
    }
    out[(int64_t)rq * HD + dd] = from_f32<T>(A / L);
  }
}

// Keys per split: aim for enough work-groups to fill the chip, at least 128
// keys per split.
static int decode_kps(int rows, int hkv, int keys) {
  int64_t groups = (int64_t)rows * hkv;
  int splits = 1;
  while (groups * splits < 2048 && keys / (splits * 2) >= 128) splits *= 2;
  return (keys + splits - 1) / splits;
}

// Waves decode_wave_kernel aims at over the whole grid.
constexpr int kWaveTarget = 2048;

// The decode rows' attention over the shared prompt prefix (one query head
// per KV head, 128 or more rows): a work-group of one wave takes 16 decode
// rows of one head as the queries of
//   S^T = K Q^T   (v_mfma_f32_16x16x32_bf16; lane l holds keys 4 (l / 16) + i
//                 and 16 on of row l % 16), then
//   O^T += V^T P^T, the key order permuted so that the B operand is the lane's
//                 own probabilities, the A operand by two LDS transpose reads
//                 of the staged V tile.
// Every prefix key is visible.  32-key tiles, the next one fetched into
// registers under the current one.  The tails were attended first and left
// part_splits partial slots per (row, query head) in `part` (unnormalised
// output, running max, sum); they are folded in by log-sum-exp and the
// attention output is written.
__global__ void __launch_bounds__(64)
prefix_attn_mfma_kernel(const float* __restrict__ q, const bf16_t* __restrict__ kpre, const bf16_t* __restrict__ vpre,
                        int P, int rows, int hq, bf16_t* __restrict__ out, float qscale,
                        const float* __restrict__ part, int part_splits) {
  constexpr int HD = 128, NT = 64;
  constexpr int KT = 32;             // keys per staged tile
  constexpr int KS = HD / 32, DT = HD / 16, CPK = HD / 8;
  constexpr int PF_KROW = HD + 8;    // K tile row (bf16), padded
  constexpr int PF_VROW = HD + 16;   // V tile row (bf16), padded: the 8-byte transpose reads of a
                                     // half wave (eight rows) fall on distinct banks
  __shared__ __attribute__((aligned(16))) bf16_t Ks[KT * PF_KROW];
  __shared__ __attribute__((aligned(16))) bf16_t Vs[KT * PF_VROW];
  const int h = blockIdx.y;
  const int fr = threadIdx.x & 15, fg = threadIdx.x >> 4;
  const int t = blockIdx.x * 16 + fr;      // this lane's decode row
  const bool qvalid = t < rows;
  // Q^T fragments: lane holds Q[t][32 s + 8 fg .. +8] for k-step s (scaled,
  // bf16); loaded from a clamped row, unconditionally, so all go out at once
  bf16x8 qf[KS];
  {
    const float sc = qvalid ? qscale : 0.f;
    const float4* qr = reinterpret_cast<const float4*>(q + ((int64_t)min(t, rows - 1) * hq + h) * HD);
    float4 qv[2 * KS];
#pragma unroll
    for (int st = 0; st < KS; ++st) {
      qv[2 * st] = qr[8 * st + 2 * fg];
      qv[2 * st + 1] = qr[8 * st + 2 * fg + 1];
    }
#pragma unroll
    for (int st = 0; st < KS; ++st) {
      const float4 a = qv[2 * st], b = qv[2 * st + 1];
      qf[st][0] = (__bf16)(a.x * sc); qf[st][1] = (__bf16)(a.y * sc);
      qf[st][2] = (__bf16)(a.z * sc); qf[st][3] = (__bf16)(a.w * sc);
      qf[st][4] = (__bf16)(b.x * sc); qf[st][5] = (__bf16)(b.y * sc);
      qf[st][6] = (__bf16)(b.z * sc); qf[st][7] = (__bf16)(b.w * sc);
    }
  }
  f32x4 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  const bf16_t* kp = kpre + (int64_t)h * P * HD;
  const bf16_t* vp = vpre + (int64_t)h * P * HD;
  // a tile is 32 keys x CPK chunks of 8 dims; thread chunks c = tid + NT i
  constexpr int CPT = (KT * CPK + NT - 1) / NT;
  uint4 kreg[CPT], vreg[CPT];
  auto fetch = [&](int kb) {
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int c = threadIdx.x + NT * i;
      const int key = kb + c / CPK, cc = c % CPK;
      kreg[i] = vreg[i] = make_uint4(0, 0, 0, 0);
      if (c < KT * CPK && key < P) {
        kreg[i] = *reinterpret_cast<const uint4*>(kp + (int64_t)key * HD + cc * 8);
        vreg[i] = *reinterpret_cast<const uint4*>(vp + (int64_t)key * HD + cc * 8);
      }
    }
  };
  // Lane i of a group names dims dt 16 + 4 (i & 3) .. + 3 of key
  // 4 fg + (i >> 2) (and 16 keys on), so it receives dim dt 16 + i of keys
  // 4 fg .. + 3 (and 16 + 4 fg .. + 3): the A operand rows of O^T += V^T P^T
  const bf16_t* vb0 = &Vs[(4 * fg + (fr >> 2)) * PF_VROW + 4 * (fr & 3)];
  // the staged tile's keys kb .. kb + 31
  auto compute = [&](int kb) {
    // S^T for key tiles 0 (keys kb..kb+15) and 1 (kb+16..kb+31)
    f32x4 st[2];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      st[kt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const bf16x8 kf = *reinterpret_cast<const bf16x8*>(&Ks[(kt * 16 + fr) * PF_KROW + 32 * s + 8 * fg]);
        st[kt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[s], st[kt], 0, 0, 0);
      }
    }
    // tile maximum for row t (this lane's column)
    float mt = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int key = kb + kt * 16 + 4 * fg + i;
        const bool ok = qvalid && key < P;
        st[kt][i] = ok ? st[kt][i] : -INFINITY;
        mt = fmaxf(mt, st[kt][i]);
      }
    mt = fmaxf(mt, __shfl_xor(mt, 16, 64));
    mt = fmaxf(mt, __shfl_xor(mt, 32, 64));
    const float mn = fmaxf(m, mt);
    const float corr = (mn == -INFINITY) ? 1.f : exp2_or_zero(m - mn);
    float ls = 0.f;
    bf16x8 pf;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float p = (mn == -INFINITY) ? 0.f : exp2_or_zero(st[kt][i] - mn);
        ls += p;
        pf[kt * 4 + i] = (__bf16)p;
      }
    ls += __shfl_xor(ls, 16, 64);
    ls += __shfl_xor(ls, 32, 64);
    l = l * corr + ls;
    m = mn;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      o[dt] *= corr;
      const i16x4 lo = lds_read_tr16(vb0 + dt * 16);
      const i16x4 hi = lds_read_tr16(vb0 + 16 * PF_VROW + dt * 16);
      o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tr16_pair(lo, hi), pf, o[dt], 0, 0, 0);
    }
  };
  fetch(0);
  for (int kb = 0; kb < P; kb += KT) {
    // stage K [key][dim] and V [key][dim]
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int c = threadIdx.x + NT * i;
      if (KT * CPK % NT == 0 || c < KT * CPK) {
        const int j = c / CPK, cc = c % CPK;
        *reinterpret_cast<uint4*>(&Ks[j * PF_KROW + cc * 8]) = kreg[i];
        *reinterpret_cast<uint4*>(&Vs[j * PF_VROW + cc * 8]) = vreg[i];
      }
    }
    lds_barrier();
    if (kb + KT < P) fetch(kb + KT);
    compute(kb);
    lds_barrier();
  }
  if (qvalid) {
    // fold in the tail partials of (row t, head h): slot s holds the
    // unnormalised output, its maximum and its sum
    const float* pr = part + ((int64_t)t * hq + h) * part_splits * (HD + 2);
    float mx = m;
    for (int sp = 0; sp < part_splits; ++sp) mx = fmaxf(mx, pr[sp * (HD + 2) + HD]);
    const float c0 = exp2_or_zero(m - mx);
    float L = l * c0;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[dt] *= c0;
    for (int sp = 0; sp < part_splits; ++sp) {
      const float* ps = pr + sp * (HD + 2);
      const float cs = exp2_or_zero(ps[HD] - mx);
      L += ps[HD + 1] * cs;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int i = 0; i < 4; ++i) o[dt][i] += ps[dt * 16 + 4 * fg + i] * cs;
    }
    const float inv = 1.0f / L;
    bf16_t* orow = out + ((int64_t)t * hq + h) * HD;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int i = 0; i < 4; ++i) orow[dt * 16 + 4 * fg + i] = f32_to_bf16(o[dt][i] * inv);
  }
}

// Whether the shared prefix is attended by the batched MFMA kernel: one query
// head per KV head (more take the row groups from 64 rows), from 128 rows
// (below that it costs more than the L2 reads it saves).
static bool prefix_by_mfma(int dtype, int hd, int g, int P, int rows) {
  return dtype == SR_BF16 && hd == 128 && g == 1 && P > 0 && rows >= 128;
}

// Partial slots needed for `keys` = prefix + maximal tail (upper bound for
// both the combined and the split-prefix forms).
int decode_attn_splits(int rows, int hkv, int keys) {
  int kps = decode_kps(rows, hkv, keys);
  const int old_form = (keys + kps - 1) / kps + (keys + 63) / 64;
  // the key-split kernel: splits <= the waves it wants per (row, KV head),
  // which grow with the key count
  const int64_t pairs = std::max<int64_t>(1, (int64_t)rows * hkv);
  const int wave_form_max = (int)std::max<int64_t>(1, std::min<int64_t>(kWaveTarget / pairs, (keys + 31) / 32));
  return std::max(old_form, wave_form_max);
}

// Work split of decode_wave_kernel over the 32-key blocks of a prefix of P
// and a tail of lt keys, for rows x hkv (row, KV head) pairs: about
// kWaveTarget waves in all (one round of resident waves: LDS holds ten per CU
// at head_dim 128), each with at least two blocks; NW waves per work-group (1,
// 2, 4 or 8) and `splits` work-groups per pair, each wave bpw blocks.  Where
// eight waves per pair already give a thousand waves, one work-group of eight
// takes the pair (no split partials, no merge launch).
struct WavePlan {
  int nw, splits, bpw;
};
static WavePlan wave_plan(int rows, int hkv, int P, int lt) {
  const int64_t pairs = std::max<int64_t>(1, (int64_t)rows * hkv);
  const int blocks = std::max(1, (P + 31) / 32 + (lt + 31) / 32);
  int want = (int)std::max<int64_t>(1, kWaveTarget / pairs);
  want = std::max(1, std::min(want, blocks / 2));
  if (want > 8 && pairs * 8 >= 1024) want = 8;
  WavePlan w;
  w.nw = want >= 8 ? 8 : (want >= 4 ? 4 : (want >= 2 ? 2 : 1));
  const int per = (want + w.nw - 1) / w.nw * w.nw;    // waves per pair
  w.bpw = (blocks + per - 1) / per;
  w.splits = std::max(1, (blocks + w.nw * w.bpw - 1) / (w.nw * w.bpw));
  return w;
}

// Whether decode_wave_kernel takes these keys (bf16, head_dim 64 or 128,
// 1, 2, 4 or 8 query heads per KV head).
static bool wave_form(int dtype, int hd, int g) {
  return dtype == SR_BF16 && (hd == 64 || hd == 128) && (g == 1 || g == 2 || g == 4 || g == 8);
}

// Whether decode_group_kernel takes the launch: bf16, head_dim 64 or 128, 2,
// 4 or 8 query heads per KV head, a prefix, and from 64 rows (fewer rows
// give too few work-groups without splitting).  Waves per row: two where
// that stays within about kWaveTarget waves (not for 2 query heads per KV
// head: eight rows a group already make eight waves), else one.
constexpr int kGroupMinRows = 64;
static bool group_form(int dtype, int hd, int g, int P, int rows) {
  return dtype == SR_BF16 && (hd == 64 || hd == 128) && (g == 2 || g == 4 || g == 8) && P > 0 &&
         rows >= kGroupMinRows;
}
static int group_wpr(int g, int rows, int hkv) {
  const int R = 16 / g;
  const int64_t waves1 = (int64_t)((rows + R - 1) / R) * hkv * R;
  return (g != 2 && waves1 * 2 <= kWaveTarget + kWaveTarget / 8) ? 2 : 1;
}

template <int HD, int G>
static void launch_group(const DecodeAttnArgs& a, float qscale, hipStream_t s) {
  constexpr int R = 16 / G;
  const int wpr = group_wpr(G, a.rows, a.hkv);
  dim3 grid(1, a.hkv, (a.rows + R - 1) / R);
#define SR_GROUP(W)                                                                                               \
  SR_LAUNCH((decode_group_kernel<HD, G, W>), grid, dim3(64 * R * W), 0, s, a.q, (const bf16_t*)a.kpre,  \
                     (const bf16_t*)a.vpre, a.P, (bf16_t*)a.ktail, (bf16_t*)a.vtail, a.cap, a.lt, a.hq, a.hkv,   \
                     a.rows, 1, a.part, (bf16_t*)a.out, qscale, a.qpart, a.qsplits, a.qkv_dim, a.rope)
  if constexpr (G != 2) {
    if (wpr == 2) SR_GROUP(2);
    else SR_GROUP(1);
  } else {
    SR_GROUP(1);
  }
#undef SR_GROUP
  SR_CHECK_LAUNCH();
}

template <int HD, int G>
static void launch_wave(const DecodeAttnArgs& a, bool prefix, const WavePlan& w, bool direct, float qscale,
                        hipStream_t s) {
#define SR_WAVE(NW)                                                                                              \
  SR_LAUNCH((decode_wave_kernel<HD, G, NW>), dim3(w.splits, a.hkv, a.rows), dim3(64 * NW), 0, s, a.q,  \
                     (const bf16_t*)a.kpre, (const bf16_t*)a.vpre, a.P, (bf16_t*)a.ktail, (bf16_t*)a.vtail,       \
                     a.cap, a.lt, a.hq, a.hkv, w.bpw, (int)prefix, w.splits, a.part, direct ? (bf16_t*)a.out : nullptr, \
                     qscale, a.qpart, a.qsplits, a.qkv_dim, a.rope, a.qout)
  if (w.nw == 8) SR_WAVE(8);
  else if (w.nw == 4) SR_WAVE(4);
  else if (w.nw == 2) SR_WAVE(2);
  else SR_WAVE(1);
#undef SR_WAVE
  SR_CHECK_LAUNCH();
}

template <typename T, int HD, int G>
static void launch_decode(const DecodeAttnArgs& a, hipStream_t s) {
  const float qscale = kLog2e / sqrtf((float)HD);
  int splits = 0;
  if constexpr (std::is_same<T, bf16_t>::value && (HD == 64 || HD == 128)) {
    SR_REQUIRE(!a.qpart || (a.lt >= 1 && a.rope && a.qsplits >= 1), SR_ERR_INTERNAL,
               "fused QKV finalize needs a new key");
    if constexpr (G != 1) {
      if (group_form(a.dtype, HD, G, a.P, a.rows)) {
        launch_group<HD, G>(a, qscale, s);
        return;
      }
    }
    // the key-split kernel over the keys past the prefix pass's, then the
    // prefix pass or (several splits without it) the merge
    const bool pre = prefix_by_mfma(a.dtype, HD, G, a.P, a.rows);
    const int pkeys = pre ? 0 : a.P;
    if (pkeys + a.lt > 0) {
      const WavePlan w = wave_plan(a.rows, a.hkv, pkeys, a.lt);
      splits = w.splits;
      const bool direct = !pre && splits == 1;
      if (!direct)
        SR_REQUIRE((size_t)a.rows * a.hq * splits * (HD + 2) <= a.part_cap, 5, "attention partial buffer too small");
      DecodeAttnArgs b = a;
      if (!pre) b.qout = nullptr;  // only the prefix pass reads q back
      launch_wave<HD, G>(b, !pre, w, direct, qscale, s);
    }
    if constexpr (HD == 128 && G == 1) {
      // The batched pass over the shared prefix (16 rows per work-group) runs
      // last: the tails left partial slots and it folds them into its own
      // result, so no merge pass is needed.
      if (pre) {
        SR_LAUNCH(prefix_attn_mfma_kernel, dim3((a.rows + 15) / 16, a.hkv), dim3(64), 0, s, a.q, (const bf16_t*)a.kpre,
                  (const bf16_t*)a.vpre, a.P, a.rows, a.hq, (bf16_t*)a.out, qscale, a.part, splits);
        SR_CHECK_LAUNCH();
        return;
      }
    }
  } else {
    SR_REQUIRE(!a.qpart, SR_ERR_INTERNAL, "fused QKV finalize without the MFMA decode kernels");
    const int keys = a.P + a.lt;
    const int kps = decode_kps(a.rows, a.hkv, keys);
    splits = (keys + kps - 1) / kps;
    if (splits > 1)
      SR_REQUIRE((size_t)a.rows * a.hq * splits * (HD + 2) <= a.part_cap, 5,
                 "attention partial buffer too small");
    SR_LAUNCH((decode_attn_kernel<T, HD, G>), dim3(splits, a.hkv, a.rows), dim3(256), 0, s,
                       a.q, (const T*)a.kpre, (const T*)a.vpre, a.P, (const T*)a.ktail,
                       (const T*)a.vtail, a.cap, a.lt, a.hq, a.hkv, kps, splits, a.part,
                       splits == 1 ? (T*)a.out : (T*)nullptr, qscale);
    SR_CHECK_LAUNCH();
  }
  if (splits > 1) {
    SR_LAUNCH((decode_merge_kernel<T, HD>), dim3(a.rows * a.hq), dim3(HD), 0, s, a.part, splits, (T*)a.out);
    SR_CHECK_LAUNCH();
  }
}

template <typename T, int HD>
static void decode_by_group(const DecodeAttnArgs& a, hipStream_t s) {
  switch (a.hq / a.hkv) {
    case 1: launch_decode<T, HD, 1>(a, s); break;
    case 2: launch_decode<T, HD, 2>(a, s); break;
    case 4: launch_decode<T, HD, 4>(a, s); break;
    case 8: launch_decode<T, HD, 8>(a, s); break;
    default: SR_REQUIRE(false, 3, "query heads per KV head must be 1, 2, 4 or 8");
  }
}

template <typename T>
static void decode_by_hd(const DecodeAttnArgs& a, hipStream_t s) {
  switch (a.hd) {
    case 32: decode_by_group<T, 32>(a, s); break;
    case 64: decode_by_group<T, 64>(a, s); break;
    case 128: decode_by_group<T, 128>(a, s); break;
    default: SR_REQUIRE(false, 3, "head_dim must be 32, 64 or 128");
  }
}

// Whether decode_attn sums the QKV partials itself (the MFMA streaming form:
// bf16, head_dim 128, 1, 2, 4 or 8 query heads per KV head).
bool decode_attn_fuses_qkv(const DecodeAttnArgs& a) {
  if (a.hkv <= 0 || a.hq % a.hkv) return false;
  const int g = a.hq / a.hkv;
  return (g == 1 || g == 2 || g == 4 || g == 8) && a.lt >= 1 &&
         wave_form(a.dtype, a.hd, g);
}

void decode_attn(const DecodeAttnArgs& a, hipStream_t s) {
  if (a.rows <= 0) return;
  if (a.dtype == SR_BF16) decode_by_hd<bf16_t>(a, s);
  else decode_by_hd<float>(a, s);
}

// Split partials (floats) the launch of decode_attn for these arguments
// writes, following the dispatch above (without the fused QKV finalize).
size_t decode_attn_part_floats(const DecodeAttnArgs& a) {
  if (a.rows <= 0 || a.hkv <= 0 || a.hq % a.hkv) return 0;
  const int g = a.hq / a.hkv;
  const size_t per = (size_t)a.rows * a.hq * (a.hd + 2);
  if (group_form(a.dtype, a.hd, g, a.P, a.rows)) return 0;
  if (wave_form(a.dtype, a.hd, g)) {
    const bool pre = prefix_by_mfma(a.dtype, a.hd, g, a.P, a.rows);
    const int pkeys = pre ? 0 : a.P;
    if (pkeys + a.lt <= 0) return 0;
    const WavePlan w = wave_plan(a.rows, a.hkv, pkeys, a.lt);
    return (!pre && w.splits == 1) ? 0 : per * w.splits;
  }
  const int keys = a.P + a.lt;
  const int kps = decode_kps(a.rows, a.hkv, keys);
  const int splits = (keys + kps - 1) / kps;
  return splits > 1 ? per * splits : 0;
}

// ---- decode attention without caller-provided scratch
// For callers that cannot allocate device memory: the split partials go to
// this file-scope array instead of a caller buffer.  Each device that runs
// the library holds its own copy until the process ends; host code reaches
// it only through the address hipGetSymbolAddress reports for the current
// device (the array's name on the host is not a device address).  Every call
// on one device shares the array, so calls that overlap on a device race.
// Every partial slot is written before it is read, so nothing is cleared.
static __device__ __align__(256) float scratch[kStaticScratchFloats];

static std::mutex g_scratch_mu;
static float* g_scratch_dev[kMaxDevices] = {};

float* static_scratch_of_current_device() {
  int dev = -1;
  SR_HIP(hipGetDevice(&dev));
  SR_REQUIRE(dev >= 0 && dev < kMaxDevices, SR_ERR_UNSUPPORTED, "device index beyond the static scratch table");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void* p = nullptr;
    SR_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    SR_REQUIRE(p != nullptr, SR_ERR_DEVICE, "no device address for the static scratch array");
    g_scratch_dev[dev] = static_cast<float*>(p);
  }
  return g_scratch_dev[dev];
}

// --------------------------------------------------------------- prefill
// 256 threads = QB queries x G heads x 4 threads; thread `sub` of a
// (query, head) pair owns dimensions sub, sub + 4, sub + 8, ...
template <typename T, int HD, int G>
__global__ void __launch_bounds__(256)
prefill_attn_kernel(const float* __restrict__ q, const T* __restrict__ kpre, const T* __restrict__ vpre,
                    int P, const T* __restrict__ kown, const T* __restrict__ vown, int lr, int cap, int t0,
                    int hq, int hkv, T* __restrict__ out, float qscale) {
  constexpr int TPQ = 4, DPT = HD / TPQ, QB = 64 / G, KT = 32;
  constexpr int EPL = Vec16<T>::N, CPR = HD / EPL;
  __shared__ float Ks[KT][HD];
  __shared__ float Vs[KT][HD];
  const int qb = blockIdx.x, h = blockIdx.y, row = blockIdx.z;
  const int tid = threadIdx.x;
  const int sub = tid % TPQ, pair = tid / TPQ, g = pair % G, qi = pair / G;
  const int t = qb * QB + qi;
  const bool qvalid = t < lr;
  const int qh = h * G + g;
  float qv[DPT], acc[DPT];
#pragma unroll
  for (int d = 0; d < DPT; ++d) {
    qv[d] = qvalid ? q[(((int64_t)row * lr + t) * hq + qh) * HD + d * TPQ + sub] * qscale : 0.f;
    acc[d] = 0.f;
  }
  float m = -INFINITY, l = 0.f;
  const int tlast = min(lr, (qb + 1) * QB) - 1;
  const int nkeys = P + t0 + tlast + 1;
  const T* kp = kpre + (int64_t)h * P * HD;
  const T* vp = vpre + (int64_t)h * P * HD;
  const T* ko = kown + ((int64_t)row * hkv + h) * cap * HD;
  const T* vo = vown + ((int64_t)row * hkv + h) * cap * HD;
  for (int kb = 0; kb < nkeys; kb += KT) {
    for (int idx = tid; idx < KT * CPR; idx += 256) {
      const int j = idx / CPR, c = idx % CPR;
      const int key = kb + j;
      float kf[EPL], vf[EPL];
      if (key < nkeys) {
        const T* kr = key < P ? kp + (int64_t)key * HD : ko + (int64_t)(key - P) * HD;
        const T* vr = key < P ? vp + (int64_t)key * HD : vo + (int64_t)(key - P) * HD;
        Vec16<T>::load(kr + c * EPL, kf);
        Vec16<T>::load(vr + c * EPL, vf);
      } else {
#pragma unroll
        for (int e = 0; e < EPL; ++e) kf[e] = vf[e] = 0.f;
      }
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        Ks[j][c * EPL + e] = kf[e];
        Vs[j][c * EPL + e] = vf[e];
      }
    }
    __syncthreads();
    float s[KT];
    float mt = -INFINITY;
#pragma unroll
    for (int j = 0; j < KT; ++j) {
      float d = 0.f;
#pragma unroll
      for (int dd = 0; dd < DPT; ++dd) d = fmaf(qv[dd], Ks[j][dd * TPQ + sub], d);
      d += __shfl_xor(d, 1, 64);
      d += __shfl_xor(d, 2, 64);
      const int key = kb + j;
      const bool ok = qvalid && key <= P + t0 + t;
      s[j] = ok ? d : -INFINITY;
      mt = fmaxf(mt, s[j]);
    }
    const float mn = fmaxf(m, mt);
    if (mn != -INFINITY) {
      const float corr = exp2_or_zero(m - mn);
      l *= corr;
#pragma unroll
      for (int dd = 0; dd < DPT; ++dd) acc[dd] *= corr;
#pragma unroll
      for (int j = 0; j < KT; ++j) {
        const float p = exp2_or_zero(s[j] - mn);
        l += p;
#pragma unroll
        for (int dd = 0; dd < DPT; ++dd) acc[dd] = fmaf(p, Vs[j][dd * TPQ + sub], acc[dd]);
      }
      m = mn;
    }
    __syncthreads();
  }
  if (qvalid) {
    T* o = out + (((int64_t)row * lr + t) * hq + qh) * HD;
#pragma unroll
    for (int dd = 0; dd < DPT; ++dd) o[dd * TPQ + sub] = from_f32<T>(acc[dd] / l);
  }
}


// --------------------------------------------------------- prefill (MFMA)
// bf16 flash attention with v_mfma_f32_32x32x16_bf16, head_dim 64 or 128.
// Work-group = one row, one KV head, QB blocks of 32 queries; wave w computes
// query head (kvh * G + w % G) for query block w / G, so the G QB waves share
// every staged K/V tile.
//   S^T = K Q^T   (keys x queries): lane l holds, of every 32 keys, the 16
//                 with (key / 4) % 2 = l / 32 for query l % 32, so a query's
//                 softmax state lives in lanes l and l + 32.
//   O^T += V^T P^T (dims x queries): the contraction visits the keys of a
//                 16-key chunk in the order the lane holds them (0-3 and 8-11
//                 of it for l < 32, 4-7 and 12-15 for the others), so the B
//                 operand is the lane's own eight probabilities; the A operand
//                 comes from the V tile by two LDS transpose reads.
// KT-key tiles go memory -> LDS by global_load_lds, four stages deep, one
// barrier per tile; the scores of the next 32 keys are formed under the
// probabilities of these; 16-byte chunks sit XOR-swizzled in the LDS rows (K:
// the fragment reads of eight neighbouring keys, V: the transpose reads of a
// half wave, on distinct banks).  Queries and outputs pass through LDS too, so
// that memory sees whole rows.  Online softmax in base 2 relative to each
// column's exact maximum.  (A maximum up to 2^8 stale spares most rescalings of
// the 64 accumulators, 844 -> 795 us at the longest case below, but puts the
// output 5 % further off: the largest probability is then rounded to bf16
// where it would be exactly 1.)
// Four waves and 32-key tiles, two work-groups a CU (eight waves and 64-key
// tiles with 8 query heads a KV head): eight waves in one work-group were
// 5-17 % slower on short responses and at head_dim 64.
// Against 16-query waves with tiles staged through registers, head_dim 128:
// 103 rows x 32 heads x 507 queries after 384 keys 1198 -> 856 us, 512 rows
// of 128 queries after 256 keys 873 -> 685 us (2.8 TB/s of queries, outputs and
// keys), one prompt of 256 15.4 -> 12.0 us.  What is left is issue: VALU
// (16 exponentials of 32 keys take as long as half their MFMAs), MFMA and LDS
// waits overlap only across the two waves of a SIMD.
constexpr int PF_NST = 4;            // stages

template <int HD, int G, int QB, int KT>
__global__ void __launch_bounds__(64 * G * QB, 2)
prefill_attn_mfma_kernel(const float* __restrict__ q, const bf16_t* __restrict__ kpre,
                         const bf16_t* __restrict__ vpre, int P, const bf16_t* __restrict__ kown,
                         const bf16_t* __restrict__ vown, int rows, int lr, int cap, int t0, int hq, int hkv,
                         bf16_t* __restrict__ out, float qscale) {
  constexpr int NW = G * QB;
  constexpr int KS = HD / 16, DT = HD / 32, CPK = HD / 8;
  constexpr int TILE = KT * HD;                // bf16 elements of a K (or V) tile
  constexpr int RPI = 64 / CPK;                // keys per copy instruction (1 KB)
  constexpr int DPW = KT / RPI / NW;        // copies per wave of a K (or V) tile
  static_assert(HD == 64 || HD == 128, "head_dim");
  static_assert(DPW * RPI * NW == KT, "copies divide the tile");
  __shared__ __attribute__((aligned(1024))) bf16_t lds[PF_NST * 2 * TILE];
  // A 1-D grid of 8 C work-groups, dealt round-robin to the 8 XCDs: XCD x
  // takes the consecutive logical blocks [x C, (x + 1) C), ordered query
  // block fastest (last block, the longest, first), so the query blocks that
  // read the same row's keys share one L2.
  const int ngq = (lr + 32 * QB - 1) / (32 * QB), total = ngq * hkv * rows;
  const int per_xcd = (total + 7) / 8;
  const int pid = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (pid >= total) return;
  const int qg = ngq - 1 - pid % ngq;
  const int h = (pid / ngq) % hkv;
  const int row = pid / (ngq * hkv);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int fr = lane & 31, fh = lane >> 5;
  const int b0 = (qg * QB + wave / G) * 32;     // first query of the wave
  const int qh = h * G + wave % G;
  const int t = b0 + fr;                        // this lane's query
  const int nkeys = P + t0 + min(lr, (qg + 1) * QB * 32);           // of the work-group's last query
  const int wkeys = b0 < lr ? P + t0 + min(lr, b0 + 32) : 0;        // of this wave's
  const int ntile = (nkeys + KT - 1) / KT;

  // The wave's 32 query rows, 16 bytes per lane along whole rows (from
  // clamped rows; results of rows past the end are not stored)
  constexpr int LPR = HD / 4, RPQ = 64 / LPR, NQ = 32 / RPQ;   // lanes per row, rows per load, loads
  float4 qv[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int tq = min(b0 + RPQ * i + lane / LPR, lr - 1);
    qv[i] = reinterpret_cast<const float4*>(q + (((int64_t)row * lr + tq) * hq + qh) * HD)[lane % LPR];
  }

  // Copies: instruction i of a wave moves keys RPI (wave + NW i) .. of the
  // tile; lane l writes slot l % CPK of key l / CPK and fetches the chunk
  // stored there.  Keys past the last are clamped (their scores are masked).
  const bf16_t* kp = kpre + (int64_t)h * P * HD;
  const bf16_t* vp = vpre + (int64_t)h * P * HD;
  const bf16_t* ko = kown + ((int64_t)row * hkv + h) * cap * HD;
  const bf16_t* vo = vown + ((int64_t)row * hkv + h) * cap * HD;
  auto vswz = [](int k) { return HD == 128 ? (k & 3) << 2 : ((k >> 1) & 1) << 2; };
  auto issue = [&](int tile, int buf) {
    bf16_t* kd = lds + buf * 2 * TILE;
    bf16_t* vd = kd + TILE;
#pragma unroll
    for (int i = 0; i < DPW; ++i) {
      const int r0 = RPI * (wave + NW * i);
      const int r = r0 + lane / CPK, sl = lane % CPK;
      const int j = min(tile * KT + r, nkeys - 1);
      const int64_t off = (int64_t)(j < P ? j : j - P) * HD;
      dma16(reinterpret_cast<const char*>((j < P ? kp : ko) + off + 8 * (sl ^ (r & (CPK - 1)))), kd + r0 * HD);
      dma16(reinterpret_cast<const char*>((j < P ? vp : vo) + off + 8 * (sl ^ vswz(r))), vd + r0 * HD);
    }
  };
  auto wait_barrier = [](auto n) {
    constexpr int N = decltype(n)::value;
    if constexpr (N == 0) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else if constexpr (N == 2) asm volatile("s_waitcnt vmcnt(2) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else if constexpr (N == 4) asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else if constexpr (N == 8) asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else static_assert(N < 0, "add this wait count");
  };

  // LDS element offsets: the K fragment of key fr (chunk 2 s + fh), and the
  // four dims dt 32 + 16 (l / 16 % 2) + 4 (l % 4) .. of V key 4 fh + l % 16 / 4
  bf16x8 qf[KS];
  int koff[KS];
  uint32_t vbase[DT];   // LDS bytes, in the first stage's V tile
#pragma unroll
  for (int s = 0; s < KS; ++s) koff[s] = fr * HD + 8 * ((2 * s + fh) ^ (fr & (CPK - 1)));
  {
    const int vk = 4 * fh + ((lane & 15) >> 2);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
      vbase[dt] = lds_addr(lds + TILE + vk * HD +
                           8 * ((4 * dt + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ vswz(vk)) + 4 * (lane & 1));
  }

  f32x16 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[dt][e] = 0.f;
  // The running maximum starts at the lowest finite score: while a column has
  // seen only scores of -inf (an infinite key, products that overflow), their
  // probabilities are exp2(-inf) = 0, where -inf - -inf would be NaN.
  float m = -FLT_MAX, l = 0.f;

  auto zero = [](f32x16& sc) {
#pragma unroll
    for (int e = 0; e < 16; ++e) sc[e] = 0.f;
  };
  // Half a tile: the scores `sc` of the 32 keys from `key` on are there (V
  // rows from byte VOFF of the V tile); the scores of the next 32 keys (K rows
  // at `kn`) are formed into `sn`.  Per 16-key chunk: the K fragments and V
  // of the chunk are read under the O MFMAs of the chunk before, then every
  // score MFMA runs beside a share of the chunk's probabilities.
  constexpr int KC = KS / 2;     // score MFMAs of a chunk
  auto half = [&](auto voff, int key, const uint32_t (&va)[DT], const bf16_t* kn, f32x16& sc, f32x16& sn) {
    constexpr int VOFF = decltype(voff)::value;
    bf16x8 kf[KC], pf;
    i16x4 lo[DT], hi[DT];
    auto read_k = [&](int c) {
#pragma unroll
      for (int s = 0; s < KC; ++s) kf[s] = *reinterpret_cast<const bf16x8*>(kn + koff[c * KC + s]);
    };
    auto scores = [&](int c) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < KC; ++s) {
        sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], qf[c * KC + s], sn, 0, 0, 0);
#pragma unroll
        for (int e = s * 8 / KC; e < (s + 1) * 8 / KC; ++e) {
          const float p = __builtin_amdgcn_exp2f(sc[8 * c + e] - m);
          l += p;
          pf[e] = (__bf16)p;
        }
      }
#pragma unroll
      for (int s = 0; s < KC; ++s) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 8 / KC, 0);
        __builtin_amdgcn_sched_group_barrier(0x400, 8 / KC, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 12 / KC, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    auto output = [&] {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tr16_pair(lo[dt], hi[dt]), pf, o[dt], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    };
    read_k(0);
    lds_read_tr16_pairs<DT, VOFF, VOFF + 8 * HD * 2>(va, lo, hi);
    if (key + 31 > P + t0 + b0) {   // the diagonal (wave-uniform)
      asm volatile("");             // (a branch, not 32 selects on every tile)
      const int lim = P + t0 + t - key - 4 * fh;   // last visible key, from this lane's first
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (8 * (e >> 2) + (e & 3) > lim) sc[e] = -INFINITY;
    }
    float mt = sc[0];
#pragma unroll
    for (int e = 1; e < 16; ++e) mt = fmaxf(mt, sc[e]);
    mt = fmaxf(mt, other_half(mt));
    if (__any(mt > m)) {
      const float mn = fmaxf(m, mt);
      const float corr = __builtin_amdgcn_exp2f(m - mn);
      l *= corr;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) o[dt] *= corr;
      m = mn;
    }
    zero(sn);
    scores(0);
    read_k(1);
    output();
    lds_read_tr16_pairs<DT, VOFF + 16 * HD * 2, VOFF + 24 * HD * 2>(va, lo, hi);
    scores(1);
    output();
  };
  constexpr int CPW = 2 * DPW;   // copies per wave and tile
  // Before tile i: tile i + 1 landed too (its first scores are formed under
  // tile i; only the copies of i + 2 may still fly), and every wave is done
  // with tile i - 1, whose buffer takes tile i + 3.
  auto sync = [&](int tile) {
    if (tile + 2 < ntile) wait_barrier(std::integral_constant<int, CPW>{});
    else wait_barrier(std::integral_constant<int, 0>{});
    if (tile + PF_NST - 1 < ntile) issue(tile + PF_NST - 1, (tile + PF_NST - 1) % PF_NST);
  };
  auto kstage = [&](int tile) { return lds + (tile % PF_NST) * 2 * TILE; };
  auto vstage = [&](int tile, uint32_t (&va)[DT]) {
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) va[dt] = vbase[dt] + (uint32_t)(tile % PF_NST) * (2 * TILE * 2);
  };
  // Tiles 0 and 1 go out first; the scaled bf16 queries pass through the
  // buffers of tiles 2 and 3 (a 32-row slice per wave, chunks placed like
  // K's) into fragments: lane holds Q[t][16 s + 8 fh .. + 8].
  issue(0, 0);
  if (ntile > 1) issue(1, 1);
  bf16_t* const slice = lds + wave * 32 * HD;
  {
    bf16_t* qs = slice + 2 * 2 * TILE;
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      const int r = RPQ * i + lane / LPR, c4 = lane % LPR;
      const bf16x4 v = {(__bf16)(qv[i].x * qscale), (__bf16)(qv[i].y * qscale), (__bf16)(qv[i].z * qscale),
                        (__bf16)(qv[i].w * qscale)};
      *reinterpret_cast<bf16x4*>(qs + r * HD + 8 * ((c4 >> 1) ^ (r & (CPK - 1))) + 4 * (c4 & 1)) = v;
    }
#pragma unroll
    for (int s = 0; s < KS; ++s) qf[s] = *reinterpret_cast<const bf16x8*>(qs + koff[s]);
  }
  f32x16 sa, sb;
  zero(sa);
  wait_barrier(std::integral_constant<int, 0>{});   // tiles 0 and 1, and every wave's queries read
  if (ntile > 2) issue(2, 2);
  if (ntile > 3) issue(3, 3);
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    const bf16x8 kf = *reinterpret_cast<const bf16x8*>(lds + koff[s]);
    sa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[s], sa, 0, 0, 0);
  }
  // 64 keys a round; the scores formed past the last tile are those of a
  // stale buffer and never used
  for (int kb = 0, tile = 0; kb < nkeys; kb += 64) {
    if (kb > 0) sync(tile);
    uint32_t va[DT];
    if (kb < wkeys) {   // else beyond this wave's last query
      vstage(tile, va);
      half(std::integral_constant<int, 0>{}, kb, va, KT == 64 ? kstage(tile) + 32 * HD : kstage(tile + 1), sa, sb);
    }
    if constexpr (KT == 32) {
      ++tile;
      if (tile < ntile) sync(tile);
    }
    if (kb + 32 < wkeys) {
      if constexpr (KT == 32) vstage(tile, va);
      half(std::integral_constant<int, KT == 64 ? 32 * HD * 2 : 0>{}, kb + 32, va, kstage(tile + 1), sb, sa);
    }
    ++tile;
  }
  l += other_half(l);
  const float inv = 1.0f / l;
  wait_barrier(std::integral_constant<int, 0>{});   // every wave is done with the tiles
  // The outputs pass through the wave's slice of LDS (chunks placed like
  // K's), so that a row leaves as one contiguous run.
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const bf16x4 v = {(__bf16)(o[dt][4 * g] * inv), (__bf16)(o[dt][4 * g + 1] * inv),
                        (__bf16)(o[dt][4 * g + 2] * inv), (__bf16)(o[dt][4 * g + 3] * inv)};
      *reinterpret_cast<bf16x4*>(slice + fr * HD + 8 * ((4 * dt + g) ^ (fr & (CPK - 1))) + 4 * fh) = v;
    }
  const bool wide = (reinterpret_cast<uintptr_t>(out) & 15) == 0;
#pragma unroll
  for (int i = 0; i < 32 / RPI; ++i) {
    const int r = RPI * i + lane / CPK, c = lane % CPK;
    const uint4 v = *reinterpret_cast<const uint4*>(slice + r * HD + 8 * (c ^ (r & (CPK - 1))));
    if (b0 + r >= lr) continue;
    bf16_t* dst = out + (((int64_t)row * lr + b0 + r) * hq + qh) * HD + 8 * c;
    if (wide) {
      *reinterpret_cast<uint4*>(dst) = v;
    } else {
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int k = 0; k < 8; ++k) dst[k] = (bf16_t)(w[k >> 1] >> (16 * (k & 1)));
    }
  }
}

template <typename T, int HD, int G>
static void launch_prefill(const PrefillAttnArgs& a, hipStream_t s) {
  constexpr int QB = 64 / G;
  const float qscale = kLog2e / sqrtf((float)HD);
  dim3 grid((a.lr + QB - 1) / QB, a.hkv, a.rows);
  SR_LAUNCH((prefill_attn_kernel<T, HD, G>), grid, dim3(256), 0, s, a.q, (const T*)a.kpre,
                     (const T*)a.vpre, a.P, (const T*)a.kown, (const T*)a.vown, a.lr, a.cap, a.t0, a.hq,
                     a.hkv, (T*)a.out, qscale);
  SR_CHECK_LAUNCH();
}

template <typename T, int HD>
static void prefill_by_group(const PrefillAttnArgs& a, hipStream_t s) {
  switch (a.hq / a.hkv) {
    case 1: launch_prefill<T, HD, 1>(a, s); break;
    case 2: launch_prefill<T, HD, 2>(a, s); break;
    case 4: launch_prefill<T, HD, 4>(a, s); break;
    case 8: launch_prefill<T, HD, 8>(a, s); break;
    default: SR_REQUIRE(false, 3, "query heads per KV head must be 1, 2, 4 or 8");
  }
}

template <typename T>
static void prefill_by_hd(const PrefillAttnArgs& a, hipStream_t s) {
  switch (a.hd) {
    case 32: prefill_by_group<T, 32>(a, s); break;
    case 64: prefill_by_group<T, 64>(a, s); break;
    case 128: prefill_by_group<T, 128>(a, s); break;
    default: SR_REQUIRE(false, 3, "head_dim must be 32, 64 or 128");
  }
}

template <int HD, int G>
static void launch_prefill_mfma(const PrefillAttnArgs& a, hipStream_t s) {
  const float qscale = kLog2e / sqrtf((float)HD);
  constexpr int QB = G <= 4 ? 4 / G : 1;   // query blocks per work-group
  const int64_t total = (int64_t)((a.lr + 32 * QB - 1) / (32 * QB)) * a.hkv * a.rows;
  SR_REQUIRE(total <= (int64_t)INT32_MAX - 8, SR_ERR_UNSUPPORTED, "prefill attention grid too large");
  dim3 grid((unsigned)(8 * ((total + 7) / 8)));
  SR_LAUNCH((prefill_attn_mfma_kernel<HD, G, QB, G <= 4 ? 32 : 64>), grid, dim3(64 * G * QB), 0, s, a.q,
            (const bf16_t*)a.kpre, (const bf16_t*)a.vpre, a.P, (const bf16_t*)a.kown, (const bf16_t*)a.vown, a.rows,
            a.lr, a.cap, a.t0, a.hq, a.hkv, (bf16_t*)a.out, qscale);
  SR_CHECK_LAUNCH();
}

void prefill_attn(const PrefillAttnArgs& a, hipStream_t s) {
  if (a.rows <= 0 || a.lr <= 0) return;
  // The matrix-core kernel copies keys and values 16 bytes a lane straight into
  // LDS; rows off a 16-byte boundary take the vector kernel, whose global loads
  // accept any address.
  const bool mfma = a.dtype == SR_BF16 &&
                    ((reinterpret_cast<uintptr_t>(a.kown) | reinterpret_cast<uintptr_t>(a.vown) |
                      (a.P > 0 ? reinterpret_cast<uintptr_t>(a.kpre) | reinterpret_cast<uintptr_t>(a.vpre) : 0)) &
                     15) == 0;
  if (mfma && a.hd == 128) {
    switch (a.hq / a.hkv) {
      case 1: launch_prefill_mfma<128, 1>(a, s); return;
      case 2: launch_prefill_mfma<128, 2>(a, s); return;
      case 4: launch_prefill_mfma<128, 4>(a, s); return;
      case 8: launch_prefill_mfma<128, 8>(a, s); return;
      default: break;
    }
  }
  if (mfma && a.hd == 64) {
    switch (a.hq / a.hkv) {
      case 1: launch_prefill_mfma<64, 1>(a, s); return;
      case 2: launch_prefill_mfma<64, 2>(a, s); return;
      case 4: launch_prefill_mfma<64, 4>(a, s); return;
      case 8: launch_prefill_mfma<64, 8>(a, s); return;
      default: break;
    }
  }
  if (a.dtype == SR_BF16) prefill_by_hd<bf16_t>(a, s);
  else prefill_by_hd<float>(a, s);
}

}  // namespace sr
