// The rejection cut of section 4.2 (eqs. cutoff-threshold and accepted-set)
// and the stream compaction that packs the survivors' KV rows and state.
//
// Ranking: total order (score descending, candidate index ascending, NaN
// lowest).  A row's rank is the number of rows that precede it; the `keep`
// rows of rank < keep are accepted.  Scores are mapped to order-preserving
// unsigned keys (NaN -> 0, +0 and -0 equal), so ranks are integer-exact.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace sr {

constexpr int kCutThreads = 1024;
constexpr int kCutMax = 4096;
constexpr int kCutPer = kCutMax / kCutThreads;

__device__ __forceinline__ uint32_t order_key(float f) {
  if (f != f) return 0u;
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7FFFFFFFu) == 0u) u = 0u;  // -0 == +0
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ bool precedes(uint32_t ka, int ca, uint32_t kb, int cb) {
  return ka > kb || (ka == kb && ca < cb);
}
// The same order as one unsigned comparison: row a precedes row b when its
// word is larger (key descending, then candidate ascending).
__device__ __forceinline__ uint64_t order_word(float score, int cand) {
  return ((uint64_t)order_key(score) << 32) | (~(uint32_t)cand ^ 0x80000000u);
}

// Exclusive block scan of per-thread counts (NT threads); returns the
// exclusive prefix of this thread and writes the total to *total.
template <int NT = kCutThreads>
__device__ int block_excl_scan(int v, int* wsum, int* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int inc = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    int t = __shfl_up(inc, o, 64);
    if (lane >= o) inc += t;
  }
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  int off = 0, tot = 0;
  for (int w = 0; w < NT / 64; ++w) {
    if (w < wave) off += wsum[w];
    tot += wsum[w];
  }
  __syncthreads();
  *total = tot;
  return off + inc - v;
}

// Lanes that share the count of one row when `rows` rows are ranked by 1024
// threads at a time: a power of two, at most a wave.
__device__ __forceinline__ int lanes_per_row(int rows) {
  int t = 64;
  while (t > 1 && rows * t > kCutThreads) t >>= 1;
  return t;
}

// rank[i - i0] = rows preceding row i, for i in [i0, i1); words: LDS [b].
// A row's count is shared by `tpr` neighbouring lanes, which read
// neighbouring words.
__device__ void rank_rows(const uint64_t* words, int b, int i0, int i1, int tpr, int* rank) {
  const int sub = threadIdx.x % tpr, per = kCutThreads / tpr;
  for (int base = i0; base < i1; base += per) {   // uniform trip count
    const int i = base + threadIdx.x / tpr;
    int n = 0;
    if (i < i1) {
      const uint64_t w = words[i];
#pragma unroll 8
      for (int j = sub; j < b; j += tpr) n += words[j] > w ? 1 : 0;
    }
    for (int o = tpr >> 1; o > 0; o >>= 1) n += __shfl_xor(n, o, 64);
    if (i < i1 && sub == 0) rank[i - i0] = n;
  }
}

// Each work-group ranks kSelectRows rows against all of them, 16 lanes a
// row: 512 rows take 8 work-groups of 32 comparisons a lane (one work-group
// whose threads each counted four whole rows took 51 us).
constexpr int kSelectRows = 64;

__global__ void __launch_bounds__(kCutThreads)
select_kernel(const float* __restrict__ score, const int32_t* __restrict__ cand, int b, int keep,
              int32_t* __restrict__ accept) {
  __shared__ uint64_t words[kCutMax];
  __shared__ int rank[kSelectRows];
  for (int i = threadIdx.x; i < b; i += kCutThreads) words[i] = order_word(score[i], cand[i]);
  __syncthreads();
  const int i0 = blockIdx.x * kSelectRows, i1 = min(b, i0 + kSelectRows);
  rank_rows(words, b, i0, i1, kCutThreads / kSelectRows, rank);
  __syncthreads();
  for (int i = i0 + threadIdx.x; i < i1; i += kCutThreads) accept[i] = rank[i - i0] < keep ? 1 : 0;
}

void select_topk(const float* score, const int32_t* cand, int b, int keep, int32_t* accept,
                 hipStream_t s) {
  SR_REQUIRE(b >= 1 && b <= kCutMax, 3, "cut supports 1..4096 rows");
  SR_LAUNCH(select_kernel, dim3((b + kSelectRows - 1) / kSelectRows), dim3(kCutThreads), 0, s, score, cand, b, keep,
            accept);
  SR_CHECK_LAUNCH();
}

__global__ void __launch_bounds__(kCutThreads) cut_kernel(CutArgs a) {
  __shared__ uint64_t words[kCutMax];
  __shared__ int rank[kCutMax];
  __shared__ int wsum[kCutThreads / 64];
  for (int i = threadIdx.x; i < a.b; i += kCutThreads) words[i] = order_word(a.score[i], a.cand[i]);
  __syncthreads();
  rank_rows(words, a.b, 0, a.b, lanes_per_row(a.b), rank);
  __syncthreads();
  int acc[kCutPer], dn[kCutPer];
  int nd = 0, nc = 0;
#pragma unroll
  for (int k = 0; k < kCutPer; ++k) {
    const int i = threadIdx.x * kCutPer + k;
    acc[k] = (i < a.b && rank[i] < a.keep) ? 1 : 0;
    dn[k] = (i < a.b && a.done[i]) ? 1 : 0;
    if (i < a.b) a.accept[i] = acc[k];
    nd += dn[k];
    nc += (acc[k] && !dn[k]) ? 1 : 0;
  }
  const int i_base = *a.i_count;
  int tot_done, tot_cont;
  int pd = block_excl_scan(nd, wsum, &tot_done);
  int pc = block_excl_scan(nc, wsum, &tot_cont);
#pragma unroll
  for (int k = 0; k < kCutPer; ++k) {
    const int i = threadIdx.x * kCutPer + k;
    if (i >= a.b) continue;
    if (dn[k]) {  // completed rows join I whether accepted or not
      const int slot = i_base + pd++;
      a.i_cand[slot] = a.cand[i];
      a.i_score[slot] = a.score[i];
      a.i_len[slot] = a.len[i];
    } else if (acc[k]) {
      const int j = pc++;
      a.src_row[j] = i;
      a.cand_out[j] = a.cand[i];
      a.len_out[j] = a.len[i];
      a.tok_out[j] = a.next_tok[i];
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    *a.i_count = i_base + tot_done;
    *a.count = tot_cont;
  }
}

void cut(const CutArgs& a, hipStream_t s) {
  SR_REQUIRE(a.b >= 1 && a.b <= kCutMax, 3, "cut supports 1..4096 rows");
  SR_LAUNCH(cut_kernel, dim3(1), dim3(kCutThreads), 0, s, a);
  SR_CHECK_LAUNCH();
}

// keep_flag -> packed source rows and count (single work-group).
__global__ void __launch_bounds__(kCutThreads)
pack_flags_kernel(const int32_t* __restrict__ flag, int b, int32_t* __restrict__ src_row,
                  int32_t* __restrict__ count) {
  __shared__ int wsum[kCutThreads / 64];
  int f[kCutPer], n = 0;
#pragma unroll
  for (int k = 0; k < kCutPer; ++k) {
    const int i = threadIdx.x * kCutPer + k;
    f[k] = (i < b && flag[i] != 0) ? 1 : 0;
    n += f[k];
  }
  int tot;
  int p = block_excl_scan(n, wsum, &tot);
#pragma unroll
  for (int k = 0; k < kCutPer; ++k) {
    const int i = threadIdx.x * kCutPer + k;
    if (f[k]) src_row[p++] = i;
  }
  if (threadIdx.x == 0) *count = tot;
}

// KV compaction: the grid walks the 16 KB chunks of the kept rows' (block, row,
// head) runs, so a row that is not kept costs no work-group and the number of
// kept rows stays on the device; a chunk's four loads per thread go out before
// its stores.
// From a row list (the generation loop) every chunk gets a work-group of its
// own, up to kListGrid: copy bound, and a work-group that walks many chunks
// waits for its stores between them (103 of 512 rows, 32 layers of 8 x 128 bf16,
// 127 tokens, 3.4 GB moved: 677 us, with 2048 work-groups 724).
// From flags (FLAGS): below kPackBytes of rows that may move, 2048 work-groups
// pack the flags into LDS lists of their own (and the first one writes src_row
// and new_count), which saves a launch (68 MB moved: 13.7 against 14.8 us); from
// there one work-group packs them first and the list form follows (the 3.4 GB
// above: 679 against 724 us; 429 MB: 82 against 88).
constexpr int kCompactThreads = 256;
constexpr int kCompactUnroll = 4;
constexpr int kFlagGrid = 2048;      // eight work-groups per CU
constexpr int kListGrid = 65536;
constexpr int64_t kPackBytes = 512LL << 20;

template <bool FLAGS>
__global__ void __launch_bounds__(kCompactThreads)
compact_kernel(const uint8_t* __restrict__ src, int64_t src_block, uint8_t* __restrict__ dst,
               int64_t dst_block, const int32_t* __restrict__ keep_flag, int b, const int32_t* __restrict__ src_row,
               const int32_t* __restrict__ count, int32_t* __restrict__ src_row_out, int32_t* __restrict__ count_out,
               int hkv, int row_bytes, int cap_src, int cap_dst, int len) {
  __shared__ uint16_t list[FLAGS ? kCutMax : 1];
  __shared__ int wsum[kCompactThreads / 64];
  int kept;
  if constexpr (FLAGS) {
    // thread t packs flags [t per, (t + 1) per)
    const bool first = blockIdx.x == 0 && blockIdx.y == 0;
    const int per = (b + kCompactThreads - 1) / kCompactThreads;
    const int f0 = min(b, (int)threadIdx.x * per), f1 = min(b, f0 + per);
    int n = 0;
    for (int i = f0; i < f1; ++i) n += keep_flag[i] != 0 ? 1 : 0;
    int p = block_excl_scan<kCompactThreads>(n, wsum, &kept);
    for (int i = f0; i < f1; ++i)
      if (keep_flag[i] != 0) {
        list[p] = (uint16_t)i;
        if (first) src_row_out[p] = i;
        ++p;
      }
    if (first && threadIdx.x == 0) *count_out = kept;
    __syncthreads();
  } else {
    kept = *count;
  }
  const int n16 = (int)((int64_t)len * row_bytes / 16);   // 16-byte units of a run
  constexpr int CH = kCompactThreads * kCompactUnroll;    // units of a chunk
  const int nch = (n16 + CH - 1) / CH;
  const int blk = blockIdx.y;
  const uint32_t total = (uint32_t)kept * hkv * nch;      // chunks of a block
  for (uint32_t w = blockIdx.x; w < total; w += gridDim.x) {
    const uint32_t run = w / (uint32_t)nch;
    const int c = (int)(w - run * nch);
    const int j = (int)(run / (uint32_t)hkv), h = (int)(run - j * hkv);
    const int i = FLAGS ? list[j] : src_row[j];
    const uint4* s4 = reinterpret_cast<const uint4*>(src + blk * src_block + (((int64_t)i * hkv + h) * cap_src) * row_bytes);
    uint4* d4 = reinterpret_cast<uint4*>(dst + blk * dst_block + (((int64_t)j * hkv + h) * cap_dst) * row_bytes);
    const int k0 = c * CH + threadIdx.x;
    uint4 v[kCompactUnroll];
#pragma unroll
    for (int u = 0; u < kCompactUnroll; ++u) v[u] = s4[min(k0 + u * kCompactThreads, n16 - 1)];
#pragma unroll
    for (int u = 0; u < kCompactUnroll; ++u)
      if (k0 + u * kCompactThreads < n16) d4[k0 + u * kCompactThreads] = v[u];
  }
}

void compact(const CompactArgs& a, hipStream_t s) {
  if (a.keep_flag) SR_REQUIRE(a.b >= 1 && a.b <= kCutMax, 3, "compaction supports 1..4096 rows");
  const int row_bytes = a.hd * a.elem_bytes;
  const bool moves = a.max_rows > 0 && a.len > 0;
  if (!moves && !a.keep_flag) return;
  if (moves) SR_REQUIRE(row_bytes % 16 == 0, 3, "KV row must be a multiple of 16 bytes");
  const int64_t units = (int64_t)a.len * row_bytes / 16;
  const int64_t nch = (units + kCompactThreads * kCompactUnroll - 1) / (kCompactThreads * kCompactUnroll);
  const int64_t chunks = std::max<int64_t>(1, (int64_t)a.max_rows * a.hkv * nch);
  SR_REQUIRE(units <= INT32_MAX / 2 && chunks <= INT32_MAX, SR_ERR_UNSUPPORTED, "KV pool too large to compact");
  const int blocks = moves ? 2 * a.n_layers : 1;
  const bool pack = a.keep_flag && moves && (int64_t)a.max_rows * a.hkv * a.len * row_bytes * blocks >= kPackBytes;
  if (pack) {
    SR_LAUNCH(pack_flags_kernel, dim3(1), dim3(kCutThreads), 0, s, a.keep_flag, a.b, a.scratch_src_row, a.new_count);
    SR_CHECK_LAUNCH();
  }
  const bool flags = a.keep_flag && !pack;   // (without tokens to move, one work-group still packs them)
  const int32_t* src_row = pack ? a.scratch_src_row : a.src_row;
  const int32_t* count = pack ? a.new_count : a.count;
  const dim3 grid((unsigned)std::min<int64_t>(chunks, std::max(1, (flags ? kFlagGrid : kListGrid) / blocks)), blocks);
#define SR_COMPACT(FLAGS)                                                                                             \
  SR_LAUNCH(compact_kernel<FLAGS>, grid, dim3(kCompactThreads), 0, s, (const uint8_t*)a.src,                          \
            a.src_block * a.elem_bytes, (uint8_t*)a.dst, a.dst_block * a.elem_bytes, a.keep_flag, a.b, src_row, count, \
            a.scratch_src_row, a.new_count, a.hkv, row_bytes, a.cap_src, a.cap_dst, moves ? a.len : 0)
  if (flags) SR_COMPACT(true);
  else SR_COMPACT(false);
#undef SR_COMPACT
  SR_CHECK_LAUNCH();
}

// Best of n (score, cand) pairs; n read from the device.
__global__ void __launch_bounds__(kCutThreads)
argmax_kernel(const float* __restrict__ score, const int32_t* __restrict__ cand,
              const int32_t* __restrict__ n_dev, int n_max, int32_t* __restrict__ best) {
  __shared__ uint32_t sk[kCutThreads / 64];
  __shared__ int sc[kCutThreads / 64], si[kCutThreads / 64];
  const int n = min(*n_dev, n_max);
  uint32_t bk = 0;
  int bc = 0x7FFFFFFF, bi = -1;
  for (int i = threadIdx.x; i < n; i += kCutThreads) {
    const uint32_t k = order_key(score[i]);
    const int c = cand[i];
    if (bi < 0 || precedes(k, c, bk, bc)) { bk = k; bc = c; bi = i; }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const uint32_t ok = __shfl_xor(bk, o, 64);
    const int oc = __shfl_xor(bc, o, 64), oi = __shfl_xor(bi, o, 64);
    if (oi >= 0 && (bi < 0 || precedes(ok, oc, bk, bc))) { bk = ok; bc = oc; bi = oi; }
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) { sk[wave] = bk; sc[wave] = bc; si[wave] = bi; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 0; w < kCutThreads / 64; ++w)
      if (si[w] >= 0 && (bi < 0 || precedes(sk[w], sc[w], bk, bc))) { bk = sk[w]; bc = sc[w]; bi = si[w]; }
    best[0] = bi;
  }
}

void argmax_best(const float* score, const int32_t* cand, const int32_t* n_dev, int n_max,
                 int32_t* best, hipStream_t s) {
  SR_LAUNCH(argmax_kernel, dim3(1), dim3(kCutThreads), 0, s, score, cand, n_dev, n_max, best);
  SR_CHECK_LAUNCH();
}

}  // namespace sr
