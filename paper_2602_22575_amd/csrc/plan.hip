// S2O ranking stage for gfx950 (paper Sec. 3.1, Alg. 1, Eqs. (1)-(2)).
//
//   kguide_kernel        partial sums of the first key segment (k_guide = k_mean[0]).
//   pool_sq_sort_kernel  one workgroup per (z, h, segment): a single pass over the
//                        segment's Q rows gives q_mean and s_Q; the S scores are then
//                        Argsort-ed in LDS (block_sort) -> Q_perm.
//   mean_guide_kernel,   small inputs: the same work in two launches instead of three, s_Q and
//   score_sort_kernel    Q_perm beside the scores (pool_segment, guide_part, score_block).
//   score_kernel         s_K[n, t] = <q_mean[n], K[t]> as an MFMA contraction per KV head:
//                        columns = (query head of the group, segment), rows = key tokens
//                        staged through LDS.  q_mean is split exactly into three bf16 terms
//                        so that bf16 MFMA reproduces the fp32 x bf16 products exactly (fp32
//                        accumulation).  The scores are stored (in the caller's s_K array or
//                        in scratch) together with one sampled score per 32 tokens.
//   threshold_kernel     only if some row is longer than one LDS sort: cuts every such row into
//                        score ranges of about equal population, from the sample.
//   row_sort_kernel      a row, or one score range of it, is collected in LDS by streaming over
//                        the row's scores, sorted there (block_sort), and the token indices are
//                        written at their final ranks -> KV_perm.  The number of keys above the
//                        range, counted on the way, is its first rank: nothing is exchanged
//                        between workgroups.
//   split_sort_kernel    many long rows: a workgroup takes whole rows, deals the keys of a row out
//                        to its ranges first and sorts range after range.
//
// Measured against the form this replaces, which scattered (key, token) pairs of all rows to
// buckets in memory, packed the buckets into spans and sorted those (eight launches of its own,
// Llama head shape, us for the whole ranking): 4K tokens in 512-token segments 77 -> 26, 8K in 1024
// 110 -> 40, 32K in 2048 277 -> 174, 64K in 1024 1005 -> 725, 128K in 2048 1808 -> 1401, and 3700 -> 1440 where
// far-off scores had sent the old spans to their bitonic network.
//
// Argsort semantics: descending score, ties by ascending index, -0 == +0.
#include <float.h>

#include <type_traits>

#include "s2o_internal.h"

namespace s2o {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kD = 128;
constexpr int kSampleStride = 32;  // one sampled score per this many tokens
constexpr int kChunkMax = 1024;    // key tokens per score workgroup (halved while the grid is too small)
constexpr int kSub = 128;          // key tokens per LDS tile of the score kernel
constexpr int kScoreWaves = 4;     // wavefronts (row blocks of 32) of a score workgroup.  8 would let all 4 x 64 rows
                                   // of a KV head at 128K share one pass over its K rows (295 against 307 us alone),
                                   // but an 8-wavefront workgroup of 200 registers needs a whole CU at once and
                                   // starves beside the own-segment pass on the second stream (up to 3 ms)
constexpr int kKStride = 136;      // bf16 elements per K row in LDS (272 B)
constexpr int kGuideParts = 8;     // workgroups per KV head summing the first key segment
constexpr int kOneEach = 256;      // query rows (workgroups) that leave every CU with one at most: 256 CUs

// float -> uint32 whose unsigned order is the float order (-0 canonicalised to +0)
__device__ inline uint32_t ordered_u32(float f) {
  uint32_t u = __float_as_uint(f);
  if (u == 0x80000000u) u = 0u;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ inline float ordered_to_float(uint32_t o) {
  return __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
}

__device__ inline float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ inline float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// ---------------------------------------------------------------------------------------
constexpr int kMapBins = 256;      // linear pieces of the map
// Shapes of the LDS sort: threads and keys per thread; 36 fine buckets per thread, that is 36 / kPer per key for a
// full set: 4.5, 2.8, 2.8, 9, 5.1, 3.6 and 2.3 for the shapes below.
template <int kT, int kPer>
struct SortShape {
  static constexpr int kThreads = kT, kPerThread = kPer, kCap = kT * kPer;
  static constexpr int kWords = 12 * kT;                         // bucket words, three buckets each
  static constexpr size_t pow2(size_t v) { size_t p = 1; while (p < v) p <<= 1; return p; }
  // byte offsets: bucket words, (score, token) pairs (+ 64 behind them), misc
  static constexpr size_t kListAt = 4 * (size_t)kWords, kTailAt = kListAt + 8 * ((size_t)kCap + 64);
  static constexpr size_t kFallback = 8 * pow2(kCap);            // the bitonic network uses everything below misc
  static constexpr size_t kMiscAt = kTailAt > kFallback ? kTailAt : kFallback;
  static constexpr size_t kLds = kMiscAt + 256;
};
using SmallSort = SortShape<256, 8>;     // 2048 keys, 29 KB: five workgroups per CU
using MidSort = SortShape<512, 13>;      // 6656 keys, 77 KB: two per CU
using LargeSort = SortShape<1024, 13>;   // 13312 keys, 153 KB: one per CU
using Sort4K = SortShape<1024, 4>;       // rows that fit one sort, besides the ones above: launch_plan
using Sort7K = SortShape<1024, 7>;
using Sort10K = SortShape<1024, 10>;
using QuerySort = SortShape<512, 16>;    // 8192 keys, 89 KB: one per CU

// Rows longer than the sort's capacity are cut into ranges of this many keys on average.  The
// cuts come from a 1-in-32 sample, so the population of a range of the medium shape scatters by
// about 8 % of the mean: the capacity is 4.3 sigma away, and a range in 100000 does not fit (with
// a 1-in-64 sample and ranges of 0.8 of the capacity it was one in 100, and collecting those
// again cost 140 us at 128K).  A range that does not fit is cut again (row_sort_kernel).
__host__ __device__ inline int range_target(int cap) { return cap - 7 * (cap / 25); }
__host__ __device__ inline int row_ranges(int64_t len, int cap) {
  return len <= cap ? (len > 0 ? 1 : 0) : (int)((len + range_target(cap) - 1) / range_target(cap));
}

// Split rows: a long row is taken by one workgroup, which first deals its keys out to one region
// per range (cap pairs each, in its own part of the scratch) and then sorts range after range;
// the longest rows first.  Alternatively every (row, range) is a piece of its own whose workgroup
// scans the whole row for its keys: no pairs in memory, and enough pieces when there are few
// rows, but a row of 128K tokens is scanned 27 times.
//
// Splitting takes as long as its longest row, or as all rows on kSplitGroups workgroups: about 9 us
// per range.  Scanning takes (4.2 sum(r) + 0.71 sum(r^2)) / 512 us over the rows' ranges r (fitted to
// 120 shapes from 24K to 256K tokens).  Below kSplitRows rows the longest row decides, and with r
// spread evenly up to the longest row's (causal) or the same for all rows (non-causal, where up to 512
// rows take one round and more take two) the line lies where split_pays puts it.  Measured on both
// sides (us for the whole ranking, splitting / scanning; rows x ranges of the longest): causal 1020 x 7
// 195 / 191, 744 x 14 383 / 384, 1008 x 14 401 / 427, 508 x 28 491 / 482, 744 x 27 748 / 887, 1020 x 28
// 649 / 894, 255 x 55 773 / 688, 511 x 55 893 / 1276; non-causal 512 x 7 194 / 172, 960 x 7 335 / 308,
// 384 x 14 352 / 339, 512 x 14 342 / 396, 768 x 14 529 / 584, 192 x 28 756 / 738, 256 x 28 477 / 555,
// 512 x 28 667 / 1041, 960 x 28 1240 / 1918.  From kSplitRows rows on: 2016 x 27 1440 / 1900, 2016 x 14
// 754 / 845; below kSplitRanges ranges: 736 x 5 179 / 160.
constexpr int kSplitGroups = 512;  // workgroups of the medium shape that fit the 256 CUs at once
constexpr int kSplitRows = 1024;
constexpr int kSplitRanges = 6;
inline bool split_pays(int64_t rows, int64_t ranges, int non_causal) {
  if (ranges < kSplitRanges) return false;
  if (rows >= kSplitRows) return true;
  if (non_causal) return rows * (ranges + 6) >= (rows > kSplitGroups ? 15000 : 8000);
  return rows * (ranges + 9) >= 19500;
}
constexpr int kMaxSplit = 256;      // ranges of a split row at most (L <= 1M tokens: 219)
constexpr size_t kSplitLds = 8 * kMaxSplit;   // a row's range counts and lower ends, behind the sort's LDS

struct Scratch {
  float* kguide;      // [Z*Hkv][kGuideParts][128] partial column sums of the first key segment
  uint16_t* qsplit;   // [Z*H*N][3][128] bf16
  float* samples;     // [Z*H*N][L/32] one score per 32 tokens of the row's prefix
  float* thr;         // [Z*H*N][max_ranges + 2] descending; entry r = lower end of range r; then the sample's
                      // highest and lowest score (from entry [ranges of the row] on)
  float* sk;          // [Z*H*P] s_K, used when the caller does not ask for the scores
  uint32_t* ticket;   // next row to take, and number of ranges left over (split rows)
  int2* left_over;    // [rows][max_ranges] (row_id | range << 24, rank behind the range) of the ranges whose keys
                      // did not fit their region (split rows)
  uint64_t* pairs;    // [groups][max_ranges][cap] (score, token) pairs by range (split rows)
  int cap;            // keys of one LDS sort
  int max_ranges;     // ranges of the longest row
  int groups;         // workgroups of the splitting kernel
  bool split;         // long rows are split by one workgroup each, not scanned once per range
  int chunk;          // key tokens per score workgroup: kChunkMax, less for short sequences
  size_t total;
};

static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

static Scratch carve(void* base, int Z, int H, int Hkv, int L, int S, int non_causal) {
  const int64_t N = L / S;
  const int64_t rows = (int64_t)Z * H * N;
  const int64_t P = kv_rows_total(N, S, L, non_causal);
  Scratch s;
  // one workgroup per (KV head, 128 rows, chunk): keep at least ~1024 of them in the grid
  {
    const int64_t rbg = ((int64_t)(H / Hkv) * N + 32 * kScoreWaves - 1) / (32 * kScoreWaves);
    s.chunk = kChunkMax;
    while (s.chunk > kSub && (int64_t)Z * Hkv * rbg * ((L + s.chunk - 1) / s.chunk) < 1024) s.chunk /= 2;
  }
  const int64_t longest = non_causal ? L : (int64_t)L - S;
  s.cap = longest <= SmallSort::kCap ? SmallSort::kCap
          : longest > MidSort::kCap && longest <= LargeSort::kCap ? LargeSort::kCap : MidSort::kCap;
  s.max_ranges = row_ranges(longest, s.cap);
  const int64_t long_rows = (int64_t)Z * H * (non_causal ? N : N - 1);
  s.split = split_pays(long_rows, s.max_ranges, non_causal);
  s.groups = (int)(long_rows < kSplitGroups ? long_rows : kSplitGroups);
  size_t off = 0;
  // (integer arithmetic: the size query carves from a null base)
  auto take = [&](size_t bytes) { size_t o = off; off += align256(bytes); return (char*)((uintptr_t)base + o); };
  s.kguide = (float*)take((size_t)Z * Hkv * kGuideParts * kD * 4);
  s.qsplit = (uint16_t*)take((size_t)rows * 3 * kD * 2);
  s.samples = (float*)take((size_t)rows * (L / kSampleStride) * 4);
  s.thr = (float*)take((size_t)rows * (s.max_ranges + 2) * 4);
  s.ticket = (uint32_t*)take(64);
  s.left_over = (int2*)take(s.split ? (size_t)rows * s.max_ranges * 8 : 0);
  s.sk = (float*)take((size_t)Z * H * P * 4);
  s.pairs = (uint64_t*)take(s.split ? (size_t)s.groups * s.max_ranges * s.cap * 8 : 0);
  // the size reported to callers stays at no less than 8 bytes per ranked key
  s.total = off > (size_t)Z * H * P * 8 ? off : align256((size_t)Z * H * P * 8);
  return s;
}

size_t plan_scratch_bytes(int Z, int H, int Hkv, int L, int S, int non_causal) {
  return carve(nullptr, Z, H, Hkv, L, S, non_causal).total;
}

// ---------------------------------------------------------------------------------------
// Built-in scratch for callers that cannot allocate (s2o_plan_static): one array per GPU, held
// from the moment the library is loaded there until the process ends.  The name below is a
// host-side stand-in, not a device address: host code only ever uses the address that
// hipGetSymbolAddress reports for the current device.
static __device__ __align__(256) unsigned char scratch[kStaticPlanScratchBytes];

hipError_t static_plan_scratch(void** ptr) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  return hipSuccess;
}

// ---------------------------------------------------------------------------------------
// A broken invariant (see the S2O_PLAN_* bits) is recorded in the caller's status word, which
// the first kernel of the call clears.
__device__ inline void raise(const PlanArgs& a, uint32_t bit) {
  if (a.status) atomicOr(reinterpret_cast<unsigned int*>(a.status), bit);
}

// Partial column sums of the first key segment: workgroup (z, g, part) adds the rows of its
// eighth of the segment; the consumers add the eight partial sums in a fixed order, so k_guide
// is reproducible bit for bit without a serial pass over the segment by one workgroup.
__device__ __forceinline__ void guide_part(const PlanArgs& a, const Scratch& sc, int block) {
  __shared__ float red[16][kD];
  if (block == 0 && threadIdx.x == 0) {
    if (a.status) *a.status = 0;
    sc.ticket[0] = 0u;
    sc.ticket[1] = 0u;
  }
  const int unit = block / kGuideParts, part = block % kGuideParts;
  const int z = unit / a.Hkv, g = unit % a.Hkv;
  const int c = threadIdx.x & 15, r = threadIdx.x >> 4;
  const uint16_t* Kh = a.K + z * a.ks[0] + g * a.ks[1];
  const int rows = a.S / kGuideParts;            // S is a multiple of 64
  const int end = (part + 1) * rows;
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int row0 = part * rows + r; row0 < end; row0 += 16 * 4) {   // four loads in flight
    u32x4 v4[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      v4[u] = *reinterpret_cast<const u32x4*>(Kh + (int64_t)min(row0 + 16 * u, end - 1) * a.ks[2] + 8 * c);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (row0 + 16 * u < end) {
        const u32x4 v = v4[u];
#pragma unroll
        for (int q = 0; q < 4; ++q) { acc[2 * q] += bf16_lo(v[q]); acc[2 * q + 1] += bf16_hi(v[q]); }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) red[r][8 * c + j] = acc[j];
  __syncthreads();
  if (threadIdx.x < kD) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) s += red[i][threadIdx.x];
    sc.kguide[(int64_t)block * kD + threadIdx.x] = s;
  }
}

__global__ __launch_bounds__(256) void kguide_kernel(PlanArgs a, Scratch sc) { guide_part(a, sc, (int)blockIdx.x); }

// ---------------------------------------------------------------------------------------
// Sum over the lanes up to and including this one (data-parallel-primitive moves, no LDS).
__device__ __forceinline__ uint32_t wave_inclusive_sum(uint32_t x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);    // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);    // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);    // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);    // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15 -> rows 1, 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31 -> rows 2, 3
  return x;
}

// The value of another lane of a row of 16: rotated by up to 15 lanes, or neighbours swapped (data-parallel-primitive
// moves, which the compiler folds into the instruction that uses them).
constexpr int kRotated = 0x120, kSwapped = 0xb1;
template <int kControl>
__device__ __forceinline__ float lane_move(float x) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), kControl, 0xf, 0xf, true));
}

// op over all 64 lanes, in every lane (op: a minimum or maximum, whose order does not matter).  As six shuffles, LDS
// round trips one after the other at the head of every sort that has to find its range: whole ranking, us, 32 heads, 4K in
// 512 26.5 / 26.0, 7360 in 320 52.5 / 51.8, 64K in 1024 with scores 741 / 735.
template <class Op>
__device__ __forceinline__ float wave_reduce(float x, Op op) {
  x = op(x, lane_move<kRotated + 8>(x));
  x = op(x, lane_move<kRotated + 4>(x));
  x = op(x, lane_move<kRotated + 2>(x));
  x = op(x, lane_move<kRotated + 1>(x));
  const u32x2 p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = op(__uint_as_float(p.x), __uint_as_float(p.y));
  const u32x2 q = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return op(__uint_as_float(q.x), __uint_as_float(q.y));
}
__device__ __forceinline__ float wave_min(float x) { return wave_reduce(x, [](float a, float b) { return fminf(a, b); }); }
__device__ __forceinline__ float wave_max(float x) { return wave_reduce(x, [](float a, float b) { return fmaxf(a, b); }); }

// A value that is the same in every lane, as the scalar it is.
__device__ __forceinline__ uint32_t uniform(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }
// The same value, but unknown to the optimiser from here on: what is computed from it is not
// kept in registers across phases (or hoisted out of a loop that normally runs once).
__device__ __forceinline__ int fresh(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// In-LDS bitonic sort of n2 (power of two) 64-bit keys, ascending.
__device__ inline void bitonic_sort_lds(uint64_t* keys, int n2, int tid, int nthreads) {
  for (int k = 2; k <= n2; k <<= 1) {
    for (int jj = k >> 1; jj > 0; jj >>= 1) {
      for (int t = tid; t < (n2 >> 1); t += nthreads) {
        const int i = ((t & ~(jj - 1)) << 1) | (t & (jj - 1));
        const int l = i | jj;
        const uint64_t x = keys[i], y = keys[l];
        const bool up = (i & k) == 0;
        if ((x > y) == up) { keys[i] = y; keys[l] = x; }
      }
      __syncthreads();
    }
  }
}

// LDS of one sort.
template <class Shape>
struct SortLds {
  uint32_t* word;     // [kWords] three 6-bit bucket counters, later the words' first place above them;
                      // then the list of keys that share a bucket
  uint64_t* list;     // [kCap + 64] (score, token) pairs: as collected, then in bucket order, then (tokens) in final order
  uint64_t* all;      // everything below misc, for the bitonic network
  uint32_t* misc;     // 64 words
  uint64_t* map;      // [kMapBins] (the list's area, free while the keys are in registers) first bucket word
                      // and bucket words of a linear piece, as floats
  __device__ explicit SortLds(unsigned char* smem) {
    word = reinterpret_cast<uint32_t*>(smem);
    list = reinterpret_cast<uint64_t*>(smem + Shape::kListAt);
    all = reinterpret_cast<uint64_t*>(smem);
    misc = reinterpret_cast<uint32_t*>(smem + Shape::kMiscAt);
    map = list;
  }
};

// x moved into [0, hi], NaN to 0: what a conversion to an unsigned integer is defined for.  Scores
// lie outside a sampled range as a matter of course, and a range may be infinite or denormal.
__device__ __forceinline__ float within(float x, float hi) { return __builtin_amdgcn_fmed3f(x, 0.f, hi); }

// What the sort takes for a score: NaN (an input error) counts as -inf.
__device__ __forceinline__ float sort_score(float s) { return s == s ? s : -INFINITY; }
__device__ __forceinline__ uint64_t pair_of(float s, uint32_t tok) { return ((uint64_t)tok << 32) | __float_as_uint(s); }
__device__ __forceinline__ float pair_score(uint64_t p) { return __uint_as_float((uint32_t)p); }
__device__ __forceinline__ uint32_t pair_token(uint64_t p) { return (uint32_t)(p >> 32); }
// 1 if pair p comes before the key (s, tok), else 0; no branches
__device__ __forceinline__ uint32_t ahead_of(uint64_t p, float s, uint32_t tok) {
  return (uint32_t)(pair_score(p) > s) | ((uint32_t)(pair_score(p) == s) & (uint32_t)(pair_token(p) < tok));
}

// Sorts n keys (1 <= n <= kCap) by (score descending, token ascending) and writes the tokens to
// out[0..n).  Key t + e * kThreads is (f[e], tok[e]) of thread t.  Every thread of the workgroup
// calls it after a barrier behind which the LDS is free; a caller that uses the LDS again puts a
// barrier in front.  bounded: all scores are known to lie in [flo, fhi]; otherwise the range is
// found first.
//
// Linear time: a monotone map of the score to 36 x kThreads fine buckets (two to five per key, 18 in the sort of up to 512) by
// one counting atomic, which also ranks the key inside its bucket, a scan of the counters, and
// every key is put at its bucket's place.  What is left is the order inside a bucket: keys that
// share one, a quarter to a half, are listed, and a full set of lanes works on the list: each is
// compared with its bucket's pairs and its token put at its final place.  (Comparing from where
// the keys are, three lanes in four idle, took 37 instead of 17 vector instructions per 64 keys.)
// A bucket of over 60 keys (many equal scores, or an outlier that stretches the range) sends the
// whole set to a bitonic network instead, and so does a list of more than kWords (full buckets
// everywhere).
//
// What bounds it is LDS and vector instructions alike: per 64 keys one atomic, one random 4-byte
// read and one random 8-byte write, 9 to 12 clocks each, the list about the same again; and about
// 60 vector instructions.  Three 6-bit counters and the 14-bit place share a word so that one
// read gives all of them.  Wavefronts without keys in a row of kThreads skip it.
template <class Shape>
__device__ __forceinline__ void block_sort(const SortLds<Shape>& m, int n, float (&f)[Shape::kPerThread],
                                           uint32_t (&tok)[Shape::kPerThread], bool bounded, float flo, float fhi,
                                           int32_t* out) {
  constexpr int T = Shape::kThreads, kPer = Shape::kPerThread, kWaves = T / 64;
  constexpr int kW = Shape::kWords / T;             // bucket words of a thread
  static_assert(Shape::kCap <= 16384 && kW % 4 == 0, "packing of the bucket words");
  static_assert(3 * Shape::kWords >= 2 * Shape::kCap, "the list of keys that share a bucket has to fit kWords");
  const int tid = fresh(threadIdx.x), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int left = n - tid;                               // key e exists iff e * T < left
  uint32_t* const wlo = m.misc;                     // [16]
  uint32_t* const whi = m.misc + 16;                // [16]
  uint32_t* const wsum = m.misc + 32;               // [16]
  uint32_t* const crowded = m.misc + 48;
  uint32_t* const nlist = m.misc + 49;
  u32x4* const w4 = reinterpret_cast<u32x4*>(m.word);
  {
    const u32x4 z = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int k = 0; k < kW / 4; ++k) w4[tid + k * T] = z;
  }
  if (tid == 0) { *crowded = 0u; *nlist = 0u; }
  // scale: bucket words per unit of the score for a bounded set, map pieces per unit otherwise;
  // 0 (everything in the first) for an empty or infinite range
  float scale;
  if (bounded) {
    const float range = fhi - flo;
    scale = range > 0.f ? ((float)Shape::kWords - 0.5f) / range : 0.f;   // below kWords for every score of the range
    __syncthreads();
  } else {
    float lo = INFINITY, hi = -INFINITY;
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      const bool mine = tid + e * T < n;
      lo = fminf(lo, mine ? f[e] : INFINITY);
      hi = fmaxf(hi, mine ? f[e] : -INFINITY);
    }
    lo = wave_min(lo);
    hi = wave_max(hi);
    if (lane == 0) { wlo[wave] = __float_as_uint(lo); whi[wave] = __float_as_uint(hi); }
    uint32_t* const hist = reinterpret_cast<uint32_t*>(m.map) + kMapBins;   // (the upper half of the map's area)
    for (int i = tid; i < kMapBins; i += T) hist[i] = 0u;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      lo = fminf(lo, __uint_as_float(wlo[w]));
      hi = fmaxf(hi, __uint_as_float(whi[w]));
    }
    flo = lo; fhi = hi;
    const float range = fhi - flo;
    scale = range > 0.f ? ((float)kMapBins - 0.5f) / range : 0.f;
    // The first and the last range of a row, and whole rows, are far from evenly filled (tails, a
    // few far-off keys).  Half of the buckets are spread over the score range evenly, the other
    // half follows a sample, the first key of every thread.
    if (tid < n) atomicAdd(&hist[(uint32_t)within((fhi - f[0]) * scale, (float)(kMapBins - 1))], 1u);
    __syncthreads();
    if (tid < 64) {                                 // one wavefront, four pieces per lane; 1/16 bucket words, exact in fp32
      const u32x4 c = reinterpret_cast<const u32x4*>(hist)[tid];
      const uint32_t per_bin = 8u * Shape::kWords / kMapBins, per_key = (8u * Shape::kWords - 16u) / (uint32_t)min(n, T);
      uint32_t at = wave_inclusive_sum(c[0] + c[1] + c[2] + c[3]) - (c[0] + c[1] + c[2] + c[3]);
      at = at * per_key + 4u * tid * per_bin;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t len = per_bin + c[k] * per_key;
        // (the wavefront has read every count of the upper half before the first is overwritten)
        m.map[4 * tid + k] = ((uint64_t)__float_as_uint((float)len * 0.0625f) << 32) | __float_as_uint((float)at * 0.0625f);
        at += len;
      }
    }
    __syncthreads();
  }
  left = fresh(left);
  // ---- count: pk = word | shift of the counter << 14 | rank << 19
  uint32_t pk[kPer], old[kPer];
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    if (e * T < left) {
      float y = (fhi - f[e]) * scale;
      if (!bounded) {                               // monotone: a piece ends where the next one begins
        y = within(y, (float)kMapBins - 0.25f);     // (at most kMapBins - 0.5 but for rounding and infinities)
        const uint32_t b = (uint32_t)y;
        const uint64_t piece = m.map[b];
        y = fmaf(__uint_as_float((uint32_t)(piece >> 32)), y - (float)b, __uint_as_float((uint32_t)piece));
      }
      y = within(y, (float)Shape::kWords - 0.25f);
      const uint32_t w = (uint32_t)y;
      const uint32_t sh = __umul24((uint32_t)(3.0f * __builtin_amdgcn_fractf(y)), 6u);   // (three fractions are below 3)
      // (24-bit: a 32-bit multiply takes four times as long)
      old[e] = atomicAdd(&m.word[w], 1u << (sh & 31u));
      pk[e] = (fresh(sh) << 14) | w;              // (not folded into a multiply)
    }
  }
  uint32_t most = 0;
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    if (e * T < left) {
      const uint32_t r = __builtin_amdgcn_ubfe(old[e], pk[e] >> 14, 6u);
      most = max(most, r);
      pk[e] |= r << 19;
    }
  }
  if (most >= 60u) *crowded = 1u;
  __syncthreads();
  // ---- first place of every word's first bucket, into the word
  {
    u32x4 x[kW / 4];
    uint32_t s[kW], run = 0;
#pragma unroll
    for (int k = 0; k < kW / 4; ++k) x[k] = w4[kW / 4 * tid + k];
#pragma unroll
    for (int k = 0; k < kW; ++k) {
      const uint32_t w = x[k / 4][k % 4];
      s[k] = run;
      run += (w & 63u) + __builtin_amdgcn_ubfe(w, 6u, 6u) + __builtin_amdgcn_ubfe(w, 12u, 6u);
    }
    const uint32_t incl = wave_inclusive_sum(run);
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    uint32_t base = incl - run;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) base += w < wave ? wsum[w] : 0u;
#pragma unroll
    for (int k = 0; k < kW; ++k) x[k / 4][k % 4] |= (base + s[k]) << 18;
#pragma unroll
    for (int k = 0; k < kW / 4; ++k) w4[kW / 4 * tid + k] = x[k];
  }
  const bool fallback = __builtin_amdgcn_readfirstlane((int)*crowded) != 0;
  __syncthreads();
  if (!fallback) {
    left = fresh(left);
    // ---- place.  A key alone in its bucket is where it belongs; the others go to a list:
    // first place of the bucket | population << 14 | rank << 20
#pragma unroll
    for (int e = 0; e < kPer; ++e)
      if (e * T < left) old[e] = m.word[pk[e] & 0x3fffu];
    uint32_t shared = 0;                            // bit e: key e shares its bucket
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      if (e * T < left) {
        const uint32_t sh = __builtin_amdgcn_ubfe(pk[e], 14u, 5u), r = pk[e] >> 19;
        const uint32_t below = old[e] & ((1u << sh) - 1u);
        const uint32_t p0 = (old[e] >> 18) + (below & 63u) + (below >> 6), c = __builtin_amdgcn_ubfe(old[e], sh, 6u);
        m.list[p0 + r] = pair_of(f[e], tok[e]);
        pk[e] = p0 | (c << 14) | (r << 20);
        shared |= c > 1u ? 1u << e : 0u;
      }
    }
    __syncthreads();                                // the bucket words are free now: the list goes there
    {
      const uint32_t cnt = (uint32_t)__builtin_popcount(shared);
      const uint32_t incl = wave_inclusive_sum(cnt);
      const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
      uint32_t at = 0;
      if (lane == 0) at = atomicAdd(nlist, total);
      at = uniform(at);
      if (at + total <= (uint32_t)Shape::kWords) {
        at += incl - cnt;
#pragma unroll
        for (int e = 0; e < kPer; ++e)
          if (shared & (1u << e)) m.word[at++] = pk[e];
      }
    }
    __syncthreads();
    const int listed = (int)uniform(*nlist);
    if (listed <= Shape::kWords) {                  // (a list that does not fit: full buckets everywhere)
      constexpr int kHold = Shape::kWords / T;      // listed keys of a thread
      const int mine = listed - tid;                // listed key k exists iff k * T < mine
      uint32_t to[kHold], tk[kHold];
#pragma unroll
      for (int k = 0; k < kHold; ++k) {
        if (k * T < mine) {
          const uint32_t w = m.word[tid + k * T], p0 = w & 0x3fffu, c = __builtin_amdgcn_ubfe(w, 14u, 6u);
          const uint64_t me = m.list[p0 + (w >> 20)];
          const float s = pair_score(me);
          tk[k] = pair_token(me);
          to[k] = p0;
          uint64_t x[3];
#pragma unroll
          for (int q = 0; q < 3; ++q) x[q] = m.list[p0 + q];   // (pairs past the bucket come later than it)
#pragma unroll
          for (int q = 0; q < 3; ++q) to[k] += (uint32_t)q < c ? ahead_of(x[q], s, tk[k]) : 0u;
#pragma unroll 1
          for (uint32_t q = 3; q < c; ++q) to[k] += ahead_of(m.list[p0 + q], s, tk[k]);
        }
      }
      __syncthreads();
      uint32_t* const token = reinterpret_cast<uint32_t*>(m.list) + 1;
#pragma unroll
      for (int k = 0; k < kHold; ++k)
        if (k * T < mine) token[2 * to[k]] = tk[k];
      __syncthreads();
      for (int i = tid; i < n; i += T) out[i] = (int32_t)token[2 * i];
      return;
    }
    __syncthreads();
  }
  int n2 = 1;
  while (n2 < n) n2 <<= 1;
  for (int i = n + tid; i < n2; i += T) m.all[i] = ~0ull;
#pragma unroll
  for (int e = 0; e < kPer; ++e)
    if (tid + e * T < n) m.all[tid + e * T] = ((uint64_t)(~ordered_u32(f[e])) << 32) | tok[e];
  __syncthreads();
  bitonic_sort_lds(m.all, n2, tid, T);
  for (int i = tid; i < n; i += T) out[i] = (int32_t)(uint32_t)m.all[i];
}

// ---------------------------------------------------------------------------------------
// One workgroup per (z, h, n) = row_id: q_mean (kMean), s_Q and Q_perm (kSort) of the segment in
// one pass over Q.  Sixteen rows at a time, each by 16 lanes with 8 columns (256 threads) or 32 lanes
// with 4 (512 threads, which the sorts of more than 2048 queries need).  The sums are taken in one
// order whatever the number of threads: a product's 8-column chain runs on from the even lane to the
// odd one.
template <class Shape, bool kMean, bool kSort>
__device__ __forceinline__ void pool_segment(const PlanArgs& a, const Scratch& sc, int64_t row_id, unsigned char* smem) {
  constexpr int T = Shape::kThreads, kLanes = T / 16, kCols = kD / kLanes;
  static_assert(T == 256 || T == 512, "the row loop is written for 16 or 32 lanes a row");
  typedef uint32_t Piece __attribute__((ext_vector_type(kCols / 2)));
  float* sq = reinterpret_cast<float*>(smem);                       // [S] scores; the sort's LDS later
  float* red = sq + (kSort ? Shape::kCap : 0);                      // [wavefronts][128]
  static_assert(!kSort || 4 * (size_t)Shape::kCap + T / 64 * 4 * kD <= Shape::kLds, "the partial sums fit behind the scores");

  const int G = a.H / a.Hkv;
  const int n = (int)(row_id % a.N);                                // row_id = (z*H + h)*N + n
  const int h = (int)((row_id / a.N) % a.H);
  const int z = (int)(row_id / ((int64_t)a.N * a.H));
  const int g = h / G;
  const int tid = threadIdx.x, c = tid % kLanes, r = tid / kLanes;
  const uint16_t* Qs = a.Q + z * a.qs[0] + h * a.qs[1] + (int64_t)n * a.S * a.qs[2];
  // k_guide = mean of the first key segment, from the partial sums in a fixed order
  const float* kg = sc.kguide + ((int64_t)z * a.Hkv + g) * kGuideParts * kD + kCols * c;
  float kgv[kCols];
  if constexpr (kSort) {
#pragma unroll
    for (int j = 0; j < kCols; ++j) {
      float t = 0.f;
#pragma unroll
      for (int pp = 0; pp < kGuideParts; ++pp) t += kg[pp * kD + j];
      kgv[j] = t * (1.0f / (float)a.S);
    }
  }
  if (kSort && a.k_guide && n == 0 && h % G == 0 && r == 0) {
#pragma unroll
    for (int j = 0; j < kCols; ++j) a.k_guide[((int64_t)z * a.Hkv + g) * kD + kCols * c + j] = kgv[j];
  }

  // Four rows of a thread per trip (S is a multiple of 64: no tail).  Where a CU has one workgroup, or its
  // workgroups are large, memory latency bounds the pass and the next trip's loads are on their way during a
  // trip (us for the whole ranking without / with: 256 rows of 512 queries 31.1 / 29.6, of 1024 50.8 / 47.0, 128 of
  // 1024 161 / 156, 128 of 2048 without causality 81.5 / 74.6).  One pass over Q by 256 threads has several
  // workgroups on a CU from 257 rows on: 512 rows of 1024 90.1 / 91.6, 552 of 320 60.1 / 61.6.
  const bool ahead = !(kMean && kSort && T == 256) || (Shape::kCap > 512 && gridDim.x <= kOneEach);
  auto load = [&](Piece (&x)[4], int row0) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      x[u] = *reinterpret_cast<const Piece*>(Qs + (int64_t)(row0 + 16 * u) * a.qs[2] + kCols * c);
  };
  float acc[kCols] = {};
  Piece v4[4];
  auto trip = [&](int row0) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int row = row0 + 16 * u;
      const Piece v = v4[u];
      float x[kCols];
#pragma unroll
      for (int q = 0; q < kCols / 2; ++q) { x[2 * q] = bf16_lo(v[q]); x[2 * q + 1] = bf16_hi(v[q]); }
      if constexpr (kMean) {
#pragma unroll
        for (int j = 0; j < kCols; ++j) acc[j] += x[j];
      }
      if constexpr (!kSort) continue;
      auto chain = [&](float t) {
#pragma unroll
        for (int j = 0; j < kCols; ++j) t = fmaf(x[j], kgv[j], t);
        return t;
      };
      float dot = chain(0.f);
      // Moves between lanes inside the additions: as shuffles, through LDS, they bounded the pass.  Whole ranking, us,
      // shuffles / moves: 32 heads, 4K in 512 29.3 / 27.0, 8K in 1024 47.1 / 42.4, 16K in 4096 104 / 75; 8 heads, 16K in 8192 167 /
      // 109; 12 over 4, 5K in 1024 without causality 37 / 30; 128K in 2048 1413 / 1410 (bound by Q from memory).
      if constexpr (kLanes == 32) {
        const float even = lane_move<kSwapped>(dot);
        dot = chain((c & 1) ? even : 0.f);        // complete in the odd lanes
        const u32x2 p = __builtin_amdgcn_permlane16_swap(__float_as_uint(dot), __float_as_uint(dot), false, false);
        dot = __uint_as_float(p.x) + __uint_as_float(p.y);
      }
      // plus that of lane c ^ 8, then ^ 4, ^ 2 (and ^ 1): the sums repeat with that period, so a rotation is enough
      dot += lane_move<kRotated + 8>(dot);
      dot += lane_move<kRotated + 4>(dot);
      dot += lane_move<kRotated + 2>(dot);
      if constexpr (kLanes == 16) dot += lane_move<kRotated + 1>(dot);
      if (c == kLanes / 16 - 1) sq[row] = dot;
    }
  };
  if (ahead) {
    load(v4, r);
    for (int at = 64; at < a.S; at += 64) {
      Piece next[4];
      load(next, at + r);
      trip(at - 64 + r);
#pragma unroll
      for (int u = 0; u < 4; ++u) v4[u] = next[u];
    }
    trip(a.S - 64 + r);
  } else {
    for (int at = 0; at < a.S; at += 64) {
      load(v4, at + r);
      trip(at + r);
    }
  }
  // ---- q_mean: column sums over the wavefront's four row groups, then over the wavefronts
#pragma unroll
  for (int j = 0; j < kCols; ++j) {
    if constexpr (kLanes == 16) {
      const u32x2 p = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[j]), __float_as_uint(acc[j]), false, false);
      acc[j] = __uint_as_float(p.x) + __uint_as_float(p.y);
    }
    const u32x2 p = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[j]), __float_as_uint(acc[j]), false, false);
    acc[j] = __uint_as_float(p.x) + __uint_as_float(p.y);
  }
  if (kMean && (tid & 63) < kLanes) {
#pragma unroll
    for (int j = 0; j < kCols; ++j) red[(tid >> 6) * kD + kCols * c + j] = acc[j];
  }
  __syncthreads();
  if (kMean && tid < kD) {
    float p[4];
#pragma unroll
    for (int w = 0; w < 4; ++w)
      p[w] = kLanes == 16 ? red[w * kD + tid] : red[2 * w * kD + tid] + red[(2 * w + 1) * kD + tid];
    float s = (p[0] + p[1]) + (p[2] + p[3]);
    s *= 1.0f / (float)a.S;
    if (a.q_mean) a.q_mean[row_id * kD + tid] = s;
    // exact three-way bf16 split (truncation keeps every step exact in fp32)
    const uint32_t u = __float_as_uint(s);
    const float hi = __uint_as_float(u & 0xffff0000u);
    const float r1 = s - hi;
    const float mid = __uint_as_float(__float_as_uint(r1) & 0xffff0000u);
    const float lo = r1 - mid;
    uint16_t* qs = sc.qsplit + row_id * 3 * kD;
    qs[tid] = (uint16_t)(__float_as_uint(hi) >> 16);
    qs[kD + tid] = (uint16_t)(__float_as_uint(mid) >> 16);
    qs[2 * kD + tid] = (uint16_t)(__float_as_uint(lo) >> 16);   // 8 bits left: exact
  }
  if constexpr (!kSort) return;
  float f[Shape::kPerThread];
  uint32_t tok[Shape::kPerThread];
#pragma unroll
  for (int e = 0; e < Shape::kPerThread; ++e) {
    const int i = tid + e * T;
    tok[e] = (uint32_t)i;
    f[e] = i < a.S ? sq[i] : 0.f;
  }
  // (Not from the row loop: the wait for the next rows at the end of a trip would cover the trip's stores.
  // Whole ranking, 8 heads, three segments of 6144 queries, stored there / here 154 / 133 us, 32 heads, 8 of 4096
  // 179 / 152.)
  if (a.s_q) {
#pragma unroll
    for (int e = 0; e < Shape::kPerThread; ++e)
      if (tid + e * T < a.S) a.s_q[row_id * a.S + tid + e * T] = f[e];
  }
#pragma unroll
  for (int e = 0; e < Shape::kPerThread; ++e) f[e] = sort_score(f[e]);
  __syncthreads();                                // the scores and partial sums have been read
  const SortLds<Shape> m(smem);
  block_sort<Shape>(m, a.S, f, tok, false, 0.f, 0.f, a.q_perm + row_id * a.S);
}

// (Two workgroups per CU where the sort's LDS allows it.)
template <class Shape>
__global__ __launch_bounds__(Shape::kThreads, Shape::kThreads == 512 ? (Shape::kLds <= 81920 ? 4 : 2) : 1)
void pool_sq_sort_kernel(PlanArgs a, Scratch sc) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  pool_segment<Shape, true, true>(a, sc, blockIdx.x, smem);
}

// Short sequences: the first launch takes q_mean of all rows and, in further workgroups, k_guide's
// partial sums, neither of which needs the other; s_Q and its Argsort then run beside the scores
// (score_sort_kernel).
constexpr size_t kMeanLds = 4 * kD * sizeof(float);
__global__ __launch_bounds__(256) void mean_guide_kernel(PlanArgs a, Scratch sc, int rows) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  if ((int)blockIdx.x < rows) pool_segment<SortShape<256, 2>, true, false>(a, sc, blockIdx.x, smem);
  else guide_part(a, sc, (int)blockIdx.x - rows);
}

// ---------------------------------------------------------------------------------------
// s_K scoring.  Workgroup = (z, g, group of kScoreWaves row blocks, chunk of sc.chunk tokens);
// a wavefront owns one row block of the group (32 rows of the contraction's N side) and keeps
// its q_mean split fragments in registers for the whole chunk; the chunk's K rows pass through
// LDS in tiles of kSub tokens shared by the wavefronts.  Row r of KV head g is a (query head,
// segment n) and needs tokens t < n*S.
//   A (32 tokens x 16 dims): K tile rows from LDS, lane (token = l%32, hh = l/32) reads dims
//                            16*kk + 8*hh .. +8
//   B (16 dims x 32 rows)  : q_mean split terms, lane (row = l%32, hh) holds the same dims
//   C (32 tokens x 32 rows): register i of lane l = [token 8*(i/4) + 4*hh + i%4][row l%32],
//                            so a lane sees one row only and its meta data are scalars
// What bounds it: matrix instructions, at two wavefronts per SIMD, and stores of 16 bytes one after the other
// (64K tokens, 32 heads, 1024-token segments: 140 us; without the stores 97, with a third of the products as
// well 56).  And two waits that nothing needs: the compiler guards the q_mean fragments, loaded in front of the
// loop, with a wait for the next tile's K rows before a tile's first product, and the wait that puts those rows
// down covers the scores stored since.  Two chains of 32 tokens side by side: +-0.  Stored as whole lines after a turn through LDS: 1 to
// 3 % faster there, 2 us slower at 8K and 16K.
__device__ __forceinline__ void score_block(const PlanArgs& a, const Scratch& sc, int block, unsigned char* smem) {
  uint16_t* Kt = reinterpret_cast<uint16_t*>(smem);                          // [kSub][kKStride]

  const int G = a.H / a.Hkv;
  const int R = G * a.N;
  const int nchunks = (a.L + sc.chunk - 1) / sc.chunk;
  // all work on one KV head goes to one XCD (block ids are dealt round-robin to the 8 XCDs):
  // the row blocks of a head read the same K chunks
  int unit, rest;
  {
    const int U = a.Z * a.Hkv, b = block;
    if (U % 8 == 0) {
      const int xcd = b & 7, idx = b >> 3, per = U / 8;
      unit = (idx % per) * 8 + xcd;
      rest = idx / per;
    } else {
      unit = b % U;
      rest = b / U;
    }
  }
  const int chunk = rest % nchunks;
  const int rbg = rest / nchunks;
  const int g = unit % a.Hkv, z = unit / a.Hkv;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m_ = lane & 31, hh = lane >> 5;
  // (shifted by the chunk: the wavefronts with the shorter rows are not always on the same SIMD)
  const int rb = kScoreWaves * rbg + ((wave + chunk) & (kScoreWaves - 1));

  // Row r: with several groups of row blocks all heads of a segment follow one another, so that a group's
  // rows are about equally long and the groups of short rows leave most chunks alone (all segments of a head
  // in a row: every group has long rows, and half of its wavefronts, always on the same two SIMDs, have
  // nothing to do beyond the middle of the sequence.  This kernel, 256 rows a KV head, 64K tokens 156 -> 140 us,
  // 128K 294 -> 259).  A single group has every row in any order, and without causality all rows are equally
  // long.  From 256 segments on a head has groups of its own, and by head the rows of a block are neighbours:
  // whole ranking, by head / by segment, 4 heads over one, 129 segments of 320 144 / 138 us, 200 of 64 85 / 82, but
  // 3 over one, 256 of 512 522 / 530, 12 over 4, 320 of 64 421 / 429; without causality 16 over one, 128 of 320 0.96.
  const bool by_segment = R > 32 * kScoreWaves && a.N < 64 * kScoreWaves && !a.non_causal;
  const int inner = by_segment ? G : a.N;         // row r = (r / inner, r % inner); one division a row
  // longest of the rows first .. first + count - 1 (the last one's, but if a run by head wraps it
  // contains a last segment)
  auto run_limit = [&](int first, int count) {
    const int last = min(first + count, R) - 1;
    if (first > last) return 0;
    const int u = last / inner, v = last - u * inner;
    const int n = by_segment ? u : last - first > v ? a.N - 1 : v;
    return (int)kv_row_len(n, a.S, a.L, a.non_causal);
  };
  // token limits: of the workgroup's rows and of this wavefront's rows
  const int lim_wg = run_limit(32 * kScoreWaves * rbg, 32 * kScoreWaves);
  const int lim_wave = run_limit(32 * rb, 32);
  const int t_begin = chunk * sc.chunk;
  if (t_begin >= lim_wg) return;
  const int t_end = min(t_begin + sc.chunk, lim_wg);

  // this lane's row
  const int r = 32 * rb + m_, rr = min(r, R - 1);
  const int u = rr / inner, v = rr - u * inner, n = by_segment ? u : v;
  const int lim = r < R ? (int)kv_row_len(n, a.S, a.L, a.non_causal) : 0;
  const int64_t zh = (int64_t)z * a.H + g * G + (by_segment ? v : u);
  const int64_t row_id = zh * a.N + n;
  const int64_t base = zh * kv_rows_total(a.N, a.S, a.L, a.non_causal) + kv_row_start(n, a.S, a.L, a.non_causal);
  float* skdst = (a.s_k ? a.s_k : sc.sk) + base;

  // B fragments: 3 split terms x 8 contraction steps
  bf16x8 bq[3][8];
  {
    const uint16_t* qs = sc.qsplit + row_id * 3 * kD;
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int kk = 0; kk < 8; ++kk)
        bq[t][kk] = *reinterpret_cast<const bf16x8*>(qs + t * kD + 16 * kk + 8 * hh);
  }
  const int samples_per_row = a.L / kSampleStride;

  // K tile loader: thread (c, q) moves 16-byte chunk c of rows q, q+16, ...
  const uint16_t* Kh = a.K + z * a.ks[0] + g * a.ks[1];
  const int c = tid & 15, q = tid >> 4;
  constexpr int kLoadRows = 4 * kScoreWaves;      // tile rows one pass of the loader covers
  u32x4 kreg[kSub / kLoadRows];
  auto load_tile = [&](int t0) {
#pragma unroll
    for (int s = 0; s < kSub / kLoadRows; ++s) {
      const int t = min(t0 + q + kLoadRows * s, a.L - 1);
      kreg[s] = *reinterpret_cast<const u32x4*>(Kh + (int64_t)t * a.ks[2] + 8 * c);
    }
  };
  auto store_tile = [&]() {
#pragma unroll
    for (int s = 0; s < kSub / kLoadRows; ++s)
      *reinterpret_cast<u32x4*>(Kt + (q + kLoadRows * s) * kKStride + 8 * c) = kreg[s];
  };

  load_tile(t_begin);
  for (int t0 = t_begin; t0 < t_end; t0 += kSub) {
    __syncthreads();                       // previous tile fully consumed
    store_tile();
    __syncthreads();
    if (t0 + kSub < t_end) load_tile(t0 + kSub);
    if (t0 < lim_wave) {
#pragma unroll 1
      for (int sb = 0; sb < kSub / 32; ++sb) {
        f32x16 acc;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = 0.f;
        bf16x8 ka[8];
#pragma unroll
        for (int kk = 0; kk < 8; ++kk)
          ka[kk] = *reinterpret_cast<const bf16x8*>(Kt + (32 * sb + m_) * kKStride + 16 * kk + 8 * hh);
        // smallest term first so that the large products meet an accumulator that already
        // holds the corrections
#pragma unroll
        for (int tt = 2; tt >= 0; --tt)
#pragma unroll
          for (int kk = 0; kk < 8; ++kk)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[kk], bq[tt][kk], acc, 0, 0, 0);
        // lim is a multiple of 64, so a 32-token block is valid for this row as a whole or not at all
        if (t0 + 32 * sb < lim) {
          // sample: one token of the 32, its place among eight varying from block to block
          const int blk = (t0 + 32 * sb) / kSampleStride;
          if (((blk >> 2) & 1) == hh) {
            const float v = (blk & 2) ? ((blk & 1) ? acc[15] : acc[10]) : ((blk & 1) ? acc[5] : acc[0]);
            sc.samples[row_id * samples_per_row + blk] = v;
          }
          // the four registers of a group are four consecutive tokens
#pragma unroll
          for (int i4 = 0; i4 < 4; ++i4) {
            const int t = t0 + 32 * sb + 8 * i4 + 4 * hh;
            const f32x4 v = {acc[4 * i4], acc[4 * i4 + 1], acc[4 * i4 + 2], acc[4 * i4 + 3]};
            *reinterpret_cast<f32x4*>(skdst + t) = v;
          }
        }
      }
    }
  }
}

__global__ __launch_bounds__(64 * kScoreWaves) void score_kernel(PlanArgs a, Scratch sc) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  score_block(a, sc, (int)blockIdx.x, smem);
}

// The scores and, in workgroups of their own in front, s_Q and Q_perm of all rows.
constexpr size_t kScoreLds = (size_t)kSub * kKStride * 2;
template <class Shape>
__global__ __launch_bounds__(64 * kScoreWaves) void score_sort_kernel(PlanArgs a, Scratch sc, int rows) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  static_assert(Shape::kLds <= kScoreLds && Shape::kThreads == 64 * kScoreWaves, "one launch shape for both");
  if ((int)blockIdx.x < rows) pool_segment<Shape, false, true>(a, sc, blockIdx.x, smem);
  else score_block(a, sc, (int)blockIdx.x - rows, smem);
}

__device__ inline int64_t row_base(const PlanArgs& a, int64_t zh, int n) {
  return zh * kv_rows_total(a.N, a.S, a.L, a.non_causal) + kv_row_start(n, a.S, a.L, a.non_causal);
}

// Per row longer than one LDS sort: the lower ends of its score ranges.  A linear histogram of
// the sampled scores is cut at equal shares, interpolating inside a bin.  Nothing depends on the
// cuts being good but the balance between workgroups, and row_sort_kernel cuts again where a
// range does not fit; they only have to be in descending order and finite, so that -inf, and NaN
// which counts as -inf, belong to the last range whatever the sample holds.
constexpr int kThrBins = 1024;
__global__ __launch_bounds__(256) void threshold_kernel(PlanArgs a, Scratch sc) {
  __shared__ uint32_t hist[kThrBins + 1];
  __shared__ float red[8];
  __shared__ uint32_t wsum[4];
  const int64_t row_id = blockIdx.x;
  const int n = (int)(row_id % a.N);
  const int len = (int)kv_row_len(n, a.S, a.L, a.non_causal);
  const int nr = row_ranges(len, sc.cap);
  if (nr <= 1) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int ns = len / kSampleStride;
  const float* smp = sc.samples + row_id * (a.L / kSampleStride);
  float lo = INFINITY, hi = -INFINITY;
  for (int i = tid; i < ns; i += 256) { const float v = smp[i]; lo = fminf(lo, v); hi = fmaxf(hi, v); }
  lo = wave_min(lo);
  hi = wave_max(hi);
  if (lane == 0) { red[wave] = lo; red[4 + wave] = hi; }
  for (int i = tid; i <= kThrBins; i += 256) hist[i] = 0u;
  __syncthreads();
  lo = fminf(fminf(red[0], red[1]), fminf(red[2], red[3]));
  hi = fmaxf(fmaxf(red[4], red[5]), fmaxf(red[6], red[7]));
  const float width = (hi - lo) / (float)kThrBins;
  const float inv = width > 0.f ? 1.0f / width : 0.f;
  for (int i = tid; i < ns; i += 256)
    atomicAdd(&hist[(uint32_t)within((hi - smp[i]) * inv, (float)(kThrBins - 1))], 1u);
  __syncthreads();
  // exclusive scan, four bins per thread
  uint32_t v[4], run = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) { v[k] = run; run += hist[4 * tid + k]; }
  const uint32_t incl = wave_inclusive_sum(run);
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  uint32_t base = incl - run;
  for (int w = 0; w < wave; ++w) base += wsum[w];
#pragma unroll
  for (int k = 0; k < 4; ++k) hist[4 * tid + k] = base + v[k];
  if (tid == 255) hist[kThrBins] = base + run;
  __syncthreads();
  float* out = sc.thr + row_id * (sc.max_ranges + 2);
  if (tid == 0) { out[nr] = hi; out[nr + 1] = lo; }
  for (int r = tid; r < nr; r += 256) {
    // position (r + 1) / nr of the sample: the last bin that starts at or before it
    const float at = (float)ns * ((float)(r + 1) / (float)nr);
    int b = 0;
#pragma unroll
    for (int step = kThrBins / 2; step > 0; step >>= 1)
      if ((float)hist[b + step] <= at) b += step;
    const float in = (float)(hist[b + 1] - hist[b]);
    const float frac = in > 0.f ? fminf((at - (float)hist[b]) / in, 1.0f) : 0.f;
    const float t = hi - ((float)b + frac) * width;
    out[r] = t >= -FLT_MAX ? t : -FLT_MAX;        // (NaN: there are infinities in the sample, or nothing but NaN)
  }
}

// A piece of the ranking of one row: score range r of the nr the row is cut into.
struct RowItem {
  int len, r, nr;
  int64_t base, row_id;    // of the row in s_K / KV_perm; (z*H + h)*N + n
  bool valid;
};

// Workgroup list (none in memory): rows n and N-n of a head are taken together, their lengths add
// up to N*S, so every pair needs about the same number of pieces (`slots`; a few hold nothing).
// The pieces of a pair go to workgroups whose ids land on one XCD (block ids are dealt round-robin
// to the 8 XCDs) and that work on them at about the same time: the row is read from HBM once
// and from that XCD's L2 for every further range.
__device__ __forceinline__ RowItem row_item(const PlanArgs& a, const Scratch& sc, int slots, int pairs, int xcd, int idx) {
  RowItem it;
  it.valid = false;
  it.len = 0; it.r = 0; it.nr = 0; it.base = 0; it.row_id = 0;
  const int ZH = a.Z * a.H, u = (idx / slots) * 8 + xcd;
  if (u >= ZH * pairs) return it;
  int r = idx % slots, n = u / ZH;
  const int zh = u % ZH;
  if (!a.non_causal) {
    const int p = n;
    n = a.N - 1 - p;
    const int first = row_ranges((int64_t)n * a.S, sc.cap);
    if (r >= first) { r -= first; n = 1 + p < n ? 1 + p : 0; }
  }
  it.len = (int)kv_row_len(n, a.S, a.L, a.non_causal);
  it.nr = row_ranges(it.len, sc.cap);
  it.r = r;
  it.base = row_base(a, zh, n);
  it.row_id = (int64_t)zh * a.N + n;
  it.valid = r < it.nr;
  return it;
}

// Deals a row's keys out to its ranges' regions: cells of 6144 keys are bucketed in LDS (a table
// over 256 linear pieces of the score gives the range but for three comparisons), counted with
// replicated counters, staged range by range and copied out as runs of a few hundred pairs.
// counts[r] = keys of range r (regions hold the first kCap at most; a range with more is
// incomplete there); lower[r] = its lower end.
template <class Shape>
__device__ __forceinline__ void split_row(const SortLds<Shape>& m, uint32_t* counts, float* lower, const float* sk, int len,
                                          int nr, const float* thr, uint64_t* regions) {
  constexpr int T = Shape::kThreads, kCap = Shape::kCap, kVec = 3, kCell = 4 * kVec * T, kLut = 256;
  constexpr int kCounters = 4 * T, kIdShift = 20;      // tokens are below 2^20
  static_assert(kCell <= Shape::kCap, "a cell is staged in the pair list");
  static_assert(Shape::kWords >= 4 * kLut + kMaxSplit + kCounters, "tables");
  const int tid = fresh(threadIdx.x), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  u32x4* const lut = reinterpret_cast<u32x4*>(m.word);                     // three thresholds to compare with, range
  uint32_t* const delta = m.word + 4 * kLut;                               // [nr] region slot - staging slot
  uint32_t* const cnt = m.word + 4 * kLut + kMaxSplit;                     // [nr][rep] counters, then first staging slots
  u32x4* const c4 = reinterpret_cast<u32x4*>(cnt);
  uint32_t* const wsum = m.misc;
  uint32_t rs = 5;                               // 2^rs copies of the counters against conflicts, rotated by range
  while ((nr << rs) > kCounters) --rs;
  const uint32_t rep = (uint32_t)(4 * wave + (lane & 3)), rmask = (1u << rs) - 1u;
  const float hi = thr[nr], range = hi - thr[nr + 1];
  const float inv = range > 0.f ? ((float)kLut - 0.5f) / range : 0.f;
  __syncthreads();                               // the previous row is out of LDS
  if (tid < nr + 3) lower[tid] = tid < nr - 1 ? thr[tid] : -INFINITY;
  if (tid < nr) counts[tid] = 0u;
  __syncthreads();
  if (tid < kLut) {
    // keys of piece b lie below the upper end of piece b - 1, whatever the rounding
    const float end = tid == 0 ? INFINITY : hi - (float)(tid - 1) * (range / ((float)kLut - 0.5f));
    uint32_t id = 0;
    for (int k = 0; k < nr - 1; ++k) id += lower[k] > end ? 1u : 0u;
    const u32x4 l = {__float_as_uint(lower[id]), __float_as_uint(lower[id + 1]), __float_as_uint(lower[id + 2]), id};
    lut[tid] = l;
  }
  f32x4 v[kVec];
  auto load = [&](int t0) {
#pragma unroll
    for (int q = 0; q < kVec; ++q)
      v[q] = *reinterpret_cast<const f32x4*>(sk + min(t0 + 4 * (q * T + tid), len - 4));
  };
  load(0);
  for (int t0 = 0; t0 < len; t0 += kCell) {
    {
      const u32x4 z = {0u, 0u, 0u, 0u};
      c4[tid] = z;
    }
    __syncthreads();                             // also: the table is there, the previous cell has been copied out
    uint32_t at[4 * kVec];                       // counter | rank << 16
    float s[4 * kVec];
    uint32_t further = 0;                        // bit k: the range of key k lies beyond the table's three
#pragma unroll
    for (int k = 0; k < 4 * kVec; ++k) {
      s[k] = sort_score(v[k / 4][k & 3]);
      const u32x4 l = lut[(uint32_t)within((hi - s[k]) * inv, (float)(kLut - 1))];
      at[k] = l[3] + (s[k] < __uint_as_float(l[0]) ? 1u : 0u) + (s[k] < __uint_as_float(l[1]) ? 1u : 0u) +
              (s[k] < __uint_as_float(l[2]) ? 1u : 0u);
      if (s[k] < __uint_as_float(l[2])) further |= 1u << k;
    }
    if (further != 0u) {
#pragma unroll
      for (int k = 0; k < 4 * kVec; ++k)
        if (further & (1u << k))
          while (s[k] < lower[at[k]]) ++at[k];   // (ends at the last range: nothing is below -inf)
    }
#pragma unroll
    for (int k = 0; k < 4 * kVec; ++k) at[k] = (at[k] << rs) + ((rep + at[k]) & rmask);
    if (t0 + kCell < len) load(t0 + kCell);
#pragma unroll
    for (int k = 0; k < 4 * kVec; ++k)
      if (t0 + 4 * ((k / 4) * T + tid) < len) at[k] |= atomicAdd(&cnt[at[k]], 1u) << 16;
    __syncthreads();
    {
      u32x4 x = c4[tid];
      const uint32_t run = x[0] + x[1] + x[2] + x[3];
      const uint32_t incl = wave_inclusive_sum(run);
      if (lane == 63) wsum[wave] = incl;
      __syncthreads();
      uint32_t base = incl - run;
#pragma unroll
      for (int w = 0; w < T / 64; ++w) base += w < wave ? wsum[w] : 0u;
#pragma unroll
      for (int k = 0; k < 4; ++k) { const uint32_t c = x[k]; x[k] = base; base += c; }
      c4[tid] = x;
    }
    __syncthreads();
    const int ncell = min(kCell, len - t0);
    if (tid < nr) {
      const uint32_t begin = cnt[tid << rs], end = tid + 1 < nr ? cnt[(tid + 1) << rs] : (uint32_t)ncell;
      const uint32_t have = counts[tid], c = end - begin;
      // (a staging slot is below a region's size, so a delta is never negative)
      delta[tid] = have + c <= (uint32_t)kCap ? (uint32_t)(tid * kCap) + have - begin : 0xffffffffu;
      counts[tid] = have + c;
    }
#pragma unroll
    for (int k = 0; k < 4 * kVec; ++k) {
      const int t = t0 + 4 * ((k / 4) * T + tid) + (k & 3);
      if (t < len) {
        const uint32_t slot = at[k] & 0xffffu;
        m.list[cnt[slot] + (at[k] >> 16)] = pair_of(s[k], (uint32_t)t | ((slot >> rs) << kIdShift));
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4 * kVec; ++k) {
      const int i = tid + k * T;
      if (i < ncell) {
        const uint64_t x = m.list[i];
        const uint32_t d = delta[pair_token(x) >> kIdShift];
        if (d != 0xffffffffu) regions[d + (uint32_t)i] = x & ((1ull << (32 + kIdShift)) - 1ull);
      }
    }
  }
  __syncthreads();                               // the regions are complete
}

// Ranks rows longer than one sort: a workgroup takes row after row, deals its keys out to the
// ranges' regions (split_row) and sorts range after range from there.  A range that did not fit
// its region is left to row_sort_kernel.
//
// What bounds it: LDS and vector instructions at 16 wavefronts per CU: a range of 4600 keys takes 9
// us to sort and 3 us to arrive, a cell of 6144 keys 7.7 us to deal out, two workgroups per CU.
// The rows are taken from a ticket, the longest first, so that the last ones to finish are short.
// 128K, 2016 rows: 935 us, against 1370 us with one piece per (row, range) and a scan each.
template <class Shape>
__global__ __launch_bounds__(Shape::kThreads, 4) void split_sort_kernel(PlanArgs a, Scratch sc, int nrows) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int T = Shape::kThreads, kPer = Shape::kPerThread, kCap = Shape::kCap;
  const SortLds<Shape> m(smem);
  uint32_t* const counts = reinterpret_cast<uint32_t*>(smem + Shape::kLds);            // [max_ranges]
  float* const lower = reinterpret_cast<float*>(smem + Shape::kLds + 4 * kMaxSplit);   // [max_ranges + 3], the last -inf
  uint32_t* const taken = m.misc + 52;
  uint64_t* const regions = sc.pairs + (int64_t)blockIdx.x * sc.max_ranges * kCap;
  for (;;) {
    if (threadIdx.x == 0) *taken = atomicAdd(&sc.ticket[0], 1u);
    __syncthreads();
    const int idx = (int)uniform(*taken);
    if (idx >= nrows) break;
    const int zh = idx % (a.Z * a.H), n = a.N - 1 - idx / (a.Z * a.H);
    const int len = (int)kv_row_len(n, a.S, a.L, a.non_causal), nr = row_ranges(len, kCap);
    const int64_t base = row_base(a, zh, n), row_id = (int64_t)zh * a.N + n;
    const float* const sk = (a.s_k ? a.s_k : sc.sk) + base;
    const float* const thr = sc.thr + row_id * (sc.max_ranges + 2);
    if (nr > 1) split_row<Shape>(m, counts, lower, sk, len, nr, thr, regions);
    int rank = 0;                                // first rank of the range
    for (int r = 0; r < nr; ++r) {
      const int tid = fresh(threadIdx.x);
      const int count = nr > 1 ? (int)uniform(counts[r]) : len;
      if (count > kCap) {
        if (tid == 0) sc.left_over[atomicAdd(&sc.ticket[1], 1u)] = make_int2((int)((uint32_t)row_id | ((uint32_t)r << 24)), rank + count);
      } else if (count > 0) {
        float f[kPer], fa = 0.f, fb = 0.f;
        uint32_t tok[kPer];
        const bool bounded = r > 0 && r < nr - 1;
        if (bounded) { fa = lower[r - 1]; fb = lower[r]; }
        __syncthreads();                         // the previous keys are out of LDS
        if (nr > 1) {
          const uint64_t* const src = regions + (int64_t)r * kCap;
#pragma unroll
          for (int e = 0; e < kPer; ++e) {
            const uint64_t x = src[tid + e * T]; // (whatever lies past the count is not looked at)
            f[e] = pair_score(x);
            tok[e] = pair_token(x);
          }
        } else {                                 // the whole row fits
#pragma unroll
          for (int e = 0; e < kPer; ++e) {
            const int i = tid + e * T;
            tok[e] = (uint32_t)i;
            f[e] = sort_score(sk[min(i, len - 1)]);
          }
        }
        block_sort<Shape>(m, count, f, tok, bounded, fb, fa, a.kv_perm + base + rank);
      }
      rank += count;
    }
    if (rank != len && threadIdx.x == 0) raise(a, 2u);
    __syncthreads();                             // the ticket word may be written again
  }
}

// Ranks the rows of KV_perm, one (row, score range) after the other.  Range r of a row holds the
// scores s with thr[r] <= s < thr[r-1] (the first range has no upper end, the last one takes
// all the rest, NaN included).
//
// kWhole     every row fits one sort.  Nothing but the row itself is read, so the rows go to the workgroups in order of
//            their length, longest first, there and back.  (As pairs of a long and a short one on one XCD, as a scan's
//            pieces go, some workgroups had four rows where others had two: whole ranking, us, pairs / there and back,
//            32 heads, 7360 tokens in 320 63.7 / 56.6, 8K in 256 80 / 74, 12K in 512 83.6 / 77.2, 12 heads 54.4 / 45.0.)
// kScan      a range's keys are collected by scanning the row (two comparisons per score); the
//            number of keys above the range, counted on the way, is its first rank.
// kLeftOver  the same for the ranges that split_sort_kernel has listed: normally none.
//
// What bounds it: LDS and vector instructions; a scan reads the row from L2.  A workgroup takes
// piece after piece: a new workgroup could only start at an old one's end.
enum RowMode { kWhole, kScan, kLeftOver };

template <class Shape, RowMode kMode>
__global__ __launch_bounds__(Shape::kThreads, 4) void row_sort_kernel(PlanArgs a, Scratch sc, int slots, int pairs) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int T = Shape::kThreads, kPer = Shape::kPerThread, kCap = Shape::kCap;
  constexpr int kVec = 4, kTrip = 4 * kVec * T;  // 16-byte loads per thread and trip of a scan, scores per trip
  constexpr uint32_t kBottom = 0x007fffffu, kTop = 0xff800001u;   // ordered_u32: -inf; one past +inf
  const SortLds<Shape> m(smem);
  const float* const scores = a.s_k ? a.s_k : sc.sk;
  const int xcd = (int)blockIdx.x & 7;
  // items of all workgroups, or of this XCD's (kScan)
  const int ZH = a.Z * a.H, nrows = a.non_causal ? ZH * a.N : ZH * (a.N - 1);
  const int nitems = kMode == kLeftOver ? (int)uniform(sc.ticket[1]) : kMode == kWhole ? nrows : (ZH * pairs + 7) / 8 * slots;
  const int stride = kMode == kScan ? (int)gridDim.x >> 3 : (int)gridDim.x;
  uint32_t* const cursor = m.misc + 50;          // keys collected
  uint32_t* const nabove = m.misc + 51;          // keys above the range
  for (int first_idx = 0; first_idx < nitems; first_idx += stride) {
    int idx = first_idx + (kMode == kScan ? (int)blockIdx.x >> 3 : (int)blockIdx.x);
    if (kMode == kWhole && (first_idx / stride & 1) != 0) idx = first_idx + stride - 1 - (int)blockIdx.x;
    if (idx >= nitems) continue;
    RowItem cur;
    int end = 0;                                 // rank behind the range, as the splitter counted it
    if (kMode == kLeftOver) {
      const int2 it = sc.left_over[idx];
      const uint32_t at = uniform((uint32_t)it.x);
      const int n = (int)(at & 0xffffffu) % a.N;
      cur.row_id = (int64_t)(at & 0xffffffu);
      cur.r = (int)(at >> 24);
      end = (int)uniform((uint32_t)it.y);
      cur.len = (int)kv_row_len(n, a.S, a.L, a.non_causal);
      cur.nr = row_ranges(cur.len, kCap);
      cur.base = row_base(a, cur.row_id / a.N, n);
      cur.valid = true;
    } else if (kMode == kWhole) {
      const int n = a.N - 1 - idx / ZH, zh = idx % ZH;
      cur.len = (int)kv_row_len(n, a.S, a.L, a.non_causal);
      cur.r = 0; cur.nr = 1;
      cur.base = row_base(a, zh, n);
      cur.row_id = (int64_t)zh * a.N + n;
      cur.valid = true;
    } else {
      cur = row_item(a, sc, slots, pairs, xcd, idx);
    }
    if (!cur.valid) continue;
    const float* const sk = scores + cur.base;
    int32_t* const out = a.kv_perm + cur.base;
    const int len = cur.len, nr = kMode == kWhole ? 1 : cur.nr;
    const bool last = cur.r == nr - 1;
    // the range as [lo, hi) in the order of ordered_u32 (one past +inf: no upper end)
    uint32_t range_lo = kBottom, hi = kTop;
    if (kMode != kWhole) {
      const float* const thr = sc.thr + cur.row_id * (sc.max_ranges + 2);
      if (!last) range_lo = uniform(ordered_u32(thr[cur.r]));
      if (cur.r > 0) hi = max(uniform(ordered_u32(thr[cur.r - 1])), range_lo);
    }
    uint32_t lo = range_lo;
    // The whole range at once; if its keys do not fit, its upper part first.
    for (bool more = hi > lo || last; more; more = hi > lo) {
      const int tid = fresh(threadIdx.x), lane = tid & 63;
      float f[kPer];
      uint32_t tok[kPer];
      int count = len, first = 0;
      const bool bounded = hi != kTop && lo != kBottom;
      const float fa = hi == kTop ? __uint_as_float(0x7fc00000u) : ordered_to_float(hi);   // s >= NaN is false
      const float fb = ordered_to_float(lo);
      __syncthreads();                           // the previous keys are out of LDS
      if (nr == 1) {                             // the whole row fits
#pragma unroll
        for (int e = 0; e < kPer; ++e) {
          const int i = tid + e * T;
          tok[e] = (uint32_t)i;
          f[e] = sort_score(sk[min(i, len - 1)]);
        }
        hi = lo;
      } else if (kMode != kWhole) {
        f32x4 v[kVec];
        auto load = [&](f32x4 (&x)[kVec], int t0) {
          const int tid_ = fresh(threadIdx.x);
#pragma unroll
          for (int q = 0; q < kVec; ++q)
            x[q] = *reinterpret_cast<const f32x4*>(sk + min(t0 + 4 * (q * T + tid_), len - 4));
        };
        load(v, 0);
        if (tid == 0) { *cursor = 0u; *nabove = 0u; }
        __syncthreads();
        const uint64_t rest = lo == kBottom && last ? ~0ull : 0ull;   // the last part takes NaN scores, too
        const uint32_t list_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)m.list;
        uint32_t above = 0;
        // one trip: compare, rank the hits among the wavefront's, append them
        auto trip = [&](int t0, auto whole_, auto last_) {
          constexpr bool kWhole = decltype(whole_)::value, kLast = decltype(last_)::value;
          uint64_t in[kVec][4];
          uint32_t mine = 0;
#pragma unroll
          for (int q = 0; q < kVec; ++q) {
            const uint64_t valid = kWhole ? ~0ull : __builtin_amdgcn_ballot_w64(t0 + 4 * (q * T + tid) < len);
            uint64_t up[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              up[e] = __builtin_amdgcn_ballot_w64(v[q][e] >= fa) & valid;
              if (kLast) in[q][e] = ~up[e] & valid;   // NaN scores, too
              else in[q][e] = __builtin_amdgcn_ballot_w64(v[q][e] >= fb) & valid & ~up[e];
            }
            // Per-lane counts, one more where the lane's bit is set: additions with the mask as carry.
            // A vector instruction may read a mask two wait states after the comparison that wrote it,
            // and a data-parallel move a register two after the addition that did; the compiler keeps
            // neither for a text, so the text idles at both ends.  (Left to the compiler the additions
            // are two selects and an addition for two masks.)
            asm("s_nop 1\n\t"
                "v_addc_co_u32 %[up], vcc, 0, %[up], %[u0]\n\t"
                "v_addc_co_u32 %[in], vcc, 0, %[in], %[i0]\n\t"
                "v_addc_co_u32 %[up], vcc, 0, %[up], %[u1]\n\t"
                "v_addc_co_u32 %[in], vcc, 0, %[in], %[i1]\n\t"
                "v_addc_co_u32 %[up], vcc, 0, %[up], %[u2]\n\t"
                "v_addc_co_u32 %[in], vcc, 0, %[in], %[i2]\n\t"
                "v_addc_co_u32 %[up], vcc, 0, %[up], %[u3]\n\t"
                "v_addc_co_u32 %[in], vcc, 0, %[in], %[i3]\n\t"
                "s_nop 1"
                : [up] "+v"(above), [in] "+v"(mine)
                : [u0] "s"(up[0]), [u1] "s"(up[1]), [u2] "s"(up[2]), [u3] "s"(up[3]),
                  [i0] "s"(in[q][0]), [i1] "s"(in[q][1]), [i2] "s"(in[q][2]), [i3] "s"(in[q][3])
                : "vcc");
          }
          const uint32_t incl = wave_inclusive_sum(mine);
          const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
          uint32_t at = 0;
          if (lane == 0) at = atomicAdd(cursor, total);
          at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
          if (at + total > (uint32_t)kCap) return;   // the count says so
          uint32_t dst = list_lds + 8u * (at + incl - mine), t = (uint32_t)(t0 + 4 * tid);
#pragma unroll
          for (int q = 0; q < kVec; ++q) {
            // (score, token) pairs from every lane of each mask, to the lane's next place
            uint32_t tk;
            asm volatile(
                "s_mov_b64 exec, %[i0]\n\t"
                "v_add_u32 %[tk], %[d], %[t]\n\t"
                "ds_write2_b32 %[dst], %[s0], %[tk] offset1:1\n\t"
                "v_add_u32 %[dst], 8, %[dst]\n\t"
                "s_mov_b64 exec, %[i1]\n\t"
                "v_add3_u32 %[tk], %[t], %[d], 1\n\t"
                "ds_write2_b32 %[dst], %[s1], %[tk] offset1:1\n\t"
                "v_add_u32 %[dst], 8, %[dst]\n\t"
                "s_mov_b64 exec, %[i2]\n\t"
                "v_add3_u32 %[tk], %[t], %[d], 2\n\t"
                "ds_write2_b32 %[dst], %[s2], %[tk] offset1:1\n\t"
                "v_add_u32 %[dst], 8, %[dst]\n\t"
                "s_mov_b64 exec, %[i3]\n\t"
                "v_add3_u32 %[tk], %[t], %[d], 3\n\t"
                "ds_write2_b32 %[dst], %[s3], %[tk] offset1:1\n\t"
                "v_add_u32 %[dst], 8, %[dst]\n\t"
                "s_mov_b64 exec, -1"
                : [dst] "+v"(dst), [tk] "=&v"(tk)
                : [i0] "s"(in[q][0]), [i1] "s"(in[q][1]), [i2] "s"(in[q][2]), [i3] "s"(in[q][3]), [t] "v"(t),
                  [s0] "v"(v[q][0]), [s1] "v"(v[q][1]), [s2] "v"(v[q][2]), [s3] "v"(v[q][3]), [d] "s"(4 * q * T)
                : "memory");
          }
        };
        auto scan = [&](auto last_) {
          int t0 = 0;
          for (; t0 + kTrip <= len; t0 += kTrip) {
            f32x4 w[kVec];                     // the next trip's scores are on their way during a trip
            load(w, t0 + kTrip);
            trip(t0, std::true_type{}, last_);
#pragma unroll
            for (int q = 0; q < kVec; ++q) v[q] = w[q];
          }
          if (t0 < len) trip(t0, std::false_type{}, last_);
        };
        if (lo == kBottom && last) scan(std::true_type{});
        else scan(std::false_type{});
        {
          const uint32_t sum = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_sum(above), 63);
          if (lane == 0) atomicAdd(nabove, sum);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the appended pairs, which the compiler does not know of
        __syncthreads();
        count = (int)uniform(*cursor);
        first = (int)uniform(*nabove);
        if (count > kCap && hi - lo > 1u) {    // too many: the upper half of the range
          lo += (hi - lo) / 2;
          continue;
        }
        if (count > kCap) {                    // more equal scores than fit: they keep their order
          uint32_t done = 0;
          for (int t1 = 0; t1 < len; t1 += T) {
            const int t = t1 + tid;
            const float s = t < len ? sk[t] : 0.f;
            const bool mine = t < len && !(s >= fa) && (s >= fb || rest != 0ull);
            const uint64_t hits = __builtin_amdgcn_ballot_w64(mine);
            if (lane == 0) m.misc[tid >> 6] = (uint32_t)__builtin_popcountll(hits);
            __syncthreads();
            uint32_t at = done + (uint32_t)__builtin_popcountll(hits & ((1ull << lane) - 1ull));
            for (int k = 0; k < T / 64; ++k) {
              const uint32_t c = m.misc[k];
              at += k < (tid >> 6) ? c : 0u;
              done += c;
            }
            if (mine && first + at < (uint32_t)len) out[first + at] = t;
            __syncthreads();
          }
        }
#pragma unroll
        for (int e = 0; e < kPer; ++e) {
          const uint64_t x = m.list[tid + e * T];   // (whatever lies past the count is not looked at)
          f[e] = sort_score(pair_score(x));
          tok[e] = pair_token(x);
        }
        __syncthreads();
        if (tid == 0 && ((rest != 0ull && first + count != len) || (kMode == kLeftOver && lo == range_lo && first + count != end)))
          raise(a, 2u);
        if (first + count > len) { raise(a, 8u); count = 0; }
        hi = lo;
        lo = range_lo;
      }
      if (count > 0 && count <= kCap) block_sort<Shape>(m, count, f, tok, bounded, fb, fa, out + first);
    }
  }
}

// ---------------------------------------------------------------------------------------
template <class Shape>
static int64_t sorts_per_cu() {
  const int64_t by_lds = 163840 / (int64_t)Shape::kLds, by_threads = 2048 / Shape::kThreads;
  return by_lds < by_threads ? by_lds : by_threads;
}

template <class Shape>
static void launch_whole_rows(const PlanArgs& a, const Scratch& sc, int cus, hipStream_t stream) {
  const int64_t rows = (int64_t)a.Z * a.H * (a.non_causal ? a.N : a.N - 1), fit = cus * sorts_per_cu<Shape>();
  hipLaunchKernelGGL((row_sort_kernel<Shape, kWhole>), dim3((unsigned)(rows < fit || fit < 1 ? rows : fit)),
                     dim3(Shape::kThreads), Shape::kLds, stream, a, sc, 1, 1);
}

static void launch_scan(const PlanArgs& a, const Scratch& sc, int cus, hipStream_t stream) {
  int slots = 1, pairs = a.N;
  if (a.non_causal) {
    slots = row_ranges(a.L, MidSort::kCap);
  } else {
    pairs = a.N / 2;                             // rows 1 .. N-1: (N-1, 1), (N-2, 2), ..., the middle one alone
    for (int p = 0; p < pairs; ++p) {
      const int hi = a.N - 1 - p, lo = 1 + p;
      const int k = row_ranges((int64_t)hi * a.S, MidSort::kCap) + (lo < hi ? row_ranges((int64_t)lo * a.S, MidSort::kCap) : 0);
      slots = k > slots ? k : slots;
    }
  }
  const int64_t per_xcd = ((int64_t)a.Z * a.H * pairs + 7) / 8 * slots;
  const int64_t fit = cus / 8 * sorts_per_cu<MidSort>();
  const int64_t groups = per_xcd < fit || fit < 1 ? per_xcd : fit;
  hipLaunchKernelGGL((row_sort_kernel<MidSort, kScan>), dim3((unsigned)(8 * groups)), dim3(MidSort::kThreads), MidSort::kLds,
                     stream, a, sc, slots, pairs);
}

static void launch_split_sort(const PlanArgs& a, const Scratch& sc, hipStream_t stream) {
  const int64_t rows = (int64_t)a.Z * a.H * (a.non_causal ? a.N : a.N - 1);
  hipLaunchKernelGGL(split_sort_kernel<MidSort>, dim3((unsigned)sc.groups),
                     dim3(MidSort::kThreads), MidSort::kLds + kSplitLds, stream, a, sc, (int)rows);
  hipLaunchKernelGGL((row_sort_kernel<MidSort, kLeftOver>), dim3(kSplitGroups), dim3(MidSort::kThreads), MidSort::kLds,
                     stream, a, sc, 1, 1);
}


// Small inputs: s_Q and its Argsort run beside the scores, k_guide beside q_mean -- one launch less
// in the chain, and the query sort out of it, for a second read of Q that the caches serve.  us for the whole
// ranking, sort in front / beside, 32 heads over 8 (20 is what the calls take): 64 rows of 512 23.8 / 19.2, 256 of 256
// 25.9 / 20.8, 256 of 512 29.8 / 26.2, 128 of 1024 31.9 / 31.6, 320 of 64 22.8 / 20.1, 384 of 128 24.3 / 20.3.  Alone it also gains
// a little beyond these lines (192 of 768 31.3 / 30.6, 256 of 768 36.3 / 35.3, 320 of 512 34.8 / 32.0; 256 of 1024 40.0 / 41.9), but
// a layer runs it beside the own-segment pass, where the larger second launch and the second read weigh more.  A
// layer up to its walk, 32, 8 and 4 heads: 320 rows of 64 0.95, 0.94, 0.96, of 128 0.97, 0.96, 0.94; on the other side
// 256 of 768 0.98, 1.01, 1.00, 512 of 256 0.98, 1.05, 1.00, 320 of 512 1.00, 0.98, 1.00.
constexpr int64_t kBesideRows = 384;
constexpr int64_t beside_queries(int64_t rows) { return rows <= kOneEach ? 1 << 17 : 1 << 16; }
using PoolSort512 = SortShape<256, 2>;

hipError_t launch_plan(const PlanArgs& a, hipStream_t stream) {
  const Scratch sc = carve(a.scratch, a.Z, a.H, a.Hkv, a.L, a.S, a.non_causal);
  if (sc.total > a.scratch_bytes) return hipErrorInvalidValue;
  const int64_t rows = (int64_t)a.Z * a.H * a.N;
  if (rows * (sc.max_ranges + 8) > 0x7fffffff || (sc.split && sc.max_ranges > kMaxSplit - 3)) return hipErrorInvalidValue;
  const int G = a.H / a.Hkv;
  int cus = 0;
  // dynamic LDS limits of the kernels that need more than the default
  {
    static std::mutex mu;
    static uint64_t done = 0;
    const hipError_t se = once_per_device(mu, done, [] {
      const struct { const void* f; size_t lds; } big[] = {
          {reinterpret_cast<const void*>(&pool_sq_sort_kernel<MidSort>), MidSort::kLds},
          {reinterpret_cast<const void*>(&pool_sq_sort_kernel<QuerySort>), QuerySort::kLds},
          {reinterpret_cast<const void*>(&row_sort_kernel<MidSort, kWhole>), MidSort::kLds},
          {reinterpret_cast<const void*>(&row_sort_kernel<MidSort, kScan>), MidSort::kLds},
          {reinterpret_cast<const void*>(&row_sort_kernel<MidSort, kLeftOver>), MidSort::kLds},
          {reinterpret_cast<const void*>(&split_sort_kernel<MidSort>), MidSort::kLds + kSplitLds},
          {reinterpret_cast<const void*>(&row_sort_kernel<Sort10K, kWhole>), Sort10K::kLds},
          {reinterpret_cast<const void*>(&row_sort_kernel<Sort4K, kWhole>), Sort4K::kLds},
          {reinterpret_cast<const void*>(&row_sort_kernel<Sort7K, kWhole>), Sort7K::kLds},
          {reinterpret_cast<const void*>(&row_sort_kernel<LargeSort, kWhole>), LargeSort::kLds}};
      static_assert(2 * (MidSort::kLds + kSplitLds) <= 163840, "two workgroups per CU");
      for (const auto& b : big) {
        const hipError_t e = hipFuncSetAttribute(b.f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)b.lds);
        if (e != hipSuccess) return e;
      }
      return hipSuccess;
    });
    if (se != hipSuccess) return se;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
  }

  const dim3 block(256);
  const int guide_blocks = a.Z * a.Hkv * kGuideParts;
  int64_t score_blocks = 0;
  if (a.N > 1 || a.non_causal) {
    const int RB = (G * a.N + 31) / 32;
    const int RBG = (RB + kScoreWaves - 1) / kScoreWaves;
    const int nchunks = (a.L + sc.chunk - 1) / sc.chunk;
    score_blocks = (int64_t)a.Z * a.Hkv * RBG * nchunks;
  }
  if (a.S <= SmallSort::kCap && rows <= kBesideRows && rows * a.S <= beside_queries(rows)) {
    hipLaunchKernelGGL(mean_guide_kernel, dim3((unsigned)(rows + guide_blocks)), block, kMeanLds, stream, a, sc, (int)rows);
    const dim3 grid((unsigned)(rows + score_blocks));
    if (a.S <= PoolSort512::kCap)
      hipLaunchKernelGGL(score_sort_kernel<PoolSort512>, grid, block, kScoreLds, stream, a, sc, (int)rows);
    else
      hipLaunchKernelGGL(score_sort_kernel<SmallSort>, grid, block, kScoreLds, stream, a, sc, (int)rows);
  } else {
    hipLaunchKernelGGL(kguide_kernel, dim3(guide_blocks), block, 0, stream, a, sc);
    const dim3 grid((unsigned)rows);
    if (a.S <= PoolSort512::kCap)
      hipLaunchKernelGGL(pool_sq_sort_kernel<PoolSort512>, grid, block, PoolSort512::kLds, stream, a, sc);
    else if (a.S <= SmallSort::kCap)
      hipLaunchKernelGGL(pool_sq_sort_kernel<SmallSort>, grid, block, SmallSort::kLds, stream, a, sc);
    // Above 2048 queries 512 threads sort: with 256 and 32 keys each there is about one bucket per key,
    // and from 5.4K queries on the list of keys that share one overflows into the bitonic network.  32
    // segments of 4096 88 -> 78 us, of 5632 277 -> 105, of 8192 326 -> 149; 2048 of 5632 1426 -> 687.
    else if (a.S <= MidSort::kCap)
      hipLaunchKernelGGL(pool_sq_sort_kernel<MidSort>, grid, dim3(MidSort::kThreads), MidSort::kLds, stream, a, sc);
    else
      hipLaunchKernelGGL(pool_sq_sort_kernel<QuerySort>, grid, dim3(QuerySort::kThreads), QuerySort::kLds, stream, a, sc);
    if (score_blocks > 0)
      hipLaunchKernelGGL(score_kernel, dim3((unsigned)score_blocks), dim3(64 * kScoreWaves), kScoreLds, stream, a, sc);
  }
  if (score_blocks > 0) {
    if (sc.max_ranges > 1)
      hipLaunchKernelGGL(threshold_kernel, dim3((unsigned)rows), dim3(256), 0, stream, a, sc);
    if (sc.max_ranges == 1) {
      const int64_t longest = a.non_causal ? a.L : (int64_t)a.L - a.S;
      // With at most a row a CU, 1024 threads sort it; with more, two smaller workgroups share a CU where rows fit them.  Above
      // 6656 keys one sort has the CU whatever its shape, and the smallest that holds the rows has the fewest empty
      // turns.  Whole ranking, us, 32 heads unless said, in shapes of 2048, 6656 and 13312 keys only / with 4096, 7168
      // and 10240 as well: rows of 3584, a row a CU 27.0 / 26.6 (more rows 38.0 / 42.3: not taken), 6400 (16 rows, no causality) 27.8 / 25.8,
      // 7040 57.1 / 52.6, 7936 73.5 / 70.6, 8704 66.9 / 64.8, 9216 55.6 / 54.1.  Up to 6656 keys a workgroup of 1024
      // threads does not fit beside one of the own-segment pass, one of 512 does; a layer that runs the two at once shows nothing of
      // it.  22 layers with at most a row a CU, rows of 2560 to 6400 keys, captured in a graph, time in 1024 / in 512 threads: whole layer
      // 0.983 to 1.003 (8 heads, 6656 in 512 122.0 / 123.1 us, 32 heads, 4K in 512 153.6 / 155.3), up to its walk 0.983 to
      // 1.010, the ranking alone 0.960 to 0.997.
      const int64_t krows = (int64_t)a.Z * a.H * (a.non_causal ? a.N : a.N - 1);
      if (longest <= SmallSort::kCap) launch_whole_rows<SmallSort>(a, sc, cus, stream);
      else if (krows <= kOneEach && longest <= Sort4K::kCap) launch_whole_rows<Sort4K>(a, sc, cus, stream);
      else if (krows > kOneEach && longest <= MidSort::kCap) launch_whole_rows<MidSort>(a, sc, cus, stream);
      else if (longest <= Sort7K::kCap) launch_whole_rows<Sort7K>(a, sc, cus, stream);
      else if (longest <= Sort10K::kCap) launch_whole_rows<Sort10K>(a, sc, cus, stream);
      else launch_whole_rows<LargeSort>(a, sc, cus, stream);
    } else if (!sc.split) launch_scan(a, sc, cus, stream);
    else launch_split_sort(a, sc, stream);
  }
  return hipGetLastError();
}

}  // namespace s2o
