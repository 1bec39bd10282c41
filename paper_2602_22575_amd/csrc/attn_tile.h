// Per-wavefront building blocks shared by the S2O attention kernels for gfx950 (local.hip:
// own-segment pass, paper Alg. 2; prefix.hip: prefix walk, paper Alg. 3, and both in one launch):
// one wavefront = 32 query rows against one 64-token key tile staged in LDS.
//
// MFMA formulation (v_mfma_f32_16x16x32_bf16), transposed so that a query row lives in four
// lanes and the P operand of the second product comes from the first one's accumulators:
//   S^T[n, m] = sum_d K[n, d] Q[m, d]        A = K tile rows from LDS, B = Q from registers
//   O^T[d, m] = sum_n V^T[d, n] P^T[n, m]    A = V^T from LDS,        B = P from the S^T
//                                            accumulators (no data movement)
// Lane l = (m = l % 16, g = l / 16).  A 16x16 accumulator block holds, in register i of lane
// l, the element [row 4*g + i][column m]; a wavefront's 32 rows are two column blocks.  The B operand of
// the PV product takes registers 0..3 of two neighbouring S^T blocks as its 8 contraction slots, so slot (g, jj)
// is key 16*(jj/4) + 4*g + jj%4 of the 32-key step.
//
// Why this shape: a long walk is bound by the chip's power limit, and the 32x32x16 instruction reads and
// writes twice the accumulators for the same products.  Bare MFMAs on N(0,1) operands at that limit: 16x16x32
// 2000 to 2090 TFLOP/s, 32x32x16 1800 to 1860 (zero operands: 2475 both).  An operand fragment out of LDS is 1 KB and feeds two
// instructions where it fed one: the LDS traffic is the same.  The kernels' times with this and the read order
// below / with 32x32x16, same card: contiguous 8K x 32 heads 848 / 907 us, 32K causal without a stop rule
// 6470 / 6940, at 5e-3 1151 / 1193, own segments of 1024 tokens at 16K 186 / 217.  In cycles it costs: twice the
// products to issue, and less vector work beside them.  On zero data, which draws little power, 8K contiguous 650 / 632,
// causal walks at 1e-37 8K 374 / 361, 32K 5665 / 5429, 128K 101.2 / 90.0 ms (without votes 96.2 / 89.5), single launch
// 32K 6563 / 6193, own segments 128K 1896 / 1844; on Gaussian data where a CU has a workgroup or two of short runs: own
// segments alone, one head, 4K in 1024 25.5 / 24.6, 4 heads, 8K in 1024 27.3 / 26.3, 32 heads, 8K in 64 47.5 / 45.9 (in 256
// 47.2 / 48.4, in 1024 94.8 / 98.5).
//
// K and V tiles sit row-major (token rows of 256 bytes) in LDS, written there directly by
// global_load_lds (no staging registers): a wavefront instruction deposits 4 gathered rows
// as 1 KB, lane l at byte 16*l, so rows cannot be padded; bank conflicts are avoided by an XOR
// swizzle instead: the sixteen 16-byte chunks of row r are stored at slot chunk ^ swz(r)
// (each lane fetches, from global memory, the chunk that belongs at its LDS slot), with
// swz(r) = 4*(r%4) + 2*((r/4 + r/8)%2) + (r/8)%2: the 16 rows that 16 lanes of a K read touch land on 16
// different chunks, also where the hardware takes rows 0..3, 12..15 of one chunk and 4..11 of the next together, and so do
// the 8 rows x 32 bytes that half a wavefront touches in a transposing V read.  (The counter of bank conflicts at 128K, 5e-3: 0 in the
// own-segment pass and 8e6 clocks in the walk; with 2*((r/4)%2) in the middle 1.4e8 and 3.6e8, and the walk 1.00 to 1.015 of the time.)
// The K operand is a plain 16-byte read of a row; the V^T operand is read with the
// transposing LDS load ds_read_b64_tr_b16: within each group of 16 lanes, lane i receives
// element (i % 4) of the four 8-byte rows pointed to by lanes i/4, 4 + i/4, 8 + i/4 and
// 12 + i/4, so pointing lane r of group g at (key 4*g + r/4, dims 4*(r%4)..+3) hands every
// lane the four keys of its contraction slots at its own head dimension.
//
// Online softmax: logits are kept in base-2 units (raw score * softmax_scale * log2 e).
// m_ref is the reference maximum the accumulated terms are expressed in; it follows the true
// running maximum lazily: terms are only rescaled when the maximum has grown by more than
// kLazy (2^8), so that in the common case a tile costs no pass over the accumulator.  Any
// reference gives the same result; tile masses and the stop test are ratios in one common
// reference.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace s2o {
namespace tile {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(1))) void gvoid;
typedef __attribute__((address_space(3))) void lvoid;

constexpr int kD = 128;                  // head dim
constexpr int kBN = 64;                  // key tile
constexpr int kRowsPerWave = 32;         // query rows of one wavefront
constexpr int kRowElems = kD;            // K and V rows sit unpadded in LDS (256 B)
constexpr int kTileElems = kBN * kRowElems;
constexpr int kBlockBytes = 16 * kRowElems * 2;   // 16 rows of a tile
constexpr float kLazy = 8.0f;

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  bf16x2 t = {(__bf16)lo, (__bf16)hi};
  return __builtin_bit_cast(uint32_t, t);
}

__device__ __forceinline__ int swz(int r) { return ((r & 3) << 2) | ((((r >> 2) ^ (r >> 3)) & 1) << 1) | ((r >> 3) & 1); }

// Byte offset, inside its 256-byte global row, of the chunk that lane `lane` of a 4-row load
// instruction must fetch so that it lands at the right (swizzled) LDS slot; `row0` is the
// first of the 4 tile rows the instruction covers (lane l covers row row0 + l/16).
__device__ __forceinline__ int load_chunk_offset(int lane, int row0) {
  return 16 * ((lane & 15) ^ swz(row0 + (lane >> 4)));
}

// One 4-row load instruction: 64 lanes x 16 bytes from global memory straight into LDS.
__device__ __forceinline__ void load_rows_to_lds(const char* lane_src, uint16_t* lds_row0) {
  __builtin_amdgcn_global_load_lds((const gvoid*)lane_src, (lvoid*)lds_row0, 16, 0, 0);
}

// Q fragments of a lane's two rows (16 apart in the wavefront): dims 32*kk + 8*g .. +8 for the 4 contraction steps.
__device__ __forceinline__ void load_q(const uint16_t* qrow0, const uint16_t* qrow1, int g, bf16x8 (&qf)[4][2]) {
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    qf[kk][0] = *reinterpret_cast<const bf16x8*>(qrow0 + 32 * kk + 8 * g);
    qf[kk][1] = *reinterpret_cast<const bf16x8*>(qrow1 + 32 * kk + 8 * g);
  }
}

// ---------------------------------------------------------------------------------------
// Explicitly scheduled operand reads.
//
// The compiler cannot tell an LDS read of one tile buffer from the asynchronous global->LDS
// load that is filling another, so it drains every outstanding global load (s_waitcnt
// vmcnt(0)) before any LDS read it knows about: a tile fetch issued at the top of a step
// would be waited for at the step's first operand read, with the whole memory latency
// exposed.  The operand reads below are therefore issued from inline assembly, which the
// compiler's wait insertion does not look into, and every fragment is handed to its MFMA
// through an explicit `s_waitcnt lgkmcnt(n)` that names how many younger LDS reads may still be
// in flight (LDS reads complete in order).  The kernels wait for their own tile fetches
// themselves (wait_fetches) right before the barrier that publishes a tile.
//
// Addresses: one VGPR per fragment slot (the swizzle makes them lane-dependent), fixed for the
// whole kernel; tile buffer and sub-block are selected with the instruction's immediate offset.
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

__device__ __forceinline__ uint32_t lds_address(const void* p) { return (uint32_t)(uintptr_t)(lvoid*)p; }

template <int kOff>
__device__ __forceinline__ void lds_issue_b128(bf16x8& d, uint32_t addr) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(d) : "v"(addr), "n"(kOff) : "memory");
}
template <int kOff>
__device__ __forceinline__ void lds_issue_tr64(u32x2& d, uint32_t addr) {
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(d) : "v"(addr), "n"(kOff) : "memory");
}
// All global->LDS tile loads (and every other global load) of this wavefront have landed.
__device__ __forceinline__ void wait_tile_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// The same wait, for all but the kYoungest most recent vector-memory instructions of the
// wavefront (they complete in order), through the builtin, so that the compiler's own bookkeeping
// of outstanding loads sees it.
template <int kYoungest>
__device__ __forceinline__ void wait_fetches() {
  // s_waitcnt immediate: vmcnt in bits 3..0 and 15..14, every other counter left at its maximum
  __builtin_amdgcn_s_waitcnt((kYoungest & 15) | ((kYoungest >> 4) << 14) | 0x0f70);
  asm volatile("" ::: "memory");
}

// acc += a * b (kFirst: acc = a * b), the first product of a fragment behind its wait: the fragment is there once at
// most kYounger LDS reads issued after it are outstanding.  With the builtin the
// compiler is free to give the result registers of its own, which costs a copy of the 64-register O^T per key tile,
// and to move products away from the reads they stand between; in assembly the operand is tied.
// The compiler then no longer sees an MFMA and inserts no wait states around it.  In front: an
// MFMA must not read a register in the two issue slots after a VALU instruction wrote it, and
// the compiler does place moves of the operands right before the statement -- hence the wait and the idle
// slot (a second product's operands have passed the first one's).  Behind: the next MFMA on the same
// accumulator needs none; before anything else reads or writes it, mfma_settle() must have run or
// as much other work lie between.
template <int kYounger, bool kFirst>
__device__ __forceinline__ void mfma_wait(f32x4& acc, const bf16x8& a, const bf16x8& b) {
  if constexpr (kFirst)
    asm volatile("s_waitcnt lgkmcnt(%3)\n\ts_nop 0\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(acc) : "v"(a), "v"(b), "n"(kYounger));
  else
    asm volatile("s_waitcnt lgkmcnt(%3)\n\ts_nop 0\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b), "n"(kYounger));
}
template <bool kFirst>
__device__ __forceinline__ void mfma_next(f32x4& acc, const bf16x8& a, const bf16x8& b) {
  if constexpr (kFirst) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(acc) : "v"(a), "v"(b));
  else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}

// Byte addresses of a lane's operand fragments inside a tile that starts at LDS address `base`
// (a multiple of 256).  The swizzle is an XOR on the 16-byte chunk index, i.e. on address bits
// 4..7, so the slots follow from one address each by an XOR with a constant: K step kk =
// k[0] ^ (kk << 6), V dims block db = v[0] ^ (db << 5).  All twelve are kept: an XOR at the point of
// use sits between the read and the MFMA that waits for it.
struct OperandAddr {
  uint32_t k[4];      // K operand of contraction step kk, keys 0..15 (next 16: + kBlockBytes)
  uint32_t v[8];      // V^T operand: [16-dim block], keys 0..15 (next 16: + kBlockBytes)
  __device__ __forceinline__ void init(int lane, uint32_t base) {
    const int m_ = lane & 15, g = lane >> 4;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) k[kk] = (base + 2u * (uint32_t)(m_ * kRowElems + 8 * (g ^ swz(m_)))) ^ (uint32_t)(kk << 6);
    // lane r of group g points at key 4*g + r/4, dims 4*(r%4)..+3
    const int rl = 4 * g + (m_ >> 2);
#pragma unroll
    for (int db = 0; db < 8; ++db)
      v[db] = (base + 2u * (uint32_t)(rl * kRowElems + 8 * (((m_ & 3) >> 1) ^ swz(rl)) + 4 * (m_ & 1))) ^ (uint32_t)(db << 5);
  }
  // the same fragments in a tile kb / vb bytes further on (multiples of 256; may be "negative")
  __device__ __forceinline__ void shift(uint32_t kb, uint32_t vb) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) k[kk] += kb;
#pragma unroll
    for (int db = 0; db < 8; ++db) v[db] += vb;
  }
  __device__ __forceinline__ OperandAddr at(uint32_t kb, uint32_t vb) const {
    OperandAddr r = *this;
    r.shift(kb, vb);
    return r;
  }
};

constexpr int kTileBytes = kTileElems * 2;          // 16 KB
constexpr int kVStepBytes = 2 * kBlockBytes;        // one 32-key contraction step of a V tile

// The 16 K-fragment reads and 32 V^T-fragment reads of one step form one issue sequence (K
// fragments in pairs p = 2*kk + (32-key half), then V fragments c = 8*st + db of two reads each), so that the
// first V fragments are already on their way while the last score MFMAs run:
//   the K reads of the pairs 0..kKAhead-1 up front; after the MFMAs of pair p the K reads of pair
//   p + kKAhead, or, once those are exhausted, the reads of two V fragments; the PV product
//   starts by requesting the rest of the first kVAhead V fragments and then, after the MFMAs
//   of fragment c, requests fragment c + kVAhead.
// A fragment feeds two MFMAs of 16 clocks, and a wavefront waits with its second until the first has gone into
// the pipe: a read stands behind each of them, not two behind both (contiguous 8K x 32 heads 0.98 of the time, on
// zero data 0.95).  3 and 6 or 4 and 8 ahead: 1.00 to 1.02 of the time.
// While its products run, a wavefront has priority over the other one of its SIMD, which is in its softmax or
// at a barrier then: walk at 1e-3, 32K, 0.98 of the time, own-segment pass 0.97; without a stop rule 1.00.  (The other way round
// 0.98, 0.99, 1.01.)
constexpr int kKAhead = 2;     // pairs of K fragments in flight
constexpr int kVAhead = 4;     // V fragments in flight (2 transposing reads each)
constexpr int kVEarly = 2 * kKAhead;   // V fragments requested during the score MFMAs
constexpr int kProductPriority = 1;

// LDS reads issued before the score MFMAs of pair p wait for their fragments
constexpr int issued_at_qk(int p, bool with_v) {
  const int k_reads = 2 * (p + kKAhead < 8 ? p + kKAhead : 8);
  const int v_frags = with_v && p + kKAhead > 8 ? 2 * (p + kKAhead - 8) : 0;
  return k_reads + 2 * v_frags;
}

template <int kKOff, int p, int e>
__device__ __forceinline__ void issue_k_fragment(const OperandAddr& oa, bf16x8 (&ka)[8][2]) {
  lds_issue_b128<kKOff + (2 * (p & 1) + e) * kBlockBytes>(ka[p][e], oa.k[p >> 1]);
}
template <int kKOff, int p>
__device__ __forceinline__ void issue_k_pair(const OperandAddr& oa, bf16x8 (&ka)[8][2]) {
  issue_k_fragment<kKOff, p, 0>(oa, ka);
  issue_k_fragment<kKOff, p, 1>(oa, ka);
}
template <int kVOff, int c, int e>
__device__ __forceinline__ void issue_v_half(const OperandAddr& oa, u32x2 (&vf)[16][2]) {
  lds_issue_tr64<kVOff + (c >> 3) * kVStepBytes + e * kBlockBytes>(vf[c][e], oa.v[c & 7]);
}
template <int kVOff, int c>
__device__ __forceinline__ void issue_v_fragment(const OperandAddr& oa, u32x2 (&vf)[16][2]) {
  issue_v_half<kVOff, c, 0>(oa, vf);
  issue_v_half<kVOff, c, 1>(oa, vf);
}

// The K reads of the first kKAhead pairs of the K tile at byte offset kKOff from the addresses in `oa`.  A caller
// may have other work between these and qk_tile_begun, but `ka` is in flight there while the compiler takes it as
// loaded: no instruction may touch it, not even a copy or a spill.  So that work must be short and far from the
// limit of the registers.  (LDS reads in between do no harm: they complete in order, and the waits are only
// stricter for them.)  tests/test_asm_reads_in_flight.py looks for such instructions in the built code.
template <int kKOff>
__device__ __forceinline__ void qk_tile_begin(const OperandAddr& oa, bf16x8 (&ka)[8][2]) {
  static_for<0, kKAhead>([&](auto p_) { issue_k_pair<kKOff, decltype(p_)::value>(oa, ka); });
}
// S^T = K Q^T for that tile, its first reads requested by qk_tile_begin.  kWithV: also
// start the V^T reads of fragments 0..kVEarly-1 of the V tile at byte offset kVOff.
template <int kKOff, int kVOff, bool kWithV>
__device__ __forceinline__ void qk_tile_begun(const OperandAddr& oa, const bf16x8 (&qf)[4][2], f32x4 (&s)[4][2],
                                              u32x2 (&vf)[16][2], bf16x8 (&ka)[8][2]) {
  __builtin_amdgcn_s_setprio(kProductPriority);
  static_for<0, 8>([&](auto p_) {
    constexpr int p = decltype(p_)::value, kk = p >> 1, kb = 2 * (p & 1);
    constexpr int kYounger = issued_at_qk(p, kWithV) - (2 * p + 2);
    // (one read, or two of a V fragment, behind the first and behind the third product)
    auto issue = [&](auto e_) {
      constexpr int e = decltype(e_)::value;
      if constexpr (p + kKAhead < 8) issue_k_fragment<kKOff, p + kKAhead, e>(oa, ka);
      else if constexpr (kWithV) issue_v_fragment<kVOff, 2 * (p + kKAhead - 8) + e>(oa, vf);
    };
    mfma_wait<kYounger, kk == 0>(s[kb][0], ka[p][0], qf[kk][0]);
    issue(std::integral_constant<int, 0>{});
    mfma_next<kk == 0>(s[kb][1], ka[p][0], qf[kk][1]);
    mfma_next<kk == 0>(s[kb + 1][0], ka[p][1], qf[kk][0]);
    issue(std::integral_constant<int, 1>{});
    mfma_next<kk == 0>(s[kb + 1][1], ka[p][1], qf[kk][1]);
  });
  if constexpr (!kWithV) {
    __builtin_amdgcn_s_setprio(0);
    asm volatile("s_nop 15\n\ts_nop 3"
                 : "+v"(s[0][0]), "+v"(s[0][1]), "+v"(s[1][0]), "+v"(s[1][1]), "+v"(s[2][0]), "+v"(s[2][1]), "+v"(s[3][0]), "+v"(s[3][1]));
  }
}
template <int kKOff, int kVOff, bool kWithV>
__device__ __forceinline__ void qk_tile_sched(const OperandAddr& oa, const bf16x8 (&qf)[4][2], f32x4 (&s)[4][2],
                                              u32x2 (&vf)[16][2]) {
  bf16x8 ka[8][2];
  qk_tile_begin<kKOff>(oa, ka);
  qk_tile_begun<kKOff, kVOff, kWithV>(oa, qf, s, vf, ka);
}
// The results of all products are in their registers.
__device__ __forceinline__ void mfma_settle(f32x4 (&o)[2][8]) {
  asm volatile("s_nop 15\n\ts_nop 3"
               : "+v"(o[0][0]), "+v"(o[0][1]), "+v"(o[0][2]), "+v"(o[0][3]), "+v"(o[0][4]), "+v"(o[0][5]), "+v"(o[0][6]),
                 "+v"(o[0][7]), "+v"(o[1][0]), "+v"(o[1][1]), "+v"(o[1][2]), "+v"(o[1][3]), "+v"(o[1][4]), "+v"(o[1][5]),
                 "+v"(o[1][6]), "+v"(o[1][7]));
}

// O^T += V^T P^T.  kEarly: fragments 0..kVEarly-1 were requested by qk_tile_sched; the softmax of the step then
// stands between these products and whatever touches O^T next.
template <int kVOff, bool kEarly>
__device__ __forceinline__ void pv_tile_sched(const OperandAddr& oa, const bf16x8 (&pb)[2][2], f32x4 (&o)[2][8],
                                              u32x2 (&vf)[16][2]) {
  if constexpr (!kEarly) __builtin_amdgcn_s_setprio(kProductPriority);
  static_for<(kEarly ? kVEarly : 0), kVAhead>([&](auto c_) { issue_v_fragment<kVOff, decltype(c_)::value>(oa, vf); });
  static_for<0, 16>([&](auto c_) {
    constexpr int c = decltype(c_)::value, st = c >> 3, db = c & 7;
    // V reads issued so far: fragments 0..kVAhead-1 and fragment c' + kVAhead after every earlier c'
    constexpr int frags = (c + kVAhead < 16 ? c + kVAhead : 16);
    const u32x4 w = {vf[c][0].x, vf[c][0].y, vf[c][1].x, vf[c][1].y};
    const bf16x8 vfrag = __builtin_bit_cast(bf16x8, w);
    mfma_wait<2 * frags - (2 * c + 2), false>(o[0][db], vfrag, pb[st][0]);
    if constexpr (c + kVAhead < 16) issue_v_half<kVOff, c + kVAhead, 0>(oa, vf);
    mfma_next<false>(o[1][db], vfrag, pb[st][1]);
    if constexpr (c + kVAhead < 16) issue_v_half<kVOff, c + kVAhead, 1>(oa, vf);
  });
  __builtin_amdgcn_s_setprio(0);
  if constexpr (!kEarly) mfma_settle(o);
}

// The same two products alone, for a step with one of them.
template <int kKOff>
__device__ __forceinline__ void qk_tile_only(const OperandAddr& oa, const bf16x8 (&qf)[4][2], f32x4 (&s)[4][2]) {
  u32x2 none[16][2];
  qk_tile_sched<kKOff, 0, false>(oa, qf, s, none);
}
template <int kVOff>
__device__ __forceinline__ void pv_tile_only(const OperandAddr& oa, const bf16x8 (&pb)[2][2], f32x4 (&o)[2][8]) {
  u32x2 vf[16][2];
  pv_tile_sched<kVOff, false>(oa, pb, o, vf);
}

// A query row lives in the four lanes l % 16 + 16*{0..3}, which hold its values in pairs of rows 16
// apart.  Row statistics are kept by *home* lanes instead: lane l has those of the wavefront's row
// l % 16 + 16 * (l / 32) (two lanes each).  v_permlane32_swap exchanges the upper half of one register with
// the lower half of another: of (x0, x1), the values of the two rows, it makes the two that a home
// lane has to combine first; of (x, x) the home values of both rows in every lane.
// v_permlane16_swap does the same to the odd and even groups of 16 lanes.
__device__ __forceinline__ int home_row(int lane) { return (lane & 15) + 16 * (lane >> 5); }
__device__ __forceinline__ float row_max(float x0, float x1) {
  const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x0), __float_as_uint(x1), false, false);
  const float x = fmaxf(__uint_as_float(r.x), __uint_as_float(r.y));
  const u32x2 q = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(q.x), __uint_as_float(q.y));
}
__device__ __forceinline__ float row_sum(float x0, float x1) {
  const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x0), __float_as_uint(x1), false, false);
  const float x = __uint_as_float(r.x) + __uint_as_float(r.y);
  const u32x2 q = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(q.x) + __uint_as_float(q.y);
}
__device__ __forceinline__ void both_rows(int x, int (&r)[2]) {
  const u32x2 p = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)x, false, false);
  r[0] = (int)p.x; r[1] = (int)p.y;
}
__device__ __forceinline__ void both_rows(float x, float (&r)[2]) {
  const u32x2 p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  r[0] = __uint_as_float(p.x); r[1] = __uint_as_float(p.y);
}

// What a tile's score step hands to its PV step and to the row statistics.  All of the lane's home row, but
// the reference, which every lane needs for both of its rows.
struct TileStats {
  float alpha;     // factor that moves the old terms to the reference used for this tile (1 if unchanged)
  float mass;      // the tile's softmax mass, in that reference
  float prev;      // the row's mass so far, in that reference
  float m_use[2];  // the reference maximum used for this tile
  bool grow;       // the reference moved: the accumulator needs alpha
};

// Softmax numerators of a tile (left in s) and the row statistics.  kMask: apply the causal
// mask, the tile starting at key position key0 of the segment and the lane's home row being qoff.
template <bool kMask>
__device__ __forceinline__ TileStats softmax_tile(f32x4 (&s)[4][2], float c2, const float (&m_ref)[2], float l_run, int key0,
                                                  int qoff, int lane) {
  int q[2] = {0, 0};
  if (kMask) both_rows(qoff, q);
  float mx[2] = {-INFINITY, -INFINITY};
#pragma unroll
  for (int kb = 0; kb < 4; ++kb)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int kpos = key0 + 16 * kb + 4 * (lane >> 4) + i;
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) {
        if (kMask && kpos > q[cb]) s[kb][cb][i] = -INFINITY;     // CausalMask
        mx[cb] = fmaxf(mx[cb], s[kb][cb][i]);
      }
    }
  const float top = row_max(mx[0], mx[1]) * c2;
  const float m_old = lane < 32 ? m_ref[0] : m_ref[1];
  TileStats t;
  t.grow = top > m_old + kLazy;
  const float m_new = t.grow ? top : m_old;
  both_rows(m_new, t.m_use);
  float sum[2] = {0.f, 0.f};
#pragma unroll
  for (int kb = 0; kb < 4; ++kb)
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float pe = __builtin_amdgcn_exp2f(fmaf(s[kb][cb][i], c2, -t.m_use[cb]));
        s[kb][cb][i] = pe;
        sum[cb] += pe;
      }
  t.mass = row_sum(sum[0], sum[1]);
  t.alpha = t.grow ? __builtin_amdgcn_exp2f(m_old - m_new) : 1.0f;
  t.prev = l_run * t.alpha;
  return t;
}

// The common tile of a ranked walk raises no row's maximum by much, and then the reference does
// not move: the numerators can be formed against the current reference straight away, without
// the pass that finds the tile's maximum first (17 instructions and a cross-lane exchange that
// the exponentials would have to wait for).  Whether that was admissible shows in the mass
// itself: a numerator is at most the mass, so a mass of at most kMassLimit bounds every bf16
// P value and every accumulator term by it.  `redo` (a larger mass, an overflow to infinity, or
// a row that has no reference yet) tells the caller to score the tile again and take
// softmax_tile.
//
// The reference decides at which scale the bf16 rounding of P falls, so the limit is part of the
// result.  kMassLimit lets the reference lag by up to 2^16: the walk under the stop rule, but for the
// single launch.  The other loops (no stop rule, single launch) give the bits that softmax_tile gives
// for every tile: for them `redo` is already set by a mass above kSameMass, and confirm_redo drops it
// again unless some numerator is near 2^kLazy, where softmax_tile would move the reference.  (A
// row's mass is above kSameMass at every few tiles of a top-k walk; scoring all of these again cost
// 6 % of it.)
constexpr float kMassLimit = 65536.0f, kSameMass = 128.0f;
constexpr float kSameMax = 240.0f;       // 2^kLazy less the rounding of logits up to 2^16
static_assert(kLazy == 8.0f && 64.0f * kSameMax < kMassLimit, "kSameMax lies just below 2^kLazy");
__device__ __forceinline__ bool confirm_redo(const f32x4 (&s)[4][2], float mass) {
  float mx = 0.f;
#pragma unroll
  for (int kb = 0; kb < 4; ++kb)
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) mx = fmaxf(mx, s[kb][cb][i]);
  return !(mx <= kSameMax && mass <= kMassLimit);    // of any lane that holds a part of the row (NaN: confirmed)
}
template <bool kExactReference>
__device__ __forceinline__ TileStats softmax_tile_keep_reference(f32x4 (&s)[4][2], float c2, const float (&m_ref)[2],
                                                                 float l_run, bool& redo) {
  TileStats t;
  t.grow = false;
  t.m_use[0] = m_ref[0]; t.m_use[1] = m_ref[1];
  t.alpha = 1.0f;
  t.prev = l_run;
  float sum[2] = {0.f, 0.f};
#pragma unroll
  for (int kb = 0; kb < 4; ++kb)
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float pe = __builtin_amdgcn_exp2f(fmaf(s[kb][cb][i], c2, -m_ref[cb]));
        s[kb][cb][i] = pe;
        sum[cb] += pe;
      }
  t.mass = row_sum(sum[0], sum[1]);
  redo = !(t.mass <= (kExactReference ? kSameMass : kMassLimit));
  return t;
}

// P^T fragments (bf16) of both rows for the two 32-key contraction steps
__device__ __forceinline__ void pack_p(const f32x4 (&s)[4][2], bf16x8 (&pb)[2][2]) {
#pragma unroll
  for (int st = 0; st < 2; ++st)
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
      u32x4 w;
#pragma unroll
      for (int q = 0; q < 4; ++q) w[q] = pack_bf16x2(s[2 * st + (q >> 1)][cb][2 * (q & 1)], s[2 * st + (q >> 1)][cb][2 * (q & 1) + 1]);
      pb[st][cb] = __builtin_bit_cast(bf16x8, w);
    }
}

// rare: move the accumulator to a new reference maximum (O^T *= alpha)
__device__ __forceinline__ void rescale(f32x4 (&o)[2][8], float al, bool gr) {
  if (__builtin_amdgcn_ballot_w64(gr) != 0ull) {
    mfma_settle(o);
    float alpha[2];
    both_rows(al, alpha);
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int db = 0; db < 8; ++db)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          // in place: as plain C++ the products get registers of their own and the common path
          // (no rescale) pays for the merge with a copy of the whole accumulator per key tile
          float x = o[cb][db][i];
          asm volatile("v_mul_f32 %0, %1, %0" : "+v"(x) : "v"(alpha[cb]));
          o[cb][db][i] = x;
        }
  }
}

__device__ __forceinline__ void zero_acc(f32x4 (&o)[2][8]) {
#pragma unroll
  for (int cb = 0; cb < 2; ++cb)
#pragma unroll
    for (int db = 0; db < 8; ++db)
#pragma unroll
      for (int i = 0; i < 4; ++i) o[cb][db][i] = 0.f;
}

// State buffers: a row's accumulator is kept as 128 fp32 in the order of the head's dims = four 128-byte lines.
//
// lines_from_acc regroups the accumulators of a wavefront's 32 consecutive rows through two
// wavefront-private 4 KB LDS areas: afterwards lane L holds in acc_line(q, k) the 16-byte
// piece L % 8 of line q of row 8k + L / 8, and a store instruction of store_acc_lines writes 8
// whole lines.  Stored straight from the accumulator layout an instruction would put 64 bytes
// into each of 16 lines: the same bytes in twice as many write requests, which is what the
// own-segment pass then waits for.  (LDS serves a wavefront's accesses in order: the reads
// behind the writes need no wait of their own.)
__device__ __forceinline__ f32x4& acc_line(f32x4 (&o)[2][8], int q, int k) { return o[k >> 1][2 * q + (k & 1)]; }
__device__ __forceinline__ const f32x4& acc_line(const f32x4 (&o)[2][8], int q, int k) { return o[k >> 1][2 * q + (k & 1)]; }
__device__ __forceinline__ void lines_from_acc(f32x4 (&o)[2][8], uint32_t area0, uint32_t area1, int lane) {
  // LDS accesses in assembly, like the fragment reads: the compiler would put a wait for every
  // outstanding global load in front of them (it cannot tell them from a global->LDS load's target)
  const int m_ = lane & 15, g = lane >> 4, grp = lane >> 3, piece = lane & 7;
  // row r sits at line r ^ (r / 8 % 2), its pieces rotated by r: the 16 rows of a write land on 16 bank groups
  const uint32_t wr = (uint32_t)((m_ ^ (m_ >> 3)) * 128 + ((g ^ (m_ & 7)) << 4));
  const uint32_t rd = (uint32_t)(grp * 128 + ((piece ^ grp) << 4));
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int q = 2 * pass + half;
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int e = 0; e < 2; ++e)
          asm volatile("ds_write_b128 %0, %1" :: "v"((half ? area1 : area0) + 2048u * cb + (wr ^ (uint32_t)(e << 6))), "v"(o[cb][2 * q + e]) : "memory");
    }
    f32x4 r[2][4];
#pragma unroll
    for (int half = 0; half < 2; ++half)
#pragma unroll
      for (int k = 0; k < 4; ++k)
        asm volatile("ds_read_b128 %0, %1" : "=v"(r[half][k]) : "v"((half ? area1 : area0) + (rd ^ (uint32_t)((k & 1) << 7)) + 1024u * k) : "memory");
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(r[0][0]), "+v"(r[0][1]), "+v"(r[0][2]), "+v"(r[0][3]), "+v"(r[1][0]), "+v"(r[1][1]),
                   "+v"(r[1][2]), "+v"(r[1][3])
                 :: "memory");
#pragma unroll
    for (int half = 0; half < 2; ++half)
#pragma unroll
      for (int k = 0; k < 4; ++k) acc_line(o, 2 * pass + half, k) = r[half][k];
  }
}
// `wave_rows` = the accumulator state of the wavefront's first row; o as left by lines_from_acc.
__device__ __forceinline__ void store_acc_lines(float* wave_rows, const f32x4 (&o)[2][8], int lane) {
  float* p = wave_rows + (lane >> 3) * kD + (lane & 7) * 4;
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int k = 0; k < 4; ++k) *reinterpret_cast<f32x4*>(p + 8 * k * kD + 32 * q) = acc_line(o, q, k);
}
// sp0, sp1 = accumulator states of the lane's two rows + 4 * (lane / 16)
__device__ __forceinline__ void load_acc(const float* sp0, const float* sp1, f32x4 (&o)[2][8]) {
#pragma unroll
  for (int db = 0; db < 8; ++db) {
    o[0][db] = *reinterpret_cast<const f32x4*>(sp0 + 16 * db);
    o[1][db] = *reinterpret_cast<const f32x4*>(sp1 + 16 * db);
  }
}

// Normalise a wavefront's 32 output rows and store them as whole rows: the rows are regrouped
// through a wavefront-private 8 KB LDS area (32 rows x 256 bytes, the 16-byte chunks of a row
// rotated by the row number against bank conflicts), so that a store instruction writes 4
// complete rows (8 lines) where the accumulator layout would give 32 bytes to each of 16
// lines.  `tok` = the home row's destination (a token index), `inv` its factor; `head` +
// tok * row_stride is the row's address.
__device__ __forceinline__ void store_o_rows(uint16_t* head, int64_t row_stride, int tok, unsigned char* area,
                                             int lane, const f32x4 (&o)[2][8], float inv) {
  const int m_ = lane & 15, g = lane >> 4;
  float factor[2];
  both_rows(inv, factor);
#pragma unroll
  for (int cb = 0; cb < 2; ++cb)
#pragma unroll
    for (int db = 0; db < 8; ++db) {            // dims 16*db + 4*g + (0..3) of row 16*cb + m_
      u32x2 w;
      w.x = pack_bf16x2(o[cb][db][0] * factor[cb], o[cb][db][1] * factor[cb]);
      w.y = pack_bf16x2(o[cb][db][2] * factor[cb], o[cb][db][3] * factor[cb]);
      *reinterpret_cast<u32x2*>(area + (16 * cb + m_) * 256 + (((2 * db + (g >> 1)) ^ m_) << 4) + 8 * (g & 1)) = w;
    }
  const int sub = lane >> 4, chunk = lane & 15;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int row = 4 * k + sub;
    const u32x4 v = *reinterpret_cast<const u32x4*>(area + row * 256 + ((chunk ^ (row & 15)) << 4));
    const int t = __builtin_amdgcn_ds_bpermute(4 * ((row & 15) + 32 * (k >> 2)), tok);
    *reinterpret_cast<u32x4*>(head + (int64_t)t * row_stride + 8 * chunk) = v;
  }
}

// block id -> (head index z*H + h, segment counted from the last, position inside the
// segment's run of `per_seg` workgroups); false: an id that only rounds the grid up.  Longest
// prefixes first.  Consecutive block ids are dealt round-robin to the 8 XCDs, each with its own
// L2: workgroups of one (z, h, segment) walk the same keys at about the same time, so they are
// given ids that land on one XCD (their K/V tiles then hit in that L2).  What an XCD is dealt is
// fixed, while heads stop at lengths that differ by more than 3x and those of a KV group stop
// alike: the launch takes as long as the XCD with the longest share.
//
// Heads a multiple of 8: a segment's heads go to the 8 XCDs in turn, shifted by 4 from one
// segment to the next and by 1 every second segment, so that an XCD's share of every group is
// spread evenly over long and short prefixes.  (Shifted by 1 per segment, as before, an XCD had
// the long-walking groups in its 4 longest segments or in its 4 shortest: 32 heads, 8K tokens, 8 segments:
// the longest share 1.18 -> 1.03 of the mean, walk 324 -> 295 us; 32K with two of 8 groups walking
// four times as far 1.07 -> 1.02, 3290 -> 3090 us.)
// Otherwise: runs of up to 4 of a segment's workgroups go to the XCDs in turn, shifted by 1
// every 8 runs.  Dealt out one by one every XCD fetches every tile for itself: walk at 1e-3 with this /
// with runs, 4 heads, 64K tokens, 1024-token segments 1187 / 889 us, 128K in 512 1593 / 1212; 12 heads, 64K in 2048
// 1976 / 1877, 8K in 256 175 / 171.  Whole segments share a little more and
// balance less (4 heads, 64K in 2048: 881 one by one, 864 in runs, 905 whole; 12 heads, 32K in 2048 1341, 1238, 1265).
// Few workgroups are the exception that is left: 20 heads, 8K in 1024 166 one by one, 169 in runs.
// Shorter runs where all walks are of one length (alike) and an XCD would get so many more workgroups than one
// by one that some of its 32 CUs have another one: 5248 tokens without causality, 12 heads (492 workgroups, 41 a
// head) 224 us in runs of 4, which give an XCD 65 for its 64 places, 146 in runs of 3, 151 one by one; 6 heads 113 in
// runs of 4, 106 of 2, 107 one by one; 36 heads 506 in runs of 4, 465 of 3; 4 heads, 11 segments of 1280 574 in runs of 4,
// 369 of 2.
// (Runs per segment and workgroups per run come from the host: a division takes 0.15 us of a walk that
// may take 20.)
struct WalkGrid {
  int per_seg, run, runs;
  int64_t blocks;
};
inline WalkGrid walk_grid(int64_t ZH, int64_t N, int per_seg, bool alike) {
  WalkGrid g;
  g.per_seg = per_seg;
  const int64_t one = (ZH * N * per_seg + 7) / 8;               // workgroups of an XCD, one by one
  for (int longest = 4;; --longest) {
    g.runs = (per_seg + longest - 1) / longest;
    g.run = (per_seg + g.runs - 1) / g.runs;
    const int64_t share = (ZH * N * g.runs + 7) / 8 * g.run;    // ... of the fullest XCD, in runs
    if (longest == 1 || !alike || (share + 31) / 32 == (one + 31) / 32) break;
  }
  g.blocks = ZH % 8 == 0 ? ZH * N * per_seg : (ZH * N * g.runs + 7) / 8 * 8 * g.run;
  return g;
}
__device__ __forceinline__ bool map_block(int b, int ZH, int N, const WalkGrid& w, int& zh, int& nr, int& pos) {
  const int xcd = b & 7, idx = b >> 3;
  if (ZH % 8 == 0) {
    const int per = ZH / 8, unit = idx / w.per_seg;
    pos = idx % w.per_seg;
    nr = unit / per;
    zh = ((xcd - 4 * (nr & 1) - (nr >> 1)) & 7) + 8 * (unit % per);
    return true;
  }
  const int k = idx / w.run, r = 8 * k + ((xcd - k) & 7), unit = r / w.runs;
  pos = (r % w.runs) * w.run + idx % w.run;
  nr = unit / ZH;
  zh = unit % ZH;
  return nr < N && pos < w.per_seg;
}

}  // namespace tile
}  // namespace s2o
