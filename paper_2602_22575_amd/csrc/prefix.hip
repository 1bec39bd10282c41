// S2O prefix walk (paper Sec. 3.3, Alg. 3; Alg. 4 when the query order is the identity) for
// gfx950, resuming every query row from the state (accumulator, l, m) that the own-segment
// pass (Alg. 2, local.hip) left in the state buffers.
//
// One workgroup = 4 wavefronts = 128 permuted query rows of one (batch, head, segment): two
// query tiles of 64 rows or one of 128, 32 rows per wavefront.  The wavefronts of a segment
// walk the same KV_perm row, so a gathered 64-token K/V tile is staged in LDS once per
// workgroup.  MFMA formulation, LDS layouts, the explicitly scheduled operand reads and the
// base-2 online softmax with lazy rescaling are in attn_tile.h; the early-stop vote is taken
// one tile late, the PV product of a tile waiting for it.
//
// Tile pipeline.  Because the PV product of tile k runs during step k+1, V tile k is only
// needed one step after K tile k, so it is also fetched one step later: step k reads K(k) and
// V(k-1) while K(k+1) and V(k) arrive.  Two K and two V buffers (64 KB) then suffice, and with
// 4 wavefronts of under 256 registers two workgroups share a CU.
// A step is:   read the votes on tile k-1 and the tokens of tile k+1  ->  request the first K
// fragments  ->  issue the fetches of K(k+1), V(k) and of the token indices of tile k+2  ->  scores of
// tile k, PV of tile k-1, then the softmax of tile k  ->  wait for the wavefront's own fetches  ->
// barrier.  The fetches are issued first and waited for last, so they have the whole step to land;
// nothing between depends on them (the indices loaded in step k are first touched at the top of
// step k+1).  What bounds a step is the chip's power limit where a walk is long, and before that
// the two wavefronts of a SIMD taking turns: one's products beside the other's softmax.
//
// Walk with votes, us, before / after the softmax was kept behind the PV products, votes and tokens
// came with one LDS round trip in a loop without inner loops, and K was requested before the fetches
// (0.97, 0.96 and 0.98 to 1.00 of the time in turn; 32 heads): 8K at 1e-3 309 / 284, 32K at 5e-3 1319 / 1267, at
// 1e-37 8064 / 7694, 128K at 2e-2 2576 / 2519, at 5e-3 4789 / 4629, at 1e-3 12092 / 11435; 128-row tiles, 128K, half
// of the heads unstructured 20942 / 19734; one head, 2K 23.3 / 21.7.  (All before the steps went in pairs, below, and
// with 32x32x16 products; prefetch depth and wavefront priority of the present ones: attn_tile.h.)
//
// Other splits of the work, with the present products, 32 heads, time / this kernel's.  64 rows a wavefront, one
// wavefront a SIMD, softmax by hand between its products (half the LDS reads and fetches): 1.00 at contiguous 8K,
// 1.19 on zero data, 1.03 to 1.6 where walks are short: one wavefront issues too slowly.  256 rows a
// workgroup of 8 wavefronts (half the fetches), with a barrier a step 1.03 (zero data 1.22), with arrival counters in LDS and four
// buffers each 1.06 (1.28): two independent workgroups are what keeps one's products beside the other's softmax.
//
// The wait that ends a step goes through the builtin (wait_fetches): behind a wait it cannot see,
// the compiler guards the accumulator, loaded from the state in front of the loop, with waits of
// its own for all fetches in flight, in the middle of every step.  Walk without a stop rule,
// contiguous 8K keys x 32 heads: 1090 -> 1000 us together with the PV product moved one step
// late as in the walk with votes (with either one alone 1065 to 1088).  In the walk with votes, 32
// heads, time against a wait in assembly text: 128K at 2e-2 0.97, at 5e-3 0.99, at 1e-3 0.99 to 1.01,
// 32K at 5e-3 0.98; where no tile is skipped (1e-37, say) 1.01 at 32K and 1.02 to 1.03 at 128K, since
// what a step then spends is power, not cycles.  A threshold of 0 or less has no votes to take.
//
// The single-launch form (no state buffer) runs the own-segment tiles through the same
// pipeline first.  It is bound by the matrix products: a query tile in permuted order has rows
// anywhere in the segment and needs all S/64 own tiles where one in original order stops at its
// diagonal, which is why a caller with a state buffer gets two launches.  Single launch against two,
// 32 heads, 16K tokens, threshold 5e-3 (time, two launches = 1), permuted order: segments of 64 tokens 0.89, of
// 256 0.92, of 512 0.96, of 1024 1.08, of 2048 1.20, of 4096 1.39, of 8192 1.53; original order 0.86 to 0.93.
// Against the 8-wavefront workgroups (one per CU, operand reads placed by the compiler) it replaces:
// permuted order 0.82 to 0.89 from 512-token segments on, original order 0.74 to 0.86; 16K tokens,
// 32 heads, original order, threshold 5e-3, with the ranking 1028 -> 697 us.
#include "attn_tile.h"
#include "s2o_internal.h"

namespace s2o {

namespace {

using namespace tile;

constexpr int kWaves = 4, kThreads = 64 * kWaves;
constexpr int kVBytes0 = 2 * kTileBytes;                           // K x2 at 0, V x2 behind them
constexpr size_t kPrefixLds = (size_t)(4 * kTileBytes) + 64 + 4 * kWaves * 64;   // + vote flags + index ring

// min(max(x, 0), hi) in one instruction (the compiler emits two: it cannot know that hi >= 0)
__device__ __forceinline__ uint32_t clamp_token(int x, int hi) {
  int r;
  asm("v_med3_i32 %0, %1, 0, %2" : "=v"(r) : "v"(x), "s"(hi));
  return (uint32_t)r;
}

// kNoStop: every prefix tile is folded in (stop_mode 2, the paper's kernel C; a state buffer and a
// threshold of 0 or less), as an instantiation of its own, so that neither loop's registers weigh on the other.
// kMapped: the walk follows a KV_perm row (always, except the non-causal walk in storage order,
// which then does not carry the map's registers and selects).
// kOwn: the single-launch form for callers without a state buffer.  The key tiles of the
// segment itself are folded in first, with the causal mask per row, and the state never leaves
// the registers.  Tiles are numbered through: 0 .. nloc-1 the own segment's, then the prefix's.
// kExactReference: the softmax reference moves as in softmax_tile (see attn_tile.h).
template <bool kNoStop, bool kMapped, bool kOwn, bool kExactReference>
__global__ __launch_bounds__(kThreads, 2) void s2o_prefix_kernel(const AttnArgs a, const WalkGrid grid) {
  extern __shared__ __attribute__((aligned(256))) unsigned char smem[];   // OperandAddr needs a 256-byte base
  uint16_t* Ks = reinterpret_cast<uint16_t*>(smem);
  uint16_t* Vt = Ks + 2 * kTileElems;
  uint8_t* vote = reinterpret_cast<uint8_t*>(Vt + 2 * kTileElems);   // stop votes: two sets of one byte per wavefront
  int* own_tiles = reinterpret_cast<int*>(vote) + kWaves;     // kOwn: own-segment tiles per wavefront
  int32_t* ring = reinterpret_cast<int32_t*>(smem + 4 * kTileBytes + 64);   // map entries: 4 tiles x kWaves x 16

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int BM = a.BM;                                   // query tile rows: 64 or 128
  const int tpw = BM == 64 ? 2 : 1;                      // query tiles per workgroup
  const int TJ = a.S >> (BM == 64 ? 6 : 7);              // query tiles per segment

  int zh_, nr, jg;
  if (!map_block(blockIdx.x, a.Z * a.H, a.N, grid, zh_, nr, jg)) return;
  if (kOwn) jg = grid.per_seg - 1 - jg;   // original order: the tiles with most own-segment keys first
  const int n = a.N - 1 - nr, z = a.Z == 1 ? 0 : zh_ / a.H, h = zh_ - z * a.H;
  const int g = h / (a.H / a.Hkv);
  const uint16_t* Qh = a.Q + z * a.qs[0] + h * a.qs[1];
  const uint16_t* Kh = a.K + z * a.ks[0] + g * a.ks[1];
  const uint16_t* Vh = a.V + z * a.vs[0] + g * a.vs[1];
  uint16_t* Oh = a.O + z * a.os[0] + h * a.os[1];
  const int64_t zh = (int64_t)z * a.H + h;
  const int32_t* kvrow = a.kv_perm + zh * kv_rows_total(a.N, a.S, a.L, a.non_causal) +
                         kv_row_start(n, a.S, a.L, a.non_causal);
  const int nS = n * a.S;
  // key tiles this segment's row of KV_perm lists: its prefix, or everything without causality
  const int nK_all = (int)(kv_row_len(n, a.S, a.L, a.non_causal) / kBN);
  // prefix tiles this launch may walk: at most the budget
  const int ntiles = a.max_tiles > 0 ? min(nK_all, a.max_tiles) : nK_all;

  // wavefront -> (query tile of the workgroup, 32-row part); the parts of a tile are
  // wavefronts tile, tile + tpw, ...
  const int tile_l = tpw == 2 ? wave & 1 : 0, part = tpw == 2 ? wave >> 1 : wave;
  const int j = jg * tpw + tile_l;              // this wavefront's permuted query tile
  const bool active = j < TJ;

  // ---- the home row of this lane
  int qoff;
  {
    const int r = min(j, TJ - 1) * BM + kRowsPerWave * part + home_row(lane);
    qoff = a.use_q_perm ? a.q_perm[(zh * a.N + n) * a.S + r] : r;
    qoff = min(max(qoff, 0), a.S - 1);
  }
  // own-segment tiles: of the workgroup, of this wavefront; row_lo = the wavefront's first row
  int nloc = 0, myn = 0, row_lo = 0;
  if constexpr (kOwn) {
    int lo = qoff, hi = qoff;
#pragma unroll
    for (int d : {1, 2, 4, 8, 32}) { lo = min(lo, __shfl_xor(lo, d)); hi = max(hi, __shfl_xor(hi, d)); }
    row_lo = __builtin_amdgcn_readfirstlane(lo);
    myn = active ? __builtin_amdgcn_readfirstlane(hi) / kBN + 1 : 0;
    if (lane == 0) own_tiles[wave] = myn;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) nloc = max(nloc, __builtin_amdgcn_readfirstlane(own_tiles[w]));
  }
  const int nall = nloc + ntiles;               // tiles of this launch

  // ---- loader: every wavefront moves 16 rows of K and 16 rows of V per step, 4 rows per
  // instruction (lane l of group gi moves a chunk of tile row 16*wave + 4*gi + l/16).  The map
  // entries of its rows travel through a small ring in LDS, private to the wavefront: the 16
  // entries of tile t+2 are requested (global -> LDS, like the tiles) at the top of step t and
  // first read at the top of step t+1, so no register holds an index across a step and no
  // fetch ever waits for an index load.  Ring position 4*(l/16) + gi holds the entry of row
  // 4*gi + l/16, so a lane gets its four tokens with one 16-byte read.
  const uint32_t k_stride_bytes = (uint32_t)(a.ks[2] * 2), v_stride_bytes = (uint32_t)(a.vs[2] * 2);
  uint32_t goff[4];
#pragma unroll
  for (int gi = 0; gi < 4; ++gi) goff[gi] = (uint32_t)load_chunk_offset(lane, 16 * wave + 4 * gi);
  auto ring_slot = [&](int t) { return ring + (t & 3) * (16 * kWaves) + 16 * wave; };
  // (lane l < 16 requests the entry of tile row 16*wave + 4*(l%4) + l/4)
  auto fetch_index = [&](int t) {       // map entries of tile t (clamped tile number) -> ring; ntiles > 0
    if (kMapped && (!kOwn || (t >= nloc && t < nall)) && lane < 16) {
      // scalar base + 32-bit lane offset: no 64-bit per-lane pointer is kept across the walk
      // The lane's offset is worked out again at every call (opaque lane id): kept across the
      // walk it would be a 64-bit per-lane pointer, two registers that the allocator spills
      // and reloads inside the step, behind a wait for every fetch in flight.
      int l = lane;
      asm volatile("" : "+v"(l));
      const uint32_t row4 = (uint32_t)(4 * (16 * wave + 4 * (l & 3) + ((l >> 2) & 3)));
      const char* tile_idx = reinterpret_cast<const char*>(kvrow + (int64_t)min(t - nloc, ntiles - 1) * kBN);
      __builtin_amdgcn_global_load_lds((const gvoid*)(tile_idx + (uint64_t)row4), (lvoid*)ring_slot(t), 4, 0, 0);
    }
  };
  auto tokens = [&](int t, uint32_t (&tok)[4]) {   // this lane's four tokens of tile t, clamped to the sequence
    if (kOwn && t < nloc) {             // the segment's own keys
#pragma unroll
      for (int gi = 0; gi < 4; ++gi)
        tok[gi] = (uint32_t)min(nS + t * kBN + 16 * wave + 4 * gi + (lane >> 4), a.L - 1);
    } else if (kMapped) {
      const int4 e = *reinterpret_cast<const int4*>(ring_slot(t) + 4 * (lane >> 4));
      const int ev[4] = {e.x, e.y, e.z, e.w};
#pragma unroll
      for (int gi = 0; gi < 4; ++gi) tok[gi] = clamp_token(ev[gi], a.L - 1);
    } else {                            // no map (non-causal only): the keys in storage order
#pragma unroll
      for (int gi = 0; gi < 4; ++gi)
        tok[gi] = (uint32_t)min(min(t, ntiles - 1) * kBN + 16 * wave + 4 * gi + (lane >> 4), a.L - 1);
    }
  };
  auto load_k = [&](int t, const uint32_t (&tok)[4]) {   // K tile t -> buffer t & 1
    uint16_t* kd = Ks + (t & 1) * kTileElems;
#pragma unroll
    for (int gi = 0; gi < 4; ++gi)
      load_rows_to_lds(reinterpret_cast<const char*>(Kh) + (uint64_t)(__umul24(tok[gi], k_stride_bytes) + goff[gi]),
                       kd + (16 * wave + 4 * gi) * kRowElems);
  };
  auto load_v = [&](int t, const uint32_t (&tok)[4]) {   // V tile t -> buffer t & 1
    uint16_t* vd = Vt + (t & 1) * kTileElems;
#pragma unroll
    for (int gi = 0; gi < 4; ++gi)
      load_rows_to_lds(reinterpret_cast<const char*>(Vh) + (uint64_t)(__umul24(tok[gi], v_stride_bytes) + goff[gi]),
                       vd + (16 * wave + 4 * gi) * kRowElems);
  };
  // the fetches of step t (top of the step): K(t+1), V(t), indices of tile t+2
  // A wavefront calls fetch_step for t = 0, 1, 2, ... in turn (working or draining), so the
  // tokens of tile t, which V(t) needs, are the ones the previous call worked out for K(t):
  // they stay in four registers instead of being read from the ring and clamped again.
  uint32_t tok_cur[4] = {0, 0, 0, 0};
  auto fetch_step_of = [&](int t, const uint32_t (&tn)[4]) {      // tn: the tokens of tile t + 1
    if (t + 1 < nall) load_k(t + 1, tn);
    load_v(t, tok_cur);
#pragma unroll
    for (int gi = 0; gi < 4; ++gi) tok_cur[gi] = tn[gi];
    fetch_index(t + 2);
  };
  auto fetch_step = [&](int t) {
    uint32_t tn[4];
    tokens(t + 1, tn);
    fetch_step_of(t, tn);
  };
  if (nall > 0) {
    fetch_index(0);
    fetch_index(1);
    if (!kOwn) wait_tile_loads();
    tokens(0, tok_cur);
    load_k(0, tok_cur);
  }

  // ---- the Q fragments of the row
  int rows[2];                                  // the lane's two rows
  both_rows(qoff, rows);
  bf16x8 qf[4][2];
  load_q(Qh + (int64_t)(nS + rows[0]) * a.qs[2], Qh + (int64_t)(nS + rows[1]) * a.qs[2], lane >> 4, qf);
  OperandAddr oa;
  oa.init(lane, lds_address(smem));

  // ---- online-softmax state and output accumulator O^T[d-block], resumed from the state
  // buffers (row (z, h, l) -> accumulator, l, m).  The statistics are needed by the first
  // softmax; the accumulator only by the first PV product, one step later: its 512 bytes per
  // row are requested after the first tile's scores have been issued and arrive behind them.
  const float c2 = a.scale_log2e;
  // Without causality there is no own-segment pass: every row starts from the empty state.
  // Neither is there a state to resume in the single-launch form.
  const int64_t st_row = zh * a.L + nS + qoff;
  float m_ref[2] = {-INFINITY, -INFINITY}, l_run = 0.f;
  const bool no_state = kOwn || a.non_causal;
  if (!no_state) { both_rows(a.st_m[st_row], m_ref); l_run = a.st_l[st_row]; }
  f32x4 o[2][8];
  const float* st_acc_rows[2];
  for (int cb = 0; cb < 2; ++cb) st_acc_rows[cb] = a.st_acc + (zh * a.L + nS + rows[cb]) * kD + 4 * (lane >> 4);
  auto init_acc = [&] {
    if (no_state) zero_acc(o);
    else load_acc(st_acc_rows[0], st_acc_rows[1], o);
  };
  int committed = 0, issued = 0;

  f32x4 s[4][2];
  TileStats ts;
  auto softmax = [&] { ts = softmax_tile<false>(s, c2, m_ref, l_run, 0, 0, lane); };

  // ---- prefix tiles in KV_perm order with the early-stop rule: the query tile continues iff
  // some row's tile mass reaches tau * (mass so far).  The wavefronts of a tile vote through
  // LDS; the vote on tile k is written before the barrier that ends step k and read at the
  // start of step k+1, where the PV product of tile k is then run, dropped, or folded in as
  // the last one.  The statistics (l, m) are advanced speculatively, and on a drop the mass l is
  // rolled back: nothing reads m_ref after a stop, and the accumulator is only ever touched (rescaled
  // included) by a tile that is kept.  Every wavefront runs
  // one barrier per step; one whose query tile has stopped (or that has none) drops into a
  // drain loop that only keeps fetching tiles for the others.
  bf16x8 pb_pend[2][2];
  float alpha_pend = 1.f, l_save = 0.f;
  bool grow_pend = false;
  auto vote_word = [&](int step) { return vote + kWaves * (step & 1); };
  auto publish = [&](int step) {        // after softmax of tile `step`: vote + speculative stats
    const bool keep = __builtin_amdgcn_ballot_w64(ts.mass >= a.tau * ts.prev) != 0ull;
    vote_word(step)[wave] = keep ? 1 : 0;
    l_save = l_run;
    l_run = ts.prev + ts.mass; m_ref[0] = ts.m_use[0]; m_ref[1] = ts.m_use[1];
    alpha_pend = ts.alpha; grow_pend = ts.grow;
    pack_p(s, pb_pend);
    ++issued;
  };
  // The four wavefronts' votes of a step come with one 4-byte read; a query tile's wavefronts are
  // tile_l, tile_l + tpw, ...
  struct Votes { uint32_t mine, any; };
  const uint32_t my_votes = tpw == 1 ? 0xffffffffu : tile_l == 0 ? 0x00ff00ffu : 0xff00ff00u;
  auto votes_of = [&](uint32_t word) {
    const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)word);
    return Votes{w & my_votes, w};
  };
  auto read_votes = [&](int step) { return votes_of(*reinterpret_cast<const uint32_t*>(vote_word(step))); };
  // The same together with the tokens of tile step + 2: one LDS round trip at the top of a step.
  const uint32_t vote_lds = lds_address(vote), ring_lds = lds_address(ring) + 64 * wave + 16 * (lane >> 4);
  auto read_votes_and_tokens = [&](int step, uint32_t (&tok)[4]) {
    uint32_t w;
    if constexpr (kMapped) {
      u32x4 e;
      asm volatile("ds_read_b32 %0, %2\n\tds_read_b128 %1, %3\n\ts_waitcnt lgkmcnt(0)"
                   : "=&v"(w), "=&v"(e)
                   : "v"(vote_lds + kWaves * (step & 1)), "v"(ring_lds + 64 * kWaves * ((step + 2) & 3)) : "memory");
#pragma unroll
      for (int gi = 0; gi < 4; ++gi) tok[gi] = clamp_token((int)e[gi], a.L - 1);
    } else {
      asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(w) : "v"(vote_lds + kWaves * (step & 1)) : "memory");
      tokens(step + 2, tok);
    }
    return votes_of(w);
  };
  auto end_step = [&] {                 // this wavefront's fetches have landed; everyone's after the barrier
    wait_fetches<0>();
    __syncthreads();
  };

  // Step `it` reads K(it) in K buffer it & 1 and V(it-1), whose PV product is due, in V buffer
  // (it-1) & 1.  The walk's loops come in pairs of steps with the buffers as constants in the reads'
  // offsets: moving the operand addresses (sixteen then, with 32x32x16 products) to the other buffers at the end of every step took
  // 4 to 6 % of a walk without votes (8K contiguous 998 / 961 us, 32K causal 7472 / 7000, top-k at 16K 525 / 505)
  // and 1.5 to 2 % of one with votes (32 heads, 128K at 5e-3 4601 / 4495, 32K at 1e-37 7656 / 7497); the
  // own-segment tiles of the single launch 1 % (32K 2406 / 2368, 16K in original order 642 / 637; without a stop
  // rule, both loops, 16K in original order 2122 / 2092, 8 heads 642 / 619, 4K x 4 heads 112 / 106).
  bool acc_loaded = false, pending = false;
  int it = 0;
  typedef std::integral_constant<int, 0> Even;
  typedef std::integral_constant<int, 1> Odd;
  auto k_at = [&](int it_) { return oa.at((uint32_t)((it_ & 1) * kTileBytes), 0u); };
  auto v_at = [&](int it_) { return oa.at(0u, (uint32_t)(kVBytes0 + (it_ & 1) * kTileBytes)); };
  auto pv_last = [&] {                          // V(it-1), alone
    rescale(o, alpha_pend, grow_pend);
    pv_tile_only<0>(v_at(it - 1), pb_pend, o);
  };
  auto fold = [&] {                             // a tile that is kept without a vote
    pack_p(s, pb_pend);
    alpha_pend = ts.alpha; grow_pend = ts.grow;
    if constexpr (kExactReference) {
      l_run = fmaf(l_run, ts.alpha, ts.mass);   // (one rounding, written out: as prev + mass it is up to the compiler)
    } else {
#pragma clang fp contract(off)
      l_run = ts.prev + ts.mass;                // (two roundings, as in the walk with votes)
    }
    m_ref[0] = ts.m_use[0]; m_ref[1] = ts.m_use[1];
    pending = true;
  };
  // The softmax of a step behind the first.  Left to itself the compiler puts it between the PV products.
  // The two wavefronts of a SIMD then get in each other's way; kept behind them, one's products run beside
  // the other's softmax (a step of the walk with votes took 3810 and 4550 clocks on the two, one without votes,
  // where a branch kept them apart anyway, 3300; the barrier alone 0.97 of the walk's time).
  auto softmax_step = [&](auto par) {
    __builtin_amdgcn_sched_barrier(0);
    bool redo;
    ts = softmax_tile_keep_reference<kExactReference>(s, c2, m_ref, l_run, redo);
    if (__builtin_amdgcn_ballot_w64(redo) != 0ull &&       // rare: the tile may move some row's reference
        !(kExactReference && __builtin_amdgcn_ballot_w64(confirm_redo(s, ts.mass)) == 0ull)) {
      qk_tile_only<decltype(par)::value * kTileBytes>(oa, qf, s);
      softmax();
    }
  };

  if constexpr (kOwn) {
    // ---- the segment's own tiles (Pass-1: dense, causal mask where a row ends inside the tile).
    // A wavefront without a query tile (myn = 0) only fetches.
    zero_acc(o);
    acc_loaded = true;
    wait_fetches<0>();
    __syncthreads();                            // K tile 0 has landed
    auto own_step = [&](auto par) {
      constexpr int kK = decltype(par)::value * kTileBytes, kV = kVBytes0 + kTileBytes - kK;
      fetch_step(it);
      if (it < myn) {
        if (pending) {
          u32x2 vfr[16][2];
          qk_tile_sched<kK, kV, true>(oa, qf, s, vfr);
          rescale(o, alpha_pend, grow_pend);
          pv_tile_sched<kV, true>(oa, pb_pend, o, vfr);
        } else {
          qk_tile_only<kK>(oa, qf, s);
        }
        const bool masked = it * kBN + kBN - 1 > row_lo;
        ts = masked ? softmax_tile<true>(s, c2, m_ref, l_run, it * kBN, qoff, lane)
                    : softmax_tile<false>(s, c2, m_ref, l_run, it * kBN, qoff, lane);
        fold();
      } else if (pending) {                     // this wavefront's last tile, one step after its scores
        rescale(o, alpha_pend, grow_pend);
        pv_tile_only<kV>(oa, pb_pend, o);
        pending = false;
      }
      wait_fetches<0>();
      __syncthreads();
      ++it;
    };
    while (it + 1 < nloc) { own_step(Even{}); own_step(Odd{}); }
    if (it < nloc) own_step(Even{});
    if (pending) {
      pv_last();
      pending = false;
    }
  }

  if (kNoStop && ntiles > 0) {
    // ---- every prefix tile is folded in: no votes
    if (!kOwn) {
      init_acc(); acc_loaded = true;
      wait_fetches<0>();                          // K tile 0 has landed
      __syncthreads();
    }
    fetch_step(it);                               // first tile: scores only
    if (active) {
      qk_tile_only<0>(k_at(it), qf, s);
      softmax();
      fold();
    }
    wait_fetches<0>();
    __syncthreads();
    ++it;
    auto step = [&](auto par) {
      constexpr int kK = decltype(par)::value * kTileBytes, kV = kVBytes0 + kTileBytes - kK;
      fetch_step(it);
      if (active) {
        u32x2 vfr[16][2];
        qk_tile_sched<kK, kV, true>(oa, qf, s, vfr);
        rescale(o, alpha_pend, grow_pend);
        pv_tile_sched<kV, true>(oa, pb_pend, o, vfr);
        softmax_step(par);
        fold();
      }
      wait_fetches<0>();
      __syncthreads();
      ++it;
    };
    if (kOwn && (it & 1) == 0 && it < nall) step(Even{});
    while (it + 1 < nall) { step(Odd{}); step(Even{}); }
    if (it < nall) step(Odd{});
    if (active) {
      pv_last();
      committed = issued = ntiles;
    }
  } else if (ntiles > 0) {
    if (!kOwn) end_step();                        // K tile 0 has landed
    bool wg_done = false;
    if (active) {
      // first tile: scores only
      fetch_step(it);
      qk_tile_only<0>(k_at(it), qf, s);
      if (!kOwn) { init_acc(); acc_loaded = true; }
      softmax();
      publish(it);
      end_step();
      ++it;
      // One step; false: this query tile stops here.  The stop's own work stands behind the loop: with the
      // last PV product inside, the compiler hoists what the loop does not have registers for.
      Votes votes = {1u, 1u};
      auto step = [&](auto par) -> bool {
        constexpr int kK = decltype(par)::value * kTileBytes, kV = kVBytes0 + kTileBytes - kK;
        uint32_t tn[4];
        votes = read_votes_and_tokens(it - 1, tn);
        if (votes.mine == 0) return false;
        bf16x8 ka[8][2];
        qk_tile_begin<kK>(oa, ka);              // on their way while the fetches are issued
        fetch_step_of(it, tn);
        u32x2 vfr[16][2];
        qk_tile_begun<kK, kV, true>(oa, qf, s, vfr, ka);
        rescale(o, alpha_pend, grow_pend);
        pv_tile_sched<kV, true>(oa, pb_pend, o, vfr);
        ++committed;
        softmax_step(par);
        publish(it);
        wait_fetches<0>();
        __syncthreads();
        ++it;
        return true;
      };
      for (bool odd = !kOwn || (it & 1) != 0; it < nall; odd = true) {
        if (odd) {
          if (!step(Odd{})) break;
          if (it >= nall) break;
        }
        if (!step(Even{})) break;
      }
      if (it == nall) votes = read_votes(nall - 1);   // the last tile: its vote is visible now
      wg_done = it == nall || votes.any == 0;
      if (votes.mine == 0 && a.stop_mode == 0) {
        l_run = l_save;
      } else {
        pv_last();
        ++committed;
      }
    }
    // ---- drain: keep the tile pipeline fed until every query tile of the workgroup has stopped
    if (!wg_done) {
      for (; it < nall; ++it) {
        if (it > nloc && read_votes(it - 1).any == 0) break;
        fetch_step(it);
        vote_word(it)[wave] = 0;
        end_step();
      }
    }
  }

  if (active) {
    if (!acc_loaded) init_acc();                 // no prefix tile was walked (first segment)
    // normalise and scatter to the original row
    // (every wavefront of the workgroup is past the last barrier: the K buffers are idle)
    store_o_rows(Oh, a.os[2], nS + qoff, smem + wave * 8192, lane, o, 1.0f / l_run);
    if (lane == 0 && part == 0) {
      const int64_t ci = zh * (a.L / BM) + (int64_t)n * TJ + j;
      if (a.computed) a.computed[ci] = committed;
      if (a.skipped) a.skipped[ci] = nK_all - issued;
    }
  }
}

}  // namespace

hipError_t launch_prefix(const AttnArgs& a, hipStream_t stream) {
  static std::mutex mu;
  static uint64_t done = 0;
  const hipError_t se = once_per_device(mu, done, [] {
    const void* fns[8] = {reinterpret_cast<const void*>(&s2o_prefix_kernel<false, true, false, false>),
                          reinterpret_cast<const void*>(&s2o_prefix_kernel<true, true, false, false>),
                          reinterpret_cast<const void*>(&s2o_prefix_kernel<true, true, false, true>),
                          reinterpret_cast<const void*>(&s2o_prefix_kernel<false, false, false, false>),
                          reinterpret_cast<const void*>(&s2o_prefix_kernel<true, false, false, false>),
                          reinterpret_cast<const void*>(&s2o_prefix_kernel<true, false, false, true>),
                          reinterpret_cast<const void*>(&s2o_prefix_kernel<false, true, true, true>),
                          reinterpret_cast<const void*>(&s2o_prefix_kernel<true, true, true, true>)};
    for (const void* f : fns) {
      const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kPrefixLds);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  });
  if (se != hipSuccess) return se;
  const int TJ = a.S / a.BM;
  const int tpw = kWaves / (a.BM / kRowsPerWave);
  const int JG = (TJ + tpw - 1) / tpw;
  const WalkGrid grid = walk_grid((int64_t)a.Z * a.H, a.N, JG, a.non_causal || a.N == 1);
  if (grid.blocks <= 0 || grid.blocks > 0x7fffffff) return hipErrorInvalidValue;
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid.blocks), dim3(kThreads), kPrefixLds, stream, a, grid);
  };
  // A threshold of 0 or less never stops, so nothing is lost by leaving the votes out (us with /
  // without them, 32 heads: 8K 448 / 418, 32K 7296 / 6587, 128K 125166 / 110741).  The reference then
  // still moves as in the walk with votes, and the results keep its bits.  (The single launch's
  // normaliser is rounded otherwise without votes: there the votes stay.)
  const bool rule = a.stop_mode != 2, no_stop = !rule || a.tau <= 0.f;
  if (a.passes == 0) !rule ? launch(s2o_prefix_kernel<true, true, true, true>) : launch(s2o_prefix_kernel<false, true, true, true>);
  else if (a.kv_perm)
    !no_stop ? launch(s2o_prefix_kernel<false, true, false, false>)
             : rule ? launch(s2o_prefix_kernel<true, true, false, false>) : launch(s2o_prefix_kernel<true, true, false, true>);
  else
    !no_stop ? launch(s2o_prefix_kernel<false, false, false, false>)
             : rule ? launch(s2o_prefix_kernel<true, false, false, false>) : launch(s2o_prefix_kernel<true, false, false, true>);
  return hipGetLastError();
}

}  // namespace s2o
