// The row-splitting bf16 kernels (internal to libaspd): many rows per KV head (branch chunks, whole sequences).
#pragma once

#include "attn_bf16_math.h"

namespace {

// ---------------------------------------------------------------------------------------------
// bf16, many rows per KV head (branch chunks, prefills, whole sequences): the waves of a workgroup split
// the ROWS instead of the keys.  Every group of ROWS_PPS pairs of pages is loaded once per workgroup,
// cooperatively and straight into LDS, two groups ahead, for all waves to read; each wave keeps its own 32 rows
// (Q operands, accumulators, softmax state, all in registers) for the whole segment, so there is no
// reduction across waves.  One barrier per group.  With NW waves a row group holds NW * 32 rows, and the
// pages of a KV head are fetched once per that many rows.
//
// What bounds it is the issue slots of a SIMD (two waves): MFMA and vector instructions of both waves go
// through them.  So the products run on 32x32x16 MFMA tiles (half the MFMA instructions of 16x16x32 at the
// same rate, and one softmax row per lane instead of two), the running reference is tested on the sum of the
// weights (which is needed anyway) instead of on a maximum of the scores, and the pair loop is pipelined: a
// step issues the score products of pair p + 1 and the value products of pair p - 1, which depend on nothing
// in it, beside the softmax of pair p, so that a wave by itself keeps the matrix unit and the vector unit
// busy together.  Measured against 16x16x32 tiles without the pipeline: 64 whole sequences (18.8 TFLOP) 22.1 -> 20.8 ms,
// where the matrix unit's share of the cycles went from 41 % to 53 % and the shader clock from 1.91 to 1.58 GHz (the
// launch runs into the power limit); prompts of 90 to 2000 tokens 403 -> 225 us a layer.  (Since then, with fewer reads past the
// L2 and shorter starts: 16.7 ms, 58 % at 1.89 GHz, and 125 us.)
//
// 32x32x16 layout: S^T[key][row] = K * Q^T, lane (c, h) = (lane % 32, lane / 32) holds, of row c, the keys
// 8 b + 4 h + j (b, j = 0 .. 3) of the pair, which is the B-operand layout of O^T[d][row] = V^T * P^T when the
// eight keys of a lane's k-slice are taken in that order; V^T comes from the LDS transpose read.
// ---------------------------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(16))) float f32x16;

template <int D>
struct RowsCfg {
  static constexpr int CH = D / 8;          // 16-byte chunks per row
  static constexpr int PAGE_U4 = 16 * CH;
  static constexpr int KSTEPS = D / 16;     // k-steps of the score product
  static constexpr int MT = D / 32;         // 32-wide d-tiles of the value product
  static constexpr int PAGE_B = PAGE_U4 * 16;
  static constexpr int PAIR_B = 2 * PAGE_B;               // both pages of a pair: 32 consecutive rows
  static constexpr int STAGE_B = 2 * ROWS_PPS * PAIR_B;   // K pairs, then V pairs
  // Pages lie in LDS as they do in the cache (they are loaded straight into it, 64 x 16 bytes in a row per
  // instruction), but for the order of the 16-byte chunks inside a row, which is chosen so that no read has a bank
  // conflict: a K operand read takes one chunk of sixteen rows at a time, a transposing V read 64 bytes of four.
  static __device__ __forceinline__ int kswz(int row) { return D == 128 ? (row & 15) : ((row >> 1) & 7); }
  static __device__ __forceinline__ int vswz(int row) { return D == 128 ? 4 * (row & 3) : 4 * ((row >> 1) & 1); }
};
// Groups in LDS: the one being computed, two on their way (three stages would do; four make the ring a mask).  One group
// ahead is too few where row groups are light and the read rate of the chip counts, a third one only costs scalar registers.
// Groups ahead 1 / 2 / 3, whole steps, us: 64 sequences x 8000 tokens, two layers, 52 rows per KV head 806 / 776 / 778, 256
// rows 1203 / 1207 / 1210, 64 rows of head size 64 292 / 242 / 243; 39 sequences of up to 500 tokens at 8/8 heads 343 / 352 /
// 357, 12 of up to 1000 at 32/8 149 / 149 / 153; the 64-sequence chunk 1727 / 1739 / 1754; prompts 433 / 434 / 436.
constexpr int ROWS_BUFS = 4;

template <int D>
constexpr size_t rows_smem_bytes() { return (size_t)ROWS_BUFS * RowsCfg<D>::STAGE_B; }

// One wave's 32 rows: lane (c, h) keeps the statistics of row c (its share of the sum) and O^T[32 mt + 8 b + 4 h +
// j][c] in acc[mt][4 b + j].
template <int D>
struct Rows32 {
  f32x16 acc[D / 32];
  float m_run, l_run;
  float neg_ref;  // minus the running reference, 0 while there is none
  float limit;    // weight sum above which the references are raised; below any sum before and at the second raise
};

// Largest weight sum of a lane's sixteen keys before the row's reference is raised (see rows_raise).  A thousand would be
// as safe in fp32 and in the bf16 operand.  What the value decides is the rounding of the weights: the weight of the
// key that gave the reference is 1 and has no error, and where few keys carry a row the error of the largest weights
// is that of the output.  With 20, and with the references raised at the second pair in any case (so that they are
// the largest of 64 scores at least), the error against float64 is 0.1 to 4 % below that of references taken from a
// group of 64 keys and raised at a score 2^6 above (as before the 32x32x16 tiles) for queries ~ N(0, 1) and N(0, 36),
// 3 to 8 % for N(0, 4).  With 1024 and the first pair's maximum it was 0.8, 4 to 8 and 10 % above.  The raise at the
// second pair costs about 1 us a launch (three short whole sequences, two layers 143.0 -> 144.5 us, eight prompts
// 438 -> 444) and 0.6 % of the 64-sequence ones (chunk 1790 -> 1801 us, whole sequences 23.81 -> 23.94 ms).
constexpr float ROWS_SUM_MAX = 20.f;

// V operand: two transposing reads, eight rows apart.
template <int D>
__device__ __forceinline__ bf16x8 rows_v_operand(uint32_t at) {
  const s16x4 a = lds_operand_transposed(at);
  const s16x4 b = lds_operand_transposed(at + 8 * D * 2);
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Weights of one pair against the rows' lazily raised references (log2 domain, scaled scores; a reference is
// not necessarily the row maximum).  The weights are computed first and their sum, which the row needs anyway,
// tells whether a reference has to go up: while no lane's sixteen weights sum to more than ROWS_SUM_MAX none of
// them exceeds it.  Otherwise, while a row of the wave has no reference, and once more after that, the references are
// raised to the largest score so far, the accumulators rescaled and the weights formed again.  (Testing the sum costs
// one comparison per pair; the maximum it replaces cost eight instructions and the wait states in front of them.)
template <int D>
__device__ __forceinline__ float rows_weights(const f32x16& s, const Rows32<D>& rs, bf16x8 (&p)[2], float scale_log2) {
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const float w = __builtin_amdgcn_exp2f(fmaf(s[i], scale_log2, rs.neg_ref));
    sum += w;
    p[i >> 3][i & 7] = (__bf16)w;
  }
  return sum;
}
// The references go up to the largest score so far; returns the sum of the weights formed again.
template <int D>
__device__ __forceinline__ float rows_raise(const f32x16& s, Rows32<D>& rs, bf16x8 (&p)[2], float scale_log2) {
  float lo[8], hi[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    lo[i] = s[i];
    hi[i] = s[8 + i];
  }
  float mx = fmaxf(max8(lo), max8(hi));
  mx = over_halves(mx, [](float x, float y) { return fmaxf(x, y); }) * scale_log2;  // scale > 0: the maximum commutes with it
  const float m_new = fmaxf(rs.m_run, mx);
  const float ref = exp2_safe_ref(m_new);
  const float alpha = __builtin_amdgcn_exp2f(rs.m_run - ref);
  rs.m_run = m_new;
  rs.neg_ref = -ref;
  rs.l_run *= alpha;
#pragma unroll
  for (int mt = 0; mt < D / 32; ++mt) rs.acc[mt] *= alpha;
  rs.limit = __any(m_new == -INFINITY) ? -2.f : (rs.limit < -1.f ? -1.f : ROWS_SUM_MAX);
  return rows_weights<D>(s, rs, p, scale_log2);
}

// SEQ: the rows are tokens of a whole multi-stage sequence (aspd_attn_full_sequence): each brings the first
// slot of its own stage (a.row_base) and the first slot of its own branch there (a.row_lo), which are all of
// what it sees: [0, base) and [lo, slot].  Otherwise all rows belong to the sequence's running stage, which
// starts at it.L, and owner tags tell whose a slot of that stage is.
// take_from: a counter that thread 0 adds one to before it writes its rows (so that the answer, which it returns, does not
// have to be waited for), or null.
// result: asked at the end whether the segment is a whole item, and where its partial result goes otherwise.
struct Result {
  bool complete;
  float* pslot;
};
template <int D, int NW, bool SEQ, typename ResultOf>
__device__ __forceinline__ int segment_rows(const AttnArgs& a, char* smem, const Seg& it, ResultOf result,
                                            int* take_from) {
  using C = RowsCfg<D>;
  constexpr int PPS = ROWS_PPS;
  static_assert(PPS == 2 && NW == 4 * PPS, "one wave per page of a group");
  constexpr int LPT = C::PAGE_U4 / 64;      // 16-byte loads per lane and page
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 31;
  const int h = lane >> 5;
  const int R = it.nq * a.G;                       // rows of the whole row group
  const int page0 = it.page0, page1 = it.page1;
  const int Rw = min(32, R - wave * 32);           // rows this wave owns (<= 0: none)
  const bool wave_active = Rw > 0;

  const uint32_t lds0 = lds_address(smem);  // [ROWS_BUFS] stages
  typedef const __attribute__((address_space(4))) int32_t* const_i32;  // (block tables: no kernel writes them)
  const const_i32 bt = (const_i32)(uintptr_t)(a.kv.block_tables + (long)it.s * a.kv.max_blocks_per_seq);
  const uint8_t* owner_row = (!SEQ && a.slot_owner) ? uniform_ptr(a.slot_owner + (long)it.s * a.owner_stride) : nullptr;
  // The rows of a group are packed in the order of their slots: the last row's slot bounds what any row
  // of the group may see.  Slots past it have never been written (the tail of the last page) and may hold
  // anything; their V rows are cleared on the way into LDS (zero weight times a NaN would be a NaN).
  const int last_slot = load_word_uniform(a.logical_slot + it.q0 + it.nq - 1);

  // Pairs of pages of the segment, numbered without the ones no row of the group sees: whole sequences lay a
  // stage's branches one after the other, so between the start of a stage and the first branch that the group
  // has rows in lies a run of sibling tokens.  (Under the shared mask, without owner tags, rows see their siblings.)
  int npairs = (page1 - page0 + 1) >> 1;
  int hole_at = npairs, hole = 0;
  if (SEQ && a.slot_owner) {
    const int b0 = load_word_uniform(a.row_base + it.q0), b1 = load_word_uniform(a.row_base + it.q0 + it.nq - 1);
    const int lo0 = load_word_uniform(a.row_lo + it.q0);
    const int first = page0 >> 1;  // (a piece starts with a whole pair)
    const int from = max(((b0 + 31) >> 5) - first, 0), to = min((lo0 >> 5) - first, npairs);
    if (b0 == b1 && to > from) {
      hole_at = from;
      hole = min(to - from, npairs - 1);  // (a piece that the group sees nothing of keeps one pair, all of it masked)
      hole_at = min(hole_at, npairs - hole);
    }
    npairs -= hole;
  }
  auto page_of_pair = [&](int p) -> int { return page0 + 2 * (p < hole_at ? p : p + hole); };

  // ---- staging.  Group i holds the K pages of pairs 2 i + 1 and 2 i + 2 and the V pages of pairs 2 i - 1 and
  // 2 i (what the two steps of the group multiply); wave w fetches one page of it.  Pages outside the segment
  // are fetched as the nearest one inside.  Their scores are not used; V pages that a step multiplies all the same, with
  // weight zero (pair -1 by the first full step, the second page of an odd last pair), are zeros in LDS.
  const bool l_is_k = wave < 4;
  const int l_pair = (wave >> 1) & 1;
  const int n_last = npairs - 1;
  auto page_of_group = [&](int i) -> int {
    const int p = min(max(2 * i + l_pair + (l_is_k ? 1 : -1), 0), n_last);
    return min(page_of_pair(p) + (wave & 1), page1 - 1);
  };
  const char* const pool = (const char*)(l_is_k ? a.kv.k : a.kv.v) + (long)it.h * C::PAGE_B;
  const uint32_t l_at = lds0 + (l_is_k ? 0 : PPS * C::PAIR_B) + l_pair * C::PAIR_B + (wave & 1) * C::PAGE_B;
  // Which 16 bytes of its page the lane fetches with the first load; with the k-th, 1024 k bytes on, and with the
  // chunk order of the rows there (bit 2 of a K row's order changes with every load).
  uint32_t goff;
  {
    const int row = lane / C::CH;
    goff = row * (D * 2) + ((lane % C::CH ^ (l_is_k ? C::kswz(row) : C::vswz(row))) << 4);
  }
  const uint32_t goff_flip = l_is_k ? 64 : 0;

  auto buffer_of = [&](int i) -> int { return i & (ROWS_BUFS - 1); };
  const int i_last = npairs >> 1;
  // Block ids of the wave's pages of groups ids_from .. ids_from + 63, one per lane.  (A scalar load per group was waited for
  // with the first operands of the next: LDS reads and scalar loads are counted together.  64-sequence chunk 1 449 -> 1 438
  // us, 64 whole sequences 24.0 -> 23.9 ms.)
  int ids_from = -1;
  int ids = bt[page_of_group(ids_from + lane)];

  // ---- the loads of the start: this wave's row descriptors and Q operands, which go straight to registers, then its pages
  // of the first two groups.  They return in that order, and a wait for a descriptor, which the compiler counts without
  // the pages it does not know of, ends when the Q operands are there at the latest: what the rows have in common is
  // worked out while the pages are on their way (first scores 7.1 -> 5.3 us after the launch's start; launches, us: stage
  // opening over 12 sequences 59.6 -> 58.9, eight prompts 138.3 -> 137.3, three whole sequences 45.5 -> 45.1).
  __syncthreads();  // LDS of the previous segment is free
  bf16x8 qr[C::KSTEPS];
  int slot, branch = 0, base = it.L, lo = 0;
  {
    const int rr = min(wave * 32 + c, R - 1);  // padding rows (and idle waves) repeat the last row
    const int qi = div_by_g(a, rr), q = it.q0 + qi;
    const int head = it.h * a.G + rr - qi * a.G;
    slot = a.logical_slot[q];
    if (SEQ) {
      // (no owner tags: the shared mask, every row is treated like a main-branch row)
      base = a.slot_owner ? a.row_base[q] : -1;
      lo = a.slot_owner ? a.row_lo[q] : -1;
    } else {
      branch = a.q_branch[q];
    }
    const u32x4* qsrc = (const u32x4*)a.q + ((long)q * a.kv.num_q_heads + head) * C::CH + h;
#pragma unroll
    for (int t = 0; t < C::KSTEPS; ++t) qr[t] = __builtin_bit_cast(bf16x8, qsrc[2 * t]);
  }
  auto send = [&](int i) {  // one group after the other
    if (i > i_last) return;
    if (i - ids_from == 64) {
      ids_from = i;
      ids = bt[page_of_group(i + lane)];
      __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0), here: where the register is read it would be waited for in every group
      asm volatile("" : "+v"(ids));
    }
    const int block = __builtin_amdgcn_readlane(ids, i - ids_from);
    const char* src = pool + (long)min(max(block, 0), a.kv.num_blocks - 1) * a.kv.num_kv_heads * C::PAGE_B;
#pragma unroll
    for (int k = 0; k < LPT; ++k) load_to_lds(src + k * 1024, goff ^ (k * goff_flip), l_at + buffer_of(i) * C::STAGE_B + k * 1024);
  };
  auto clear_v = [&](int i, int k) {
    *(__attribute__((address_space(3))) u32x4*)(uintptr_t)(l_at + buffer_of(i) * C::STAGE_B + k * 1024 + lane * 16) =
        u32x4{0u, 0u, 0u, 0u};
  };
  const int first_branch = !SEQ && a.cu_branches ? load_word_uniform(a.cu_branches + it.s) : 0;
  send(-1);
  if (!l_is_k && l_pair == 0) {  // V of pair -1, which the first full step multiplies with weights zero
#pragma unroll
    for (int k = 0; k < LPT; ++k) clear_v(0, k);
    // (no load in flight for group 0 here: this wave's wait for group -1, whose V pages nobody reads, may come up early)
  } else {
    send(0);
  }

  int tag = 0;
  if (SEQ) {
    if (base < 0) base = lo = slot;
  } else {
    tag = (branch < 0 || !a.cu_branches) ? 0 : branch - first_branch + 1;
  }
  // What the wave's rows have in common decides which pairs need a mask and which can be left out:
  //   mask_from  every key below this slot is visible to every row (below every row's stage and slot);
  //   slot_hi    no key above this slot is visible to any row;
  //   base_hi    the latest stage start among the rows.  A row of an earlier stage lies below it, so keys
  //              from base_hi on are visible, if at all, only to the rows of that latest stage, and only
  //              from their branches: [own_lo, own_hi] is the range of those rows' tags, or own_lo the first
  //              slot any of their branches starts at.
  // Rows lie in the order of their slots, and so of their stages and, within one, of their branches: the first and the last
  // row tell all of it.  (Padding rows are the last again.)  Steps with 23 exchanges between lanes instead -> this,
  // us: one chunk of 140 rows behind 2 721 138.2 -> 136.3, one short prompt 49.2 -> 47.2, eight prompts 371.6 -> 366.4, stage
  // opening 258.2 -> 255.5.
  auto of_lane = [](int v, int l) -> int { return __builtin_amdgcn_readlane(v, l); };
  const int base_hi = SEQ ? of_lane(base, 31) : it.L;
  const int mask_from = min(of_lane(slot, 0), SEQ ? of_lane(base, 0) : it.L), slot_hi = of_lane(slot, 31);
  const int own_lo = SEQ ? of_lane(lo, __builtin_ctz((unsigned)__ballot(base == base_hi))) : of_lane(tag, 0);
  const int own_hi = of_lane(tag, 31);

  Rows32<D> rs;
  rs.m_run = -INFINITY;
  rs.l_run = 0.f;
  rs.neg_ref = 0.f;
  rs.limit = -2.f;
#pragma unroll
  for (int mt = 0; mt < C::MT; ++mt)
#pragma unroll
    for (int i = 0; i < 16; ++i) rs.acc[mt][i] = 0.f;

  // LDS addresses of this lane in the stage of the current group (next_group moves them on): K operand of k-step t (row
  // c, chunk 2 t + h), V operand of d-tile mt (key 4 h + (lane % 16) / 4, then the same plus 8; d 32 mt + 16 (lane / 16
  // % 2) + 4 (lane % 4))
  uint32_t ka[C::KSTEPS], va[C::MT];
  {
    const uint32_t first = lds0 + (ROWS_BUFS - 1) * C::STAGE_B;  // group -1
#pragma unroll
    for (int t = 0; t < C::KSTEPS; ++t) ka[t] = first + c * (D * 2) + (((2 * t + h) ^ C::kswz(c)) << 4);
    const int key = 4 * h + ((lane & 15) >> 2);
#pragma unroll
    for (int mt = 0; mt < C::MT; ++mt)
      va[mt] = first + PPS * C::PAIR_B + key * (D * 2) +
               (((4 * mt + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ C::vswz(key)) << 4) + 8 * (lane & 1);
    // (one set of them, that moves: the compiler would keep those of the first stage beside these)
#pragma unroll
    for (int t = 0; t < C::KSTEPS; ++t) asm volatile("" : "+v"(ka[t]));
#pragma unroll
    for (int mt = 0; mt < C::MT; ++mt) asm volatile("" : "+v"(va[mt]));
  }
  auto next_group = [&](int i) {  // from group i's stage to the next
    const int d = buffer_of(i) == ROWS_BUFS - 1 ? -(ROWS_BUFS - 1) * C::STAGE_B : C::STAGE_B;
#pragma unroll
    for (int t = 0; t < C::KSTEPS; ++t) ka[t] += d;
#pragma unroll
    for (int mt = 0; mt < C::MT; ++mt) va[mt] += d;
  };
  auto k_operand = [&](int u, int t) { return lds_operand(ka[t] + u * C::PAIR_B); };
  auto v_operand = [&](int u, int j) { return rows_v_operand<D>(va[j % C::MT] + u * C::PAIR_B + (j / C::MT) * C::PAGE_B); };

  // owner tags of a group's K pairs that reach into the branch region
  auto tags_of = [&](int i, u32x4 (&t)[PPS][2]) {
    if (SEQ || !owner_row) return;
#pragma unroll
    for (int u = 0; u < PPS; ++u) {
      const int p = 2 * i + 1 + u;
      const int P = page0 + 2 * p;
      if (p >= 0 && p < npairs && (P + 2) * ASPD_BLOCK > mask_from) {
        t[u][0] = load_tags_uniform(owner_row + P * ASPD_BLOCK);
        t[u][1] = load_tags_uniform(owner_row + min(P + 1, page1 - 1) * ASPD_BLOCK);  // stays inside the owner row
      }
    }
  };
  auto lane_own = [&](const u32x4 (&t)[2], uint32_t (&own)[4]) {  // the tags of the lane's sixteen keys
#pragma unroll
    for (int b = 0; b < 4; ++b) own[b] = h ? t[b >> 1][2 * (b & 1) + 1] : t[b >> 1][2 * (b & 1)];
  };
  // Whether the wave's rows see pair p at all (bit 0) and whether some of them only in part (bit 1).
  auto look = [&](int p, const u32x4 (&t)[2]) -> int {
    if (p < 0 || p >= npairs) return 0;
    const int P = page_of_pair(p);
    const int k0 = P * ASPD_BLOCK;
    if (k0 > slot_hi) return 0;
    if (k0 + 2 * ASPD_BLOCK <= mask_from && P + 1 < page1) return 1;
    if (k0 >= base_hi) {  // wholly inside the latest stage: is any key of a branch that the wave has rows in?
      if (SEQ) {
        if (k0 + 2 * ASPD_BLOCK <= own_lo) return 0;
      } else if (owner_row && own_lo > 0) {
        uint32_t own[4];
        lane_own(t, own);
        uint32_t over = 0xffffffffu;  // how far the lane's tags lie above own_lo at least (below it: very far)
#pragma unroll
        for (int i = 0; i < 16; ++i) over = min(over, ((own[i >> 2] >> (8 * (i & 3))) & 0xff) - (uint32_t)own_lo);
        const bool mine = over <= (uint32_t)(own_hi - own_lo);
        if (!__any(mine)) return 0;
      }
    }
    return 3;
  };

  f32x16 s0, s1;         // scores of the pair whose weights are next (even, odd)
  bf16x8 p0[2], p1[2];   // weights of the pair whose value products are next (even, odd)
  u32x4 tg[PPS][2];      // owner tags of the group's K pairs
  u32x4 tc[2];           // owner tags of the pair whose weights are next
  int see_prev = 0, see = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) s0[i] = s1[i] = 0.f;
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int i = 0; i < 8; ++i) p0[u][i] = p1[u][i] = (__bf16)0.f;
  tc[0] = tc[1] = u32x4{0, 0, 0, 0};
#pragma unroll
  for (int u = 0; u < PPS; ++u) tg[u][0] = tg[u][1] = u32x4{0, 0, 0, 0};

  // Step p (slot u of its group): scores of pair p + 1 (into `s_next`), value products of pair p - 1 (weights `p_prev`),
  // softmax of pair p.  In a full step all three take part.  Its order is written out, one slot per matrix
  // instruction, and held by the scheduling barriers: score and value products in turn (neighbours never wait for each
  // other), LDS operands some products ahead of their use, and in every slot its share of the softmax.  Left to
  // itself the compiler fetches each operand right before its product, and the wave waits for LDS sixteen times a step.
  constexpr int NP = C::KSTEPS;  // score products of a pair, and as many value products
  constexpr int RK = 4, RV = 2;  // score and value products their operands are fetched ahead
  static_assert(NP == 2 * C::MT && NP % RK == 0 && NP % RV == 0 && 16 % (2 * NP) == 0, "slots of a full step");
  bf16x8 kf[RK], vf[RV];
  f32x16 z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = 0.f;
  auto fetch_first = [&](int u) {
#pragma unroll
    for (int t = 0; t < RK; ++t) kf[t] = k_operand(u, t);
#pragma unroll
    for (int t = 0; t < RV; ++t) vf[t] = v_operand(u, t);
  };
  // `ahead`: the operands are there, and the first ones of slot 1 are fetched on the way.  The exponents are formed a slot
  // before their weights, so that nothing in a slot waits for anything in it, and the additions are held where they stand
  // (left to itself the compiler puts all sixteen, one waiting for the other, behind the last product).  Three whole
  // sequences 129.8 -> 126.7 us, 64-sequence chunk 1 438 -> 1 426, eight prompts 375.6 -> 371.7, 64 whole sequences 23.9 ->
  // 23.7 ms.
  auto step_full = [&](int u, bool ahead, const f32x16& s_cur, f32x16& s_next, const bf16x8 (&p_prev)[2], bf16x8 (&p_cur)[2]) {
    constexpr int PER = 16 / (2 * NP);  // weights per slot
    float sum[2] = {0.f, 0.f}, x[PER], w_last = 0.f;
    auto exponent = [&](int i) { return fmaf(s_cur[i], a.scale_log2, rs.neg_ref); };
    auto weights = [&](int slot_index) {
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        const int i = slot_index * PER + e;
        const float w = __builtin_amdgcn_exp2f(x[e]);
        if (i + PER < 16) x[e] = exponent(i + PER);
        p_cur[i >> 3][i & 7] = (__bf16)w;
        if (i > 0) {
          sum[i & 1] += w_last;
          asm volatile("" : "+v"(sum[i & 1]));
        }
        w_last = w;
        // (converted here and not after the test of the sum, where sixteen registers would hold them until then)
        if ((i & 7) == 7) asm volatile("" : "+v"(p_cur[i >> 3]));
      }
    };
#pragma unroll
    for (int e = 0; e < PER; ++e) x[e] = exponent(e);
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      s_next = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[j % RK], qr[j], j == 0 ? z : s_next, 0, 0, 0);
      if (j + RK < NP) kf[j % RK] = k_operand(u, j + RK);
      else if (ahead) kf[j % RK] = k_operand(1, j + RK - NP);
      weights(2 * j);
      __builtin_amdgcn_sched_barrier(0);
      rs.acc[j % C::MT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[j % RV], p_prev[j / C::MT], rs.acc[j % C::MT], 0, 0, 0);
      if (j + RV < NP) vf[j % RV] = v_operand(u, j + RV);
      else if (ahead) vf[j % RV] = v_operand(1, j + RV - NP);
      weights(2 * j + 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    return sum[0] + sum[1] + w_last;
  };
  // The same for pairs that need a mask or are not seen at all, one part after the other.
  auto step = [&](int p, int u, const u32x4 (&tn)[2], f32x16& s_cur, f32x16& s_next, const bf16x8 (&p_prev)[2],
                  bf16x8 (&p_cur)[2]) {
    const int see_next = look(p + 1, tn);
    if (see_prev) {
#pragma unroll
      for (int t = 0; t < RV; ++t) vf[t] = v_operand(u, t);
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        rs.acc[j % C::MT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[j % RV], p_prev[j / C::MT], rs.acc[j % C::MT], 0, 0, 0);
        if (j + RV < NP) vf[j % RV] = v_operand(u, j + RV);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (see) {
      if (see & 2) {
        // No short-circuits: they become branches on the execution mask, one behind the other for sixteen keys, which took
        // more than the rest of a masked pair (1 000 to 1 600 cycles of it by the clock in the kernel).  Four layers,
        // before -> after: 8/8 heads, 27 sequences of 200 to 430 tokens, chunks of 4 to 16 in 2 to 8 branches
        // 213.6 -> 200.3 us; 16/4 heads of 64, 20 sequences of 100 to 2500: 226.1 -> 205.6.
        const int k0 = page_of_pair(p) * ASPD_BLOCK + 4 * h;
        const int n_end = min(slot, page1 * ASPD_BLOCK - 1) - k0;
        const int n_base = (SEQ || tag != 0 ? base : 0x7fffffff) - k0, n_lo = lo - k0;
        uint32_t own[4];
        lane_own(tc, own);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int e = 8 * (i >> 2) + (i & 3);
          const int o = (int)((own[i >> 2] >> (8 * (i & 3))) & 0xff);
          const int vis = (int)(e <= n_end) & ((int)(e < n_base) | (SEQ ? (int)(e >= n_lo) : (int)(o == tag)));
          s_cur[i] = vis ? s_cur[i] : -INFINITY;
        }
      }
      float sum = rows_weights<D>(s_cur, rs, p_cur, a.scale_log2);
      if (__any(sum > rs.limit)) sum = rows_raise<D>(s_cur, rs, p_cur, a.scale_log2);
      rs.l_run += sum;
    }
    if (see_next) {
#pragma unroll
      for (int t = 0; t < RK; ++t) kf[t] = k_operand(u, t);
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        s_next = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[j % RK], qr[j], j == 0 ? z : s_next, 0, 0, 0);
        if (j + RK < NP) kf[j % RK] = k_operand(u, j + RK);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    see_prev = see;
    see = see_next;
    tc[0] = tn[0];
    tc[1] = tn[1];
  };

  // One barrier per group: every wave has its page of the group in LDS, and is done with the stage that the group two
  // further on goes to.  The V rows of slots past the last row's or past the segment are cleared before it: they may
  // hold anything, or an infinity that belongs to another slot, and zero times either would be a NaN.
  const int v_last = min(last_slot, page1 * ASPD_BLOCK - 1);
  auto arrive = [&](int i, bool tail) {
    if (i + 1 <= i_last) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LPT) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (tail && !l_is_k) {
      const int key0 = (page_of_pair(2 * i - 1 + l_pair) + (wave & 1)) * ASPD_BLOCK;
      if (key0 + ASPD_BLOCK > v_last + 1) {
#pragma unroll
        for (int k = 0; k < LPT; ++k)
          if (key0 + (64 * k + lane) / C::CH > v_last) clear_v(i, k);
      }
    }
    __syncthreads();
    send(i + 2);
  };
  auto general_groups = [&](int from, int to) {
    for (int i = from; i < to; ++i) {
      tags_of(i, tg);
      arrive(i, true);
      if (wave_active) {
        if (i >= 0) step(2 * i, 0, tg[0], s0, s1, p1, p0);
        step(2 * i + 1, 1, tg[1], s1, s0, p0, p1);
      }
      next_group(i);
    }
  };
  // Groups whose two steps touch only pairs that every row of this wave sees in full (the leading pairs that lie
  // below mask_from): pairs 2 i - 1 .. 2 i + 2.  The range differs between the waves of a workgroup; every group
  // costs one barrier and is staged the same way in either kind of step.
  const int open_pairs = min(hole_at, (min(page1, mask_from / ASPD_BLOCK) - page0) >> 1);
  const int i_open = wave_active ? (open_pairs - 1) >> 1 : 0;  // 2 i + 2 <= open_pairs - 1
  // The Q operands are there since the first descriptor was; the compiler would wait for them where they are first used,
  // and with them for the group that is sent for in between.
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int t = 0; t < C::KSTEPS; ++t) asm volatile("" : "+v"(qr[t]));
  general_groups(-1, 0);  // (the scores of pair 0)
  int i = 0;
  if (i_open > 0) {
    for (; i < i_open; ++i) {
      arrive(i, false);
      fetch_first(0);
      float sum = step_full(0, true, s0, s1, p1, p0);
      if (__any(sum > rs.limit)) sum = rows_raise<D>(s0, rs, p0, a.scale_log2);
      rs.l_run += sum;
      sum = step_full(1, false, s1, s0, p0, p1);
      if (__any(sum > rs.limit)) sum = rows_raise<D>(s1, rs, p1, a.scale_log2);
      rs.l_run += sum;
      next_group(i);
    }
    see_prev = 1;
    tags_of(i - 1, tg);
    see = look(2 * i, tg[1]);
    tc[0] = tg[1][0];
    tc[1] = tg[1][1];
  }
  general_groups(i, i_last + 1);

  // ---- every wave writes its own rows
  int taken = 0;
  if (take_from && tid == 0) taken = atomicAdd(take_from, 1);
  if (!wave_active) return taken;
  rs.l_run = over_halves(rs.l_run, [](float x, float y) { return x + y; });
  const int r = wave * 32 + c;  // row inside the row group
  const Result to = result();
  if (to.complete) {
    // Four consecutive bf16 of a row in a lane would be stored eight bytes at a time, 32 rows at once.  So halves change
    // places twice: of lanes 32 apart, which makes sixteen consecutive bytes of two, and of lanes 16 apart, which leaves four
    // lanes with 64 consecutive bytes of a row, sixteen rows at once.  (Bound by the lines that the store instructions
    // touch, 32 each before: a workgroup took 3.7 us for its 64 KB, and its next item's loads waited behind them.  One
    // attention call: eight prompts 136 -> 129 us, 256 items of four pages 18.3 -> 15.1, three whole sequences 46 -> 44.)
    const float inv = 1.f / rs.l_run;
    const int part = 2 * ((lane >> 4) & 1) + h;  // which of a row's four 16-byte pieces the lane ends up with
    char* dst[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int rr = wave * 32 + min((lane & 15) + 16 * i, Rw - 1);
      const int qi = div_by_g(a, rr);
      dst[i] = (char*)a.out + (((long)(it.q0 + qi) * a.kv.num_q_heads + it.h * a.G + rr - qi * a.G) * D) * 2 + 16 * part;
    }
    const bool first = (lane & 15) < Rw, second = (lane & 15) + 16 < Rw;
#pragma unroll
    for (int mt = 0; mt < C::MT; ++mt) {
      unsigned w[4][2];  // d = 32 mt + 8 b + 4 h + 0 .. 3
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
          const bf16x2 v = {(__bf16)(rs.acc[mt][4 * b + 2 * e] * inv), (__bf16)(rs.acc[mt][4 * b + 2 * e + 1] * inv)};
          w[b][e] = __builtin_bit_cast(unsigned, v);
        }
      u32x4 piece[2];  // of d = 32 mt + 8 (b + h) .. + 7, b = 0 and 2
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const auto x = __builtin_amdgcn_permlane32_swap(w[2 * i][e], w[2 * i + 1][e], false, false);
          const unsigned x0 = x[0], x1 = x[1];
          piece[i][e] = x0;
          piece[i][2 + e] = x1;
        }
      u32x4 lo, hi;  // rows 0 .. 15 and 16 .. 31
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const auto x = __builtin_amdgcn_permlane16_swap(piece[0][e], piece[1][e], false, false);
        const unsigned x0 = x[0], x1 = x[1];
        lo[e] = x0;
        hi[e] = x1;
      }
      if (first) *(u32x4*)(dst[0] + 64 * mt) = lo;
      if (second) *(u32x4*)(dst[1] + 64 * mt) = hi;
    }
    if (a.lse && h == 0 && c < Rw) {
      const int qi = div_by_g(a, r);
      a.lse[(long)(it.q0 + qi) * a.kv.num_q_heads + it.h * a.G + r - qi * a.G] = (rs.m_run + log2f(rs.l_run)) * LN2;
    }
  } else {
    // A row's accumulators lie in lanes c and c + 32, four floats of eight each: stores of them write half lines, which
    // costs a write-through store as much as whole ones.  So rows 16 .. 31 of one register change places with rows 0 .. 15
    // of the next, and four lanes hold sixteen consecutive floats of one row (10 sequences of up to 600 tokens, chunks
    // of 2 to 9 tokens per branch, items split over three workgroups: 33.9 -> 31.4 us a layer).
    const int row = lane & 15;
    float* dst = partial_acc(to.pslot, wave * 32 + row, D) + 8 * ((lane >> 4) & 1) + 4 * h;
#pragma unroll
    for (int mt = 0; mt < C::MT; ++mt) {
#pragma unroll
      for (int b = 0; b < 4; b += 2) {
        f32x4 lo, hi;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const auto x = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, (float)rs.acc[mt][4 * b + e]),
                                                          __builtin_bit_cast(unsigned, (float)rs.acc[mt][4 * b + 4 + e]), false, false);
          const unsigned x0 = x[0], x1 = x[1];  // (the compiler takes element 0 for a bit cast of x[1] itself)
          lo[e] = __builtin_bit_cast(float, x0);
          hi[e] = __builtin_bit_cast(float, x1);
        }
        if (row < Rw) store_device_scope_x4(dst + 32 * mt + 8 * b, lo);
        if (row + 16 < Rw) store_device_scope_x4(dst + 16 * D + 32 * mt + 8 * b, hi);
      }
    }
    if (h == 0 && c < Rw) store_device_scope_x4(partial_stat(a, to.pslot, r, D), f32x4{rs.m_run, rs.l_run, 0.f, 0.f});
  }
  return taken;
}

template <int D, int NW>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(NW / 4, NW / 4))) void attn_bf16_rows_kernel(
    AttnArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  __shared__ int merge_flag;
  constexpr int THREADS = NW * 64;
  Seg seg;
  int next;
  const int queue = load_word_uniform(a.plan + (long)PLAN_HDR * blockIdx.x + PLAN_HDR_QUEUE);
  const int nseg = plan_begin(a, &seg, &next);
  // In a plan with a queue the d-th item that is no workgroup's first is item d / nwg + 1 of workgroup d % nwg, whose
  // items stand one behind the other in the list.
  const int each = queue / a.nwg, rest = queue - each * a.nwg;
  for (int i = 1; nseg > 0;) {
    const bool complete = seg_complete(seg);
    float* pslot = partial_slot(a, blockIdx.x, seg.page0 == 0 ? 1 : 0, D);
    const int taken = segment_rows<D, NW, false>(a, smem, seg, [=]() -> Result { return {complete, pslot}; },
                                                  queue > 0 ? a.counters + QUEUE_NEXT : nullptr);
    if (!complete && !a.merge_apart) announce_partial<D, true, THREADS, D / 16, 4>(a, seg, &merge_flag);
    int at;
    if (queue == 0) {
      if (i >= nseg) break;
      at = next + i - 1;
      ++i;
    } else {
      if (threadIdx.x == 0) merge_flag = taken;
      __syncthreads();
      const int d = __builtin_amdgcn_readfirstlane(merge_flag);
      if (d >= queue) break;
      at = d % a.nwg * each + min(d % a.nwg, rest) + d / a.nwg;
    }
    seg = plan_segment(a, at);
    if (queue > 0) seg.owner = seg.w_last = seg.page0 == 0 && seg.page1 == seg.np ? (int)blockIdx.x : -1;  // whole items only
    if (!seg_ok(a, seg)) break;
  }
  if (queue == 0) return;
  // the last workgroup to leave puts the queue's words back to zero for the next launch
  if (threadIdx.x == 0) {
    const int gone = atomicAdd(a.counters + QUEUE_DONE, 1);
    if (gone == a.nwg - 1) {
      atomicExch(a.counters + QUEUE_NEXT, 0);
      atomicExch(a.counters + QUEUE_DONE, 0);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Whole sequences (teacher forcing, re-prefill): every token of the batch is a query row.  The row
// groups (qpg consecutive tokens of a sequence, one KV head) are listed in the step's plan, longest key
// range first or sequence by sequence; workgroups take them from the list as they become free (the ranges differ by two orders
// of magnitude, so no static split would balance), through counters in the workspace that the last
// workgroup to finish puts back to zero.  Every group is computed whole by one workgroup with the
// row-splitting arithmetic above, but for the longest ones of a launch that has few: their key ranges are cut (the plan's
// list of pieces says where, and is in the order of the pieces' lengths) and the workgroup that brings the last piece
// merges, as in the row-splitting kernel.  PIECES: there may be such a list, and there is room for partial results;
// otherwise every group is taken whole.
// ---------------------------------------------------------------------------------------------
template <int D, int NW, bool PIECES>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(NW / 4, NW / 4))) void attn_bf16_seq_kernel(
    AttnArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  __shared__ int next_item[2], merge_flag;
  // Of a piece: slot of its partial result (-1: the item is a whole row group), and what the merge asks for.  In LDS because
  // the loop over the pages needs the scalar registers.
  __shared__ int held[5];
  const int Hkv = a.kv.num_kv_heads;
  static_assert(SEQ_HDR_PIECES == 4 && SEQ_HDR_HEADS == 5 && SEQ_HDR_PLACES == 6, "in one load with the row groups");
  const i32x8 hdr = load_words8(a.plan);
  const int n_groups = hdr[0];
  // (places of partial results and arrivals were given away for so many heads: with others, or with fewer places, two row
  // groups would count on one word)
  const bool listed = (int)(hdr[SEQ_HDR_HEADS] == Hkv) & (int)(hdr[SEQ_HDR_PLACES] <= a.parts);
  const int n_pieces = PIECES && listed ? min(hdr[SEQ_HDR_PIECES], SEQ_ENTRIES) : 0;
  const int32_t* items = a.plan + SEQ_PLAN_HDR + ((a.NQ + 3) & ~3);
  // Queues.  One per XCD (SEQ_QUEUE_ITEMS), so that the row groups that stream the same pages are on one L2: queue x has the
  // heads of class x modulo a power of two, and where that is less than the queues every second, fourth or eighth row group;
  // head by head.  A workgroup whose queue is empty turns to the next.  With few items, and with pieces, whose order is that of
  // their lengths, there is one for all: who is free next matters more.  64 whole sequences of 1 100 to 9 400 tokens, one
  // queue -> one per XCD: hits in L2 4 -> 89 %, 78 -> 6.4 GB read past it, the clock at the power limit 1.56 -> 1.89 GHz, 21.3
  // -> 16.7 ms (1 130 TFLOP/s).  With fewer heads than XCDs those of a class all stream their head's pages, each for its own row
  // groups, and it gains less: 16 sequences of 4 000 to 12 000 with 2 heads 4.00 -> 3.76 ms, 12 of 8 000 to 16 000 with one
  // 6.40 -> 5.98, 24 of 1 500 to 4 000 with 4 heads 3.80 -> 3.46, 12 of 2 000 to 8 000 with 6 heads 3.91 -> 3.70.
  const bool by_xcd = n_pieces == 0 && (long)n_groups * Hkv >= (long)SEQ_QUEUE_ITEMS * a.nwg;
  const int classes_log2 = min(__builtin_ctz(Hkv), SEQ_QUEUES_LOG2), every_log2 = SEQ_QUEUES_LOG2 - classes_log2;
  auto groups_of = [&](int x) -> int { return (n_groups - (x >> classes_log2) + (1 << every_log2) - 1) >> every_log2; };
  auto length_of = [&](int x) -> int { return by_xcd ? groups_of(x) * (Hkv >> classes_log2) : (n_pieces > 0 ? n_pieces : n_groups) * Hkv; };
  // Item i of queue x; false for one that no plan of the library's own holds (a workgroup that is handed anything else
  // stays inside the call's arrays).
  auto item_of = [&](int x, int i, Seg* seg, int* piece, int* pieces) -> bool {
    int group, head, part = 0;
    *piece = 0;
    *pieces = 1;
    if (by_xcd) {
      const int n = groups_of(x), pass = Hkv >> classes_log2 > 1 ? i / n : 0;
      head = (x & ((1 << classes_log2) - 1)) + (pass << classes_log2);
      group = (x >> classes_log2) + ((i - n * pass) << every_log2);
    } else {
      group = i / Hkv;
      head = i - group * Hkv;
    }
    if (n_pieces > 0) {
      const int word = a.pieces[2 * group + 1];
      group = a.pieces[2 * group];
      *piece = word & 0xff;
      *pieces = (word >> 8) & 0xff;
      part = (int)((unsigned)word >> 16) + head * *pieces;
    }
    const bool in_list = (int)((unsigned)group < (unsigned)n_groups) & (int)(*piece < *pieces) &
                         (int)(*pieces <= SEQ_PIECES_MAX) & (int)((*pieces == 1) | (part + *pieces <= a.parts));
    const i32x4 w = *(const i32x4*)(items + 4 * (in_list ? group : 0));
    seg->s = w[0];
    seg->h = head;
    seg->q0 = w[1];
    seg->nq = w[2];
    seg->np = w[3];
    seg->page0 = 0;
    seg->page1 = seg->np;
    if (*pieces > 1) {
      const int pairs = (seg->np + 1) / 2;
      const float inv = __builtin_amdgcn_rcpf((float)*pieces);
      seg->page0 = 2 * quotient(pairs * *piece, *pieces, inv);
      seg->page1 = min(seg->np, 2 * quotient(pairs * (*piece + 1), *pieces, inv));
    }
    seg->owner = part;
    seg->w_last = part + *pieces - 1;
    seg->L = 0;
    return (int)in_list & (int)(seg->page0 < seg->page1) & (int)(seg->s >= 0) & (int)(seg->s < a.B) & (int)(seg->q0 >= 0) &
           (int)(seg->nq >= 1) & (int)(seg->nq <= a.qpg) & (int)(seg->q0 <= a.NQ - seg->nq) & (int)(seg->np >= 1) &
           (int)(seg->np <= a.kv.max_blocks_per_seq);
  };
  // The first wave finds the next item: thread 0 has taken number `taken` of queue `from`.  Past that queue's end one look at
  // all counters tells which have items left.
  int from = by_xcd ? (int)blockIdx.x % SEQ_QUEUES : 0, taken = 0;
  int* const queues = a.counters + QUEUE_XCD;
  if (threadIdx.x == 0) taken = atomicAdd(queues + from, 1);
  auto find = [&]() {  // by the whole first wave
    int e = __builtin_amdgcn_readfirstlane(taken), x = from;
    while (e >= length_of(x)) {
      unsigned left = 0;
      if (by_xcd) {
        const int other = (x + 1 + (int)threadIdx.x) % SEQ_QUEUES;
        const int gone = __hip_atomic_load(queues + other, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        left = (unsigned)__ballot(gone < length_of(other)) & ((1u << SEQ_QUEUES) - 1);
      }
      if (left == 0) {
        x = -1;
        break;
      }
      x = (x + 1 + __builtin_ctz(left)) % SEQ_QUEUES;
      if (threadIdx.x == 0) taken = atomicAdd(queues + x, 1);
      e = __builtin_amdgcn_readfirstlane(taken);
    }
    if (threadIdx.x == 0) {
      next_item[0] = x;
      next_item[1] = e;
    }
  };
  for (;;) {
    if (threadIdx.x < 64) find();
    __syncthreads();
    from = __builtin_amdgcn_readfirstlane(next_item[0]);
    if (from < 0) break;
    const int e = __builtin_amdgcn_readfirstlane(next_item[1]);
    int* const take_from = queues + from;
    Seg seg;
    int piece, pieces;
    const bool ok = item_of(from, e, &seg, &piece, &pieces);
    if (!ok) {
      __syncthreads();  // everyone has read next_item
      if (threadIdx.x == 0) taken = atomicAdd(take_from, 1);
      continue;
    }
    if (PIECES && threadIdx.x == 0) {
      held[0] = pieces > 1 ? 2 * (seg.owner + piece) + (piece == 0 ? 1 : 0) : -1;
      held[1] = seg.owner;
      held[2] = seg.w_last;
      held[3] = seg.q0;
      held[4] = seg.nq | (seg.h << 16);
    }
    taken = segment_rows<D, NW, true>(a, smem, seg, [&]() -> Result {
      if (!PIECES) return {true, nullptr};
      const int slot = __builtin_amdgcn_readfirstlane(held[0]);
      return {slot < 0, a.partial + (long)slot * a.rows_cap * (D + 4)};
    }, take_from);
    if (PIECES && held[0] >= 0) {
      Seg seg;
      seg.owner = __builtin_amdgcn_readfirstlane(held[1]);
      seg.w_last = __builtin_amdgcn_readfirstlane(held[2]);
      seg.q0 = __builtin_amdgcn_readfirstlane(held[3]);
      const int rows = __builtin_amdgcn_readfirstlane(held[4]);
      seg.nq = rows & 0xffff;
      seg.h = rows >> 16;
      announce_partial<D, true, NW * 64, D / 16, 4>(a, seg, &merge_flag);
    }
  }
  // the last workgroup to leave puts the counters back to zero for the next launch
  if (threadIdx.x == 0) {
    const int gone = atomicAdd(a.counters + QUEUE_DONE, 1);
    if (gone == (int)gridDim.x - 1) {
      for (int x = 0; x < SEQ_QUEUES; ++x) atomicExch(queues + x, 0);
      atomicExch(a.counters + QUEUE_DONE, 0);
    }
  }
}

}  // namespace
