// The streaming bf16 kernel (internal to libaspd): few rows per KV head, the waves of a workgroup split the keys
// (parallel decode, serial decode, narrow chunks).
#pragma once

#include "attn_bf16_math.h"

namespace {

// ---------------------------------------------------------------------------------------------
// Every wave takes pages of its segment, 16 keys of K and V, computes them against all rows of the row group (NT tiles of
// 16 rows) and keeps its own accumulators; the waves are combined once per segment.
//
// Large launches are bound by the page stream, small ones by the chain around it (header, first pages, combination of the
// waves, partial, merge), and that chain by instruction issue: a wave alone on its SIMD issues one instruction in eight
// to nine cycles.  Hence eight waves (two per SIMD) on single pages, where it was four on pairs of pages, with the same
// 64 KB per compute unit on their way; pages, queries and descriptors loaded straight into LDS, which leaves the waves
// 256 registers for everything else; and no cross-lane step, division or barrier that can be had otherwise.  Attention
// alone in graph replay, four waves with pairs in registers -> this, us: one sequence of 2 300 tokens 14.8 -> 9.5; 27
// mixed sequences of up to 3 000, head size 64 16.1 -> 11.7; 16 sequences of 512 to 4 096 45.2 -> 41.7; four of 16 k,
// six branches 52.2 -> 49.6, after the merge 50.7 -> 45.2; 64 sequences of up to 8 192 231 -> 219 (6.4 TB/s).
//
// S^T[key][row] = K * Q^T on 16x16x32 MFMA: lane (c, g) = (lane % 16, lane / 16) holds, of row c, the keys 4 g .. 4 g + 3
// of the page, which is the B-operand layout of O^T[d][row] = V^T * P^T on 16x16x16 MFMA, whose A operand (V^T) comes
// from the LDS transpose read.  The statistics of a row live in the four lanes c, c + 16, c + 32, c + 48.
// ---------------------------------------------------------------------------------------------
constexpr int BLK_WIN = 512;   // pages of a segment whose block ids are in LDS at once

template <int D, int NT>
struct StreamLds {
  static constexpr int NW = STREAM_NW;
  static constexpr int CH = D / 8;                        // 16-byte chunks per row
  static constexpr int PAGE_B = ASPD_BLOCK * D * 2;
  static constexpr int LPP = PAGE_B / 1024;               // loads per page
  static constexpr int STAGE_B = 2 * PAGE_B + 256;        // K page, V page, owner tags (16 bytes, loaded 16 times over)
  static constexpr int LOADS = 2 * LPP + 1;               // loads of a stage
  static constexpr int WAVE_B = 2 * STAGE_B;              // two stages, or the accumulators of two tiles
  static constexpr int RED_ROW = D + 4;                   // floats per row there (the 16 rows a wave writes at once fall
                                                          // on different banks)
  static_assert(WAVE_B >= 2 * 16 * RED_ROW * 4, "two tiles of accumulators");
  static constexpr int Q = NW * WAVE_B;                   // [16 NT] query rows, in pages of sixteen
  static constexpr int BLK = Q + NT * PAGE_B;             // [BLK_WIN] block ids of the window
  static constexpr int SLOT = BLK + BLK_WIN * 4;          // [64] logical slots of the row group's queries
  static constexpr int BRANCH = SLOT + 256;               // [64] their branches
  static constexpr int M = BRANCH + 256;                  // [16 NT][NW] references of the waves
  static constexpr int L = M + 16 * NT * NW * 4;          // [16 NT][NW] sums
  static constexpr int TAKE = L + 16 * NT * NW * 4;       // [64] next page nobody has taken (word 0; see take())
  // (more than half of a compute unit's LDS: one workgroup per compute unit, as the grid is sized for)
  static constexpr int USED = TAKE + 256;
  static constexpr int BYTES = USED > 81 * 1024 ? USED : 81 * 1024;
  // Order of the 16-byte chunks inside a row, so that no operand read has a bank conflict: a K (or Q) read takes one
  // chunk of sixteen rows at a time, a transposing V read two chunks of eight.
  static __device__ __forceinline__ int kswz(int row) { return D == 128 ? (row & 15) : ((row >> 1) & 7); }
  static __device__ __forceinline__ int vswz(int row) { return D == 128 ? 2 * (row & 7) : 2 * ((row >> 1) & 3); }
};

// Largest weight sum of a lane's four keys before the row's reference is raised (see segment_stream).  With 20, and with
// the references raised at a wave's second page in any case, the error against float64 is 1 to 14 % below that of
// references raised at a score 2^6 above (as with pairs of pages), for queries ~ N(0, 1), N(0, 4) and N(0, 36).
constexpr float STREAM_SUM_MAX = 20.f;

template <int D, int NT, bool STREAM>
__device__ __forceinline__ void segment_stream(const AttnArgs& a, char* smem, const Seg& it, bool complete, float* pslot,
                                               int id0, int id1 /* blocks of the wave's first two pages, or what was
                                               thought to be: compared with the block table before the pages count */) {
  using C = StreamLds<D, NT>;
  constexpr int NW = C::NW, THREADS = NW * 64;
  constexpr int KSTEPS = D / 32, MT = D / 16, CH = C::CH;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15;
  const int g = lane >> 4;
  const int R = it.nq * a.G;
  const int page0 = it.page0, np = it.page1 - it.page0, L = it.L;
  const uint32_t lds0 = lds_address(smem);
  const uint32_t stage0 = lds0 + wave * C::WAVE_B;

  // ---- loads of the segment's start; the small ones first, loads return in order
  // lane offsets of a page's loads: load k brings rows k * 64 / CH ...
  uint32_t koff[C::LPP], voff[C::LPP];
#pragma unroll
  for (int k = 0; k < C::LPP; ++k) {
    const int row = lane / CH + k * (64 / CH);
    koff[k] = (lane / CH) * (D * 2) + ((lane % CH ^ C::kswz(row)) << 4);
    voff[k] = (lane / CH) * (D * 2) + ((lane % CH ^ C::vswz(row)) << 4);
  }
  const int32_t* bt = a.kv.block_tables + (long)it.s * a.kv.max_blocks_per_seq + page0;
  {
    // query rows: 1024 bytes of the tile per wave and round
    const char* qsrc = (const char*)a.q + ((long)it.q0 * a.kv.num_q_heads + it.h * a.G) * (D * 2);
#pragma unroll
    for (int j0 = 0; j0 < NT * C::LPP; j0 += NW) {
      const int j = j0 + wave;
      if (j < NT * C::LPP) {
        const int row = j * (64 / CH) + lane / CH;
        const int rr = min(row, R - 1);
        const int qi = div_by_g(a, rr);
        load_to_lds(qsrc, (uint32_t)((qi * a.kv.num_q_heads + rr - qi * a.G) * (D * 2) + ((lane % CH ^ C::kswz(row)) << 4)),
                    lds0 + C::Q + j * 1024);
      }
    }
    if (wave == NW - 1) load4_to_lds(a.logical_slot + it.q0, 4 * min(lane, it.nq - 1), lds0 + C::SLOT);
    if (wave == NW - 2) load4_to_lds(a.q_branch + it.q0, 4 * min(lane, it.nq - 1), lds0 + C::BRANCH);
    load4_to_lds(bt, 4 * min(tid, np - 1), lds0 + C::BLK + wave * 256);
  }
  const char* const own_row = a.slot_owner ? (const char*)(a.slot_owner + (long)it.s * a.owner_stride)
                                           : (const char*)a.logical_slot;  // (no tags: four bytes nobody looks at)
  const uint32_t own_off = a.slot_owner ? 4 * (lane & 3) : 0;
  const int own_step = a.slot_owner ? ASPD_BLOCK : 0;
  auto issue = [&](int page /* of the segment */, int id, uint32_t at) {
    const long block = min(max(id, 0), a.kv.num_blocks - 1);
    const long from = (block * a.kv.num_kv_heads + it.h) * C::PAGE_B;
    page_to_lds<D, STREAM>((const char*)a.kv.k + from, koff, at);
    page_to_lds<D, STREAM>((const char*)a.kv.v + from, voff, at + C::PAGE_B);
    load4_to_lds(own_row + (long)(page0 + page) * own_step, own_off, at + 2 * C::PAGE_B);
  };
  int cur = wave, nxt = wave + NW;  // pages are numbered from the segment's first; past the end: none
  if (cur < np) issue(cur, id0, stage0);
  if (nxt < np) issue(nxt, id1, stage0 + C::STAGE_B);
  // the first two pages of a wave are its own, the others go to whoever is free first
  if (tid == 0) *(__attribute__((address_space(3))) int*)(uintptr_t)(lds0 + C::TAKE) = 3 * NW;
  int ahead = wave + 2 * NW;
  const int first_branch = a.cu_branches ? load_word_uniform(a.cu_branches + it.s) : 0;
  // The rows of a group are packed in the order of their slots.
  const int first_slot = load_word_uniform(a.logical_slot + it.q0);
  const int last_slot = load_word_uniform(a.logical_slot + it.q0 + it.nq - 1);
  const int mask_from = min(L, first_slot);  // keys below this slot are visible to every row of the group

  // what does not depend on the loads: LDS addresses of the lane's operands, per stage a constant further on
  uint32_t ka[KSTEPS], va[MT];
#pragma unroll
  for (int t = 0; t < KSTEPS; ++t) ka[t] = c * (D * 2) + (((4 * t + g) ^ C::kswz(c)) << 4);
  {
    const int key = 4 * g + (c >> 2);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      va[mt] = stage0 + C::PAGE_B + key * (D * 2) + (((2 * mt + ((c & 3) >> 1)) ^ C::vswz(key)) << 4) + 8 * (c & 1);
  }
  int query[NT];  // of the lane's row, within the group
#pragma unroll
  for (int n = 0; n < NT; ++n) query[n] = div_by_g(a, min(16 * n + c, R - 1));
  if (nxt < np) wait_loads<2 * C::LOADS>();
  else if (cur < np) wait_loads<C::LOADS>();
  else wait_loads<0>();
  __syncthreads();

  // ---- the rows: queries as operands, and what each row may see
  auto lds_int = [&](uint32_t at) -> int { return *(const __attribute__((address_space(3))) int*)(uintptr_t)at; };
  constexpr bool Q_HELD = NT * D <= 256;  // in registers (more of them would spill)
  bf16x8 qf[NT][KSTEPS];
  const uint32_t q_back = lds0 + C::Q - stage0;
  int slot[NT], tag[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) {
#pragma unroll
    for (int t = 0; t < KSTEPS; ++t)
      if (Q_HELD) qf[n][t] = lds_operand(lds0 + C::Q + n * C::PAGE_B + ka[t]);
    slot[n] = lds_int(lds0 + C::SLOT + 4 * query[n]);
    const int b = lds_int(lds0 + C::BRANCH + 4 * query[n]);
    tag[n] = (b < 0 || !a.cu_branches) ? 0 : b - first_branch + 1;
  }
#pragma unroll
  for (int t = 0; t < KSTEPS; ++t) ka[t] += stage0;
  f32x4 acc[NT][MT];
  float m_run[NT], l_run[NT], neg_ref[NT], limit[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    m_run[n] = -INFINITY;
    l_run[n] = 0.f;
    neg_ref[n] = 0.f;
    limit[n] = -2.f;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[n][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // Next page nobody has taken (may be past the end).  Every lane adds to a word of its own and lane 0's counts: without
  // a branch around the addition.
  auto take = [&]() -> int {
    return __hip_atomic_fetch_add((__attribute__((address_space(3))) int*)(uintptr_t)(lds0 + C::TAKE + 4 * lane), 1,
                                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  auto block_of = [&](int page, int wpages) -> int { return lds_int(lds0 + C::BLK + 4 * min(page, wpages - 1)); };

  // One page, from stage S of the wave.
  auto compute = [&](auto S, int page) {
    constexpr uint32_t at = decltype(S)::value * C::STAGE_B;
    const int k_first = (page0 + page) * ASPD_BLOCK;
    // Slots past the last row's own have never been written (the tail of the last page) and may hold anything: their V
    // rows enter the second product with weight zero, and zero times a NaN is a NaN, so they are cleared.  (Their K rows
    // only reach scores that the mask replaces.)
    if (k_first + ASPD_BLOCK > last_slot + 1) {
#pragma unroll
      for (int k = 0; k < C::LPP; ++k)
        if (k_first + lane / CH + k * (64 / CH) > last_slot)
          *(__attribute__((address_space(3))) u32x4*)(uintptr_t)(stage0 + at + C::PAGE_B + k * 1024 + lane * 16) =
              u32x4{0u, 0u, 0u, 0u};
    }
    bf16x8 kf[KSTEPS];
#pragma unroll
    for (int t = 0; t < KSTEPS; ++t) kf[t] = lds_operand(ka[t] + at);
    s16x4 vf[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) vf[mt] = lds_operand_transposed(va[mt] + at);
    f32x4 s[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) s[n] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (!Q_HELD) {
#pragma unroll
      for (int t = 0; t < KSTEPS; ++t) {
        const uint32_t q_at = ka[t] + q_back;
#pragma unroll
        for (int n = 0; n < NT; ++n) qf[n][t] = lds_operand(q_at + n * C::PAGE_B);
      }
    }
#pragma unroll
    for (int t = 0; t < KSTEPS; ++t)
#pragma unroll
      for (int n = 0; n < NT; ++n) s[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[t], qf[n][t], s[n], 0, 0, 0);
    if (k_first + ASPD_BLOCK > mask_from) {  // (only pages that reach into the branch region or past a row's slot)
      const uint32_t own = (uint32_t)lds_int(stage0 + at + 2 * C::PAGE_B + 4 * g);
      const int k0 = k_first + 4 * g;
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        // (no short-circuits: they become branches on the execution mask)
        const int n_end = slot[n] - k0, n_base = (tag[n] == 0 ? 0x7fffffff : L) - k0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int o = (int)((own >> (8 * e)) & 0xff);
          const int vis = (int)(e <= n_end) & ((int)(e < n_base) | (int)(o == tag[n]));
          s[n][e] = vis ? s[n][e] : -INFINITY;
        }
      }
    }
    // Running softmax with a lazily raised reference per row (log2 domain, scaled scores; not necessarily the row's
    // maximum; the same in the four lanes of a row).  The weights are formed first, and their sum, which the row needs
    // anyway, tells whether the reference has to go up: while no lane's four weights sum to more than STREAM_SUM_MAX none
    // of them exceeds it.
    s16x4 p[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      auto weights = [&]() -> float {
        float sum = 0.f;
        typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
        bf16x4 w4;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float w = __builtin_amdgcn_exp2f(fmaf(s[n][e], a.scale_log2, neg_ref[n]));
          sum += w;
          w4[e] = (__bf16)w;
        }
        p[n] = __builtin_bit_cast(s16x4, w4);
        return sum;
      };
      float sum = weights();
      if (__any(sum > limit[n])) {
        float mx = fmaxf(fmaxf(s[n][0], s[n][1]), fmaxf(s[n][2], s[n][3]));
        mx = over_quarters(mx, [](float x, float y) { return fmaxf(x, y); }) * a.scale_log2;  // scale > 0
        const float m_new = fmaxf(m_run[n], mx);
        const float ref = exp2_safe_ref(m_new);
        const float alpha = __builtin_amdgcn_exp2f(m_run[n] - ref);
        m_run[n] = m_new;
        neg_ref[n] = -ref;
        l_run[n] *= alpha;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[n][mt] *= alpha;
        limit[n] = __any(m_new == -INFINITY) ? -2.f : (limit[n] < -1.f ? -1.f : STREAM_SUM_MAX);
        sum = weights();
      }
      l_run[n] += sum;
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int n = 0; n < NT; ++n)
        acc[n][mt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vf[mt], p[n], acc[n][mt], 0, 0, 0);
  };

  // ---- the stream, in windows of block ids (normally one).  Pages are handed out dynamically, two hand-outs ahead: a
  // wave that gets its data sooner takes the next page sooner, so that the waves finish together whatever the memory
  // system does to each of them.
  for (int w0 = 0;;) {  // w0: first page of the window; cur, nxt and ahead count from it
    const int wpages = min(np - w0, BLK_WIN);
    if (w0 > 0) {
      __syncthreads();  // every wave is done with the previous window's ids and counter
      load4_to_lds(bt + w0, 4 * min(tid, wpages - 1), lds0 + C::BLK + wave * 256);
      if (tid == 0) *(__attribute__((address_space(3))) int*)(uintptr_t)(lds0 + C::TAKE) = 3 * NW;
      wait_loads<0>();
      __syncthreads();
      cur = wave;
      nxt = wave + NW;
      ahead = wave + 2 * NW;
    }
    {
      const int b0 = __builtin_amdgcn_readfirstlane(block_of(cur, wpages));
      const int b1 = __builtin_amdgcn_readfirstlane(block_of(nxt, wpages));
      if (w0 > 0 || (cur < wpages && b0 != id0) || (nxt < wpages && b1 != id1)) {
        wait_loads<0>();  // (pages of other blocks are on their way to the same place)
        if (cur < wpages) issue(w0 + cur, b0, stage0);
        if (nxt < wpages) issue(w0 + nxt, b1, stage0 + C::STAGE_B);
      }
    }
    auto turn = [&](auto S) {
      const int id_v = block_of(ahead, wpages), taken_v = take();
      if (nxt < wpages) wait_loads<C::LOADS>();
      else wait_loads<0>();
      compute(S, w0 + cur);
      const int id = __builtin_amdgcn_readfirstlane(id_v);
      // the stage has been read; it is refilled at once
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (ahead < wpages) issue(w0 + ahead, id, stage0 + decltype(S)::value * C::STAGE_B);
      cur = nxt;
      nxt = ahead;
      ahead = __builtin_amdgcn_readfirstlane(taken_v);
    };
    // pages are handed out in increasing order: once one is past the end, all later ones are
    while (cur < wpages) {
      turn(std::integral_constant<int, 0>{});
      if (cur >= wpages) break;
      turn(std::integral_constant<int, 1>{});
    }
    w0 += BLK_WIN;
    if (w0 >= np) break;
  }

  // ---- combine the waves.  Every wave puts its accumulators, as they are, where its stages were and its statistics
  // beside them; behind a barrier a thread takes a 16-byte chunk of a row and weighs the waves' parts itself.
  const float* const wm = (const float*)(smem + C::M);
  const float* const wl = (const float*)(smem + C::L);
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    const float l = over_quarters(l_run[n], [](float x, float y) { return x + y; });
    if (g == 0) {
      ((float*)wm)[(16 * n + c) * NW + wave] = m_run[n];
      ((float*)wl)[(16 * n + c) * NW + wave] = l;
    }
  }
  constexpr int CPR = D / 4;                     // chunks per row
  constexpr int TPP = THREADS / (16 * CPR) > 1 ? THREADS / (16 * CPR) : 1;  // tiles the threads cover at once
  static_assert(THREADS == TPP * 16 * CPR && TPP <= 2, "one chunk per thread");
  float* const red = (float*)(smem + wave * C::WAVE_B);
  const float* const red0 = (const float*)smem;
#pragma unroll
  for (int n0 = 0; n0 < NT; n0 += 2) {           // two tiles a round
    if (16 * n0 >= R) break;
    if (n0 > 0) __syncthreads();
#pragma unroll
    for (int n = n0; n < n0 + 2 && n < NT; ++n)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        *(f32x4*)&red[(16 * (n - n0) + c) * C::RED_ROW + 16 * mt + 4 * g] = acc[n][mt];
    __syncthreads();
    // (the index arithmetic below depends on nothing the main loop produces; tying it to a value defined here keeps it,
    // and the registers it needs, out of that loop)
    int tid_here = tid;
    asm volatile("" : "+v"(tid_here)::"memory");
#pragma unroll
    for (int n = n0; n < n0 + 2 && n < NT; n += TPP) {
      const int rl = 16 * (n - n0) + tid_here / CPR;  // row of the round
      const int r = 16 * n0 + rl;
      const int d0 = 4 * (tid_here % CPR);
      if (r >= R || r >= 16 * NT) continue;
      float m8[NW], mg = -INFINITY, lg = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) m8[w] = wm[r * NW + w];
#pragma unroll
      for (int w = 0; w < NW; ++w) mg = fmaxf(mg, m8[w]);
      const float mref = exp2_safe_ref(mg);
      f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float f = __builtin_amdgcn_exp2f(m8[w] - mref);
        lg += wl[r * NW + w] * f;
        o += *(const f32x4*)&red0[w * (C::WAVE_B / 4) + rl * C::RED_ROW + d0] * f;
      }
      if (complete) {
        const int qi = div_by_g(a, r);
        const long row = (long)(it.q0 + qi) * a.kv.num_q_heads + it.h * a.G + r - qi * a.G;
        const float inv = 1.f / lg;
        typedef __attribute__((ext_vector_type(4))) __bf16 out_vec;
        out_vec ov;
#pragma unroll
        for (int e = 0; e < 4; ++e) ov[e] = (__bf16)(o[e] * inv);
        *(out_vec*)((__bf16*)a.out + row * D + d0) = ov;
        if (a.lse && d0 == 0) a.lse[row] = (mg + log2f(lg)) * LN2;
      } else {
        store_device_scope_x4(partial_acc(pslot, r, D) + d0, o);
        if (d0 == 0) store_device_scope_x4(partial_stat(a, pslot, r, D), f32x4{mg, lg, 0.f, 0.f});
      }
    }
  }
}

template <int D, int NT, bool STREAM>
__global__ __launch_bounds__(STREAM_NW * 64) __attribute__((amdgpu_waves_per_eu(STREAM_NW / 4, STREAM_NW / 4))) void
attn_bf16_kernel(AttnArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  __shared__ int merge_flag;
  constexpr int NW = STREAM_NW;
  constexpr int MERGE = D == 128 ? (NT < 3 ? NT : 4) : (NT < 3 ? 1 : 2);  // the rows of a group in one round
  static_assert(2 * NW <= PLAN_IDS, "the plan carries two block ids per wave");
  // One memory round trip after the kernel starts the workgroup knows its first segment and the blocks
  // of each wave's first two pages (scalar loads of the plan header), and the pages, the block ids of
  // the whole segment, the Q rows and the row descriptors all leave together.
  Seg seg;
  int next;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int32_t* ids = a.plan + (long)PLAN_HDR * blockIdx.x + PLAN_HDR_IDS + wave;
  int id0 = load_word_uniform(ids), id1 = load_word_uniform(ids + NW);
  const int nseg = plan_begin(a, &seg, &next);
  if (nseg == 0) return;
  for (int i = 0;;) {
    // the next segment's words are on their way while this one streams
    Seg after = seg;
    if (i + 1 < nseg) after = plan_segment(a, next + i);
    const bool complete = seg_complete(seg);
    float* pslot = partial_slot(a, blockIdx.x, seg.page0 == 0 ? 1 : 0, D);
    segment_stream<D, NT, STREAM>(a, smem, seg, complete, pslot, id0, id1);
    if (!complete) announce_partial<D, true, NW * 64, MERGE, (MERGE == 4 ? 6 : 16 / MERGE)>(a, seg, &merge_flag);
    if (++i >= nseg) break;
    seg = after;
    if (!seg_ok(a, seg)) break;
    const int32_t* bt = a.kv.block_tables + (long)seg.s * a.kv.max_blocks_per_seq;
    id0 = load_word_uniform(bt + min(seg.page0 + wave, seg.page1 - 1));
    id1 = load_word_uniform(bt + min(seg.page0 + wave + NW, seg.page1 - 1));
    __syncthreads();  // LDS of the segment before is free
  }
}

}  // namespace
