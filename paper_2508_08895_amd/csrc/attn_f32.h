// The fp32 kernel (internal to libaspd).
#pragma once

#include "attn_common.h"

namespace {

// ---------------------------------------------------------------------------------------------
// fp32 path: vector ALU, fp32 throughout.  Lane (k = lane % 16, g = lane / 16) owns key k of each
// page and the g-th quarter of head_dim; a row's score is completed across the four quarters with
// two butterfly adds.  Every lane keeps a private running softmax over the keys it has seen
// (one per page) and they are combined once at the end of the segment: over the sixteen lanes of a quarter, which are a
// row of lanes, by data-parallel moves, halving the values a lane is left with at every step, then over the waves
// through LDS.
//
// Small calls only, so what bounds it is a chain of waits: block id, page, combination.  The block ids of a wave's next pages
// are fetched ahead, at head_dim 64 the pages too (at 128 they would not fit the registers beside the accumulators).
// With an LDS slot per lane (256 reads a thread at the end) and nothing fetched ahead -> now, us: 4/4 heads of 64, one
// sequence of 91 tokens 10.2 -> 8.3, two of 530 14.1 -> 12.0; 8/2 heads of 128 18.3 -> 13.6 and 27.2 -> 21.6.  The error
// against float64 went from 2.3e-7 to 1.8e-7 (sums in a tree).
// ---------------------------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ float lane_move(float v) {  // every lane has a source
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
// One step of the combination: a lane and its partner each keep one half of their N sums.
template <int CTRL, int N>
__device__ __forceinline__ void halve(float* v, bool upper) {
#pragma unroll
  for (int i = 0; i < N / 2; ++i) {
    const float give = upper ? v[i] : v[i + N / 2];
    const float keep = upper ? v[i + N / 2] : v[i];
    v[i] = keep + lane_move<CTRL>(give);
  }
}

template <int D>
__device__ void segment_f32(const AttnArgs& a, char* smem, const Seg& it, bool complete, float* pslot) {
  constexpr int QD = D / 4;        // floats per lane per key
  constexpr int OWN = QD / 16;     // ... and of a row's combined output
  constexpr bool AHEAD = D == 64;  // pages fetched ahead
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int k = lane & 15;
  const int g = lane >> 4;
  const int R = it.nq * a.G;
  const int page0 = it.page0, page1 = it.page1, L = it.L;

  float* qtile = (float*)smem;                           // [F32_ROWS][D]
  int* rowslot = (int*)(qtile + F32_ROWS * D);
  int* rowtag = rowslot + F32_ROWS;
  float* part = (float*)(rowtag + F32_ROWS);             // [NW][F32_ROWS][D] sums of the waves
  float* stat = part + NW * F32_ROWS * D;                // [NW][F32_ROWS][2] reference, sum of the weights

  const int32_t* bt = a.kv.block_tables + (long)it.s * a.kv.max_blocks_per_seq;
  const uint8_t* owner_row = a.slot_owner ? a.slot_owner + (long)it.s * a.owner_stride : nullptr;
  auto block_of = [&](int P) -> int { return bt[min(P, page1 - 1)]; };  // (past the segment: its last page again)
  struct Page {
    float k[QD], v[QD];
    int own;
  };
  auto fetch = [&](int P, int blk, Page& pg) {
    blk = min(max(blk, 0), a.kv.num_blocks - 1);
    const long off = (((long)blk * a.kv.num_kv_heads + it.h) * ASPD_BLOCK + k) * D + g * QD;
#pragma unroll
    for (int e = 0; e < QD; e += 4) {
      const float4 x = *(const float4*)((const float*)a.kv.k + off + e);
      const float4 y = *(const float4*)((const float*)a.kv.v + off + e);
      pg.k[e] = x.x; pg.k[e + 1] = x.y; pg.k[e + 2] = x.z; pg.k[e + 3] = x.w;
      pg.v[e] = y.x; pg.v[e + 1] = y.y; pg.v[e + 2] = y.z; pg.v[e + 3] = y.w;
    }
    const int j = min(P, page1 - 1) * ASPD_BLOCK + k;
    pg.own = (owner_row && j >= L && j < a.owner_stride) ? owner_row[j] : 0;
  };
  const int P0 = page0 + wave;
  int blk = block_of(P0), blk_next = block_of(P0 + NW);

  __syncthreads();
  for (int i = tid; i < F32_ROWS * D; i += THREADS) {
    const int r = i / D, d = i - r * D;
    const int rr = min(r, R - 1);
    const int qi = div_by_g(a, rr);
    const int head = it.h * a.G + rr - qi * a.G;
    qtile[i] = ((const float*)a.q)[((long)(it.q0 + qi) * a.kv.num_q_heads + head) * D + d];
  }
  if (tid < F32_ROWS) {
    const int q = it.q0 + div_by_g(a, min(tid, R - 1));
    rowslot[tid] = a.logical_slot[q];
    const int qb = a.q_branch[q];
    rowtag[tid] = (qb < 0 || !a.cu_branches) ? 0 : qb - a.cu_branches[it.s] + 1;
  }
  Page cur, next;
  if (AHEAD) fetch(P0, blk, cur);
  __syncthreads();

  float acc[F32_ROWS][QD];
  float m_run[F32_ROWS], l_run[F32_ROWS];
#pragma unroll
  for (int r = 0; r < F32_ROWS; ++r) {
    m_run[r] = -INFINITY;
    l_run[r] = 0.f;
#pragma unroll
    for (int e = 0; e < QD; ++e) acc[r][e] = 0.f;
  }
  // slots past the last row's own slot have never been written and may hold anything: see below
  int last_slot = 0;
#pragma unroll
  for (int r = 0; r < F32_ROWS; ++r) last_slot = max(last_slot, rowslot[r]);

  for (int P = P0; P < page1; P += NW) {
    // The query rows are re-read from LDS for every page: kept in registers across the loop (4 rows x
    // D / 4 values per lane) they would not fit beside the accumulators.
    asm volatile("" ::: "memory");
    const int blk_after = block_of(P + 2 * NW);
    if (AHEAD) fetch(P + NW, blk_next, next);
    else fetch(P, blk, cur);
    const int j = P * ASPD_BLOCK + k;
    if (j > last_slot) {  // zero weight times a NaN would be a NaN
#pragma unroll
      for (int e = 0; e < QD; ++e) cur.v[e] = 0.f;
    }
#pragma unroll
    for (int r = 0; r < F32_ROWS; ++r) {
      float s = 0.f;
#pragma unroll
      for (int e = 0; e < QD; ++e) s = fmaf(qtile[r * D + g * QD + e], cur.k[e], s);
      s += __shfl_xor(s, 16);
      s += __shfl_xor(s, 32);
      s *= a.scale_log2;
      const bool vis = (j <= rowslot[r]) && (j < L || rowtag[r] == 0 || cur.own == rowtag[r]);
      // No branch on vis (an invisible key enters with weight zero): the lanes of one key agree on vis
      // and on s, so their statistics stay identical, and the whole update runs with all lanes active.
      const float sv = vis ? s : -INFINITY;
      const float m_new = fmaxf(m_run[r], sv);
      const float mref = exp2_safe_ref(m_new);
      const float alpha = exp2f(m_run[r] - mref);
      const float p = exp2f(sv - mref);
      m_run[r] = m_new;
      l_run[r] = l_run[r] * alpha + p;
#pragma unroll
      for (int e = 0; e < QD; ++e) acc[r][e] = fmaf(p, cur.v[e], acc[r][e] * alpha);
    }
    blk = blk_next;
    blk_next = blk_after;
    if (AHEAD) cur = next;
  }

  // ---- combine the sixteen keys' lanes of a quarter: lane k is left with the sums of the values OWN * k ..
#pragma unroll
  for (int r = 0; r < F32_ROWS; ++r) {
    float m = fmaxf(m_run[r], lane_move<0x140>(m_run[r]));  // the lane mirrored in its row of 16,
    m = fmaxf(m, lane_move<0x141>(m));                      // in its half row,
    m = fmaxf(m, lane_move<0x4e>(m));                       // two further,
    m = fmaxf(m, lane_move<0xb1>(m));                       // one further
    const float f = exp2f(m_run[r] - exp2_safe_ref(m));
    float l = l_run[r] * f;
    l += lane_move<0x140>(l);
    l += lane_move<0x141>(l);
    l += lane_move<0x4e>(l);
    l += lane_move<0xb1>(l);
#pragma unroll
    for (int e = 0; e < QD; ++e) acc[r][e] *= f;
    halve<0x140, QD>(acc[r], k & 8);
    halve<0x141, QD / 2>(acc[r], k & 4);
    halve<0x4e, QD / 4>(acc[r], k & 2);
    halve<0xb1, QD / 8>(acc[r], k & 1);
#pragma unroll
    for (int e = 0; e < OWN; ++e) part[(wave * F32_ROWS + r) * D + g * QD + OWN * k + e] = acc[r][e];
    if (lane == 0) {  // (all lanes have the same)
      stat[2 * (wave * F32_ROWS + r)] = m;
      stat[2 * (wave * F32_ROWS + r) + 1] = l;
    }
  }
  __syncthreads();
  // one thread per (row, d)
  for (int i = tid; i < F32_ROWS * D; i += THREADS) {
    const int r = i / D, d = i - r * D;
    float m[NW], mg = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      m[w] = stat[2 * (w * F32_ROWS + r)];
      mg = fmaxf(mg, m[w]);
    }
    const float mref = exp2_safe_ref(mg);
    float lg = 0.f, o = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float f = exp2f(m[w] - mref);
      lg += stat[2 * (w * F32_ROWS + r) + 1] * f;
      o += part[(w * F32_ROWS + r) * D + d] * f;
    }
    if (r < R) {
      if (complete) {
        const int qi = div_by_g(a, r);
        const long row = (long)(it.q0 + qi) * a.kv.num_q_heads + it.h * a.G + r - qi * a.G;
        ((float*)a.out)[row * D + d] = o / lg;
        if (a.lse && d == 0) a.lse[row] = (mg + log2f(lg)) * LN2;
      } else {
        store_device_scope(partial_acc(pslot, r, D) + d, o);
        if (d == 0) {
          float* st = partial_stat(a, pslot, r, D);
          store_device_scope(st, mg);
          store_device_scope(st + 1, lg);
        }
      }
    }
  }
}

template <int D>
constexpr size_t f32_smem_bytes() {
  return (F32_ROWS * D + 2 * F32_ROWS + NW * F32_ROWS * (D + 2)) * 4;
}

// One workgroup per compute unit, one wave per SIMD, which may have all of its registers; the grid is sized for that.
template <int D>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(1, 1))) void attn_f32_kernel(AttnArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  __shared__ int merge_flag;
  Seg seg;
  int next;
  const int nseg = plan_begin(a, &seg, &next);
  for (int i = 0; i < nseg; ++i) {
    if (i > 0) {
      seg = plan_segment(a, next + i - 1);
      if (!seg_ok(a, seg)) break;
    }
    const bool complete = seg_complete(seg);
    float* pslot = partial_slot(a, blockIdx.x, seg.page0 == 0 ? 1 : 0, D);
    segment_f32<D>(a, smem, seg, complete, pslot);
    if (!complete) announce_partial<D, false, THREADS, 1, 16>(a, seg, &merge_flag);
  }
}

}  // namespace
