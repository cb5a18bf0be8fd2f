// Combining the partial results of an item that several workgroups share (internal to libaspd).
#pragma once

#include "attn_common.h"

namespace {

// ---------------------------------------------------------------------------------------------
// Items split over several workgroups: every workgroup that has written a partial for the item
// announces it on the item's counter (indexed by the workgroup in whose share the item starts);
// the one that arrives last combines all partials and writes the output.  For chunks of few
// sequences a launch behind the row-splitting kernel's combines them instead (merge_kernel), and
// nothing is announced.  No workgroup waits for another.  The partials are the "starts item" slot
// of the first workgroup and the "continues item" slots of the following ones.
// ---------------------------------------------------------------------------------------------
// A thread combines ELEMS 16-byte chunks of one row at a time, BATCH parts of each: all their loads and those of the row's
// statistics are on their way at once, and nothing goes through LDS.  Bound by the instructions issued, so a row's weights
// are worked out once for all chunks of a thread (chunks of different rows before: 10 parts of 16 rows took 4.7 us of a
// launch of 14.8; stage openings over 12 sequences, three parts of 180 rows 63.1 -> 59.9 us a layer).
template <int D, bool BF16, int THREADS, int ELEMS, int BATCH>
__device__ __forceinline__ void merge_parts(const AttnArgs& a, const Seg& it, int owner, int w_last, int first_row, int R) {
  constexpr int LPR = D / 4 / ELEMS;     // threads per row
  constexpr int ROWS = THREADS / LPR;    // rows of a round
  // (defined here, so that nothing that is worked out from it lives in registers across the main loop)
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int c0 = tid % LPR;              // the thread's chunks: c0, c0 + LPR ..
  const long stride = (long)a.rows_cap * (D + 4) * sizeof(float);
  const int nparts = w_last - owner + 1;
  const char* const first = (const char*)(a.partial) + 2 * owner * stride;
  for (int r0 = first_row; r0 < R; r0 += ROWS) {
    const int r = r0 + tid / LPR;
    const uint32_t row_at = (uint32_t)min(r, R - 1);  // (rows past the last are the last again and not stored)
    const uint32_t at = row_at * (D * 4) + c0 * 16;
    float m = -INFINITY, l = 0.f;
    f32x4 o[ELEMS];
#pragma unroll
    for (int x = 0; x < ELEMS; ++x) o[x] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int p0 = 0; p0 < nparts; p0 += BATCH) {
      f32x2 ml[BATCH];
      f32x4 po[ELEMS][BATCH];
#pragma unroll
      for (int k = 0; k < BATCH; ++k) {
        const int kk = min(p0 + k, nparts - 1);  // (parts past the last are the last again and weigh nothing)
        // the first part starts the item, the others continue it
        const char* slot = first + (kk == 0 ? 1 : 2 * kk) * stride;
        ml[k] = *(const f32x2*)(slot + (long)a.rows_cap * D * sizeof(float) + row_at * 16);  // reference, sum
#pragma unroll
        for (int x = 0; x < ELEMS; ++x) po[x][k] = *(const f32x4*)(slot + at + x * LPR * 16);
      }
      float mb = m;
#pragma unroll
      for (int k = 0; k < BATCH; ++k) mb = fmaxf(mb, ml[k][0]);
      const float mref = exp2_safe_ref(mb);
      if (p0 > 0) {
        const float f0 = __builtin_amdgcn_exp2f(m - mref);
        l *= f0;
#pragma unroll
        for (int x = 0; x < ELEMS; ++x) o[x] *= f0;
      }
#pragma unroll
      for (int k = 0; k < BATCH; ++k) {
        if (p0 + k < nparts) {
          const float f = __builtin_amdgcn_exp2f(ml[k][0] - mref);
          l += ml[k][1] * f;
#pragma unroll
          for (int x = 0; x < ELEMS; ++x) o[x] += po[x][k] * f;
        }
      }
      m = mb;
    }
    if (r < R) {
      const int qi = div_by_g(a, r);
      const long row = (long)(it.q0 + qi) * a.kv.num_q_heads + it.h * a.G + r - qi * a.G;
      const float inv = 1.f / l;
#pragma unroll
      for (int x = 0; x < ELEMS; ++x) {
        const long to = row * D + 4 * (c0 + x * LPR);
        if (BF16) {
          typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
          bf16x4 ov;
#pragma unroll
          for (int e = 0; e < 4; ++e) ov[e] = (__bf16)(o[x][e] * inv);
          *(bf16x4*)((__bf16*)a.out + to) = ov;
        } else {
          *(f32x4*)((float*)a.out + to) = o[x] * inv;
        }
      }
      if (a.lse && c0 == 0) a.lse[row] = (m + log2f(l)) * LN2;
    }
  }
  // Every load has been used or not wanted: said here, so that the compiler does not wait for one of the latter, and with
  // it for all loads it does not know of, where its register is written next.
  __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
}

// A second batch costs a second round trip to memory, so the batch is as large as the registers allow, but no larger than
// the parts there are: with two waves per SIMD the merge is bound by the instructions it issues, and every slot of a batch
// costs its loads and its arithmetic whether a part stands behind it or not.
template <int D, bool BF16, int THREADS, int ELEMS, int BATCH>
__device__ __forceinline__ void merge_item(const AttnArgs& a, const Seg& it, int owner, int w_last) {
  const int nparts = w_last - owner + 1, R = it.nq * a.G;
  if (nparts <= 2) merge_parts<D, BF16, THREADS, ELEMS, 2>(a, it, owner, w_last, 0, R);
  else if (BATCH > 3 && nparts <= 3) merge_parts<D, BF16, THREADS, ELEMS, 3>(a, it, owner, w_last, 0, R);
  else if (BATCH > 4 && nparts <= 4) merge_parts<D, BF16, THREADS, ELEMS, 4>(a, it, owner, w_last, 0, R);
  else if (BATCH > 6 && nparts <= 6) merge_parts<D, BF16, THREADS, ELEMS, 6>(a, it, owner, w_last, 0, R);
  else if (BATCH > 8 && nparts <= 8) merge_parts<D, BF16, THREADS, ELEMS, 8>(a, it, owner, w_last, 0, R);
  else if (BATCH > 12 && nparts <= 12) merge_parts<D, BF16, THREADS, ELEMS, 12>(a, it, owner, w_last, 0, R);
  else merge_parts<D, BF16, THREADS, ELEMS, BATCH>(a, it, owner, w_last, 0, R);
}

template <int D, bool BF16, int THREADS, int ELEMS, int BATCH>
__device__ __forceinline__ void announce_partial(const AttnArgs& a, const Seg& it, int* flag /* LDS */) {
  const int owner = it.owner, w_last = it.w_last;
  // the write-through stores of the partial have completed before the arrival is counted
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    const int old = atomicAdd(a.counters + owner, 1);
    const int last = (old == w_last - owner) ? 1 : 0;
    if (last) atomicExch(a.counters + owner, 0);  // every part has arrived: leave it clean for the next call
    *flag = last;
  }
  __syncthreads();
  if (*flag == 0) return;
  // Only the merging workgroup pays for an acquire at device scope (it drops whatever stale copies of
  // the partial slots its caches may hold from earlier launches); the partials themselves were
  // written through by their producers, so ordinary wide loads now fetch them.
  // One wave issues it for the workgroup: the invalidate acts on the compute unit's L1 and the XCD's L2,
  // which all waves of the workgroup share.
  if (threadIdx.x < 64) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  __syncthreads();
  merge_item<D, BF16, THREADS, ELEMS, BATCH>(a, it, owner, w_last);
}

// The merge as a launch of its own, behind one of the row-splitting kernel that has left its partial results where they are:
// every workgroup that holds a part of an item combines its share of the item's rows.  Bound by the round trips of a
// workgroup: one for every batch of parts, of every round of its rows.  So a class of parts takes all of them at once, and as
// many chunks of a row a thread as the registers then hold, which makes a round (head size 128) 64 rows up to five parts, 32
// up to twelve and 16 above: the share of a full row group is one round with 4, 5, 8 to 12 and from 16 parts on, and two with
// the others.  (One class for all from five parts on, sixteen of them at once: four rounds with five parts, most of whose
// loads were the last part again.  Four layers, one / three / six sequences behind 1 000 tokens 137 -> 108, 162 -> 126, 152
// -> 122 us.)
constexpr int MERGE_THREADS = 512;
template <int D>
__global__ __launch_bounds__(MERGE_THREADS) void merge_kernel(AttnArgs a) {
  Seg seg;
  int next;
  const int queue = load_word_uniform(a.plan + (long)PLAN_HDR * blockIdx.x + PLAN_HDR_QUEUE);
  const int nseg = plan_begin(a, &seg, &next);
  if (queue > 0) return;  // whole items
  // only the first and the last segment of a workgroup can be a part of an item
  for (int i = 0; i < min(nseg, 2); ++i) {
    if (i > 0) {
      seg = plan_segment(a, next + nseg - 2);
      if (!seg_ok(a, seg)) return;
    }
    if (seg_complete(seg)) continue;
    const int n = seg.w_last - seg.owner + 1, p = (int)blockIdx.x - seg.owner, R = seg.nq * a.G;
    const int lo = R * p / n, hi = R * (p + 1) / n;
    if (n <= 3) merge_parts<D, true, MERGE_THREADS, 4, 3>(a, seg, seg.owner, seg.w_last, lo, hi);
    else if (n <= 5) merge_parts<D, true, MERGE_THREADS, 4, 5>(a, seg, seg.owner, seg.w_last, lo, hi);
    else if (n <= 8) merge_parts<D, true, MERGE_THREADS, 2, 8>(a, seg, seg.owner, seg.w_last, lo, hi);
    else if (n <= 12) merge_parts<D, true, MERGE_THREADS, 2, 12>(a, seg, seg.owner, seg.w_last, lo, hi);
    else merge_parts<D, true, MERGE_THREADS, 1, 16>(a, seg, seg.owner, seg.w_last, lo, hi);
  }
}

}  // namespace
