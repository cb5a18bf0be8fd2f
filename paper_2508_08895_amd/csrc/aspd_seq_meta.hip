// aspd_build_sequence_meta: metadata of ALL tokens of a batch of multi-stage sequences at once
// (ASPD Fig. 5, training arrangement: the branches of a parallel stage laid one after the other;
// Eq. 4 for the position ids, Eq. 2-3 for what a token sees), for teacher-forced passes and for the
// re-prefill of a cache (Sec. 4.5.3, "Same-Re").
//
// Pure integer work.  One or more workgroups per sequence: one thread walks the sequence's runs in order (a
// few hundred at most: the walk carries the stage bookkeeping, which is inherently sequential) and
// tabulates, per run, its first slot, the position of its first token, the first slot of its stage
// and its branch number; then all threads emit the tokens, finding a token's run by binary search.
// The workgroups of a sequence (gridDim.y) all walk it and share its tokens: nothing that is written here is read
// here, and a token costs its thread three waits for memory, so that with one workgroup the longest sequence
// decided.
// A second, one-workgroup kernel lists the row groups of the attention launch, longest key range
// first, behind the per-row stage bases in the step's plan buffer.
#include <algorithm>

#include "aspd_plan.h"

namespace {

constexpr int SEQ_META_THREADS = 256;

__device__ __forceinline__ void seq_raise_fault(int32_t* fault, int bits) {
  if (fault) atomicOr(fault, bits);
}

struct LayoutView {
  const int32_t* cu_runs;
  const int32_t* run_branch;
  const int32_t* run_len;
};

__global__ __launch_bounds__(SEQ_META_THREADS) void meta_sequence_kernel(KvView kv, StateView st, StepView sp,
                                                                         LayoutView lay, int32_t* __restrict__ row_base,
                                                                         int32_t* __restrict__ row_lo,
                                                                         bool same_seq, bool same_max, int fix_n) {
  __shared__ int run_slot0[ASPD_MAX_RUNS_PER_SEQ + 1];  // first slot of every run; [nr] = tokens of the sequence
  __shared__ int run_pos0[ASPD_MAX_RUNS_PER_SEQ];       // position id of the run's first token
  __shared__ int run_base[ASPD_MAX_RUNS_PER_SEQ];       // first slot of the run's stage (branch runs)
  __shared__ int red[SEQ_META_THREADS / 64];
  __shared__ int sh_ok;
  const int s = blockIdx.x;
  const int tid = threadIdx.x;
  const int r0 = lay.cu_runs[s];
  const int nr = lay.cu_runs[s + 1] - r0;

  // packed row of this sequence's first token: the tokens of all earlier sequences
  int part = 0;
  for (int i = tid; i < r0; i += SEQ_META_THREADS) part += max(lay.run_len[i], 0);
  part = wave_scan_add(part);
  if ((tid & 63) == 63) red[tid >> 6] = part;
  // The runs as the layout gives them, for the walk below, which would otherwise wait for memory at every one of them
  // (its own words of a run take their place).
  if (nr >= 0 && nr <= ASPD_MAX_RUNS_PER_SEQ)
    for (int i = tid; i < nr; i += SEQ_META_THREADS) {
      run_base[i] = lay.run_branch[r0 + i];
      run_pos0[i] = lay.run_len[r0 + i];
    }
  __syncthreads();
  int base = 0;
#pragma unroll
  for (int w = 0; w < SEQ_META_THREADS / 64; ++w) base += red[w];

  if (tid == 0) {
    int ok = 1, faults = 0;
    int slot = 0;         // tokens laid so far
    int main_pos = 0;     // position the next main-branch token takes (Same-Seq: equals `slot` outside stages)
    int stage_first = 0;  // first slot of the running parallel stage
    int stage_start = 0;  // Eq. 4 stage_start: position of the first token of each of its branches
    int longest = 0;      // most tokens any of its branches holds
    int prev = 0;         // branch number of the previous run (0: main branch)
    if (nr < 0 || nr > ASPD_MAX_RUNS_PER_SEQ) {
      ok = 0;
      faults |= ASPD_FAULT_LAYOUT;
    }
    for (int i = 0; ok && i < nr; ++i) {
      const int b = run_base[i];
      const int n = run_pos0[i];
      if (n < 0 || b < 0 || b > ASPD_MAX_BRANCHES_PER_SEQ || (b > 1 && b != prev + 1)) {
        ok = 0;
        faults |= (b > ASPD_MAX_BRANCHES_PER_SEQ) ? ASPD_FAULT_BRANCHES : ASPD_FAULT_LAYOUT;
        break;
      }
      if (prev > 0 && b <= 1) {
        // the stage that `prev` closed ends here: where the main branch continues (Sec. 4.5.3)
        main_pos = same_seq ? slot : (same_max ? stage_start + longest : stage_start + prev * fix_n);
      }
      run_slot0[i] = slot;
      if (b == 0) {
        run_pos0[i] = same_seq ? slot : main_pos;  // Eq. 4, first case
        run_base[i] = slot;
        main_pos = run_pos0[i] + n;
      } else {
        if (b == 1) {  // a stage opens
          stage_first = slot;
          stage_start = same_seq ? slot : main_pos;
          longest = 0;
        }
        if (fix_n > 0 && n > fix_n) {
          ok = 0;
          faults |= ASPD_FAULT_INTERVAL;
          break;
        }
        run_pos0[i] = stage_start + (fix_n > 0 ? (b - 1) * fix_n : 0);  // Eq. 4, second case
        run_base[i] = stage_first;
        longest = max(longest, n);
      }
      slot += n;
      prev = b;
      if ((long)slot > (long)kv.max_blocks_per_seq * ASPD_BLOCK) {
        ok = 0;
        faults |= ASPD_FAULT_BLOCK_TABLE;
      } else if (st.slot_owner && slot > st.owner_stride) {
        ok = 0;
        faults |= ASPD_FAULT_OWNER_ROW;
      }
    }
    if (ok && prev > 0) main_pos = same_seq ? slot : (same_max ? stage_start + longest : stage_start + prev * fix_n);
    if (ok && base + slot > sp.NQ) {
      ok = 0;
      faults |= ASPD_FAULT_ROW_COUNT;
    }
    if (!ok) {
      slot = 0;
      main_pos = 0;
      faults |= ASPD_FAULT_ROW_COUNT;  // the sequence's rows are missing from the step
    }
    if (ok) run_slot0[nr] = slot;
    sh_ok = ok;
    if (blockIdx.y == 0) {
      if (faults) seq_raise_fault(st.fault, faults);
      // state: as after a merge of the last stage
      st.seq_len[s] = slot;
      st.stage_base[s] = slot;
      if (st.main_pos) st.main_pos[s] = main_pos;
      if (st.stage_open) st.stage_open[s] = 0;
      sp.cu_seq_new[s] = base;
      if (s == st.B - 1) sp.cu_seq_new[st.B] = base + slot;
    }
  }
  __syncthreads();
  if (!sh_ok) return;
  const int T = run_slot0[nr];
  for (int j = blockIdx.y * SEQ_META_THREADS + tid; j < T; j += gridDim.y * SEQ_META_THREADS) {
    // the run that holds slot j: the last one whose first slot is <= j and that is not empty
    int lo = 0, hi = nr - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (run_slot0[mid] <= j) lo = mid; else hi = mid - 1;
    }
    const int b = lay.run_branch[r0 + lo];
    const int t = j - run_slot0[lo];  // index of the token within its run (= within its branch)
    const int row = base + j;
    const int blk = kv.block_tables[(long)s * kv.max_blocks_per_seq + j / ASPD_BLOCK];
    if (blk < 0 || blk >= kv.num_blocks) seq_raise_fault(st.fault, ASPD_FAULT_BLOCK_TABLE);
    sp.q_seq[row] = s;
    sp.q_branch[row] = b - 1;
    sp.position_ids[row] = run_pos0[lo] + t;
    sp.logical_slot[row] = j;
    sp.slot_mapping[row] = (int64_t)blk * ASPD_BLOCK + j % ASPD_BLOCK;
    // Eq. 2-3: a main-branch token sees every slot up to its own; a branch token sees everything before
    // its stage and its own branch up to itself
    sp.kv_len[row] = b == 0 ? j + 1 : run_base[lo] + t + 1;
    row_base[row] = b == 0 ? j : run_base[lo];
    row_lo[row] = b == 0 ? j : run_slot0[lo];
    if (st.slot_owner) st.slot_owner[(long)s * st.owner_stride + j] = (uint8_t)b;
  }
}

// The row groups of the attention launch: `qpg` consecutive tokens of one sequence each.  A group's key
// range ends at its last token's slot, so groups late in a sequence cost more than early ones; workgroups
// take groups from the list as they become free.  Where the launch has a queue per XCD and one KV head's tokens of all
// sequences are more than an L2 holds, the groups of a sequence follow each other, so that the workgroups of an XCD stream the
// same pages, longest sequence and in it longest ranges first.  Otherwise the list starts with the longest ranges of all, so
// that the launch does not end on a long one: round t lists, for every sequence that has that many, its t-th group from the
// end.
constexpr int WORKLIST_THREADS = 1024;
__global__ __launch_bounds__(WORKLIST_THREADS) void sequence_worklist_kernel(const int32_t* __restrict__ cu_seq_new,
                                                                 const int32_t* __restrict__ seq_len, int B, int NQ,
                                                                 int qpg, int max_items, int l2_items, int num_kv_heads, int nwg,
                                                                 int parts, int pieces_at, int32_t* __restrict__ plan) {
  __shared__ int ngr[ASPD_MAX_BATCH];
  __shared__ int first_item[ASPD_MAX_BATCH + 1];
  __shared__ int wave_tot[WORKLIST_THREADS / 64], wave_long[WORKLIST_THREADS / 64], wave_pages[WORKLIST_THREADS / 64];
  const int tid = threadIdx.x;
  // (a sequence that was refused holds no token: seq_len, which the kernel before this one wrote, says so,
  // while the packed rows the layout gave it stay where they are, unwritten)
  static_assert(ASPD_MAX_BATCH <= WORKLIST_THREADS, "a thread per sequence");
  const int mine = tid < B ? (max(seq_len[tid], 0) + qpg - 1) / qpg : 0;
  const int incl = wave_scan_add(mine);
  // pages of the longest row group, and of all of them (the rule below needs no better than a group's rounded up)
  const int longest_w = wave_scan_max(tid < B ? (max(seq_len[tid], 0) + ASPD_BLOCK - 1) / ASPD_BLOCK : 0);
  const int pages_w = parts == 0 ? 0 : wave_scan_add((qpg * (mine * (mine + 1) / 2) + ASPD_BLOCK - 1) / ASPD_BLOCK);
  if ((tid & 63) == 63) {
    wave_tot[tid >> 6] = incl;
    wave_long[tid >> 6] = longest_w;
    wave_pages[tid >> 6] = pages_w;
  }
  __syncthreads();
  int first = incl - mine, acc = 0, longest = 0, total = 0;
  for (int w = 0; w < (B + 63) >> 6; ++w) {
    longest = max(longest, wave_long[w]);
    total += wave_pages[w];
    if (w < (tid >> 6)) first += wave_tot[w];
    acc += wave_tot[w];
  }
  if (tid < B) {
    ngr[tid] = mine;
    first_item[tid] = first;
  }
  if (tid == 0) {
    first_item[B] = min(acc, max_items);
    plan[0] = first_item[B];
    plan[1] = qpg;
    plan[2] = NQ;
    plan[3] = B;
    for (int i = 4; i < SEQ_PLAN_HDR; ++i) plan[i] = 0;  // (SEQ_HDR_PIECES among them)
  }
  __syncthreads();
  const int n_items = first_item[B];
  int32_t* items = plan + SEQ_PLAN_HDR + ((NQ + 3) & ~3);
  // item (s, t): group ngr[s] - 1 - t of sequence s.  Its place in the list: the items of earlier rounds
  // (min(ngr, t) of every sequence) and, in its own round, the sequences before s that still have a group; or, sequence by
  // sequence, those of the longer sequences and its own t.
  const bool in_rounds = n_items <= l2_items || n_items * num_kv_heads < SEQ_QUEUE_ITEMS * nwg;
  __shared__ int longer[ASPD_MAX_BATCH];  // items of the sequences listed before (a loop over them for every item took 20 us)
  if (!in_rounds && tid < B) {
    int before = 0;
    for (int k = 0; k < B; ++k) before += ngr[k] > mine || (ngr[k] == mine && k < tid) ? ngr[k] : 0;
    longer[tid] = before;
  }
  __syncthreads();
  int group_place = 0, group_pages = 0;  // of this thread's row group (the first one, see below)
  for (int e = tid; e < n_items; e += blockDim.x) {
    int lo = 0, hi = B - 1;  // sequence of the e-th group in sequence-major order
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (first_item[mid] <= e) lo = mid; else hi = mid - 1;
    }
    const int s = lo;
    const int gidx = e - first_item[s];     // group index within the sequence, 0 = first tokens
    const int t = ngr[s] - 1 - gidx;
    int place = 0;
    if (in_rounds) {
      for (int k = 0; k < B; ++k) place += min(ngr[k], t) + ((k < s && ngr[k] > t) ? 1 : 0);
    } else {
      place = longer[s] + t;
    }
    const int T = seq_len[s];
    const int tok0 = gidx * qpg;
    const int nq = min(qpg, T - tok0);
    if (place < n_items) {
      items[4 * place + 0] = s;
      items[4 * place + 1] = cu_seq_new[s] + tok0;
      items[4 * place + 2] = nq;
      items[4 * place + 3] = (tok0 + nq + ASPD_BLOCK - 1) / ASPD_BLOCK;  // pages up to the group's last slot
      if (e == tid) {
        group_place = place;
        group_pages = (tok0 + nq + ASPD_BLOCK - 1) / ASPD_BLOCK;
      }
    }
  }

  // ---- Few row groups, some of them long against a workgroup's share of the pages: the launch would wait for the
  // longest chain of pages, so the longest key ranges are cut into pieces of about a share, whose partial results are merged.
  // The lines: with more than two row groups per workgroup the queue evens the launch out by itself.  A piece costs its
  // start, its partial results and its share of a merge, together 40 to 45 pages' worth, so nothing is cut unless the longest
  // range is SEQ_PIECE_GAIN pages longer than a piece, no piece is shorter than SEQ_PIECE_MIN, and no range is cut that is
  // not half as long again as a piece.
  // Two layers, uncut -> cut, us: 8/8 heads of 128, two sequences of 2 000 to 6 000 tokens 268 -> 201, one of 4 000 224 ->
  // 182, three of 430 to 1 466 112 -> 95; 16/4 of 64, one of 1 500 85 -> 71, one of 4 000 172 -> 148; 32/8 of 128, one of
  // 1 500 122 -> 115.  On the other side of the line, cut all the same: 32/8, three of 430 to 1 466 (the longest 92 pages,
  // a share 44) 142 -> 150; 8/8, five of 1 000 (63 and 25) 113 -> 126; one of 700 (44 and 8) 70 -> 72.
  if (parts == 0 || n_items == 0 || n_items > SEQ_ENTRIES / 2 || n_items * num_kv_heads > 2 * nwg) return;  // (uniform)
  int target = max(SEQ_PIECE_MIN, quotient(total * num_kv_heads, nwg) + 4);  // pages of a piece
  if (longest < target + SEQ_PIECE_GAIN) return;
  static_assert(SEQ_ENTRIES / 2 <= WORKLIST_THREADS, "a row group per thread");
  __shared__ int sums[2 * (WORKLIST_THREADS / 64)];
  auto total_of = [&](int v, int* wave) -> int {  // sum over the workgroup, by all of it
    const int scan = wave_scan_add(v);
    __syncthreads();
    if ((tid & 63) == 63) wave[tid >> 6] = scan;
    __syncthreads();
    int sum = 0;
    for (int w = 0; w < (n_items + 63) >> 6; ++w) sum += wave[w];
    return sum;
  };
  int pieces = 1, cut = 0, places = 0;
  bool fits = false;
  for (int attempt = 0; attempt < 16 && !fits; ++attempt) {
    pieces = 2 * group_pages > 3 * target ? min(SEQ_PIECES_MAX, quotient(group_pages + target - 1, target)) : 1;
    cut = pieces > 1 ? pieces * num_kv_heads : 0;
    places = total_of(cut, sums);
    if (places == 0) return;
    fits = places <= min(parts, 256);
    if (!fits) target += (target >> 2) + 1;
  }
  if (!fits) return;
  // places of the partial results, and of the pieces in the list: longest first, in classes
  const int mine_cut = cut, mine_n = tid < n_items ? pieces : 0;
  const int cut_before = wave_scan_add(mine_cut) - mine_cut;
  constexpr int BINS = WORKLIST_THREADS;
  __shared__ int bins[BINS];
  bins[tid] = 0;
  __syncthreads();
  if ((tid & 63) == 63) sums[tid >> 6] = cut_before + mine_cut;
  const int length = quotient(group_pages + pieces - 1, pieces);
  const int bin = BINS - 1 - min(BINS - 1, length);
  if (mine_n > 0) atomicAdd(&bins[bin], mine_n);
  __syncthreads();
  int base = cut_before;
  for (int w = 0; w < (tid >> 6); ++w) base += sums[w];
  const int in_bin = bins[tid];
  const int bin_scan = wave_scan_add(in_bin);
  int* bin_sums = sums + WORKLIST_THREADS / 64;
  if ((tid & 63) == 63) bin_sums[tid >> 6] = bin_scan;
  __syncthreads();
  int first_of_bin = bin_scan - in_bin;
  for (int w = 0; w < (tid >> 6); ++w) first_of_bin += bin_sums[w];
  bins[tid] = first_of_bin;
  __syncthreads();
  if (mine_n > 0) {
    const int at = atomicAdd(&bins[bin], mine_n);
    for (int i = 0; i < mine_n; ++i) {
      plan[pieces_at + 2 * (at + i)] = group_place;
      plan[pieces_at + 2 * (at + i) + 1] = i | (mine_n << 8) | (base << 16);
    }
  }
  const int entries = total_of(mine_n, sums);
  if (tid == 0) {
    plan[SEQ_HDR_PIECES] = entries;
    plan[SEQ_HDR_HEADS] = num_kv_heads;
    plan[SEQ_HDR_PLACES] = places;
  }
}

}  // namespace

size_t aspd_sequence_plan_words(const aspd_kv* kv, int32_t B, int32_t NQ) {
  const int G = kv->num_q_heads / kv->num_kv_heads;
  return aspd_sequence_plan_pieces(G, B, NQ) + 2 * SEQ_ENTRIES;
}

int aspd_sequence_parts(const aspd_kv* kv, int32_t B, int32_t NQ) {
  AttnVariant v;  // (a chunk of unknown size: one of the launch shapes a workspace is sized for)
  if (!aspd_choose_variant(kv, B, NQ, 0, 0, true, true, &v) || v.kernel != KERNEL_BF16_ROWS) return 0;
  return v.nwg;
}

extern "C" size_t aspd_sequence_plan_bytes(const aspd_kv* kv, int32_t B, int32_t NQ) {
  if (aspd_check_kv(kv) != ASPD_OK || B <= 0 || B > ASPD_MAX_BATCH || NQ < 0) return 0;
  const int G = kv->num_q_heads / kv->num_kv_heads;
  if (kv->dtype != ASPD_BF16 || aspd_sequence_qpg(G) < 1) return 0;
  return aspd_sequence_plan_words(kv, B, NQ) * sizeof(int32_t);
}

extern "C" int aspd_build_sequence_meta(const aspd_kv* kv, aspd_state* state, const aspd_layout* layout,
                                        int32_t pos_mode, aspd_step* out, void* stream) {
  int rc = aspd_check_kv(kv);
  if (rc != ASPD_OK) return rc;
  if (!state || !layout || !out || state->B <= 0 || !state->stage_base_d || !state->seq_len_d) return ASPD_ERR_INVALID_ARG;
  if (state->B > ASPD_MAX_BATCH) return ASPD_ERR_UNSUPPORTED;
  const int G = kv->num_q_heads / kv->num_kv_heads;
  if (kv->dtype != ASPD_BF16 || aspd_sequence_qpg(G) < 1) return ASPD_ERR_UNSUPPORTED;
  if (layout->num_runs < 0 || !layout->cu_runs_d || (layout->num_runs > 0 && (!layout->run_branch_d || !layout->run_len_d)))
    return ASPD_ERR_INVALID_ARG;
  const int mode = pos_mode & 0xff;
  const int fix_n = mode == 2 ? (pos_mode >> 8) : 0;
  if (mode < 0 || mode > 2 || (mode == 2 && fix_n <= 0)) return ASPD_ERR_INVALID_ARG;
  if (mode != ASPD_POS_SAME_SEQ && !state->main_pos_d) return ASPD_ERR_INVALID_ARG;
  if (state->slot_owner_d && state->owner_stride <= 0) return ASPD_ERR_INVALID_ARG;
  if (out->NQ < 0 || !out->cu_seq_new_d) return ASPD_ERR_INVALID_ARG;
  if (out->NQ > 0 && (!out->q_seq_d || !out->q_branch_d || !out->position_ids_d || !out->logical_slot_d ||
                      !out->slot_mapping_d || !out->kv_len_d))
    return ASPD_ERR_INVALID_ARG;
  if (!out->plan_d || ((uintptr_t)out->plan_d & 255) ||
      out->plan_bytes < aspd_sequence_plan_words(kv, state->B, out->NQ) * sizeof(int32_t))
    return ASPD_ERR_INVALID_ARG;
  hipStream_t hs = (hipStream_t)stream;
  const int qpg = aspd_sequence_qpg(G);
  LayoutView lay{layout->cu_runs_d, layout->run_branch_d, layout->run_len_d};
  // two tokens a thread where the sequences are alike; no more workgroups than eight a compute unit
  const int share = (int)std::max(1L, std::min({((long)out->NQ / state->B + 2 * SEQ_META_THREADS - 1) / (2 * SEQ_META_THREADS),
                                                8L * aspd_device_cu_count() / state->B + 1, 32L}));
  hipLaunchKernelGGL(meta_sequence_kernel, dim3(state->B, share), dim3(SEQ_META_THREADS), 0, hs, make_view(kv), make_view(state),
                     make_view(out), lay, out->plan_d + SEQ_PLAN_HDR,
                     out->plan_d + aspd_sequence_plan_lo(G, state->B, out->NQ), mode == ASPD_POS_SAME_SEQ, mode == ASPD_POS_SAME_MAX, fix_n);
  ASPD_HIP_CHECK(hipGetLastError());
  const int max_items = state->B + out->NQ / qpg;
  hipLaunchKernelGGL(sequence_worklist_kernel, dim3(1), dim3(WORKLIST_THREADS), 0, hs, out->cu_seq_new_d, state->seq_len_d, state->B,
                     out->NQ, qpg, max_items, XCD_L2_BYTES / (2 * 2 * kv->head_dim) / qpg, kv->num_kv_heads,
                     out->max_workgroups > 0 ? std::min(out->max_workgroups, aspd_device_cu_count()) : aspd_device_cu_count(),
                     aspd_sequence_may_cut(kv, state->B, out->NQ, qpg, aspd_device_cu_count())
                         ? aspd_sequence_parts(kv, state->B, out->NQ) : 0,
                     (int)aspd_sequence_plan_pieces(G, state->B, out->NQ),
                     out->plan_d);
  ASPD_HIP_CHECK(hipGetLastError());
  out->plan_key = aspd_sequence_plan_key(qpg, state->B);
  return ASPD_OK;
}
