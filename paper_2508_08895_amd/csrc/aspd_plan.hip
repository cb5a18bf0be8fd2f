// The plan of a step's attention launches (see aspd_plan.h): which workgroup takes which run of KV
// pages of which (sequence, row group, KV head) item.  One small kernel per step; integer work.
//
// Work decomposition of the attention kernels (ASPD Sec. 3.2 Eq. 1-3 evaluate, per query row, a softmax
// over the KV slots the row may see; rows that share a sequence and a KV head share the pages they
// read): the (sequence, row group, KV head, page) space is flattened and every workgroup takes a
// contiguous share of it.  A share may cut an item: the workgroups that hold parts of one item combine
// their partial results inside the attention launch.
#include <algorithm>
#include <atomic>

#include "aspd_plan.h"

namespace {

// One workgroup; a thread per workgroup of the largest attention grid and per sequence of the largest batch.  Not more waves than
// that, and few instructions on the way of all: a wave by itself issues one in eight to nine cycles, and what every wave does
// alike (sums across the waves, the choice of a regime) was most of the kernel whatever the batch.  With sixteen waves,
// shuffles, integer and 64-bit divisions the plan of one sequence took 18 400 cycles, of 16 sequences 21 100, of 64 35 100;
// with eight, data-parallel moves and reciprocals 10 700, 14 300 and 28 100.
constexpr int PLAN_THREADS = 512;
static_assert(PLAN_THREADS >= MAX_WG && PLAN_THREADS >= ASPD_MAX_BATCH, "a thread per workgroup and per sequence");

struct PlanArgs {
  const int32_t* stage_base;
  const int32_t* seq_len;
  const int32_t* cu_seq_new;
  const int32_t* block_tables;
  int32_t*       plan;
  int            B, nwg, qpg, pad, num_kv_heads, max_blocks_per_seq, num_blocks;
  int            has_owner;
  int            w_page, w_wave;  // what a page costs: w_page, and w_wave for every wave that has rows up to four (page_cost)
  int            rows_per_query;  // query heads per KV head
  int            NQ, max_items;   // rows of the step, and the items the plan has room for
};

// Rows of a sequence whose rows are [q0, q1) of the step; none where they are not rows of the step (more new tokens than the
// caller said: the metadata refuses those sequences, and a plan is sized for the rows that the caller said).
__device__ __forceinline__ int rows_between(const PlanArgs& a, int q0, int q1) {
  return (int)(q0 >= 0) & (int)(q0 <= q1) & (int)(q1 <= a.NQ) ? q1 - q0 : 0;
}

struct Item {
  int s, rg, h;     // sequence, row group, KV head
  int np;           // pages of the item
  int lp;           // even regime: pages of it that lie wholly before stage_base (no owner tags, no masking)
  int q0, nq;       // first packed query row and number of queries of the row group
  int first_unit;   // ragged regime: flattened index of the item's first unit
};

constexpr int QUEUE_BINS = 1024;  // classes of cost, see queue_end
constexpr int QUEUE_CUT = 40;     // pages' worth of a cut, see Shares

// Per-sequence scalars in LDS and the table of share boundaries.
struct Sched {
  int* cu_units;  // [B+1] exclusive scan of the units (pages + pad, over row groups and KV heads)
  int* T;         // [B]   seq_len
  int* L;         // [B]   stage_base
  int* q0;        // [B+1] cu_seq_new
  int* ng;        // [B]   row groups
  int* wgb;       // [MAX_WG+1] first unit of every workgroup's share (ragged regime only)
};
__device__ __forceinline__ Sched sched_at(int* base, int B) {
  Sched sc;
  sc.cu_units = base;
  sc.T = base + (B + 1);
  sc.L = sc.T + B;
  sc.q0 = sc.L + B;
  sc.ng = sc.q0 + (B + 1);
  sc.wgb = sc.ng + B;
  return sc;
}
constexpr int sched_ints(int B) { return (5 * B + 2 + MAX_WG + 1 + 3) & ~3; }  // (what follows stays 16-byte aligned)

__device__ __forceinline__ int pages_of(const PlanArgs& a, const Sched& sc, int s) {
  return min((sc.T[s] + ASPD_BLOCK - 1) / ASPD_BLOCK, a.max_blocks_per_seq);
}

// Pages of a sequence's row groups in the ragged regime.  A step's rows are the last slots of the sequence, in order, so
// no row of group j sees past the group's last slot: with `held` slots before the step that is slot held + (j + 1) qpg - 1,
// and the item ends there instead of at the sequence's end (in the even regime every item has all pages of its
// sequence; pieces that no row of the group sees are written and merged as empty partials).  For an append that is long
// against what it follows (a prompt) this halves the pages: 8 prompts of 90 to 2000 tokens 225 -> 163 us a layer.
// Groups of whole pages only (qpg a multiple of 16: the lengths are then an arithmetic series, which the
// flattened index is solved for); otherwise, and where the lengths do not add up (a refused sequence), every item has
// all pages.
struct Groups {
  int n;      // row groups
  int np;     // pages of the sequence, and of the last group
  int first;  // pages of group j < n - 1: first + (j + 1) * step
  int step;
  // Units of one KV head's groups before group j (j <= n), `pad` of them in front of every group.
  __device__ __forceinline__ int before(int j, int pad) const {
    const int k = min(j, n - 1);
    return k * (first + pad) + step * (k * (k + 1) / 2) + (j == n ? np + pad : 0);
  }
  __device__ __forceinline__ int pages(int j) const { return j < n - 1 ? first + (j + 1) * step : np; }
};
__device__ __forceinline__ Groups groups_at(const PlanArgs& a, int T, int rows, int n) {
  Groups g;
  g.n = n;
  const int all = (T + ASPD_BLOCK - 1) / ASPD_BLOCK;
  g.np = min(all, a.max_blocks_per_seq);
  const bool ends = (int)(g.n > 1) & (int)(a.qpg % ASPD_BLOCK == 0) & (int)(T >= rows) & (int)(all == g.np);
  g.first = ends ? (T - rows + ASPD_BLOCK - 1) / ASPD_BLOCK : g.np;
  g.step = ends ? a.qpg / ASPD_BLOCK : 0;
  return g;
}

// Cost of a page of a row group of nq queries.  From the fifth wave on a SIMD has two, and the others wait for it.
__device__ __forceinline__ int page_cost(const PlanArgs& a, int nq) {
  const int waves = (nq * a.rows_per_query + 31) / 32;
  return a.w_page + a.w_wave * (waves > 4 ? ROWS_FULL_COST : waves);
}
// Queries of the last of a sequence's row groups.
__device__ __forceinline__ int last_group(const PlanArgs& a, int rows, int n) { return rows - (n - 1) * a.qpg; }

__device__ __forceinline__ Groups groups_of(const PlanArgs& a, const Sched& sc, int s) {
  return groups_at(a, sc.T[s], sc.q0[s + 1] - sc.q0[s], sc.ng[s]);
}

// Shares of the unit space, one per workgroup used.  A unit is a page of an item or, in the ragged
// regime, one of `pad` virtual units in front of every item: they price the fixed cost a workgroup
// pays for starting a segment (start-up, reduction, a partial to be merged), so that equal shares of
// units are about equal shares of time.  Two regimes, chosen per step:
//
// EVEN (no more items than workgroups, and pieces that come out about as long as the shares of the
// ragged regime would).  Every workgroup has exactly one segment: item i is cut evenly among
// k_i = ceil(np_i / p) workgroups of its own, with p the smallest piece length for which the pieces of
// all items fit the grid.  A workgroup pays a segment's fixed cost once, and an item that fits one piece
// needs no merge.
//
// What a page costs depends, for the row-splitting kernel, on how many of its waves have rows (page_cost), so the
// lengths compared are costs there (a stage opening over 12 sequences, where row groups have two to eight waves: the
// workgroups end between 27 and 65 us with pieces of equal pages, between 26 and 59 with pieces of equal cost).
//
// QUEUE (row-splitting kernel, more items than workgroups, and the longest workgroup no longer than a share and what a cut
// costs).  Every workgroup takes whole items, longest first: the first is given, after that whichever is next when the
// workgroup gets free.  Nothing is split or merged, and no share has to be guessed from costs.  The plan lists the items
// dealt round in that order, which is what a workgroup's header and the list say; the kernel takes them out of the list by
// its own counter.  Shares of equal pages (RAGGED) ended between 457 and 804 us in a 64-sequence chunk, this between 637 and
// 685 (median 647); in eight prompts between 87 and 149, this between 121 and 135.  Launches, us: chunk 821 -> 676, prompts
// 154 -> 136.
//
// The line has two parts.  The costliest item is no more than 1.25 of a share of the cost.  And the longest workgroup, as
// the order of the items tells it (queue_end), is no longer than the longest of RAGGED: a share of the pages at the price of
// the fullest row group, QUEUE_CUT pages for the segment that is cut off (start, partial results, their merge), and a
// twelfth of the share (workgroups that are left alone run faster than among others: the second round of 264 equal items on
// 256 workgroups takes half as long as the first).  Without the second part, items of like cost a few more than the
// workgroups took two whole rounds.  One layer, queue -> shares, us, 32/8 heads, 64 new tokens behind 8 000: 33 sequences
// 441 -> 344, 40 468 -> 404, 56 566 -> 554, 64 (whole rounds, queue) 609 | 616, 65 703 -> 639, 72 750 -> 701; behind
// 4 000: 33 253 -> 199, 48 289 -> 268, 56 (queue) 308 | 312, 72 411 -> 397; behind 1 000: 33 105 -> 95, 40 112 -> 110, 48
// (queue) 125 | 129, 72 (queue) 177 | 182; 16/4 heads of 64, 66 behind 4 000 169 -> 128.  Row groups of unlike
// fullness, where shares of equal pages are unlike: 33 sequences of 1 to 9 branches of 16 tokens (queue) 273 | 296, 52 454 | 471.
//
// RAGGED.  Workgroup w nominally takes [w * total / n, (w + 1) * total / n); a boundary inside an
// item's padding, or within `tol` units after it or before the item's end, is moved onto the item
// boundary: a sliver of a neighbouring item would cost a whole extra segment for a few pages.  The
// boundaries are tabulated in LDS (wgb), which also gives the owner of a unit by binary search.
struct Shares {
  int total, n, tol, pad;
  bool even;
  bool queue;
  int longest;      // QUEUE: cost of the costliest item
  int items;
  int piece;        // EVEN: p, the cost no piece exceeds
  double share;     // RAGGED: total / n, units per workgroup
  __device__ __forceinline__ int nominal_begin(int w) const { return min(total, (int)((double)w * share)); }
};

// Row group `rg` of sequence it->s.
__device__ __forceinline__ void set_group(const PlanArgs& a, const Sched& sc, const Groups& g, int rg, Item* it) {
  const int qs = sc.q0[it->s];
  it->rg = rg;
  it->np = g.pages(rg);
  it->q0 = qs + rg * a.qpg;
  it->nq = min(a.qpg, sc.q0[it->s + 1] - it->q0);
}

// The item that holds unit `u` (ragged regime), its sequence's groups, and the unit's index within it (padding first, then
// the pages).
__device__ Item locate(const PlanArgs& a, const Sched& sc, int pad, int u, Groups* groups, int* vpage) {
  int lo = 0, hi = a.B - 1;  // the last sequence that starts at or before u
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (sc.cu_units[mid] <= u) lo = mid; else hi = mid - 1;
  }
  Item it;
  it.s = lo;
  const Groups g = groups_of(a, sc, lo);
  const int per_head = g.before(g.n, pad);
  int rel = u - sc.cu_units[lo];
  it.h = quotient(rel, per_head);  // row groups of one KV head are neighbours: they read the same pages
  rel -= it.h * per_head;
  int rg = 0;
  if (g.step == 0) {
    if (g.n > 1) rg = quotient(rel, g.np + pad);
  } else {
    int hi_rg = g.n - 1;  // the last group that starts at or before rel
    while (rg < hi_rg) {
      const int mid = (rg + hi_rg + 1) >> 1;
      if (g.before(mid, pad) <= rel) rg = mid; else hi_rg = mid - 1;
    }
  }
  set_group(a, sc, g, rg, &it);
  const int start = g.before(rg, pad);
  *vpage = rel - start;
  it.first_unit = sc.cu_units[lo] + it.h * per_head + start;
  *groups = g;
  return it;
}

// The item after `it`; there has to be one.  (The kernel is one workgroup whose threads each walk a workgroup's share, so
// what a step of the walk takes adds up: with a look-up of every item, three divisions and two searches, the plan of a
// 64-sequence chunk took 38.0 us, 28.0 without; of eight prompts 21.7 -> 15.4, of 64 decoding sequences 22.0 -> 18.9.)
__device__ __forceinline__ void advance(const PlanArgs& a, const Sched& sc, int pad, Item* it, Groups* g) {
  it->first_unit += it->np + pad;
  int rg = it->rg + 1;
  if (rg >= g->n) {
    rg = 0;
    if (++it->h >= a.num_kv_heads) {
      it->h = 0;
      do ++it->s;  // sequences without units start where the next one does
      while (it->s < a.B - 1 && sc.cu_units[it->s + 1] <= it->first_unit);
      *g = groups_of(a, sc, it->s);
    }
  }
  set_group(a, sc, *g, rg, it);
}

// Cutting one item among its k workgroups (even regime).  A page of the branch region costs a wave
// more than a page before it (owner tags, masking, scores that are thrown away): measured between 1.1
// and 1.5 times, taken as 1.25.  The cut is therefore even in cost(p) = 4p + max(0, p - lp) rather than
// in pages: piece j starts at the first page p with cost(p) * k >= j * cost(np).
__device__ __forceinline__ int item_cut(const Item& it, int j, int k) {
  const int total = 4 * it.np + (it.np - it.lp);
  const int t = quotient(j * total + k - 1, k);
  return t <= 4 * it.lp ? (t + 3) >> 2 : it.lp + (t - 4 * it.lp + 4) / 5;
}
__device__ int share_begin(const PlanArgs& a, const Sched& sc, const Shares& sh, int w) {
  if (w <= 0) return 0;
  if (w >= sh.n) return sh.total;
  const int nominal = sh.nominal_begin(w);
  int vpage;
  Groups g;
  const Item it = locate(a, sc, sh.pad, nominal, &g, &vpage);
  const int vl = it.np + sh.pad;
  if (vpage <= sh.pad + sh.tol) return it.first_unit;
  if (vl - vpage <= sh.tol) return it.first_unit + vl;
  return nominal;
}

// EVEN: pieces of an item of np pages at page cost w, none of more than p (a piece is not shorter than
// MIN_PAGES_PER_WG pages, as far as the item allows).
__device__ __forceinline__ int even_pieces(int np, int w, int p, float rp /* 1 / p */) {
  // ceil(np w / p) by a float reciprocal, made exact by one correction (np w + p < 2^24, the estimate is off by one at
  // most)
  const int x = np * w + p - 1;
  int q = (int)((float)x * rp);
  if ((q + 1) * p <= x) ++q;
  else if (q * p > x) --q;
  return min(q, (np + MIN_PAGES_PER_WG - 1) / MIN_PAGES_PER_WG);
}
// Workgroups for one KV head of a sequence: n - 1 full row groups and a last one.
__device__ __forceinline__ int even_per_head(const PlanArgs& a, int np, int n, int nq_last, int p, float rp) {
  const int last = even_pieces(np, page_cost(a, nq_last), p, rp);
  return n > 1 ? (n - 1) * even_pieces(np, page_cost(a, a.qpg), p, rp) + last : last;
}

// QUEUE: class of a row group's cost, costliest first.
__device__ __forceinline__ int queue_bin(const PlanArgs& a, const Sched& sc, const Shares& sh, int e, int* s_out, int* rg_out,
                                         Groups* g) {
  int lo = 0, hi = a.B - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (sc.cu_units[mid] <= e) lo = mid; else hi = mid - 1;
  }
  *s_out = lo;
  *rg_out = e - sc.cu_units[lo];
  *g = groups_of(a, sc, lo);
  const int rows = sc.q0[lo + 1] - sc.q0[lo];
  const int cost = g->pages(*rg_out) * page_cost(a, *rg_out < g->n - 1 ? a.qpg : last_group(a, rows, g->n));
  const float scale = (float)(QUEUE_BINS - 1) / (float)sh.longest;
  return QUEUE_BINS - 1 - min(QUEUE_BINS - 1, (int)((float)cost * scale));
}

// Over the waves before the thread's own: the sum of what each of them has in `per_wave` (16-byte aligned; all of it on its
// way at once).
typedef int i32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ int sum_before(const int* per_wave) {
  static_assert(PLAN_THREADS == 8 * 64, "eight waves");
  const i32x4 lo = *(const i32x4*)per_wave, hi = *(const i32x4*)(per_wave + 4);
  const int wave = threadIdx.x >> 6;
  int sum = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) sum += (w < wave ? lo[w] : 0) + (w + 4 < wave ? hi[w] : 0);
  return sum;
}

// QUEUE: sorts the row groups by cost (`bins`: the first place of each class) and returns the cost of the longest workgroup.
// Its estimate: the item at rank k nwg, the first of a round, starts when the first of the workgroups gets free, which has
// taken the last of every round before; what comes after it is shorter and starts on others.  Exact for equal items, a little
// low for others.
__device__ __forceinline__ float queue_end(const PlanArgs& a, const Sched& sc, const Shares& sh, int* bins,
                                           int* scratch /* 3 * PLAN_THREADS / 64 */) {
  constexpr int NWV = PLAN_THREADS / 64;
  const int tid = threadIdx.x;
  const int groups = sc.cu_units[a.B];
  static_assert(QUEUE_BINS == 2 * PLAN_THREADS, "two bins per thread");
  bins[2 * tid] = bins[2 * tid + 1] = 0;
  __syncthreads();
  int s, rg;
  Groups g;
  for (int e = tid; e < groups; e += PLAN_THREADS) atomicAdd(&bins[queue_bin(a, sc, sh, e, &s, &rg, &g)], 1);
  __syncthreads();
  const int count[2] = {bins[2 * tid], bins[2 * tid + 1]};
  const int incl = wave_scan_add(count[0] + count[1]);
  if ((tid & 63) == 63) scratch[tid >> 6] = incl;
  __syncthreads();
  const int run = incl - count[0] - count[1] + sum_before(scratch);  // row groups of the classes before
  bins[2 * tid] = run;
  bins[2 * tid + 1] = run + count[0];
  // rounds (of nwg items) that end within the thread's classes, and the cost of the items they end with
  const float rn = __builtin_amdgcn_rcpf((float)a.nwg);
  auto rounds = [&](int items) -> int { return (int)(((float)items + 0.5f) * rn); };  // (off by one from 2^22 items on at worst)
  int first[3], ended[3], cls[2], sum = 0;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    first[i] = (run + (i > 0 ? count[0] : 0) + (i > 1 ? count[1] : 0)) * a.num_kv_heads;
    ended[i] = rounds(first[i]);
    if (i < 2) cls[i] = QUEUE_BINS - 1 - (2 * tid + i);
    if (i > 0) sum += (ended[i] - ended[i - 1]) * cls[i - 1];
  }
  const int incl_sum = wave_scan_add(sum);
  if ((tid & 63) == 63) scratch[NWV + (tid >> 6)] = incl_sum;
  __syncthreads();
  int before = incl_sum - sum + sum_before(scratch + NWV);
  int end = 0;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int k = rounds(first[i + 1] - 1);  // the last round that begins here, if one does
    if (first[i + 1] > first[i] && k * a.nwg >= first[i]) end = max(end, before + (k - ended[i] + 1) * cls[i]);
    before += (ended[i + 1] - ended[i]) * cls[i];
  }
  end = wave_scan_max(end);
  if ((tid & 63) == 63) scratch[2 * NWV + (tid >> 6)] = end;
  __syncthreads();
  const i32x4 lo = *(const i32x4*)(scratch + 2 * NWV), hi = *(const i32x4*)(scratch + 2 * NWV + 4);
#pragma unroll
  for (int w = 0; w < 4; ++w) end = max(w == 0 ? 0 : end, max(lo[w], hi[w]));
  return (float)end * ((float)sh.longest / (float)(QUEUE_BINS - 1));
}

// Fills the LDS tables and returns the shares.  All threads of the workgroup call it.  QUEUE: the kernel can take whole items
// from a queue.
template <bool QUEUE>
__device__ __forceinline__ Shares build_schedule(const PlanArgs& a, const Sched& sc,
                                                 int* scratch /* 7 * PLAN_THREADS / 64 + 2 ints */, int* bins /* QUEUE_BINS */) {
  constexpr int PER = (ASPD_MAX_BATCH + PLAN_THREADS - 1) / PLAN_THREADS;  // sequences per thread
  constexpr int NWV = PLAN_THREADS / 64;
  constexpr int ALL = 0x7fffffff;
  const int tid = threadIdx.x;
  int mine_p[PER], mine_i[PER];
  int sum_p = 0, sum_i = 0;
  int longest = 0;       // cost of the costliest item in the even regime (all pages of its sequence)
  int longest_q = 0;     // ... and whole (its row group's pages)
  int most = 0;          // for the queue regime: price of a page of the fullest row group,
  int shortest = ALL;    // ... and cost of the cheapest item
  unsigned cost16 = 0;   // of all items, whole, in units of 16 (less than 2^32 of them)
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int s = tid * PER + j;
    mine_p[j] = 0;
    mine_i[j] = 0;
    if (s < a.B) {
      const int T = a.seq_len[s];
      const int q0 = a.cu_seq_new[s];
      const int q1 = a.cu_seq_new[s + 1];
      sc.T[s] = T;
      sc.L[s] = a.stage_base[s];
      sc.q0[s] = q0;
      if (s == a.B - 1) sc.q0[a.B] = q1;
      const Groups g = groups_at(a, T, q1 - q0, quotient(rows_between(a, q0, q1) + a.qpg - 1, a.qpg));
      sc.ng[s] = g.n;
      const int np = g.np;
      if (np > 0 && g.n > 0) {
        mine_i[j] = g.n * a.num_kv_heads;
        mine_p[j] = g.before(g.n, 0) * a.num_kv_heads;
        const int w_full = page_cost(a, a.qpg), w_last = page_cost(a, last_group(a, q1 - q0, g.n));
        longest = max(longest, np * (g.n > 1 ? w_full : w_last));
        if (QUEUE) {
          most = max(most, g.n > 1 ? w_full : w_last);
          shortest = min(shortest, min(g.n > 1 ? g.pages(0) * w_full : ALL, np * w_last));
        }
        longest_q = max(longest_q, max(g.n > 1 ? g.pages(g.n - 2) * w_full : 0, np * w_last));
        cost16 += (unsigned)(((long)g.before(g.n - 1, 0) * w_full + (long)np * w_last) * a.num_kv_heads >> 4);
      }
      // (for the search below; the table is filled in for good later)
      sc.wgb[s] = mine_i[j] > 0 ? np : 0;
    }
    sum_p += mine_p[j];
    sum_i += mine_i[j];
  }
  // scans: inside the wave without LDS, across the waves through LDS (one barrier)
  const int incl_p = wave_scan_add(sum_p), incl_i = wave_scan_add(sum_i);
  longest = wave_scan_max(longest);
  longest_q = wave_scan_max(longest_q);
  cost16 = (unsigned)wave_scan_add((int)cost16);
  if (QUEUE) {
    most = wave_scan_max(most);
    shortest = ALL - wave_scan_max(ALL - shortest);
  }
  if ((tid & 63) == 63) {
    scratch[tid >> 6] = incl_p;
    scratch[NWV + (tid >> 6)] = incl_i;
    scratch[2 * NWV + (tid >> 6)] = longest;
    scratch[3 * NWV + (tid >> 6)] = longest_q;
    ((unsigned*)scratch)[4 * NWV + (tid >> 6)] = cost16;
    scratch[5 * NWV + (tid >> 6)] = most;
    scratch[6 * NWV + (tid >> 6)] = shortest;
  }
  __syncthreads();
  int run_p = incl_p - sum_p, run_i = incl_i - sum_i;  // exclusive within the wave
  int pages = 0, items = 0;
  longest = longest_q = most = 0;
  shortest = ALL;
  long cost = 0;
  const int used = (a.B + 64 * PER - 1) / (64 * PER);  // waves that hold sequences
#pragma unroll 1
  for (int w = 0; w < used; ++w) {
    const int tp = scratch[w], ti = scratch[NWV + w];
    if (w < (tid >> 6)) {
      run_p += tp;
      run_i += ti;
    }
    pages += tp;
    items += ti;
    longest = max(longest, scratch[2 * NWV + w]);
    longest_q = max(longest_q, scratch[3 * NWV + w]);
    cost += (long)((unsigned*)scratch)[4 * NWV + w] << 4;
    if (QUEUE) {
      most = max(most, scratch[5 * NWV + w]);
      shortest = min(shortest, scratch[6 * NWV + w]);
    }
  }
  if (items > a.max_items) items = pages = 0;  // rows that no metadata call has written: nothing is planned
  Shares sh;
  sh.pad = a.pad;
  sh.piece = 0;
  sh.even = false;
  sh.queue = false;
  sh.items = items;
  sh.longest = longest_q;
  const int w_full = page_cost(a, a.qpg);
  // ---- EVEN regime?  The smallest of 1 024 piece costs whose pieces fit the grid.  Fewer pieces come of a larger cost, so
  // it is found in two rounds of 32 candidates each: the first tries the largest cost of every 32, the second those of the
  // 32 that hold the answer.  16 threads share a candidate, each with its part of the sequences.  (All candidates in one
  // round, every thread with all sequences: the step of 27 mixed sequences took 7 us longer.)
  constexpr int CANDIDATES = 32;
  constexpr int SHARE = PLAN_THREADS / CANDIDATES;
  int* best = scratch + 7 * NWV;  // [2]: per round, the first candidate that fits
  if (tid < 2) best[tid] = 0x7fffffff;
  const int least = MIN_PAGES_PER_WG * page_cost(a, 1);
  const int step = max((longest - least + CANDIDATES * CANDIDATES - 2) / (CANDIDATES * CANDIDATES - 1), 1);  // (the last reaches longest)
  auto candidate = [&](int t) -> int { return min(max(longest, 1), least + t * step); };
  __syncthreads();
  if (items > 0 && items <= a.nwg) {
#pragma unroll 1
    for (int round = 0; round < 2; ++round) {
      const int t = round == 0 ? (tid / SHARE + 1) * CANDIDATES - 1 : best[0] - (CANDIDATES - 1) + tid / SHARE;
      if (round == 1 && best[0] == 0x7fffffff) break;
      const int p = candidate(t);
      const float rp = __builtin_amdgcn_rcpf((float)p);
      int need = 0;  // (at most items * pages / MIN_PAGES_PER_WG, with no more items than workgroups)
#pragma unroll 1
      for (int s = tid % SHARE; s < a.B; s += SHARE)
        if (sc.wgb[s] > 0)
          need += a.num_kv_heads *
                  even_per_head(a, sc.wgb[s], sc.ng[s], last_group(a, sc.q0[s + 1] - sc.q0[s], sc.ng[s]), p, rp);
      static_assert(SHARE == 16, "a row of lanes");
      need = row_scan_add(need);
      if (tid % SHARE == SHARE - 1 && need <= a.nwg) atomicMin(best + round, t);
      __syncthreads();
    }
  }
  if (best[1] != 0x7fffffff) {
    // pieces of this cost against what the ragged regime's longest workgroups would carry (a share and two
    // segment starts)
    sh.piece = candidate(best[1]);
    // (x <= y / n for whole numbers as x n <= y: 64-bit divisions took longer than the whole search)
    sh.even = ((long)sh.piece - a.pad * w_full) * a.nwg <= (a.w_wave ? cost : (long)pages);
  }
  __syncthreads();  // (best is read by all before anyone reuses scratch)
  if (sh.even) {
    // cu_units[s]: first workgroup of sequence s' items (the unit of this regime is the workgroup)
    sh.pad = 0;
    int mine_w[PER], sum_w = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int s = tid * PER + j;
      mine_w[j] = 0;
      if (s < a.B && mine_i[j] > 0)
        mine_w[j] = a.num_kv_heads * even_per_head(a, sc.wgb[s], sc.ng[s], last_group(a, sc.q0[s + 1] - sc.q0[s], sc.ng[s]),
                                                   sh.piece, __builtin_amdgcn_rcpf((float)sh.piece));
      sum_w += mine_w[j];
    }
    const int incl_w = wave_scan_add(sum_w);
    if ((tid & 63) == 63) scratch[tid >> 6] = incl_w;
    __syncthreads();
    int run_w = incl_w - sum_w, total_w = 0;
#pragma unroll 1
    for (int w = 0; w < used; ++w) {
      if (w < (tid >> 6)) run_w += scratch[w];
      total_w += scratch[w];
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int s = tid * PER + j;
      if (s < a.B) sc.cu_units[s] = run_w;
      run_w += mine_w[j];
    }
    if (tid == 0) sc.cu_units[a.B] = total_w;
    sh.total = total_w;
    sh.n = total_w;
    sh.tol = 0;
    sh.share = 1.0;
    __syncthreads();
    return sh;
  }
  // ---- QUEUE regime?
  float ragged = 0.f;  // cost of the longest workgroup there
  bool whole = QUEUE && items > a.nwg && 4L * sh.longest * a.nwg <= 5L * cost;
  if (whole) {
    ragged = (float)pages * (float)most / (float)a.nwg * (1.f + 1.f / 12.f) + (float)(QUEUE_CUT * w_full);
    // (some workgroup takes as many items as there are rounds: where that alone is too long, nothing has to be sorted)
    whole = (float)((items + a.nwg - 1) / a.nwg) * (float)shortest <= ragged;
  }
  if (whole) {
    // cu_units[s]: row groups of the sequences before s
    int run = run_i;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int s = tid * PER + j;
      if (s < a.B) sc.cu_units[s] = run / a.num_kv_heads;
      run += mine_i[j];
    }
    if (tid == 0) sc.cu_units[a.B] = items / a.num_kv_heads;
    __syncthreads();
    if (queue_end(a, sc, sh, bins, scratch) <= ragged) {
      sh.queue = true;
      sh.n = a.nwg;
      return sh;
    }
    __syncthreads();
  }
  sh.total = pages + sh.pad * items;
  sh.n = pages > 0 ? max(1, min(a.nwg, sh.total / MIN_PAGES_PER_WG)) : 0;
  sh.tol = min((sh.total / max(sh.n, 1)) >> 3, a.pad);
  sh.share = (double)sh.total / (double)max(sh.n, 1);
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int s = tid * PER + j;
    if (s < a.B) sc.cu_units[s] = run_p + sh.pad * run_i;
    run_p += mine_p[j];
    run_i += mine_i[j];
  }
  if (tid == 0) sc.cu_units[a.B] = sh.total;
  __syncthreads();
  for (int w = tid; w <= sh.n; w += PLAN_THREADS) sc.wgb[w] = share_begin(a, sc, sh, w);
  __syncthreads();
  return sh;
}

// RAGGED: the workgroup whose share holds unit u.
__device__ int share_owner(const Sched& sc, const Shares& sh, int u) {
  // boundaries sit within a padding's length of w * share: try the nominal owner and its neighbours first
  {
    const int g = min(sh.n - 1, max(0, (int)((float)u / (float)sh.share)));
#pragma unroll
    for (int d = -1; d <= 1; ++d) {
      const int w = g + d;
      if (w >= 0 && w < sh.n && sc.wgb[w] <= u && (w == sh.n - 1 || sc.wgb[w + 1] > u)) return w;
    }
  }
  int lo = 0, hi = sh.n - 1;  // last w with wgb[w] <= u
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (sc.wgb[mid] <= u) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// EVEN: the one segment of workgroup w, and the first and last workgroup of its item.
__device__ bool even_share(const PlanArgs& a, const Sched& sc, const Shares& sh, int w, Item* out, int* page0,
                           int* page1, int* owner, int* w_last) {
  int lo = 0, hi = a.B - 1;  // the last sequence whose first workgroup is at or before w
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (sc.cu_units[mid] <= w) lo = mid; else hi = mid - 1;
  }
  Item it;
  it.s = lo;
  it.np = pages_of(a, sc, lo);
  const int ngroups = sc.ng[lo], rows = sc.q0[lo + 1] - sc.q0[lo];
  const float rp = __builtin_amdgcn_rcpf((float)sh.piece);
  // workgroups per item: of a full row group, of the last
  const int k_full = even_pieces(it.np, page_cost(a, a.qpg), sh.piece, rp);
  const int k_last = even_pieces(it.np, page_cost(a, last_group(a, rows, ngroups)), sh.piece, rp);
  const int per_head = (ngroups - 1) * k_full + k_last;
  const int local = w - sc.cu_units[lo];
  it.h = quotient(local, per_head);    // row groups of one KV head are neighbours: they read the same pages
  const int in_head = local - it.h * per_head;
  it.rg = min(quotient(in_head, k_full), ngroups - 1);
  const int j = in_head - it.rg * k_full;
  const int k = it.rg == ngroups - 1 ? k_last : k_full;
  it.first_unit = 0;
  it.lp = a.has_owner ? min(it.np, sc.L[lo] / ASPD_BLOCK) : it.np;
  const int qs = sc.q0[lo];
  it.q0 = qs + it.rg * a.qpg;
  it.nq = min(a.qpg, sc.q0[lo + 1] - qs - it.rg * a.qpg);
  *out = it;
  *page0 = item_cut(it, j, k);
  *page1 = item_cut(it, j + 1, k);
  *owner = w - j;
  *w_last = w - j + k - 1;
  return *page1 > *page0;
}

// A workgroup's walk over its share, as an iterator: each step gives a segment and the first and last
// workgroup that hold a part of its item.
struct Walk {
  int u, end;
  Item it;      // ragged regime: the item that holds u, while u < end
  Groups g;     // its sequence's groups
  int vpage;    // index of u within it
  bool even_pending;
};
__device__ __forceinline__ Walk walk_begin(const PlanArgs& a, const Sched& sc, const Shares& sh, int w) {
  Walk wk = {};
  wk.even_pending = sh.even && w < sh.n;
  if (!sh.even && w < sh.n) {
    wk.u = sc.wgb[w];
    wk.end = sc.wgb[w + 1];
    if (wk.u < wk.end) wk.it = locate(a, sc, sh.pad, wk.u, &wk.g, &wk.vpage);
  }
  return wk;
}
__device__ __forceinline__ bool walk_next(const PlanArgs& a, const Sched& sc, const Shares& sh, int w, Walk* wk,
                                          Item* it, int* page0, int* page1, int* owner, int* w_last) {
  if (sh.even) {
    if (!wk->even_pending) return false;
    wk->even_pending = false;
    return even_share(a, sc, sh, w, it, page0, page1, owner, w_last);
  }
  // the next run of real pages in [u, end)
  while (wk->u < wk->end) {
    const int v0 = wk->vpage;
    const int v1 = min(wk->it.np + sh.pad, v0 + (wk->end - wk->u));
    *it = wk->it;
    *page0 = max(0, v0 - sh.pad);
    *page1 = max(0, v1 - sh.pad);
    wk->u += v1 - v0;
    if (wk->u < wk->end) {  // the item ends here
      advance(a, sc, sh.pad, &wk->it, &wk->g);
      wk->vpage = 0;
    }
    if (*page1 > *page0) {
      *owner = *page0 == 0 ? w : share_owner(sc, sh, it->first_unit + sh.pad);
      *w_last = *page1 == it->np ? w : share_owner(sc, sh, it->first_unit + sh.pad + it->np - 1);
      return true;
    }
  }
  return false;
}

// Segments of a workgroup that pass 1 keeps in LDS for pass 2 (8 words each); a workgroup with more is walked
// on from where pass 1 stood when the room ran out.
__host__ __device__ constexpr int plan_cached_segments(int nwg) { return nwg <= 256 ? 4 : (nwg <= 512 ? 2 : 1); }

// Block ids of the first sixteen pages of a run, for a workgroup's header.
__device__ __forceinline__ void load_ids(const PlanArgs& a, int s, int p0, int p1, int (&ids)[PLAN_IDS]) {
  const int32_t* bt = a.block_tables + (long)s * a.max_blocks_per_seq;
#pragma unroll
  for (int k = 0; k < PLAN_IDS; ++k) ids[k] = bt[min(p0 + k, p1 - 1)];  // all on their way at once
#pragma unroll
  for (int k = 0; k < PLAN_IDS; ++k) ids[k] = min(max(ids[k], 0), a.num_blocks - 1);
}
__device__ __forceinline__ void store_ids(int32_t* hdr, const int (&ids)[PLAN_IDS]) {
#pragma unroll
  for (int k = 0; k < PLAN_IDS; k += 4)
    *(i32x4*)(hdr + PLAN_HDR_IDS + k) = i32x4{ids[k], ids[k + 1], ids[k + 2], ids[k + 3]};
}

// QUEUE: headers and list from the places of the classes.  Item r in the order of costs is the first of workgroup r, and the
// (r / nwg)-th of workgroup r % nwg.
__device__ void write_queue(const PlanArgs& a, const Sched& sc, const Shares& sh, int* bins /* QUEUE_BINS */) {
  const int tid = threadIdx.x;
  const int groups = sc.cu_units[a.B];
  int s, rg;
  Groups g;
  const int extra = sh.items - a.nwg, each = extra / a.nwg, rest = extra - each * a.nwg;
  int32_t* list = a.plan + PLAN_HDR * a.nwg;
  for (int e = tid; e < groups; e += PLAN_THREADS) {
    const int bin = queue_bin(a, sc, sh, e, &s, &rg, &g);
    const int rank = atomicAdd(&bins[bin], 1) * a.num_kv_heads;
    const int q0 = sc.q0[s] + rg * a.qpg, np = g.pages(rg), nq = min(a.qpg, sc.q0[s + 1] - q0);
    int ids[PLAN_IDS];
    if (rank < a.nwg) load_ids(a, s, 0, np, ids);
    int turn = quotient(rank, a.nwg), w = rank - turn * a.nwg;
    for (int h = 0; h < a.num_kv_heads; ++h) {
      const int next = w * each + min(w, rest);
      int32_t* d = turn == 0 ? a.plan + PLAN_HDR * w : list + PLAN_SEG * (next + turn - 1);
      *(i32x4*)d = i32x4{s | (h << 16), q0, nq, 0};
      *(i32x4*)(d + 4) = i32x4{np, np, w | (w << 16), sc.L[s]};
      if (turn == 0) {
        d[PLAN_HDR_NSEG] = 1 + each + (w < rest ? 1 : 0);
        d[PLAN_HDR_NEXT] = next;
        d[PLAN_HDR_QUEUE] = extra;
        store_ids(d, ids);
      }
      if (++w == a.nwg) {
        w = 0;
        ++turn;
      }
    }
  }
}

// LDS of the plan behind the tables of the schedule.
__host__ __device__ constexpr int plan_work_ints(int nwg) {
  const int cached = nwg * plan_cached_segments(nwg) * PLAN_SEG;
  return cached > QUEUE_BINS ? cached : QUEUE_BINS;
}

// Pass 2: header and segments of workgroup w (`cnt` of them, those beyond the first from place `run` of the list on).
__device__ __forceinline__ void plan_write(const PlanArgs& a, const Sched& sc, const Shares& sh, int w, int cnt, int run,
                                           int CS, const int* seg_cache, const Walk& resume) {
  int32_t* seg_list = a.plan + PLAN_HDR * a.nwg;
  int32_t* hdr = a.plan + PLAN_HDR * w;
  hdr[PLAN_HDR_NSEG] = cnt;
  hdr[PLAN_HDR_NEXT] = run;
  hdr[PLAN_HDR_QUEUE] = 0;
  const int cached = min(cnt, CS);
  for (int i = 0; i < cached; ++i) {
    const int* c = seg_cache + (w * CS + i) * PLAN_SEG;
    const i32x4 lo = *(const i32x4*)c, hi = *(const i32x4*)(c + 4);
    int32_t* d = i == 0 ? hdr : seg_list + PLAN_SEG * (run + i - 1);
    *(i32x4*)d = lo;
    *(i32x4*)(d + 4) = hi;
    if (i == 0) {
      int ids[PLAN_IDS];
      load_ids(a, lo[0] & 0xffff, lo[3], hi[0], ids);
      store_ids(hdr, ids);
    }
  }
  if (cnt > CS) {
    Walk wk = resume;
    Item it;
    int p0, p1, owner, w_last;
    int i = CS;
    while (walk_next(a, sc, sh, w, &wk, &it, &p0, &p1, &owner, &w_last)) {
      int32_t* d = seg_list + PLAN_SEG * (run + i - 1);
      *(i32x4*)d = i32x4{it.s | (it.h << 16), it.q0, it.nq, p0};
      *(i32x4*)(d + 4) = i32x4{p1, it.np, owner | (w_last << 16), sc.L[it.s]};
      ++i;
    }
  }
}

// (Two kernels, so that the plan of a decoding step, whose instructions are fetched anew every step, has nothing of the queue
// in it: with one, the step of one sequence took 66.4 us instead of 65.7.)
template <bool QUEUE>
__global__ __launch_bounds__(PLAN_THREADS) void plan_kernel(PlanArgs a) {
  extern __shared__ int lds[];
  __shared__ __attribute__((aligned(16))) int scratch[7 * PLAN_THREADS / 64 + 2];
  __shared__ int wave_tot[PLAN_THREADS / 64];
  const Sched sc = sched_at(lds, a.B);
  int* seg_cache = lds + sched_ints(a.B);
  const int CS = plan_cached_segments(a.nwg);
  const int tid = threadIdx.x;
  const Shares sh = build_schedule<QUEUE>(a, sc, scratch, seg_cache);
  if (QUEUE && sh.queue) {
    write_queue(a, sc, sh, seg_cache);
    return;
  }

  // ---- pass 1: the segments of each workgroup (thread w: workgroup w); the first few are kept in LDS
  const int w = tid;
  int cnt = 0;
  Walk resume;  // where the walk stood after the cached segments
  if (w < a.nwg) {
    Walk wk = walk_begin(a, sc, sh, w);
    resume = wk;
    Item it;
    int p0, p1, owner, w_last;
    while (cnt < CS && walk_next(a, sc, sh, w, &wk, &it, &p0, &p1, &owner, &w_last)) {
      int* c = seg_cache + (w * CS + cnt) * PLAN_SEG;
      *(i32x4*)c = i32x4{it.s | (it.h << 16), it.q0, it.nq, p0};
      *(i32x4*)(c + 4) = i32x4{p1, it.np, owner | (w_last << 16), sc.L[it.s]};
      ++cnt;
    }
    resume = wk;
    // the rest is only counted here (most of a step of the walk is then dead code)
    if (cnt == CS)
      while (walk_next(a, sc, sh, w, &wk, &it, &p0, &p1, &owner, &w_last)) ++cnt;
  }
  // exclusive scan, over the workgroups, of the segments beyond the first
  int run = 0;
  if (!sh.even) {  // (a segment each there)
    const int extra = max(cnt - 1, 0);
    const int incl = wave_scan_add(extra);
    if ((tid & 63) == 63) wave_tot[tid >> 6] = incl;
    __syncthreads();
    run = incl - extra;
    for (int wv = 0; wv < (tid >> 6); ++wv) run += wave_tot[wv];
  }

  if (w < a.nwg) plan_write(a, sc, sh, w, cnt, run, CS, seg_cache, resume);
}

std::atomic<int> g_cu_count[64];

}  // namespace

int aspd_device_cu_count() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  const bool slot = dev >= 0 && dev < 64;
  if (slot && (n = g_cu_count[dev].load(std::memory_order_relaxed)) > 0) return n;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) return 256;
  if (slot) g_cu_count[dev].store(n, std::memory_order_relaxed);
  return n;
}

int aspd_choose_variant(const aspd_kv* kv, int32_t B, int32_t NQ, int32_t max_new_per_seq, int32_t max_workgroups,
                        bool chunk_call, bool has_owner, AttnVariant* v) {
  const int G = kv->num_q_heads / kv->num_kv_heads;
  v->has_owner = has_owner;
  v->nt = 0;
  if (kv->dtype == ASPD_BF16) {
    // Row group of the streaming kernel: `nt` MFMA tiles of 16 rows, as few as the caller's bound on new
    // tokens per sequence allows (fewer tiles leave more registers for loads in flight), three when there
    // is no bound.  A sequence with more rows than one group holds is processed in several groups.
    int tiles = NT_MAX;
    if (max_new_per_seq > 0) tiles = std::min(NT_MAX, (max_new_per_seq * G + 15) / 16);
    while (tiles < NT_MAX && 16 * tiles < G) ++tiles;
    if (G > 16 * tiles) return 0;
    // Many rows per KV head (branch chunks, prefills): the waves split the rows instead of the keys.
    const bool many_rows = (long)max_new_per_seq * G > 16 * NT_MAX;
    const bool by_rows = (long)NQ * G > 16 * NT_MAX && (many_rows || (chunk_call && max_new_per_seq == 0));
    v->kernel = by_rows ? KERNEL_BF16_ROWS : KERNEL_BF16_STREAM;
    v->nt = by_rows ? 0 : tiles;
    v->rows_cap = by_rows ? ROWS_NW * 32 : 16 * tiles;
  } else {
    if (G > F32_ROWS) return 0;
    v->kernel = KERNEL_F32;
    v->rows_cap = F32_ROWS;
  }
  v->qpg = v->rows_cap / G;
  // A segment's fixed cost (start-up, reduction across waves, partial, merge) in units of the time one
  // more page takes its workgroup.
  v->pad = v->kernel == KERNEL_BF16_STREAM ? PAD_STREAM * 128 / kv->head_dim
           : (v->kernel == KERNEL_BF16_ROWS ? PAD_ROWS : PAD_COMPUTE);
  // Grid: as many workgroups as stay resident at once (one per compute unit: every kernel here needs more
  // than half of a compute unit's LDS or registers), never more than the pages can feed, never more than
  // the caller allows.
  long nwg = aspd_device_cu_count();
  if (v->kernel == KERNEL_BF16_ROWS) nwg = std::min(nwg, (long)MAX_WG_ROWS);
  const long groups_max = (long)B + NQ / v->qpg;
  const long units_max = groups_max * kv->num_kv_heads * kv->max_blocks_per_seq;
  // (... but a workgroup per item when the items are few: four items of six pages each are done sooner by
  // four workgroups than by two that take them in turn)
  nwg = std::min(nwg, std::max((units_max + MIN_PAGES_PER_WG - 1) / MIN_PAGES_PER_WG, groups_max * kv->num_kv_heads));
  if (max_workgroups > 0) nwg = std::min(nwg, (long)max_workgroups);
  v->nwg = (int)std::max(1L, std::min(nwg, (long)MAX_WG));
  v->stream_once = max_new_per_seq > 0 && max_new_per_seq <= v->qpg;
  return 1;
}

uint64_t aspd_plan_key(const aspd_kv* kv, const AttnVariant& v, int32_t B) {
  // What a plan has to agree on with the call that reads it, besides the device arrays: which items there are and which
  // kernel takes them.  (The query heads per KV head are in qpg; the sizes of the pool and of the block tables only bound
  // what a plan holds, and the kernels check that themselves.)
  uint64_t k = 1 << 16 | (uint64_t)(kv->num_kv_heads & 0xffff);
  k = k * 4 + (uint64_t)v.kernel;
  k = k * 2 + (v.has_owner ? 1 : 0);
  k = k * 2048 + (uint64_t)v.nwg;
  k = k * 512 + (uint64_t)v.qpg;
  k = k * 256 + (uint64_t)v.pad;
  k = k * 1024 + (uint64_t)B;
  return k;  // 58 bits
}

size_t aspd_plan_words(const aspd_kv* kv, const AttnVariant& v, int32_t B, int32_t NQ) {
  const size_t items = ((size_t)B + (size_t)NQ / v.qpg) * kv->num_kv_heads;
  return (size_t)PLAN_HDR * v.nwg + (size_t)PLAN_SEG * (items + v.nwg);
}

int aspd_plan_launch(const aspd_kv* kv, const AttnVariant& v, int32_t B, int32_t NQ, const int32_t* stage_base_d,
                     const int32_t* seq_len_d, const int32_t* cu_seq_new_d, int32_t* plan_d, hipStream_t stream) {
  PlanArgs a;
  a.stage_base = stage_base_d;
  a.seq_len = seq_len_d;
  a.cu_seq_new = cu_seq_new_d;
  a.block_tables = kv->block_tables_d;
  a.plan = plan_d;
  a.B = B;
  a.nwg = v.nwg;
  a.qpg = v.qpg;
  a.pad = v.pad;
  a.num_kv_heads = kv->num_kv_heads;
  a.max_blocks_per_seq = kv->max_blocks_per_seq;
  a.num_blocks = kv->num_blocks;
  a.has_owner = v.has_owner ? 1 : 0;
  a.w_page = v.kernel == KERNEL_BF16_ROWS ? ROWS_PAGE_COST : 1;
  a.w_wave = v.kernel == KERNEL_BF16_ROWS ? 1 : 0;
  a.rows_per_query = kv->num_q_heads / kv->num_kv_heads;
  a.NQ = NQ;
  a.max_items = (int)((B + (long)NQ / v.qpg) * kv->num_kv_heads);
  const size_t lds = (size_t)(sched_ints(B) + plan_work_ints(v.nwg)) * sizeof(int);
  if (v.kernel == KERNEL_BF16_ROWS) hipLaunchKernelGGL(plan_kernel<true>, dim3(1), dim3(PLAN_THREADS), lds, stream, a);
  else hipLaunchKernelGGL(plan_kernel<false>, dim3(1), dim3(PLAN_THREADS), lds, stream, a);
  ASPD_HIP_CHECK(hipGetLastError());
  return ASPD_OK;
}
