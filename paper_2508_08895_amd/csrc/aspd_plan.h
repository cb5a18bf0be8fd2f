// The per-step plan of the attention launches (internal to libaspd, not part of the public ABI).
//
// The three attention calls of a step (ASPD Sec. 3.2-3.3: parallel decode, branch chunk, serial
// decode) split the key ranges of their (sequence, row group, KV head) items among the workgroups of
// one launch.  How they are split depends on nothing but the lengths of the batch and a few launch
// constants, so it is worked out once per step, by a small kernel that runs right after the metadata
// kernel of aspd_build_branch_meta, and every attention launch of the step (one per layer) starts from
// the result: a workgroup loads its 128-byte header and has its first pages on their way after one
// memory round trip.
//
// Layout of a plan (32-bit words), for a grid of `nwg` workgroups:
//   [0, 32 nwg)                    one header per workgroup
//   [32 nwg, 32 nwg + 8 nsegs)     the segments that are not the first of their workgroup, in the
//                                  order the workgroups walk them
// Header: words 0-7 the workgroup's first segment, 8 the number of its segments (0: nothing to do),
//   9 the index of its second segment in the list above, 10 in a plan whose items are taken from a queue the number of
//   items that are not the first of a workgroup (0 in other plans; the kernel's order of them is that of their index in
//   their workgroup, then of the workgroups), 16-31 the block ids of the first sixteen
//   pages of its first segment (read again from the block table before they count, see the kernels).
// Segment: a run of pages [page0, page1) of one item, for all rows of the item's row group:
//   0  sequence | KV head << 16        1  first packed query row of the row group
//   2  queries of the row group        3  page0        4  page1
//   5  pages of the whole item (the segment is the whole item iff page0 = 0 and page1 = this)
//   6  first | last << 16 workgroup that holds a part of the item (they combine their partial results)
//   7  stage_base of the sequence
#pragma once

#include "aspd_common.h"

constexpr int PLAN_HDR = 32;         // words per workgroup header
constexpr int PLAN_SEG = 8;          // words per segment
constexpr int PLAN_HDR_NSEG = 8;
constexpr int PLAN_HDR_NEXT = 9;
constexpr int PLAN_HDR_QUEUE = 10;
constexpr int PLAN_HDR_IDS = 16;
constexpr int PLAN_IDS = 16;

// Words of the arrival counters that the queue uses (the row-splitting kernel, whose grid is smaller, has the others).
constexpr int QUEUE_NEXT = 1022, QUEUE_DONE = 1023;
// A whole-sequence launch has a queue per XCD from SEQ_QUEUE_ITEMS items a workgroup on.  What that gains is reads past the L2
// and past the memory-side cache; what it costs is a search for work at the end, about 4 us a launch, and where row groups are
// short the order by length.  One queue -> one per XCD, two layers, us: 64 sequences of 1 100 to 9 400 (one layer) 23 900 ->
// 20 290; 9 of 2 150 to 6 900 (20 items) 1 880 -> 1 830; 13 of 1 200 to 3 200 (13) 1 359 -> 1 337; 24 of 500 to 2 000
// 1 081 -> 1 073.  Below the line: 6 of 4 000 to 6 600 (8) 522 | 524, 40 of 400 (9) 526 | 539, 33 of 190 to 370 (5) 297 | 322,
// 15 of 110 to 300 (2) 64 | 71.
constexpr int SEQ_QUEUES_LOG2 = 3, SEQ_QUEUES = 1 << SEQ_QUEUES_LOG2;
constexpr int SEQ_QUEUE_ITEMS = 12;
constexpr int XCD_L2_BYTES = 4 << 20;
constexpr int QUEUE_XCD = QUEUE_NEXT - SEQ_QUEUES;

constexpr int MAX_WG = 512;          // upper bound of any attention grid
constexpr int NT_MAX = 3;            // 16-row MFMA tiles per row group of the streaming bf16 kernel
constexpr int F32_ROWS = 4;          // rows per row group of the fp32 kernel
constexpr int ROWS_NW = 8;           // waves per workgroup of the row-splitting (chunk) kernel, 32 rows each
constexpr int MAX_WG_ROWS = 256;     // its largest grid
constexpr int MIN_PAGES_PER_WG = 16; // key ranges are not split finer than this
constexpr int PAD_STREAM = 32;       // fixed cost of a segment in pages, bandwidth-bound kernel at head_dim 128
constexpr int PAD_COMPUTE = 8;       // the same for the fp32 kernel
constexpr int PAD_ROWS = 32;         // and for the row-splitting kernel: a segment there costs about 17 us (Q operands
                                     // of 256 rows into registers, 64-128 KB of output or partial, its share of a
                                     // merge), 25-40 pages' worth.  It decides where items are cut evenly and prices
                                     // ragged shares.  One layer with 16 / 32 / 48, us: branch prefixes of 5 to 21 tokens
                                     // behind 500 to 3 000 (20 sequences) 92 / 74 / 74, behind 200 to 9 000 (40) 257 /
                                     // 240 / 248, behind 100 to 16 000 (40) 419 / 378 / 376, one prompt of 2 100 98 / 91 /
                                     // 92, four of 600 73 / 74 / 80; the mean over 71 such steps 1.020 / 1 / 1.003

// Row-splitting kernel, cost of a page: ROWS_PAGE_COST and 1 per wave that has rows up to four, ROWS_FULL_COST more from five on
// (measured in a stage opening over 12 sequences, us a page without a segment's start: 0.26 with four waves, 0.42 with five,
// 0.43 with eight).  With 1 per wave up to eight -> this, us: that step 269.3 -> 260.1, 6 sequences of 1 000 to 6 000 with
// chunks of 2 to 12 in 3 to 9 branches 123.0 -> 119.9, 30 of 1 000 to 8 000 368 -> 362; 13 other chunks between 0.989 and
// 1.009 times as long.
constexpr int ROWS_PAGE_COST = 4, ROWS_FULL_COST = 9;
static_assert(MAX_WG <= QUEUE_XCD, "queue words");

enum AttnKernel { KERNEL_F32 = 0, KERNEL_BF16_STREAM = 1, KERNEL_BF16_ROWS = 2 };

// Which kernel an attention call takes and how its launch is shaped: decided on the host from the
// cache's shape and the step's host fields, by the metadata call (which builds the plan for it) and by
// the attention call (which checks that the plan it is given was built for the same launch).
struct AttnVariant {
  int  kernel;       // AttnKernel
  int  nt;           // 16-row tiles per row group (streaming bf16 kernel)
  int  qpg;          // queries per row group
  int  rows_cap;     // rows per row group the partial slots are sized for
  int  nwg;          // workgroups of the launch
  int  pad;          // virtual pages in front of every item (ragged batches)
  bool stream_once;  // no page is read by more than one row group
  bool has_owner;    // rows may carry branch tags (all calls but serial decode)
};

// 0 when the shape is not supported.  `chunk_call`: the call is aspd_attn_branch_chunk (matters only
// when the step gives no bound on the new tokens per sequence).
int aspd_choose_variant(const aspd_kv* kv, int32_t B, int32_t NQ, int32_t max_new_per_seq, int32_t max_workgroups,
                        bool chunk_call, bool has_owner, AttnVariant* out);

// Identifies the launch a plan was built for; never 0.
uint64_t aspd_plan_key(const aspd_kv* kv, const AttnVariant& v, int32_t B);

// Words a plan for `v` may take.
size_t aspd_plan_words(const aspd_kv* kv, const AttnVariant& v, int32_t B, int32_t NQ);

// Enqueues the kernel that writes the plan of the step for launch shape `v` to plan_d.
int aspd_plan_launch(const aspd_kv* kv, const AttnVariant& v, int32_t B, int32_t NQ, const int32_t* stage_base_d,
                     const int32_t* seq_len_d, const int32_t* cu_seq_new_d, int32_t* plan_d, hipStream_t stream);

// ---- The plan of a whole-sequence step (aspd_build_sequence_meta / aspd_attn_full_sequence) -------
// Layout (32-bit words):
//   [0, 16)                 header: 0 row groups in the list, 1 tokens per row group, 2 NQ, 3 B, 4 entries in the list of
//                           pieces (0: no row group is cut), 5 the KV heads that list was made for, 6 the places of
//                           partial results it gives away (an attention call on a cache of another number of KV heads,
//                           or without room for those places, takes every row group whole)
//   [16, 16 + NQ4)          per packed row, the first slot of the row's own stage (its own slot for a
//                           main-branch row); NQ4 = NQ rounded up to a multiple of 4
//   then 4 words per row group, in the order workgroups take them: sequence, first packed row,
//                           tokens, pages of its key range
//   then NQ4 words          per packed row, the first slot of the row's own branch in its stage (its own slot
//                           for a main-branch row): a row sees [0, stage start) and [this, its own slot]
//   then 2 words per piece  where the longest row groups' key ranges are cut, in the order workgroups take them: row
//                           group, piece | pieces << 8 | place of its first head's partial results << 16
constexpr int SEQ_PLAN_HDR = 16;
constexpr int SEQ_HDR_PIECES = 4;
constexpr int SEQ_HDR_HEADS = 5;
constexpr int SEQ_HDR_PLACES = 6;
constexpr int SEQ_PIECES_MAX = 8;    // of one row group
constexpr int SEQ_ENTRIES = 1024;    // room in the list of pieces
constexpr int SEQ_PIECE_MIN = 24;    // pages of a piece, and how many more the longest row group has at least where any
constexpr int SEQ_PIECE_GAIN = 48;   // is cut
// Whether row groups may be cut at all, as far as sizes known on the host say.
static inline bool aspd_sequence_may_cut(const aspd_kv* kv, int32_t B, int32_t NQ, int qpg, int cus) {
  return kv->max_blocks_per_seq >= SEQ_PIECE_MIN + SEQ_PIECE_GAIN && ((long)B + NQ / qpg) * kv->num_kv_heads <= 2L * cus;
}
// Tokens per row group: what the row-splitting kernel holds per workgroup.
static inline int aspd_sequence_qpg(int G) { return ROWS_NW * 32 / G; }
// Identifies such a plan; no value aspd_plan_key returns has bit 62 set.
static inline uint64_t aspd_sequence_plan_key(int qpg, int32_t B) {
  return ((uint64_t)1 << 62) | ((uint64_t)qpg << 16) | (uint64_t)B;
}
size_t aspd_sequence_plan_words(const aspd_kv* kv, int32_t B, int32_t NQ);
// Index of the row groups and of the branch starts in it.
static inline size_t aspd_sequence_plan_items(int32_t NQ) { return (size_t)SEQ_PLAN_HDR + (((size_t)NQ + 3) & ~(size_t)3); }
static inline size_t aspd_sequence_plan_lo(int G, int32_t B, int32_t NQ) {
  return aspd_sequence_plan_items(NQ) + 4 * ((size_t)B + (size_t)NQ / aspd_sequence_qpg(G));
}

static inline size_t aspd_sequence_plan_pieces(int G, int32_t B, int32_t NQ) {
  return aspd_sequence_plan_lo(G, B, NQ) + (((size_t)NQ + 3) & ~(size_t)3);
}
// Pieces (over all heads) that a workspace of aspd_workspace_bytes has room for the partial results of, two slots each.
int aspd_sequence_parts(const aspd_kv* kv, int32_t B, int32_t NQ);

// Compute units of the current device (256 when there is none to ask, as on a build host).
int aspd_device_cu_count();
