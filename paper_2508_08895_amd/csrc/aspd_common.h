// Internal helpers shared by the gfx950 kernels of libaspd (not part of the public ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "aspd.h"

#define ASPD_BLOCK 16  // tokens per KV block (the only block size the kernels are written for)

#define ASPD_HIP_CHECK(expr)                       \
  do {                                             \
    hipError_t _e = (expr);                        \
    if (_e != hipSuccess) return ASPD_ERR_HIP;     \
  } while (0)

// Flat-argument views of the public structs: kernels take these by value.
struct KvView {
  const void*    k;
  const void*    v;
  const int32_t* block_tables;
  int32_t        num_blocks, num_q_heads, num_kv_heads, head_dim, max_blocks_per_seq;
};

struct StateView {
  int32_t        B, NB;
  int32_t*       stage_base;
  int32_t*       seq_len;
  const int32_t* cu_branches;
  int32_t*       branch_len;
  uint8_t*       slot_owner;
  int32_t        owner_stride;
  int32_t*       fault;
  int32_t*       main_pos;
  int32_t*       stage_open;
};

struct StepView {
  int32_t  NQ;
  int32_t  max_new_per_seq;
  int32_t* cu_new;
  int32_t* cu_seq_new;
  int32_t* q_seq;
  int32_t* q_branch;
  int32_t* position_ids;
  int32_t* logical_slot;
  int64_t* slot_mapping;
  int32_t* kv_len;
};

static inline KvView make_view(const aspd_kv* kv) {
  return KvView{kv->k_cache_d, kv->v_cache_d, kv->block_tables_d, kv->num_blocks, kv->num_q_heads,
                kv->num_kv_heads, kv->head_dim, kv->max_blocks_per_seq};
}
static inline StateView make_view(const aspd_state* st) {
  return StateView{st->B, st->NB, st->stage_base_d, st->seq_len_d, st->cu_branches_d, st->branch_len_d,
                   st->slot_owner_d, st->owner_stride, st->fault_d, st->main_pos_d, st->stage_open_d};
}
static inline StepView make_view(const aspd_step* sp) {
  return StepView{sp->NQ, sp->max_new_per_seq, sp->cu_new_d, sp->cu_seq_new_d, sp->q_seq_d, sp->q_branch_d, sp->position_ids_d,
                  sp->logical_slot_d, sp->slot_mapping_d, sp->kv_len_d};
}

// Host-side validation of the cache descriptor; returns an ASPD_* code.
int aspd_check_kv(const aspd_kv* kv);

// Inclusive scans over a row of 16 lanes and over the 64 lanes of a wave by data-parallel moves: four and six instructions a
// value, where shuffles go through LDS, three instructions and a wait each.  The last lane has the result over all
// of them.  Lanes without a source see 0.
template <typename Op>
__device__ __forceinline__ int row_scan(int v, Op op) {
  v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false));  // one lane up
  v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false));  // two
  v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false));  // four
  v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false));  // eight
  return v;
}
template <typename Op>
__device__ __forceinline__ int wave_scan(int v, Op op) {
  v = row_scan(v, op);
  v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false));  // last lane of rows 0 and 2 to rows 1 and 3
  v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false));  // lane 31 to rows 2 and 3
  return v;
}
__device__ __forceinline__ int row_scan_add(int v) {
  return row_scan(v, [](int a, int b) { return a + b; });
}
__device__ __forceinline__ int wave_scan_add(int v) {
  return wave_scan(v, [](int a, int b) { return a + b; });
}
__device__ __forceinline__ int wave_scan_max(int v) {  // of values that are not negative
  return wave_scan(v, [](int a, int b) { return a > b ? a : b; });
}

// x / d for x >= 0, d > 0 by a float reciprocal rd of d, made exact (the loops run once at most while the quotient is below
// 2^20; an integer division by a value the compiler does not know is thirty to forty instructions).
__device__ __forceinline__ int quotient(int x, int d, float rd) {
  int q = (int)((float)x * rd);
  int r = x - q * d;
  while (r < 0) {
    --q;
    r += d;
  }
  while (r >= d) {
    ++q;
    r -= d;
  }
  return q;
}
__device__ __forceinline__ int quotient(int x, int d) { return quotient(x, d, __builtin_amdgcn_rcpf((float)d)); }
