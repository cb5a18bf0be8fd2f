// aspd_rope_append: the step between the metadata and the attention call.  The position ids of
// ASPD Sec. 3.2, Eq. 4 act on the attention scores through the rotary encoding of the queries and
// keys; this kernel rotates the new tokens' Q rows in place, rotates their K rows into the paged
// cache at slot_mapping and copies their V rows there.
//
// Rotary encoding as defined by RoFormer, in the rotate-half layout: head_dim D is split into the
// pairs (i, i + D/2); pair i of a vector at position p turns by the angle p * theta^(-2i/D).
//
// Few rows: a launch is bound by its own latency; many rows: by the bytes it moves, each
// Q, K and V element read and written once.  So a row is taken in units of 16 bytes from either half of a head (VEC pairs
// whole, lanes on consecutive chunks), a thread's first units are on their way before the angles are worked
// out, and the angles (formed in double: a float product would lose 1e-3 rad at positions of a few ten
// thousand) and their sines and cosines are computed once per row and pair and shared through LDS.
// One workgroup per row: four or eight rows per workgroup (an angle for every thread) measured 3 to 8 % slower from
// 4096 rows on (32768 rows, 32/8 heads of 128: 159 against 151 us) and the same below.
// Before, a thread took 2-byte elements and each of its wave's heads had its own sines: 6000 rows 39.7 -> 28.5 us,
// 550 rows 8.7 -> 6.1 us, 4 rows 4.5 -> 2.9 us; 330000 rows 1.68 -> 1.45 ms, 5.6 TB/s (a plain copy: 4.7).
#include "aspd_common.h"

namespace {

constexpr int ROPE_THREADS = 256;

// VEC pairs per unit: 16 bytes of T, or 1 where a pointer is not aligned to 16 bytes.
template <typename T, int D, int VEC>
__global__ __launch_bounds__(ROPE_THREADS) void rope_append_kernel(KvView kv, const int32_t* __restrict__ position_ids,
                                                                   const int64_t* __restrict__ slot_mapping, T* q,
                                                                   const T* k_new, const T* v_new, double log2_theta) {
  constexpr int HALF = D / 2;
  constexpr int UPH = HALF / VEC;  // units per head
  constexpr int U = 2;             // units a thread keeps in flight
  typedef T vec __attribute__((ext_vector_type(VEC)));
  __shared__ __attribute__((aligned(16))) float cs[HALF], sn[HALF];
  const int tid = threadIdx.x;
  const long row = blockIdx.x;
  // the row's units: its Q heads, then K, then V
  const int uq = kv.num_q_heads * UPH, uk = kv.num_kv_heads * UPH, units = uq + 2 * uk;
  T* qrow = q + row * kv.num_q_heads * D;
  const T* krow = k_new + row * kv.num_kv_heads * D;
  const T* vrow = v_new + row * kv.num_kv_heads * D;
  const int pos = position_ids[row];
  const long slot = slot_mapping[row];

  vec a[U], b[U];
  auto issue = [&](int u0) {
#pragma unroll
    for (int x = 0; x < U; ++x) {
      const int u = u0 + x * ROPE_THREADS;
      if (u >= units) continue;
      const T* src = u < uq ? qrow + u / UPH * D : (u < uq + uk ? krow + (u - uq) / UPH * D : vrow + (u - uq - uk) / UPH * D);
      src += u % UPH * VEC;  // (uq and uk are multiples of UPH)
      a[x] = *(const vec*)src;
      b[x] = *(const vec*)(src + HALF);
    }
  };
  issue(tid);
  asm volatile("" ::: "memory");  // these loads leave before the angles are worked out
  if (tid < HALF) {
    const double freq = exp2(-(2.0 * tid / D) * log2_theta);
    double s, c;
    sincos((double)pos * freq, &s, &c);
    cs[tid] = (float)c;
    sn[tid] = (float)s;
  }
  __syncthreads();
  const bool placed = slot >= 0 && slot < (long)kv.num_blocks * ASPD_BLOCK;  // never write outside the pools
  const long place = placed ? ((slot / ASPD_BLOCK) * kv.num_kv_heads * ASPD_BLOCK + slot % ASPD_BLOCK) * D : 0;
  for (int u0 = tid;;) {
#pragma unroll
    for (int x = 0; x < U; ++x) {
      const int u = u0 + x * ROPE_THREADS;
      if (u >= units || (u >= uq && !placed)) continue;
      const bool is_v = u >= uq + uk;
      const int ch = u % UPH * VEC;
      T* dst = u < uq ? qrow + u / UPH * D
                      : (T*)(is_v ? kv.v : kv.k) + place + (long)((u - uq - (is_v ? uk : 0)) / UPH) * ASPD_BLOCK * D;
      vec oa = a[x], ob = b[x];
      if (!is_v) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          const float xa = (float)a[x][e], xb = (float)b[x][e];
          oa[e] = (T)(xa * cs[ch + e] - xb * sn[ch + e]);
          ob[e] = (T)(xb * cs[ch + e] + xa * sn[ch + e]);
        }
      }
      *(vec*)(dst + ch) = oa;
      *(vec*)(dst + ch + HALF) = ob;
    }
    u0 += U * ROPE_THREADS;
    if (u0 >= units) break;
    issue(u0);
  }
}

template <typename T, int D, int VEC>
void rope_launch(const KvView& kv, const aspd_step* step, void* q, const void* k_new, const void* v_new, double l2,
                 hipStream_t hs) {
  hipLaunchKernelGGL((rope_append_kernel<T, D, VEC>), dim3(step->NQ), dim3(ROPE_THREADS), 0, hs, kv, step->position_ids_d,
                     step->slot_mapping_d, (T*)q, (const T*)k_new, (const T*)v_new, l2);
}

}  // namespace

extern "C" int aspd_rope_append(const aspd_kv* kv, const aspd_step* step, void* q_d, const void* k_new_d,
                                const void* v_new_d, float rope_theta, void* stream) {
  int rc = aspd_check_kv(kv);
  if (rc != ASPD_OK) return rc;
  if (!step || step->NQ < 0) return ASPD_ERR_INVALID_ARG;
  if (step->NQ == 0) return ASPD_OK;
  if (!step->position_ids_d || !step->slot_mapping_d || !q_d || !k_new_d || !v_new_d) return ASPD_ERR_INVALID_ARG;
  if (!(rope_theta > 1.f)) return ASPD_ERR_INVALID_ARG;
  const KvView kvv = make_view(kv);
  const double l2 = log2((double)rope_theta);
  hipStream_t hs = (hipStream_t)stream;
  const bool wide = (((uintptr_t)q_d | (uintptr_t)k_new_d | (uintptr_t)v_new_d | (uintptr_t)kvv.k | (uintptr_t)kvv.v) & 15) == 0;
#define ASPD_ROPE(TYPE, DD)                                                                                       \
  do {                                                                                                            \
    if (wide) rope_launch<TYPE, DD, 16 / sizeof(TYPE)>(kvv, step, q_d, k_new_d, v_new_d, l2, hs);                 \
    else rope_launch<TYPE, DD, 1>(kvv, step, q_d, k_new_d, v_new_d, l2, hs);                                      \
  } while (0)
  if (kv->dtype == ASPD_BF16) {
    if (kv->head_dim == 128) ASPD_ROPE(__bf16, 128); else ASPD_ROPE(__bf16, 64);
  } else {
    if (kv->head_dim == 128) ASPD_ROPE(float, 128); else ASPD_ROPE(float, 64);
  }
#undef ASPD_ROPE
  ASPD_HIP_CHECK(hipGetLastError());
  return ASPD_OK;
}
