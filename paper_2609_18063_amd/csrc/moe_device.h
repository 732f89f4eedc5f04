// Device-side helpers shared by the gfx950 kernels of the MoE decode path.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include "../../include/moe_api.h"

namespace moe {

constexpr int kWave = 64;

// 16-byte vector load / store through the vector memory path.
struct alignas(16) U4 {
  uint32_t x, y, z, w;
};

__device__ __forceinline__ U4 ld16(const void* p) {
  return *reinterpret_cast<const U4*>(p);
}

// DPP lane moves (gfx9 data-parallel primitives): a few cycles each, against
// an LDS round trip for a shuffle.  Controls used: quad_perm [1,0,3,2] (0xB1)
// and [2,3,0,1] (0x4E), row_half_mirror (0x141), row_mirror (0x140),
// row_bcast15 (0x142), row_bcast31 (0x143).  `old` is the value a lane keeps
// when its row is masked off.
template <int CTRL, int ROWMASK = 0xf>
__device__ __forceinline__ float dpp_f(float old, float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(v), CTRL, ROWMASK, 0xf, false));
}
template <int CTRL, int ROWMASK = 0xf>
__device__ __forceinline__ int dpp_i(int old, int v) {
  return __builtin_amdgcn_update_dpp(old, v, CTRL, ROWMASK, 0xf, false);
}

// Sum over each row of 16 lanes; every lane of the row receives the sum.
__device__ __forceinline__ float row16_sum(float v) {
  v += dpp_f<0xB1>(0.f, v);
  v += dpp_f<0x4E>(0.f, v);
  v += dpp_f<0x141>(0.f, v);
  v += dpp_f<0x140>(0.f, v);
  return v;
}

// Sum over the 64 lanes of a wave, returned to every lane.
__device__ __forceinline__ float wave_sum(float v) {
  v = row16_sum(v);
  v += dpp_f<0x142, 0xa>(0.f, v);
  v += dpp_f<0x143, 0xc>(0.f, v);
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// Sum over groups of `width` consecutive lanes (width a power of two <= 64);
// every lane of a group receives its group's sum.
__device__ __forceinline__ float group_sum(float v, int width) {
  if (width >= 64) return wave_sum(v);
  if (width >= 2) v += dpp_f<0xB1>(0.f, v);
  if (width >= 4) v += dpp_f<0x4E>(0.f, v);
  if (width >= 8) v += dpp_f<0x141>(0.f, v);
  if (width >= 16) v += dpp_f<0x140>(0.f, v);
  if (width >= 32) v += __shfl_xor(v, 16, kWave);
  return v;
}

// Dot product of 32 int4 codes (16 bytes, even input in the low nibble) with
// 32 fp32 activations.  Codes are exact small integers in fp32.
__device__ __forceinline__ float dot32_q4(const U4& q, const float* x) {
  const uint32_t w[4] = {q.x, q.y, q.z, q.w};
  float a0 = 0.f, a1 = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t lo = w[i] & 0x0F0F0F0Fu;
    const uint32_t hi = (w[i] >> 4) & 0x0F0F0F0Fu;
    const float* xv = x + 8 * i;
    a0 = fmaf((float)(lo & 0xFFu), xv[0], a0);
    a1 = fmaf((float)(hi & 0xFFu), xv[1], a1);
    a0 = fmaf((float)((lo >> 8) & 0xFFu), xv[2], a0);
    a1 = fmaf((float)((hi >> 8) & 0xFFu), xv[3], a1);
    a0 = fmaf((float)((lo >> 16) & 0xFFu), xv[4], a0);
    a1 = fmaf((float)((hi >> 16) & 0xFFu), xv[5], a1);
    a0 = fmaf((float)(lo >> 24), xv[6], a0);
    a1 = fmaf((float)(hi >> 24), xv[7], a1);
  }
  return a0 + a1;
}

// Dot product of 8 fp16 weights with 8 fp16 activations, fp32 accumulate.
__device__ __forceinline__ float dot8_h(const U4& a, const U4& b, float acc) {
  const uint32_t wa[4] = {a.x, a.y, a.z, a.w};
  const uint32_t wb[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    __half2 ha = *reinterpret_cast<const __half2*>(&wa[i]);
    __half2 hb = *reinterpret_cast<const __half2*>(&wb[i]);
    float2 fa = __half22float2(ha);
    float2 fb = __half22float2(hb);
    acc = fmaf(fa.x, fb.x, acc);
    acc = fmaf(fa.y, fb.y, acc);
  }
  return acc;
}

__device__ __forceinline__ float2 h2f2(uint32_t bits) {
  return __half22float2(*reinterpret_cast<const __half2*>(&bits));
}

// Resolve list position k of token t to a bundle, or nullptr (status set).
__device__ __forceinline__ const moe_bundle* resolve_expert(int k, int K, int E, const int32_t* idx_t,
                                                            const int32_t* slot_of,
                                                            const moe_bundle* bundles,
                                                            uint32_t* status, bool report) {
  int e = (k < K) ? idx_t[k] : E + (k - K);
  if (k < K && (e < 0 || e >= E)) {
    if (report && status) atomicOr(status, MOE_STATUS_BAD_INDEX);
    return nullptr;
  }
  int s = slot_of[e];
  if (s < 0) {
    if (report && status) atomicOr(status, MOE_STATUS_SLOT_MISS);
    return nullptr;
  }
  return bundles + s;
}

// Largest value over the wave, returned to every lane.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  v = max(v, (uint32_t)dpp_i<0xB1>(0, (int)v));
  v = max(v, (uint32_t)dpp_i<0x4E>(0, (int)v));
  v = max(v, (uint32_t)dpp_i<0x141>(0, (int)v));
  v = max(v, (uint32_t)dpp_i<0x140>(0, (int)v));
  v = max(v, (uint32_t)dpp_i<0x142, 0xa>(0, (int)v));
  v = max(v, (uint32_t)dpp_i<0x143, 0xc>(0, (int)v));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Order key of a logit for the top-k: larger logits have larger keys (NaN as
// -inf, -0 as +0), and no key is 0 (-inf is 0x007FFFFF).
__device__ __forceinline__ uint32_t topk_key(float v) {
  if (v != v) v = -INFINITY;
  if (v == 0.f) v = 0.f;
  const uint32_t b = __float_as_uint(v);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float topk_key_value(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// Softmax-top-k of one token's logits by one wave (K <= 32, E <= 64 V). Selection
// is on the fp32 logits (the softmax is increasing), descending, ties to the lower
// index; weights are the softmax renormalized over the selected set. Lane l holds
// the V logits l V .. l V + V - 1 as order keys; each of K rounds takes the largest
// key left over the wave (ties: the lowest lane, then its lowest position, which is
// the lowest id). A round is a dozen lane moves: no barrier and no LDS. The keys are
// kept in groups of four with their largest, so that a round looks through and
// updates one group (E 1024, K 32: T = 1 10.3 us a call, T = 4096 21.0; with all 16 keys
// of a lane looked through 16.4 and 32.1).
template <int V>
__device__ __forceinline__ void wave_topk(const float* l, int E, int K, int32_t* idx, float* w) {
  constexpr int C = V < 4 ? V : 4, G = V / C;
  const int lane = threadIdx.x & 63;
  uint32_t key[V], top[G];                       // key 0: no logit, or taken (no real key is 0)
#pragma unroll
  for (int j = 0; j < V; ++j) key[j] = lane * V + j < E ? topk_key(l[lane * V + j]) : 0u;
  auto group_top = [&](int g) {
    uint32_t b = key[g * C];
#pragma unroll
    for (int j = 1; j < C; ++j) b = max(b, key[g * C + j]);
    top[g] = b;
  };
#pragma unroll
  for (int g = 0; g < G; ++g) group_top(g);
  uint32_t mk = 0;                               // lane k: the k-th largest key and its id
  int mi = 0;
  for (int k = 0; k < K; ++k) {
    uint32_t best = top[0];
#pragma unroll
    for (int g = 1; g < G; ++g) best = max(best, top[g]);
    const uint32_t m = wave_max_u32(best);
    const int win = __builtin_ctzll(__ballot(best == m));
    int g0 = G - 1;
#pragma unroll
    for (int g = G - 2; g >= 0; --g) g0 = top[g] == m ? g : g0;
    g0 = G > 1 ? __builtin_amdgcn_readlane(g0, win) : 0;  // (uniform)
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (g != g0) continue;
      int pos = C - 1;
#pragma unroll
      for (int j = C - 2; j >= 0; --j) pos = key[g * C + j] == m ? j : pos;
      const int id = __builtin_amdgcn_readlane(pos, win) + win * V + g * C;
      if (lane == k) {
        mk = m;
        mi = id;
      }
#pragma unroll
      for (int j = 0; j < C; ++j) key[g * C + j] = lane == win && j == pos ? 0u : key[g * C + j];
      group_top(g);
    }
  }
  const float v = lane < K ? topk_key_value(mk) : 0.f;
  const float mx = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0));
  const float ex = lane < K ? expf(v - mx) : 0.f;
  const float sum = wave_sum(ex);
  if (lane < K) {
    idx[lane] = mi;
    w[lane] = ex / sum;
  }
}

}  // namespace moe
