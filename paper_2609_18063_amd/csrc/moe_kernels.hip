// gfx950 kernels of the MoE decode hot path: layer input, routing / prerouting,
// int4 group-64 SwiGLU experts with the unmerged LoRA delta, combine.
//
// Data layout (all row-major, see include/moe_api.h): int4 codes [out][in/2]
// with the even input in the low nibble, (scale, zero) fp16 pairs
// [out][in/64], LoRA A [r][in] and B [out][r] fp16.
//
// Lane mapping of the int4 matvecs: a row of `in` inputs is split into 16-byte
// chunks of 32 codes; LPR = min(64, in/32) lanes share one row and each lane
// owns CPL = max(1, in/2048) chunks, so one wave instruction covers 64/LPR
// rows with fully coalesced 16-byte loads.  A lane's chunks are the same for
// every row it visits, so the 32*CPL activations it needs stay in registers.
#include <algorithm>
#include <type_traits>

#include "moe_kernels.h"
#include "moe_xchg.h"

namespace moe {

// ------------------------------------------------------------------------
// Layer input: RMS normalization to fp16.  The sum of squares, the scale and
// the product are fp64 and the product is rounded once to fp16, so the fp16
// rounding of every element does not depend on the order of the reduction.
// A few tokens are latency-bound (one load, a wave reduction, one barrier, one
// store); many are bound by memory. The row stays in registers between the sum
// and the product: d 2048, T = 1 2.1 us, T = 3100 7.8 us (4.9 TB/s); 256 threads
// with an eight-barrier tree, a second read of the row and the divide and
// square root of 1 / sqrt took 4.6 and 16.6 us.
// ------------------------------------------------------------------------

// 1 / sqrt(m) for m > 0, within a few fp64 ulps over the whole fp64 range (the
// hardware estimate refined by two Newton steps); 0 for m = inf.
__device__ __forceinline__ double rsqrt_full(double m) {
  double y = __builtin_amdgcn_rsq(m);
  y = y * (1.5 - 0.5 * (m * y) * y);
  y = y * (1.5 - 0.5 * (m * y) * y);
  return m == INFINITY ? 0.0 : y;
}

// Sum over the workgroup (whole waves), returned to every thread; red: one
// double per wave.
__device__ __forceinline__ double block_sum_f64(double v, double* red) {
  v = eng::wave_sum_f64(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) s += red[i];
  return s;
}

// d a multiple of 4, d <= 4 NV blockDim.x
template <int NV>
__global__ void __launch_bounds__(512) rmsnorm_f16_kernel(const float* __restrict__ xi, int d,
                                                          __half* __restrict__ x) {
  __shared__ double red[8];
  const float4* row = reinterpret_cast<const float4*>(xi + (size_t)blockIdx.x * d);
  uint2* out = reinterpret_cast<uint2*>(x + (size_t)blockIdx.x * d);
  const int nv = d >> 2;
  float4 v[NV];
  double acc = 0.0;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int j = threadIdx.x + i * blockDim.x;
    v[i] = j < nv ? row[j] : float4{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const double a = v[i].x, b = v[i].y, c = v[i].z, e = v[i].w;
    acc += (a * a + b * b) + (c * c + e * e);
  }
  const double r = rsqrt_full(block_sum_f64(acc, red) / (double)d + 1e-6);
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int j = threadIdx.x + i * blockDim.x;
    __half h[4] = {eng::f64_to_h((double)v[i].x * r), eng::f64_to_h((double)v[i].y * r),
                   eng::f64_to_h((double)v[i].z * r), eng::f64_to_h((double)v[i].w * r)};
    if (j < nv) out[j] = *reinterpret_cast<const uint2*>(h);
  }
}

// Any d (rows that are not whole 16-byte pieces, or longer than the registers hold).
__global__ void __launch_bounds__(256) rmsnorm_f16_any_kernel(const float* __restrict__ xi, int d,
                                                              __half* __restrict__ x) {
  __shared__ double red[4];
  const float* row = xi + (size_t)blockIdx.x * d;
  double acc = 0.0;
  for (int j = threadIdx.x; j < d; j += blockDim.x) {
    const double v = row[j];
    acc += v * v;
  }
  const double r = rsqrt_full(block_sum_f64(acc, red) / (double)d + 1e-6);
  for (int j = threadIdx.x; j < d; j += blockDim.x) x[(size_t)blockIdx.x * d + j] = eng::f64_to_h((double)row[j] * r);
}

// Router / prerouter logits of a few tokens: one row of W per wave, one token
// per grid row, two waves per workgroup, so that the rows of one token spread
// over the chip and each wave has its whole row in flight. Latency-bound: with
// the selection, 5.0 us a call at T = 1, d 2048, E 256. (The selection by the
// last workgroup to finish, behind a counter, took 21 us: its two agent-scope
// fences write back the L2, in every workgroup.)
constexpr int kRouteRows = 2;
__global__ void __launch_bounds__(64 * kRouteRows) route_rows_kernel(const __half* __restrict__ x,
                                                                     const __half* __restrict__ W, int E,
                                                                     int d, float* __restrict__ logits) {
  const int t = blockIdx.y, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int e = blockIdx.x * kRouteRows + wave;
  if (e >= E) return;
  const __half* xr = x + (size_t)t * d;
  const __half* wr = W + (size_t)e * d;
  float acc = 0.f;
#pragma unroll 4
  for (int c = lane; c < (d >> 3); c += kWave) acc = dot8_h(ld16(wr + (size_t)c * 8), ld16(xr + (size_t)c * 8), acc);
  acc = wave_sum(acc);
  if (lane == 0) logits[(size_t)t * E + e] = acc;
}

// The same for many tokens, a dense contraction on the matrix cores: a
// workgroup forms 16 MB tokens x 16 NB experts, its eight waves one eighth of
// d each (a short chain of v_mfma_f32_16x16x32_f16 per accumulator, whose
// operands are loaded straight from global memory in 64-byte row pieces); the
// eight partial sums are added in LDS as a tree. Every row is read by
// E / (16 NB) or T / (16 MB) workgroups from the L2. Rows past T or E read
// the last row and are not stored. Bound by the L2 reads of the operands at
// large T (203 MB in 31 us with 2 x 2 blocks at T = 3100, d 2048, E 256; 103 MB
// with 4 x 4 blocks, 20.5 us), by one round trip at small T. With the selection,
// at d 2048 / E 256: 8.6 us at T = 64, 12.5 at 512, 25 at 3100 (one wave per row
// and token: 9.3, 37 and 187 us). Two chains per wave keep the error against
// float64 below the row kernel's (9.4e-8 against 1.1e-7 of the logits).
typedef _Float16 mf_h8 __attribute__((ext_vector_type(8)));
typedef float mf_f4 __attribute__((ext_vector_type(4)));
constexpr int kRouteWaves = 8;
template <int MB, int NB>
__global__ void __launch_bounds__(64 * kRouteWaves) route_mfma_kernel(const __half* __restrict__ x,
                                                                      const __half* __restrict__ W, int T,
                                                                      int E, int d,
                                                                      float* __restrict__ logits) {
  __shared__ float red[kRouteWaves][MB * NB][4][kWave];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int col = lane & 15, kq = lane >> 4;
  const int nb = (E + 16 * NB - 1) / (16 * NB);
  const int e0 = (blockIdx.x % nb) * 16 * NB, t0 = (blockIdx.x / nb) * 16 * MB;
  const int kw = d / kRouteWaves;                // a multiple of 64 (d >= 512)
  const int k0 = wave * kw + kq * 8;
  const __half *xr[MB], *wr[NB];
#pragma unroll
  for (int m = 0; m < MB; ++m) xr[m] = x + (size_t)min(t0 + 16 * m + col, T - 1) * d + k0;
#pragma unroll
  for (int n = 0; n < NB; ++n) wr[n] = W + (size_t)min(e0 + 16 * n + col, E - 1) * d + k0;
  constexpr int NC = 2;                          // two chains: the k steps of even and odd index
  mf_f4 acc[NC][MB][NB];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
      for (int n = 0; n < NB; ++n) acc[c][m][n] = mf_f4{0.f, 0.f, 0.f, 0.f};
  constexpr int KS = MB * NB == 1 ? 8 : MB * NB <= 4 ? 4 : 2;  // k steps whose loads are in flight at once
  for (int k = 0; k < kw; k += 32 * KS) {
    mf_h8 a[KS][MB], b[KS][NB];
#pragma unroll
    for (int u = 0; u < KS; ++u) {
      const bool in = k + 32 * u < kw;           // uniform
#pragma unroll
      for (int n = 0; n < NB; ++n)
        b[u][n] = in ? *reinterpret_cast<const mf_h8*>(wr[n] + k + 32 * u) : mf_h8{};
#pragma unroll
      for (int m = 0; m < MB; ++m)
        a[u][m] = in ? *reinterpret_cast<const mf_h8*>(xr[m] + k + 32 * u) : mf_h8{};
    }
#pragma unroll
    for (int u = 0; u < KS; ++u)
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < NB; ++n)
          acc[u % NC][m][n] =
              __builtin_amdgcn_mfma_f32_16x16x32_f16(a[u][m], b[u][n], acc[u % NC][m][n], 0, 0, 0);
  }
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        red[wave][m * NB + n][i][lane] = acc[0][m][n][i] + acc[1][m][n][i];
  __syncthreads();
  // lane (col, kq) of block (m, n) holds tokens 16 m + 4 kq + i, expert 16 n + col
  for (int p = threadIdx.x; p < MB * NB * 256; p += 64 * kRouteWaves) {
    const int blk = p >> 8, i = (p >> 6) & 3, l = p & 63;
    float v[kRouteWaves];
#pragma unroll
    for (int q = 0; q < kRouteWaves; ++q) v[q] = red[q][blk][i][l];
    const float s = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
    const int t = t0 + 16 * (blk / NB) + 4 * (l >> 4) + i, e = e0 + 16 * (blk % NB) + (l & 15);
    if (t < T && e < E) logits[(size_t)t * E + e] = s;
  }
}

// One 512-thread workgroup per token (E <= 256, K <= 32): two-stage ranking of the keys
// (moe_xchg.h), a few barriers whatever K is.
__global__ void __launch_bounds__(512) topk_block_kernel(const float* __restrict__ logits, int E, int K,
                                                         int32_t* __restrict__ idx, float* __restrict__ w) {
  __shared__ float lg[256];
  __shared__ uint64_t keys[256];
  __shared__ int part[256];
  __shared__ uint64_t cand[128];
  __shared__ uint64_t sorted[32];
  const int t = blockIdx.x;
  if ((int)threadIdx.x < E) lg[threadIdx.x] = logits[(size_t)t * E + threadIdx.x];
  __syncthreads();
  eng::block_topk(lg, E, K, idx + (size_t)t * K, w + (size_t)t * K, keys, part, cand, sorted);
}

// One wave per token, K rounds: 3.6 us at T = 2048, K 8 and 6.2 us for a workgroup per
// token. For E 1000, K 8, T = 1, 5.4 us; a wave finding the K-th key bit by bit took 17.
template <int V>
__global__ void __launch_bounds__(256) topk_wave_kernel(const float* __restrict__ logits, int T, int E, int K,
                                                        int32_t* __restrict__ idx, float* __restrict__ w) {
  const int t = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (t >= T) return;
  wave_topk<V>(logits + (size_t)t * E, E, K, idx + (size_t)t * K, w + (size_t)t * K);
}

// Sigmoid-group selection (App. A), one 512-thread workgroup per token
// (E <= 256): sigma = sigmoid(l) in fp32, the selection score sigma + bias;
// a group's score is the sum of its two largest selection scores (its one
// score if it has one member); the top_groups best groups survive (ties to
// the lower group); the K largest surviving scores are selected with the
// engines' two-stage ranking (descending, ties to the lower id); the weights
// use the raw sigma: w = scale sigma / (sum of the selected sigma + 1e-20).
__global__ void __launch_bounds__(512) topk_sigmoid_group_kernel(const float* __restrict__ logits,
                                                                 const float* __restrict__ bias, int E,
                                                                 int K, int n_groups, int top_groups,
                                                                 float scale, int32_t* __restrict__ idx,
                                                                 float* __restrict__ w) {
  __shared__ float lg[256];
  __shared__ eng::SigmoidScratch sc;
  __shared__ uint64_t keys[256];
  __shared__ int part[256];
  __shared__ uint64_t cand[128];
  __shared__ uint64_t sorted[32];
  const int t = blockIdx.x;
  if ((int)threadIdx.x < E) lg[threadIdx.x] = logits[(size_t)t * E + threadIdx.x];
  __syncthreads();
  eng::block_topk_sigmoid_group(lg, bias, E, K, n_groups, top_groups, scale, idx + (size_t)t * K,
                                w + (size_t)t * K, sc, keys, part, cand, sorted);
}

// ------------------------------------------------------------------------
// Expert stage 1: raw int4 matvecs W_gate x, W_up x (row pairs) and the LoRA
// projections A_gate x, A_up x.
// ------------------------------------------------------------------------
template <int CPL>
__device__ __forceinline__ void load_x_lane(const __half* x, int c0, int lpr, float (&xf)[CPL][32],
                                            float (&xs)[CPL]) {
#pragma unroll
  for (int cc = 0; cc < CPL; ++cc) {
    const int c = c0 + lpr * cc;
    const U4* p = reinterpret_cast<const U4*>(x + (size_t)c * 32);
    float s = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const U4 v = p[q];
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float2 f = h2f2(w[i]);
        xf[cc][q * 8 + 2 * i] = f.x;
        xf[cc][q * 8 + 2 * i + 1] = f.y;
        s += f.x + f.y;
      }
    }
    xs[cc] = s;
  }
}

template <int LPR, int CPL, int RP>
__global__ void __launch_bounds__(256) ffn_gateup_kernel(FfnArgs a) {
  constexpr int RPI = kWave / LPR;               // rows per wave instruction
  constexpr int PAIRS_PER_WG = 4 * RP * RPI;
  const int t = blockIdx.y;
  const int nblk_w = (a.I + PAIRS_PER_WG - 1) / PAIRS_PER_WG;
  const int nblk_a = (2 * a.r + 3) / 4;
  const int nblk = nblk_w + nblk_a;
  const int k = blockIdx.x / nblk, b = blockIdx.x % nblk;
  const int n = a.n_list;
  const moe_bundle* bd = resolve_expert(k, a.K, a.E, a.idx + (size_t)t * a.K, a.slot_of,
                                        a.bundles, a.status, b == 0 && threadIdx.x == 0);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const __half* x = a.x + (size_t)t * a.d;
  const size_t tk = (size_t)t * n + k;

  if (b >= nblk_w) {
    // LoRA A rows: wave handles row rr = 4 * (b - nblk_w) + wave of [A_gate; A_up].
    const int rr = 4 * (b - nblk_w) + wave;
    if (rr >= 2 * a.r) return;
    const int p = rr / a.r, kk = rr % a.r;
    float* dst = (p == 0 ? a.ag : a.au) + tk * a.r + kk;
    const moe_proj* pr = bd ? (p == 0 ? &bd->gate : &bd->up) : nullptr;
    if (!pr || !pr->lora_a || !pr->lora_b) {
      if (lane == 0) *dst = 0.f;
      return;
    }
    const __half* arow = reinterpret_cast<const __half*>(pr->lora_a) + (size_t)kk * a.d;
    float acc = 0.f;
    for (int c = lane; c < (a.d >> 3); c += kWave)
      acc = dot8_h(ld16(arow + (size_t)c * 8), ld16(x + (size_t)c * 8), acc);
    acc = wave_sum(acc);
    if (lane == 0) *dst = acc;
    return;
  }

  const int c0 = lane % LPR;
  const int sub = lane / LPR;
  const int pair0 = b * PAIRS_PER_WG + wave * RP * RPI;
  if (!bd) {
#pragma unroll
    for (int rp = 0; rp < RP; ++rp) {
      const int i = pair0 + rp * RPI + sub;
      if (c0 == 0 && i < a.I) {
        a.gx[tk * a.I + i] = 0.f;
        a.ux[tk * a.I + i] = 0.f;
      }
    }
    return;
  }
  float xf[CPL][32], xsum[CPL];
  load_x_lane<CPL>(x, c0, LPR, xf, xsum);

  const int in_bytes = a.d >> 1;
  const int ngroups = a.d >> 6;
  const uint8_t* qg = reinterpret_cast<const uint8_t*>(bd->gate.q);
  const uint8_t* qu = reinterpret_cast<const uint8_t*>(bd->up.q);
  const uint32_t* szg = reinterpret_cast<const uint32_t*>(bd->gate.sz);
  const uint32_t* szu = reinterpret_cast<const uint32_t*>(bd->up.sz);

  U4 wq[RP][2][CPL];
  uint32_t wsz[RP][2][CPL];
#pragma unroll
  for (int rp = 0; rp < RP; ++rp) {
    int i = pair0 + rp * RPI + sub;
    i = i < a.I ? i : a.I - 1;
#pragma unroll
    for (int cc = 0; cc < CPL; ++cc) {
      const int c = c0 + LPR * cc;
      wq[rp][0][cc] = ld16(qg + (size_t)i * in_bytes + (size_t)c * 16);
      wq[rp][1][cc] = ld16(qu + (size_t)i * in_bytes + (size_t)c * 16);
      wsz[rp][0][cc] = szg[(size_t)i * ngroups + (c >> 1)];
      wsz[rp][1][cc] = szu[(size_t)i * ngroups + (c >> 1)];
    }
  }
#pragma unroll
  for (int rp = 0; rp < RP; ++rp) {
    const int i = pair0 + rp * RPI + sub;
    float res[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      float acc = 0.f;
#pragma unroll
      for (int cc = 0; cc < CPL; ++cc) {
        const float2 sz = h2f2(wsz[rp][p][cc]);
        acc += sz.x * dot32_q4(wq[rp][p][cc], xf[cc]) + sz.y * xsum[cc];
      }
      res[p] = group_sum(acc, LPR);
    }
    if (c0 == 0 && i < a.I) {
      a.gx[tk * a.I + i] = res[0];
      a.ux[tk * a.I + i] = res[1];
    }
  }
}

// ------------------------------------------------------------------------
// Expert stage 2: LoRA-B of gate / up, SwiGLU, and the slice-partial LoRA-A
// projection of down.  One wave per 64 intermediate units.
// ------------------------------------------------------------------------
__global__ void __launch_bounds__(64) ffn_h_kernel(FfnArgs a) {
  const int t = blockIdx.y;
  const int nsl = a.I >> 6;
  const int k = blockIdx.x / nsl, sl = blockIdx.x % nsl;
  const int lane = threadIdx.x;
  const int i = sl * 64 + lane;
  const int n = a.n_list;
  const size_t tk = (size_t)t * n + k;
  const moe_bundle* bd = resolve_expert(k, a.K, a.E, a.idx + (size_t)t * a.K, a.slot_of,
                                        a.bundles, a.status, false);
  float* adp = a.adpart + (tk * nsl + sl) * a.r;
  if (!bd) {
    a.h[tk * a.I + i] = 0.f;
    if (lane < a.r) adp[lane] = 0.f;
    return;
  }
  float g = a.gx[tk * a.I + i];
  float u = a.ux[tk * a.I + i];
  if (a.r > 0) {
    if (bd->gate.lora_a && bd->gate.lora_b) {
      const __half* brow = reinterpret_cast<const __half*>(bd->gate.lora_b) + (size_t)i * a.r;
      const float* av = a.ag + tk * a.r;
      float acc = 0.f;
      for (int kk = 0; kk < a.r; ++kk) acc = fmaf(__half2float(brow[kk]), av[kk], acc);
      g = fmaf(a.lora_scale, acc, g);
    }
    if (bd->up.lora_a && bd->up.lora_b) {
      const __half* brow = reinterpret_cast<const __half*>(bd->up.lora_b) + (size_t)i * a.r;
      const float* av = a.au + tk * a.r;
      float acc = 0.f;
      for (int kk = 0; kk < a.r; ++kk) acc = fmaf(__half2float(brow[kk]), av[kk], acc);
      u = fmaf(a.lora_scale, acc, u);
    }
  }
  const float hv = g / (1.f + expf(-g)) * u;
  a.h[tk * a.I + i] = hv;
  const bool has_down = a.r > 0 && bd->down.lora_a && bd->down.lora_b;
  for (int kk = 0; kk < a.r; ++kk) {
    const float p =
        has_down ? __half2float(reinterpret_cast<const __half*>(bd->down.lora_a)[(size_t)kk * a.I + i]) * hv
                 : 0.f;
    const float s = wave_sum(p);
    if (lane == 0) adp[kk] = s;
  }
}

// ------------------------------------------------------------------------
// Expert stage 3: down int4 matvec on h plus the LoRA-B of down, folded into
// the same cross-lane reduction.
// ------------------------------------------------------------------------
template <int LPR, int CPL, int RIT>
__global__ void __launch_bounds__(256) ffn_down_kernel(FfnArgs a) {
  constexpr int RPI = kWave / LPR;
  constexpr int ROWS_PER_WG = 4 * RIT * RPI;
  const int t = blockIdx.y;
  const int nblk = (a.d + ROWS_PER_WG - 1) / ROWS_PER_WG;
  const int k = blockIdx.x / nblk, b = blockIdx.x % nblk;
  const int n = a.n_list;
  const size_t tk = (size_t)t * n + k;
  const moe_bundle* bd = resolve_expert(k, a.K, a.E, a.idx + (size_t)t * a.K, a.slot_of,
                                        a.bundles, a.status, false);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int c0 = lane % LPR, sub = lane / LPR;
  const int row0 = b * ROWS_PER_WG + wave * RIT * RPI;
  float* ye = a.y_experts + tk * a.d;
  if (!bd) {
#pragma unroll
    for (int it = 0; it < RIT; ++it) {
      const int j = row0 + it * RPI + sub;
      if (c0 == 0 && j < a.d) ye[j] = 0.f;
    }
    return;
  }
  // h for this lane's chunks
  float hf[CPL][32], hsum[CPL];
  const float* hrow = a.h + tk * a.I;
#pragma unroll
  for (int cc = 0; cc < CPL; ++cc) {
    const int c = c0 + LPR * cc;
    float s = 0.f;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const float4 v = reinterpret_cast<const float4*>(hrow + (size_t)c * 32)[q];
      hf[cc][4 * q] = v.x;
      hf[cc][4 * q + 1] = v.y;
      hf[cc][4 * q + 2] = v.z;
      hf[cc][4 * q + 3] = v.w;
      s += (v.x + v.y) + (v.z + v.w);
    }
    hsum[cc] = s;
  }
  // LoRA: lane c0 owns rank components c0, c0 + LPR, ... < r
  const bool has_lora = a.r > 0 && bd->down.lora_a && bd->down.lora_b;
  constexpr int KMAX = 64 / LPR > 0 ? (64 + LPR - 1) / LPR : 1;
  float adv[KMAX];
  const int nsl = a.I >> 6;
#pragma unroll
  for (int m = 0; m < KMAX; ++m) {
    const int kk = c0 + LPR * m;
    float s = 0.f;
    if (has_lora && kk < a.r)
      for (int sl = 0; sl < nsl; ++sl) s += a.adpart[(tk * nsl + sl) * a.r + kk];
    adv[m] = s;
  }
  const int in_bytes = a.I >> 1;
  const int ngroups = a.I >> 6;
  const uint8_t* qd = reinterpret_cast<const uint8_t*>(bd->down.q);
  const uint32_t* szd = reinterpret_cast<const uint32_t*>(bd->down.sz);
  const __half* bl = has_lora ? reinterpret_cast<const __half*>(bd->down.lora_b) : nullptr;

  U4 wq[RIT][CPL];
  uint32_t wsz[RIT][CPL];
#pragma unroll
  for (int it = 0; it < RIT; ++it) {
    int j = row0 + it * RPI + sub;
    j = j < a.d ? j : a.d - 1;
#pragma unroll
    for (int cc = 0; cc < CPL; ++cc) {
      const int c = c0 + LPR * cc;
      wq[it][cc] = ld16(qd + (size_t)j * in_bytes + (size_t)c * 16);
      wsz[it][cc] = szd[(size_t)j * ngroups + (c >> 1)];
    }
  }
#pragma unroll
  for (int it = 0; it < RIT; ++it) {
    const int j = row0 + it * RPI + sub;
    const int jc = j < a.d ? j : a.d - 1;
    float acc = 0.f;
#pragma unroll
    for (int cc = 0; cc < CPL; ++cc) {
      const float2 sz = h2f2(wsz[it][cc]);
      acc += sz.x * dot32_q4(wq[it][cc], hf[cc]) + sz.y * hsum[cc];
    }
    if (has_lora) {
      float la = 0.f;
#pragma unroll
      for (int m = 0; m < KMAX; ++m) {
        const int kk = c0 + LPR * m;
        if (kk < a.r) la = fmaf(__half2float(bl[(size_t)jc * a.r + kk]), adv[m], la);
      }
      acc = fmaf(a.lora_scale, la, acc);
    }
    acc = group_sum(acc, LPR);
    if (c0 == 0 && j < a.d) ye[j] = acc;
  }
}

// ------------------------------------------------------------------------
// Stages 2 and 3 in one launch: every down workgroup forms its expert's whole h
// (LoRA-B of gate / up, SwiGLU) and A_down h in LDS, then its output rows. The
// operands that do not depend on h (gate / up sums, LoRA rows, the workgroup's
// codes) are requested before the first barrier, so the three phases wait for
// memory once. Both launches of a call, K + S 9, d 2048, I 512: 15.3 us at T = 1
// and 105 at T = 24 (three launches: 26.2 and 141); K 4, d 4096, I 1024: 23.8 and
// 172 us (32.6 and 226). Latency-bound at T = 1; passing the resolved bundle on
// from the first launch changed nothing (15.1 and 15.5 us).
// ------------------------------------------------------------------------

// sum_k b[k] av[k] over the rank, k ascending; the first 16 of b preloaded.
__device__ __forceinline__ float lora_b_dot(const U4& b0, const U4& b1, const __half* brow, const float* av,
                                            int r) {
  float acc = 0.f;
  const uint32_t w[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float2 f = h2f2(w[i]);
    if (2 * i < r) acc = fmaf(f.x, av[2 * i], acc);
    if (2 * i + 1 < r) acc = fmaf(f.y, av[2 * i + 1], acc);
  }
  for (int k = 16; k < r; ++k) acc = fmaf(__half2float(brow[k]), av[k], acc);
  return acc;
}
// elements k .. k + 7 of a row of r halves (zero past r)
__device__ __forceinline__ U4 ld_rank8(const __half* row, int k, int r) {
  U4 v{0, 0, 0, 0};
  if (k >= r) return v;
  if (r % 8 == 0) return ld16(row + k);
  uint16_t e[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) e[i] = k + i < r ? reinterpret_cast<const uint16_t*>(row)[k + i] : (uint16_t)0;
  v.x = e[0] | ((uint32_t)e[1] << 16);
  v.y = e[2] | ((uint32_t)e[3] << 16);
  v.z = e[4] | ((uint32_t)e[5] << 16);
  v.w = e[6] | ((uint32_t)e[7] << 16);
  return v;
}

// I = 32 LPR CPL <= 1024; a workgroup takes `batches` runs of 4 RIT 64 / LPR rows,
// the codes of the next run in flight while one is summed.
template <int LPR, int CPL, int RIT>
__global__ void __launch_bounds__(256) ffn_hdown_kernel(FfnArgs a, int batches) {
  constexpr int I = 32 * LPR * CPL;
  constexpr int RPI = kWave / LPR;
  constexpr int RUN = 4 * RIT * RPI;             // rows of one run
  constexpr int IPT = (I + 255) / 256;           // h rows per thread
  constexpr int PQ = I >= 512 ? I / 512 : 1;     // 8-element pieces of an A_down row per lane
  constexpr int RW = 4;                          // A_down rows per wave requested ahead (rank <= 16)
  constexpr int KMAX = 64 / LPR > 0 ? (64 + LPR - 1) / LPR : 1;
  // h in 32-element pieces, 36 floats apart (the lanes of a row read one piece
  // each: consecutive pieces on different banks)
  __shared__ __align__(16) float hs[(I / 32) * 36];
  __shared__ float av[2][64], ad[64];
  const int t = blockIdx.y;
  const int nblk = a.d / (RUN * batches);        // (powers of two)
  const int k = blockIdx.x / nblk, b = blockIdx.x % nblk;
  const int n = a.n_list, tid = threadIdx.x;
  const size_t tk = (size_t)t * n + k;
  float gv[IPT], uv[IPT];
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    const int i = tid + 256 * j;
    gv[j] = i < I ? a.gx[tk * I + i] : 0.f;
    uv[j] = i < I ? a.ux[tk * I + i] : 0.f;
  }
  const float avv = tid < 2 * a.r ? (tid < a.r ? a.ag[tk * a.r + tid] : a.au[tk * a.r + tid - a.r]) : 0.f;
  const moe_bundle* bd = resolve_expert(k, a.K, a.E, a.idx + (size_t)t * a.K, a.slot_of,
                                        a.bundles, a.status, false);
  const int wave = tid >> 6, lane = tid & 63;
  const int c0 = lane % LPR, sub = lane / LPR;
  const int row0 = b * RUN * batches + wave * RIT * RPI + sub;  // this lane's first row
  float* ye = a.y_experts + tk * a.d;
  if (!bd) {
    if (c0 == 0)
      for (int rb = 0; rb < batches; ++rb)
#pragma unroll
        for (int it = 0; it < RIT; ++it) ye[row0 + rb * RUN + it * RPI] = 0.f;
    return;
  }
  const bool has_g = a.r > 0 && bd->gate.lora_a && bd->gate.lora_b;
  const bool has_u = a.r > 0 && bd->up.lora_a && bd->up.lora_b;
  const bool has_lora = a.r > 0 && bd->down.lora_a && bd->down.lora_b;
  const __half* bg = static_cast<const __half*>(bd->gate.lora_b);
  const __half* bu = static_cast<const __half*>(bd->up.lora_b);
  const __half* al = static_cast<const __half*>(bd->down.lora_a);
  const __half* bl = static_cast<const __half*>(bd->down.lora_b);
  const uint8_t* qd = static_cast<const uint8_t*>(bd->down.q);
  const uint32_t* szd = static_cast<const uint32_t*>(bd->down.sz);

  U4 gb[IPT][2], ub[IPT][2];
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    const int i = tid + 256 * j < I ? tid + 256 * j : 0;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      gb[j][q] = has_g ? ld_rank8(bg + (size_t)i * a.r, 8 * q, a.r) : U4{0, 0, 0, 0};
      ub[j][q] = has_u ? ld_rank8(bu + (size_t)i * a.r, 8 * q, a.r) : U4{0, 0, 0, 0};
    }
  }
  U4 ar[RW][PQ];
#pragma unroll
  for (int m = 0; m < RW; ++m)
#pragma unroll
    for (int q = 0; q < PQ; ++q) {
      const int c = lane + kWave * q;
      ar[m][q] = has_lora && wave + 4 * m < a.r && c < I / 8 ? ld16(al + (size_t)(wave + 4 * m) * I + 8 * c)
                                                             : U4{0, 0, 0, 0};
    }
  U4 wq[RIT][CPL];
  uint32_t wsz[RIT][CPL];
  uint16_t bv[RIT][KMAX];                        // LoRA-B of down: rank components c0, c0 + LPR, ...
  auto load_run = [&](int rb) {
#pragma unroll
    for (int it = 0; it < RIT; ++it) {
      const int j = row0 + rb * RUN + it * RPI;
#pragma unroll
      for (int cc = 0; cc < CPL; ++cc) {
        const int c = c0 + LPR * cc;
        wq[it][cc] = ld16(qd + (size_t)j * (I / 2) + (size_t)c * 16);
        wsz[it][cc] = szd[(size_t)j * (I / 64) + (c >> 1)];
      }
#pragma unroll
      for (int m = 0; m < KMAX; ++m) {
        const int kk = c0 + LPR * m;
        bv[it][m] = has_lora && kk < a.r ? reinterpret_cast<const uint16_t*>(bl)[(size_t)j * a.r + kk] : (uint16_t)0;
      }
    }
  };
  load_run(0);

  if (tid < 2 * a.r) av[tid < a.r ? 0 : 1][tid < a.r ? tid : tid - a.r] = avv;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    const int i = tid + 256 * j;
    if (i < I) {
      float g = gv[j], u = uv[j];
      if (has_g) g = fmaf(a.lora_scale, lora_b_dot(gb[j][0], gb[j][1], bg + (size_t)i * a.r, av[0], a.r), g);
      if (has_u) u = fmaf(a.lora_scale, lora_b_dot(ub[j][0], ub[j][1], bu + (size_t)i * a.r, av[1], a.r), u);
      hs[(i >> 5) * 36 + (i & 31)] = g / (1.f + expf(-g)) * u;
    }
  }
  __syncthreads();
  // A_down h, one rank row per wave and turn
  if (has_lora) {
    for (int m = 0; wave + 4 * m < a.r; ++m) {
      const int kk = wave + 4 * m;
      // a 64-element slice is eight lanes' pieces, its products added as a balanced
      // tree; the slices are added in order (the sums of the separate h launch, bit
      // for bit)
      float s = 0.f;
#pragma unroll
      for (int q = 0; q < PQ; ++q) {
#pragma clang fp contract(off)
        const int c = lane + kWave * q;
        float v = 0.f;
        if (c < I / 8) {
          U4 a8 = {0, 0, 0, 0};
          if (m < RW) {
#pragma unroll
            for (int z = 0; z < RW; ++z)
              if (m == z) a8 = ar[z][q];
          } else {
            a8 = ld16(al + (size_t)kk * I + 8 * c);
          }
          const float* hp = hs + (c >> 2) * 36 + (c & 3) * 8;
          const float2 f0 = h2f2(a8.x), f1 = h2f2(a8.y), f2 = h2f2(a8.z), f3 = h2f2(a8.w);
          v = ((f0.x * hp[0] + f0.y * hp[1]) + (f1.x * hp[2] + f1.y * hp[3])) +
              ((f2.x * hp[4] + f2.y * hp[5]) + (f3.x * hp[6] + f3.y * hp[7]));
        }
        v += dpp_f<0xB1>(0.f, v);
        v += dpp_f<0x4E>(0.f, v);
        v += dpp_f<0x141>(0.f, v);
#pragma unroll
        for (int sl = 0; sl < 8; ++sl)
          if (8 * q + sl < I / 64) s += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 8 * sl));
      }
      if (lane == 0) ad[kk] = s;
    }
  }
  float hf[CPL][32], hsum[CPL];
#pragma unroll
  for (int cc = 0; cc < CPL; ++cc) {
    const float4* hp = reinterpret_cast<const float4*>(hs + (c0 + LPR * cc) * 36);
    float s = 0.f;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const float4 v = hp[q];
      hf[cc][4 * q] = v.x;
      hf[cc][4 * q + 1] = v.y;
      hf[cc][4 * q + 2] = v.z;
      hf[cc][4 * q + 3] = v.w;
      s += (v.x + v.y) + (v.z + v.w);
    }
    hsum[cc] = s;
  }
  __syncthreads();
  float adv[KMAX];
#pragma unroll
  for (int m = 0; m < KMAX; ++m) adv[m] = has_lora && c0 + LPR * m < a.r ? ad[c0 + LPR * m] : 0.f;
  for (int rb = 0; rb < batches; ++rb) {
    float acc[RIT];
#pragma unroll
    for (int it = 0; it < RIT; ++it) {
      acc[it] = 0.f;
#pragma unroll
      for (int cc = 0; cc < CPL; ++cc) {
        const float2 sz = h2f2(wsz[it][cc]);
        acc[it] += sz.x * dot32_q4(wq[it][cc], hf[cc]) + sz.y * hsum[cc];
      }
      if (has_lora) {
        float la = 0.f;
#pragma unroll
        for (int m = 0; m < KMAX; ++m) la = fmaf(__half2float(__ushort_as_half(bv[it][m])), adv[m], la);
        acc[it] = fmaf(a.lora_scale, la, acc[it]);
      }
    }
    if (rb + 1 < batches) load_run(rb + 1);
#pragma unroll
    for (int it = 0; it < RIT; ++it) {
      const float s = group_sum(acc[it], LPR);
      if (c0 == 0) ye[row0 + rb * RUN + it * RPI] = s;
    }
  }
}

// ------------------------------------------------------------------------
// Combine: y = sum_k w_k y_k + sum_s y_shared_s.
// ------------------------------------------------------------------------
// (four columns a thread, the loads of up to eight experts at once: one after the
// other, each waits for the expert kernel's writes in another XCD's L2 at T = 1)
__global__ void __launch_bounds__(256) combine_kernel(const float* __restrict__ ye,
                                                      const float* __restrict__ w, int K, int S,
                                                      int d, float* __restrict__ y, int accumulate) {
  const int t = blockIdx.y;
  const int j = 4 * (blockIdx.x * blockDim.x + threadIdx.x);
  if (j >= d) return;
  const int n = K + S;
  const float* base = ye + (size_t)t * n * d + j;
  const float* wt = w + (size_t)t * K;
  float4* out = reinterpret_cast<float4*>(y + (size_t)t * d + j);
  float4 old = {0.f, 0.f, 0.f, 0.f}, acc = {0.f, 0.f, 0.f, 0.f};
  if (accumulate) old = *out;
  auto group = [&](int k0, auto count) {
    constexpr int C = decltype(count)::value;
    float4 v[C];
#pragma unroll
    for (int q = 0; q < C; ++q) v[q] = *reinterpret_cast<const float4*>(base + (size_t)(k0 + q) * d);
#pragma unroll
    for (int q = 0; q < C; ++q) {
      const float f = k0 + q < K ? wt[k0 + q] : 1.f;  // (1 x v + acc is acc + v)
      acc.x = fmaf(f, v[q].x, acc.x);
      acc.y = fmaf(f, v[q].y, acc.y);
      acc.z = fmaf(f, v[q].z, acc.z);
      acc.w = fmaf(f, v[q].w, acc.w);
    }
  };
  int k0 = 0;
  for (; k0 + 8 <= n; k0 += 8) group(k0, std::integral_constant<int, 8>());
  if (k0 + 4 <= n) {
    group(k0, std::integral_constant<int, 4>());
    k0 += 4;
  }
  for (; k0 < n; ++k0) group(k0, std::integral_constant<int, 1>());
  if (accumulate) acc = float4{old.x + acc.x, old.y + acc.y, old.z + acc.z, old.w + acc.w};
  *out = acc;
}

// ------------------------------------------------------------------------
// Decode-chain stand-in for attention (one workgroup per call):
//   token start:  r = xi + rmsnorm(r)         (norm in fp64, r kept fp32)
//   layer input:  r = r + D * r[perm];  x = fp16(rmsnorm(r))
// ------------------------------------------------------------------------
// Both are one workgroup of 1024 threads and latency-bound: each thread keeps
// its d / 1024 elements in registers (NV of them) between the sum and the use
// (the mixing at d 2048: 2.9 us; with 256 threads, re-reading r, 7.6 us).
template <int NV>
__global__ void __launch_bounds__(1024) chain_token_start_kernel(const float* __restrict__ xi, int d,
                                                                 float* __restrict__ r) {
  __shared__ double red[16];
  float v[NV], xv[NV];
  double acc = 0.0;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int j = threadIdx.x + 1024 * i;
    v[i] = j < d ? r[j] : 0.f;
    xv[i] = j < d ? xi[j] : 0.f;
  }
#pragma unroll
  for (int i = 0; i < NV; ++i) acc += (double)v[i] * (double)v[i];
  const double inv = rsqrt_full(block_sum_f64(acc, red) / (double)d + 1e-6);
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int j = threadIdx.x + 1024 * i;
    if (j < d) r[j] = (float)((double)xv[i] + (double)v[i] * inv);
  }
}

template <int NV>
__global__ void __launch_bounds__(1024) chain_mix_rmsnorm_kernel(const __half* __restrict__ mix_d,
                                                                 const int32_t* __restrict__ perm, int d,
                                                                 float* __restrict__ r,
                                                                 __half* __restrict__ x) {
  extern __shared__ float rs[];
  __shared__ double red[16];
  float v[NV], m[NV];
  int p[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int j = threadIdx.x + 1024 * i;
    v[i] = j < d ? r[j] : 0.f;
    p[i] = j < d ? perm[j] : -1;
    m[i] = j < d ? __half2float(mix_d[j]) : 0.f;
  }
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int j = threadIdx.x + 1024 * i;
    if (j < d) rs[j] = v[i];
  }
  __syncthreads();
  double acc = 0.0;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    v[i] = fmaf(m[i], (p[i] >= 0 && p[i] < d) ? rs[p[i]] : 0.f, v[i]);
    acc += (double)v[i] * (double)v[i];
  }
  const double inv = rsqrt_full(block_sum_f64(acc, red) / (double)d + 1e-6);
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int j = threadIdx.x + 1024 * i;
    if (j < d) {
      r[j] = v[i];
      x[j] = eng::f64_to_h((double)v[i] * inv);
    }
  }
}

// ------------------------------------------------------------------------
// Launchers
// ------------------------------------------------------------------------
// Router logits: rows of W against one token at a time while that is little
// work (T E d; it re-reads W for every token), else the matrix cores. Whole
// calls, rows / 16 x 16 blocks: d 2048, E 256: 6.7 / 8.6 us at T = 24, 9.3 / 8.7
// at 64; d 4096, E 64: 6.7 / 11.6 at 64, 21 / 11.8 at 512; d 512, E 16: 4.8 / 5.3
// at 128, 6.1 / 5.4 at 512.
constexpr int kRouteRowsMaxT = 128;
constexpr long long kRouteRowsMaxWork = 1 << 24;
// Larger blocks read less from the L2 but leave CUs idle when few: 2 x 2 blocks
// of 16 from 160 workgroups on (16 x 16 / 32 x 32: 12.4 / 12.7 us with 128, 19 /
// 12.9 with 200), 4 x 4 from 150 on (32 x 32 / 64 x 64: 21.3 / 22.4 us with 96,
// 36 / 25 with 196).
constexpr int kRouteFill22 = 160;
constexpr int kRouteFill44 = 150;
template <int NV>
static void rmsnorm(const float* xi, int T, int d, int threads, __half* x, hipStream_t st) {
  hipLaunchKernelGGL(rmsnorm_f16_kernel<NV>, dim3(T), dim3(threads), 0, st, xi, d, x);
}

hipError_t launch_rmsnorm(const float* xi, int T, int d, __half* x, hipStream_t st) {
  if (d % 4 || d > 8192) {
    hipLaunchKernelGGL(rmsnorm_f16_any_kernel, dim3(T), dim3(256), 0, st, xi, d, x);
    return hipGetLastError();
  }
  // One or a few 16-byte pieces per thread while the rows are few, four waves a row once
  // they fill the chip several times over. 256 / 512 / 1024 threads at most (us): d 2048
  // T = 1 2.7 / 2.6, T = 512 3.3 / 3.2, T = 700 3.5 / 3.8; d 4096 T = 1 3.0 / 2.6 / 2.8,
  // T = 512 4.1 / 4.0 / 4.6, T = 700 4.5 / 4.7 / 5.8; d 8192 T = 512 5.8 / 5.3 / 5.9.
  const int most = T <= 512 ? 512 : 256;
  const int pieces = d / 4, threads = std::min(most, (pieces + 63) / 64 * 64);
  const int nv = (pieces + threads - 1) / threads;
  if (nv <= 1)
    rmsnorm<1>(xi, T, d, threads, x, st);
  else if (nv <= 2)
    rmsnorm<2>(xi, T, d, threads, x, st);
  else if (nv <= 4)
    rmsnorm<4>(xi, T, d, threads, x, st);
  else
    rmsnorm<8>(xi, T, d, threads, x, st);
  return hipGetLastError();
}

hipError_t launch_router_logits(const __half* x, const __half* W, int T, int E, int d, float* logits,
                                hipStream_t st) {
  if (T <= kRouteRowsMaxT && (long long)T * E * d <= kRouteRowsMaxWork) {
    hipLaunchKernelGGL(route_rows_kernel, dim3((E + kRouteRows - 1) / kRouteRows, T), dim3(64 * kRouteRows), 0, st,
                       x, W, E, d, logits);
    return hipGetLastError();
  }
  auto blocks = [&](int mb, int nb) { return ((T + 16 * mb - 1) / (16 * mb)) * ((E + 16 * nb - 1) / (16 * nb)); };
  if (blocks(4, 4) >= kRouteFill44)
    hipLaunchKernelGGL((route_mfma_kernel<4, 4>), dim3(blocks(4, 4)), dim3(64 * kRouteWaves), 0, st, x, W, T, E, d,
                       logits);
  else if (blocks(2, 2) >= kRouteFill22)
    hipLaunchKernelGGL((route_mfma_kernel<2, 2>), dim3(blocks(2, 2)), dim3(64 * kRouteWaves), 0, st, x, W, T, E, d,
                       logits);
  else
    hipLaunchKernelGGL((route_mfma_kernel<1, 1>), dim3(blocks(1, 1)), dim3(64 * kRouteWaves), 0, st, x, W, T, E, d,
                       logits);
  return hipGetLastError();
}

hipError_t launch_topk_sigmoid_group(const float* logits, const float* bias, int T, int E, int K,
                                     int n_groups, int top_groups, float scale, int32_t* idx, float* w,
                                     hipStream_t st) {
  if (E > 256 || K > 32 || n_groups < 1 || E % n_groups) return hipErrorInvalidValue;
  hipLaunchKernelGGL(topk_sigmoid_group_kernel, dim3(T), dim3(512), 0, st, logits, bias, E, K, n_groups,
                     top_groups, scale, idx, w);
  return hipGetLastError();
}

// A wave's time grows with K, a workgroup's with T once they fill the chip. A call,
// workgroup / wave (us): K 8: T = 1 2.7 / 2.9, T = 256 3.1 / 3.3, T = 384 3.3 / 3.3; K 16:
// T = 1 3.1 / 4.0, T = 640 4.1 / 4.4, T = 777 4.4 / 4.4; K 32: T = 1 3.6 / 6.0, T = 1024
// 5.9 / 6.6, T = 1536 7.8 / 7.3; K 6: T = 64 3.0 / 3.1, T = 256 3.1 / 3.1; K 4: T = 1 2.6 / 2.5.
constexpr int kBlockTopkMinK = 6, kBlockTopkTokens = 40;

hipError_t launch_topk(const float* logits, int T, int E, int K, int32_t* idx, float* w,
                       hipStream_t st) {
  if (E <= 256 && K >= kBlockTopkMinK && T <= kBlockTopkTokens * K) {
    hipLaunchKernelGGL(topk_block_kernel, dim3(T), dim3(512), 0, st, logits, E, K, idx, w);
    return hipGetLastError();
  }
  const dim3 grid((T + 3) / 4), block(T == 1 ? 64 : 256);
  if (E <= 256)
    hipLaunchKernelGGL(topk_wave_kernel<4>, grid, block, 0, st, logits, T, E, K, idx, w);
  else
    hipLaunchKernelGGL(topk_wave_kernel<16>, grid, block, 0, st, logits, T, E, K, idx, w);
  return hipGetLastError();
}

template <int LPR, int CPL>
static void gateup(const FfnArgs& a, int T, hipStream_t st, hipEvent_t ps, hipEvent_t pe) {
  constexpr int RP = 4;
  constexpr int PAIRS = 4 * RP * (kWave / LPR);
  const int nblk = (a.I + PAIRS - 1) / PAIRS + (2 * a.r + 3) / 4;
  if (ps && pe)
    hipExtLaunchKernelGGL((ffn_gateup_kernel<LPR, CPL, RP>), dim3(nblk * a.n_list, T), dim3(256),
                          0, st, ps, pe, 0, a);
  else
    hipLaunchKernelGGL((ffn_gateup_kernel<LPR, CPL, RP>), dim3(nblk * a.n_list, T), dim3(256), 0,
                       st, a);
}

template <int LPR, int CPL>
static void down(const FfnArgs& a, int T, hipStream_t st) {
  constexpr int RIT = 4;
  constexpr int ROWS = 4 * RIT * (kWave / LPR);
  const int nblk = (a.d + ROWS - 1) / ROWS;
  hipLaunchKernelGGL((ffn_down_kernel<LPR, CPL, RIT>), dim3(nblk * a.n_list, T), dim3(256), 0, st,
                     a);
}

// Rows per workgroup: enough runs that the launch still has 512 workgroups (two
// a CU), so that the h of a workgroup is formed for as many rows as it can be.
// Whole calls with 512 / 1024 / 2048: d 4096, I 1024, K 4: T = 4 45 / 52 / 64 us,
// T = 24 170 / 175 / 186; d 2048, I 512, K + S 9: T = 8 45 / 46.5 / 51.
// At I = 1024 a CU holds two workgroups (192 registers a lane): 513 to 1023 of them are
// a second round for a few, each with an h of its own, so up to four runs a workgroup
// are taken where that leaves one round, and up to eight for 256 workgroups beyond
// rank 32, whose h costs most. K + S 5, one run / this rule / h in a launch of its own:
// d 4096, T = 1, r 5 29.9 / 25.2 / 26.7 us, r 64 77 / 41.6 / 65; d 2048, T = 2, r 16
// 25.0 / 22.0 / 30.3; d 512, T = 8, r 64 80.5 / 41.8 / 56.
// Rank 0, whose h costs least, takes half the runs where long workgroups would be a round
// and a rest below a half: K + S 9, d 4096, T = 8 116.3 / 109.4 / 116.3; K + S 5, d 2048,
// T = 64 231 / 214 / 241.
constexpr int kHdownFill = 512;
template <int LPR, int CPL>
static void hdown(const FfnArgs& a, int T, hipStream_t st) {
  constexpr int RIT = 4;
  const int runs = a.d / (4 * RIT * (kWave / LPR));  // (d >= 512, a power of two: at least 4)
  const long long all = (long long)runs * a.n_list * T;
  int batches = 1;
  while (2 * batches <= runs && all / (2 * batches) >= kHdownFill) batches *= 2;
  if (32 * LPR * CPL > 512) {
    const int resident = a.r > 32 ? 256 : 512, most = a.r > 32 ? 8 : 4;
    while (2 * batches <= std::min(runs, most) && all / batches > resident) batches *= 2;
    if (a.r == 0 && batches >= 8 && all / batches > 512 && all / batches < 768) batches /= 2;
  }
  hipLaunchKernelGGL((ffn_hdown_kernel<LPR, CPL, RIT>), dim3(runs / batches * a.n_list, T), dim3(256), 0, st, a,
                     batches);
}

static bool dispatch_gateup(const FfnArgs& a, int T, hipStream_t st, hipEvent_t ps,
                            hipEvent_t pe) {
  switch (a.d) {
    case 256: gateup<8, 1>(a, T, st, ps, pe); return true;
    case 512: gateup<16, 1>(a, T, st, ps, pe); return true;
    case 1024: gateup<32, 1>(a, T, st, ps, pe); return true;
    case 2048: gateup<64, 1>(a, T, st, ps, pe); return true;
    case 4096: gateup<64, 2>(a, T, st, ps, pe); return true;
    case 8192: gateup<64, 4>(a, T, st, ps, pe); return true;
  }
  return false;
}

static bool dispatch_hdown(const FfnArgs& a, int T, hipStream_t st) {
  static_assert(kHdownMaxI == 1024, "the workspace's rule is this dispatch");
  switch (a.I) {
    case 256: hdown<8, 1>(a, T, st); return true;
    case 512: hdown<16, 1>(a, T, st); return true;
    case 1024: hdown<32, 1>(a, T, st); return true;
  }
  return false;
}

static bool dispatch_down(const FfnArgs& a, int T, hipStream_t st) {
  switch (a.I) {
    case 2048: down<64, 1>(a, T, st); return true;
    case 4096: down<64, 2>(a, T, st); return true;
    case 8192: down<64, 4>(a, T, st); return true;
  }
  return false;
}

// h and down in one launch up to I = 1024; beyond that a workgroup's own copy of
// h would be more work than its rows, and h gets a launch of its own.
hipError_t launch_ffn(const FfnArgs& a, int T, hipStream_t st, hipEvent_t prof_start,
                      hipEvent_t prof_stop) {
  if (!dispatch_gateup(a, T, st, prof_start, prof_stop)) return hipErrorInvalidValue;
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (dispatch_hdown(a, T, st)) return hipGetLastError();
  hipLaunchKernelGGL(ffn_h_kernel, dim3((a.I >> 6) * a.n_list, T), dim3(64), 0, st, a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (!dispatch_down(a, T, st)) return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_combine(const float* ye, const float* w, int T, int K, int S, int d, float* y,
                          int accumulate, hipStream_t st) {
  // 64 / 128 / 256 threads (us): d 2048, K + S 9: T = 16 2.5 / 2.5 / 2.6, T = 512 7.7 / 6.8 /
  // 6.6; d 512, K 2, T = 3100 5.3 / 4.3 / 4.3; d 2048, K + S 5, T = 777 - / 7.2 / 6.6.
  const int threads = T >= 64 ? 256 : 64;        // (d is a multiple of 512)
  hipLaunchKernelGGL(combine_kernel, dim3((d / 4 + threads - 1) / threads, T), dim3(threads), 0, st, ye, w, K, S, d,
                     y, accumulate);
  return hipGetLastError();
}

hipError_t launch_chain_token_start(const float* xi, int d, float* r, hipStream_t st) {
  if (d <= 2048)
    hipLaunchKernelGGL(chain_token_start_kernel<2>, dim3(1), dim3(1024), 0, st, xi, d, r);
  else if (d <= 4096)
    hipLaunchKernelGGL(chain_token_start_kernel<4>, dim3(1), dim3(1024), 0, st, xi, d, r);
  else
    hipLaunchKernelGGL(chain_token_start_kernel<8>, dim3(1), dim3(1024), 0, st, xi, d, r);
  return hipGetLastError();
}

hipError_t launch_chain_mix_rmsnorm(const __half* mix_d, const int32_t* perm, int d, float* r,
                                    __half* x, hipStream_t st) {
  const size_t lds = (size_t)d * 4;
  if (d <= 2048)
    hipLaunchKernelGGL(chain_mix_rmsnorm_kernel<2>, dim3(1), dim3(1024), lds, st, mix_d, perm, d, r, x);
  else if (d <= 4096)
    hipLaunchKernelGGL(chain_mix_rmsnorm_kernel<4>, dim3(1), dim3(1024), lds, st, mix_d, perm, d, r, x);
  else
    hipLaunchKernelGGL(chain_mix_rmsnorm_kernel<8>, dim3(1), dim3(1024), lds, st, mix_d, perm, d, r, x);
  return hipGetLastError();
}

}  // namespace moe
