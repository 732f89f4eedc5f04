// Batched decode / prefill expert path for gfx950.
//
// The math is the one-token expert FFN (Sec. 3.1, Math contract; Sec. 3.3
// unmerged LoRA) applied to every (token, expert) pair of a batch; grouping by
// expert is what makes it a dense contraction (the whole-layer executor path
// of Sec. 3.1 loads every expert of a layer for a prefill chunk).
//
//   permute   per-expert counts, scans, the tiles, and the permuted list of
//             y_experts rows (token t, list position k); x in pair order (below).
//   prep      per tile A_g x and A_u x (the LoRA-A products, once per tile
//             instead of once per column slab).
//   gate/up   per tile x 64 or 128 columns: G = X W_g^T, U = X W_u^T over the
//             tile's rows with v_mfma_f32_16x16x32_f16; int4 codes and the
//             activation rows stream into LDS through global_load_lds in
//             128-k chunks of whole row segments (a ring of two to four
//             chunks, by the tile's row count), the (s, z) rows once per
//             tile; codes are dequantized to fp16 in registers (w = s q + z,
//             one rounding); the LoRA delta is one MFMA step with K = the
//             rank (B rows against lora_scale * A x); epilogue h = silu(g) u
//             stored fp16 in pair order, and the slab's partial A_d h.
//   down      per 64 rows x 256 (or 128) columns: Y = H W_d^T the same way, LoRA-B of down
//             against lora_scale * (the sum of the slab partials of A_d h);
//             fp32 rows go straight to y_experts.
//
// A narrow gate/up or a down workgroup uses half of the CU's LDS, so two share a CU: the
// loads that start and end a tile of one overlap the streaming of the other.
// A workgroup's first copies depend only on its tile record (which carries the
// bundle's pointers) and on the tile's token list, both written by the
// permutation; the operands of the epilogue (LoRA rows, A x, the output rows)
// are requested before the copies and consumed after the k loop.
//
// Per launch at d 2048, I 512, E 256, K 8, S 1, with one workgroup permuting, narrow
// shapes only and tiles in group order / now (us, means of 20 traced calls): T = 64
// permute 6.7 / 5.3, prep 12.0 / 9.4, gate/up 49 / 42, down 32 / 26; T = 512 10.8 / 7.7,
// 19.9 / 14.9, 95 / 83, 62 / 51; T = 3100 39 / 24, 51 / 42, 274 / 221, 197 / 153. At
// d 4096, I 1024, E 64, K 4: T = 37 gate/up 64 / 45 (two workgroups a CU at 48 KB of
// ring, one at 56), T = 777 174 / 130, down 83 / 72. A gate/up workgroup of one row
// block is bound by the dequantization (13 VALU instructions per 8 codes, 0.54 us a
// chunk for the two of a CU) and by its start: 6 of its 16 us pass before its first
// chunk is there. One of eight row blocks spends 2.3 us a chunk on 1.0 us of matrix
// instructions and 0.5 us of VALU: a probe build's T = 3100 launch of 200 us took 175
// without its copies, 160 without the matrix instructions, 176 without the
// dequantization.
//
// Pair order: inside each 8-element piece the elements run [0,4,1,5,2,6,3,7],
// the order in which the packed nibbles of one code dword come out of a
// 0x000F000F mask at shifts 0, 4, 8, 12. Both MFMA operands use it, so the
// activations (x, h) are kept in pair order and the codes need no shuffle.
// Every output row depends only on its own input row, so the order of rows
// inside a group does not change any result bit.
#include <algorithm>
#include <type_traits>

#include "moe_grouped.h"

namespace moe {
namespace {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h2v __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kGK = 128;                        // k per staged chunk
constexpr int kGT = 512;                        // threads of a GEMM workgroup (8 waves)
constexpr int kGW = kGT / 64;
constexpr int kSlots = 4;                       // slots of the chunk ring, at most
constexpr int kCodeRow = kGK / 2;               // code bytes of one weight row in a chunk
constexpr int kActRow = kGK * 2;                // activation bytes of one row in a chunk
// A GEMM workgroup has eight waves; each takes NBW blocks of 16 weight rows
// against TRB blocks of 16 token rows. With NBW 2 an activation operand read
// from LDS serves two MFMAs (with one, the LDS reads of a 64-row tile take twice
// the time of the matrix cores). EU: waves per SIMD that the registers must
// allow; RING: bytes of the chunk ring.
// Gate/up, 64 gate and the 64 up columns, for groups of few rows, whose time is
// the weights': two workgroups share a CU and one's latencies hide behind the
// other's streaming.
struct GateNarrow {
  static constexpr int NBW = 1, TRB = 4, RING = 48 * 1024, EU = 4;
};
// Gate/up, 128 gate and the 128 up columns, for groups of many rows.
struct GateWide {
  static constexpr int NBW = 2, TRB = 8, RING = 96 * 1024, EU = 2;
};
// Down, 256 columns, or 128 where the (s, z) rows of 256 would leave room for one
// workgroup a CU only (k is short: half of a workgroup's time is its start and end).
struct DownWide {
  static constexpr int NBW = 2, TRB = 4, RING = 64 * 1024, EU = 4;
};
struct DownNarrow {
  static constexpr int NBW = 1, TRB = 4, RING = 48 * 1024, EU = 4;
};
template <class V>
struct Shape {
  static constexpr int NROWS = 16 * kGW * V::NBW;  // weight rows of a workgroup
  static constexpr int GATE = NROWS / 2;           // gate (and up) columns
  static constexpr int DOWN = NROWS;               // down columns
  static constexpr int TR = 16 * V::TRB;           // token rows of a tile
  static constexpr int XJ = V::TRB / 2;            // activation copies of a wave per chunk, at most
};
static_assert(Shape<GateWide>::TR == 2 * Shape<DownWide>::TR && Shape<DownNarrow>::TR == Shape<DownWide>::TR &&
                  Shape<GateNarrow>::TR == Shape<DownWide>::TR,
              "a tile is one or two parts of the prep and down launches");
static_assert(Shape<GateNarrow>::TR == kGroupMinRows && Shape<GateNarrow>::GATE == kGroupSlab, "workspace layout");
// (s, z) rows of a workgroup's weight rows, staged once per tile: k / 16 bytes a row
template <class V>
constexpr int lds_bytes(int k) {
  return V::RING + Shape<V>::NROWS * (k / 16);
}
constexpr int kLdsMax = 160 * 1024;             // LDS of a CU: the most one workgroup may take

__device__ __forceinline__ h2v as_h2(uint32_t u) { return __builtin_bit_cast(h2v, u); }
__device__ __forceinline__ h8 as_h8(U4 u) { return __builtin_bit_cast(h8, u); }

// [v0..v7] -> [v0,v4,v1,v5,v2,v6,v3,v7] (fp16 elements of a 16-byte piece)
__device__ __forceinline__ U4 perm8(U4 w) {
  U4 o;
  o.x = (w.x & 0xffffu) | (w.z << 16);
  o.y = (w.x >> 16) | (w.z & 0xffff0000u);
  o.z = (w.y & 0xffffu) | (w.w << 16);
  o.w = (w.y >> 16) | (w.w & 0xffff0000u);
  return o;
}
// Eight int4 codes of one dword (nibble m = input m) -> fp16 weights
// s q + z in pair order. A nibble masked into the mantissa of the fp16 1024
// (0x6400) gives 1024 + q from bits 0-3 and 1024 + 16 q from bits 4-7, so
// nibbles 0, 4 and 1, 5 of v and 2, 6 and 3, 7 of v >> 8 come out with one
// shift and four three-input bit operations ((x & mask) | 0x6400, truth table
// 0xEA); q = (1024 + q) - 1024 or (1024 + 16 q) / 16 - 64, both exact, then the
// fma rounds once.
__device__ __forceinline__ h8 dequant8(uint32_t v, h2v s, h2v z) {
  const uint32_t v8 = v >> 8;
  const h2v off = {(_Float16)1024.0f, (_Float16)1024.0f};
  const h2v sixteenth = {(_Float16)0.0625f, (_Float16)0.0625f}, m64 = {(_Float16)-64.0f, (_Float16)-64.0f};
  const h2v q0 = as_h2(__builtin_amdgcn_bitop3_b32(v, 0x000F000Fu, 0x64006400u, 0xEA)) - off;
  const h2v q1 = __builtin_elementwise_fma(as_h2(__builtin_amdgcn_bitop3_b32(v, 0x00F000F0u, 0x64006400u, 0xEA)),
                                           sixteenth, m64);
  const h2v q2 = as_h2(__builtin_amdgcn_bitop3_b32(v8, 0x000F000Fu, 0x64006400u, 0xEA)) - off;
  const h2v q3 = __builtin_elementwise_fma(as_h2(__builtin_amdgcn_bitop3_b32(v8, 0x00F000F0u, 0x64006400u, 0xEA)),
                                           sixteenth, m64);
  const h2v w0 = __builtin_elementwise_fma(q0, s, z);
  const h2v w1 = __builtin_elementwise_fma(q1, s, z);
  const h2v w2 = __builtin_elementwise_fma(q2, s, z);
  const h2v w3 = __builtin_elementwise_fma(q3, s, z);
  return h8{w0[0], w0[1], w1[0], w1[1], w2[0], w2[1], w3[0], w3[1]};
}

__device__ __forceinline__ f4 mfma(h8 a, h8 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// LoRA-B operand of the rank step: row `row` of B [out][r], elements
// kq*8 .. kq*8+7 of the rank (zero past r and for kq >= 2).
__device__ __forceinline__ h8 lora_b_operand(const __half* b, int row, int r, int kq) {
  h8 v = {};
  if (kq < 2) {
    const _Float16* p = reinterpret_cast<const _Float16*>(b) + (size_t)row * r + kq * 8;
    if (r == 16 || (r == 8 && kq == 0)) {
      v = as_h8(ld16(p));
    } else if (r != 8) {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (kq * 8 + e < r) v[e] = p[e];
    }
  }
  return v;
}

// ---- copies into LDS --------------------------------------------------------
// global_load_lds: each lane of the wave moves 16 bytes from its own address to
// lds + 16 * lane. The compiler does not see these as memory instructions; vm_wait
// orders them.
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)p;
}
__device__ __forceinline__ void dma16(const void* g, const void* lds) {
  uint32_t saved;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %1\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %2, off\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved)
      : "s"(lds_addr(lds)), "v"(g)
      : "memory");
}
// wait until at most N of this wave's copies are outstanding (N an immediate)
template <int N>
__device__ __forceinline__ void vm_wait_n() {
  static_assert(N >= 0 && N <= 63, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// the same for N = A * (hi ? PH : PL) with A = ahead in [0, kSlots): a short chain of
// scalar compares on uniform values instead of one case per count
template <int PH, int PL, int A = 0>
__device__ __forceinline__ void vm_wait_ahead(int ahead, bool hi) {
  if constexpr (A < kSlots) {
    if (ahead == A) {
      if (hi)
        vm_wait_n<A * PH>();
      else
        vm_wait_n<A * PL>();
      return;
    }
    vm_wait_ahead<PH, PL, A + 1>(ahead, hi);
  } else {
    vm_wait_n<0>();
  }
}

// The XOR key of a row's 16-byte pieces in LDS. ds_read_b128 serves the lanes in
// four groups of 16 (0-3, 12-15, 20-27 / 4-11, 16-19, 28-31 / the same + 32;
// measured by timing pairs of lanes that share banks), so a group holds rows
// 0-3, 12-15 of one k quarter and rows 4-11 of the next. With the quads of rows
// keyed 0, 2, 3, 1 the 16 pieces a group reads lie on all 64 banks (4.9 clocks a
// read); keyed by the row itself, pairs collide (8.5 clocks).
__device__ __forceinline__ int quad_key(int row) {
  const int b = (row >> 2) & 3;
  return ((b << 1) & 2) ^ (b >> 1) ^ (b & 2);
}
__device__ __forceinline__ int act_key(int row) { return (row & 3) | (quad_key(row) << 2); }

// ---- one tile's k loop --------------------------------------------------------
// acc[b][m] += X[rows of block m] . W[16 rows of this wave's block b]^T over
// Kdim for the MB 16-row blocks of the tile (MB a compile-time count). Chunk c
// (k in [c kGK, (c+1) kGK)) of every weight row and activation row is staged into
// a ring slot with global_load_lds, each instruction copying whole row segments
// (16 rows x 64 bytes of codes, 4 rows x 256 bytes of activations; chunks of 64 k
// and twice the slots were slower, 220 against 199 us for a T = 3100 gate/up).
// MFMA instruction j of a chunk takes, in lane (col, kq), the k values
// kq 32 + 8 j .. + 7 (one dword of codes; the same k order in both operands, so
// any order is fine); a lane uses one (s, z) group per chunk and block. The (s, z)
// rows of the whole k range are staged before chunk 0.
// wrow(row) / srow(row): the global code and (s, z) row of weight row `row`
// (block row / 16, wave row / (16 NBW)); xsrc(j, k): global address of 8
// activations (pair order) at k of the row this lane copies in its wave's j-th
// activation copy (row 4 (wave + 8 j) + lane / 16).
template <class V, int MB, typename WRow, typename SRow, typename XSrc>
__device__ __forceinline__ void tile_gemm_mb(char* ring, char* szl, int Kdim, WRow wrow, SRow srow,
                                             XSrc xsrc, f4 (*acc)[V::TRB]) {
  constexpr int NBW = V::NBW, NROWS = Shape<V>::NROWS, CR = kCodeRow, AR = kActRow;
  constexpr int CODE_B = NROWS * CR;                           // codes of a slot
  constexpr int SLOT = CODE_B + MB * 16 * AR;
  constexpr int NBUF = V::RING / SLOT;
  static_assert(NBUF >= 2 && NBUF <= kSlots, "two slots at least");
  constexpr int CODE_I = NBW;                                  // code copies per wave per chunk
  constexpr int XI = MB * 16 * AR / 1024;                      // activation copies per chunk
  constexpr int JN = kGK / 32;                                 // MFMA steps of a chunk
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int col = lane & 15, kq = lane >> 4;
  // this wave's copies per chunk: CODE_I codes and XHI or XLO activation copies
  constexpr int XLO = XI / kGW, XHI = (XI + kGW - 1) / kGW;
  const bool xhi = wave < XI % kGW;
  const int nch = Kdim / kGK;
  const int szr = Kdim / 16;                                   // (s, z) bytes per row
  const int szm = min(szr / 16, 16) - 1;                       // (Kdim is a power of two)
  auto slot = [&](int c) { return ring + (c % NBUF) * SLOT; };
  auto issue = [&](int c) {
    char* sl = slot(c);
#pragma unroll
    for (int i = 0; i < CODE_I; ++i) {
      const int b = wave * CODE_I + i;
      const int row = 16 * b + (lane >> 2), piece = (lane & 3) ^ quad_key(row);
      dma16(wrow(row) + c * CR + piece * 16, sl + b * 1024);
    }
#pragma unroll
    for (int j = 0; j < XHI; ++j) {
      const int b = wave + j * kGW;
      if (b < XI) {
        const int row = 4 * b + (lane >> 4), piece = (lane & 15) ^ act_key(row);
        dma16(xsrc(j, c * kGK + piece * 8), sl + CODE_B + b * 1024);
      }
    }
  };
  // (loads of the caller still outstanding here are older than every copy:
  // they complete before the chunks in whose wait they are counted)
  for (int b = wave; b * 1024 < NROWS * szr; b += kGW) {  // (s, z) rows
    const int o = b * 1024 + lane * 16, r = o / szr, piece = ((o % szr) >> 4) ^ (r & szm);
    dma16(srow(r) + piece * 16, szl + b * 1024);
  }
  const int pre = nch < NBUF ? nch : NBUF;
  for (int c = 0; c < pre; ++c) issue(c);
  const int row0 = wave * NBW * 16 + col;                      // this lane's first weight row
  const int akey = act_key(col);
  for (int c = 0; c < nch; ++c) {
    // chunks issued after chunk c: all of the first NBUF at c = 0, then one
    // per chunk (into the slot of chunk c - 1)
    const int ahead = c == 0 ? pre - 1 : min(nch - 1 - c, NBUF - 2);
    vm_wait_ahead<CODE_I + XHI, CODE_I + XLO>(ahead, xhi);
    __syncthreads();  // chunk c is in LDS for every wave; chunk c - 1 is consumed
    if (c > 0 && c + NBUF - 1 < nch) issue(c + NBUF - 1);
    const char* sl = slot(c);
    U4 q[NBW];
    h2v s2[NBW], z2[NBW];
#pragma unroll
    for (int i = 0; i < NBW; ++i) {
      const int row = row0 + 16 * i;
      q[i] = *reinterpret_cast<const U4*>(sl + row * CR + (kq ^ quad_key(row)) * 16);
      const int so = 2 * c + (kq >> 1);                        // (s, z) group
      const h2v sz = as_h2(*reinterpret_cast<const uint32_t*>(szl + row * szr + (((so >> 2) ^ (row & szm)) * 16) +
                                                              (so & 3) * 4));
      s2[i] = h2v{sz[0], sz[0]};
      z2[i] = h2v{sz[1], sz[1]};
    }
#pragma unroll
    for (int j = 0; j < JN; ++j) {
      h8 af[MB];
#pragma unroll
      for (int m = 0; m < MB; ++m)
        af[m] = *reinterpret_cast<const h8*>(sl + CODE_B + (16 * m + col) * AR + ((kq * JN + j) ^ akey) * 16);
#pragma unroll
      for (int i = 0; i < NBW; ++i) {
        const uint32_t word = j == 0 ? q[i].x : j == 1 ? q[i].y : j == 2 ? q[i].z : q[i].w;
        const h8 w = dequant8(word, s2[i], z2[i]);
#pragma unroll
        for (int m = 0; m < MB; ++m) acc[i][m] = mfma(af[m], w, acc[i][m]);
      }
    }
  }
  __syncthreads();  // the ring is free again
}
// mb (1 .. TRB) is the same for every thread of the workgroup
template <class V, typename WRow, typename SRow, typename XSrc>
__device__ __forceinline__ void tile_gemm(char* ring, char* szl, int Kdim, int mb, WRow wrow, SRow srow,
                                          XSrc xsrc, f4 (*acc)[V::TRB]) {
  if constexpr (V::TRB == 8) {
    if (mb > 6) {
      tile_gemm_mb<V, 8>(ring, szl, Kdim, wrow, srow, xsrc, acc);
      return;
    }
    if (mb > 4) {
      tile_gemm_mb<V, 6>(ring, szl, Kdim, wrow, srow, xsrc, acc);
      return;
    }
  }
  switch (mb) {
    case 1: tile_gemm_mb<V, 1>(ring, szl, Kdim, wrow, srow, xsrc, acc); break;
    case 2: tile_gemm_mb<V, 2>(ring, szl, Kdim, wrow, srow, xsrc, acc); break;
    case 3: tile_gemm_mb<V, 3>(ring, szl, Kdim, wrow, srow, xsrc, acc); break;
    default: tile_gemm_mb<V, 4>(ring, szl, Kdim, wrow, srow, xsrc, acc); break;
  }
}

// ---------------------------------------------------------------------------
// permute: workgroups [0, np) each count all routing ids (LDS) and scan the
// counts, so that every one knows every group's rows and tiles; each then
// writes the tile records of its share of the groups (pairs 2 t, 2 t + 1 with
// t mod np its index) and scatters the ids of those groups. Workgroups from np
// on write x in pair order.
//
// Tiles are numbered full ones first, then the last tile of each group by its
// size class (quarters of a tile), largest first: the GEMM workgroups start in
// that order, so the long ones do not end the launch.
constexpr int kPT = 1024;
constexpr int kXPieces = 4;                      // 16-byte pieces of x per thread
constexpr int kIds = 8;                          // ids a thread loads at once
__global__ void __launch_bounds__(kPT) grouped_permute_kernel(GroupedArgs a, int np) {
  const int tid = threadIdx.x;
  if ((int)blockIdx.x >= np) {
    const size_t pieces = (size_t)a.T * a.d / 8;
    const size_t p0 = (size_t)(blockIdx.x - np) * kPT * kXPieces + tid;
    U4 v[kXPieces];
#pragma unroll
    for (int q = 0; q < kXPieces; ++q) {
      const size_t p = p0 + q * kPT;
      if (p < pieces) v[q] = ld16(reinterpret_cast<const char*>(a.x) + p * 16);
    }
#pragma unroll
    for (int q = 0; q < kXPieces; ++q) {
      const size_t p = p0 + q * kPT;
      if (p < pieces) *reinterpret_cast<U4*>(reinterpret_cast<char*>(a.xp) + p * 16) = perm8(v[q]);
    }
    return;
  }
  __shared__ int cnt[kGroupMaxG];                // counts, then insertion cursors
  __shared__ int goff[kGroupMaxG];               // first permuted row of a group
  __shared__ int gfull[kGroupMaxG];              // its first full tile
  __shared__ int gnf[kGroupMaxG];                // the rows in its full tiles
  __shared__ int grem[kGroupMaxG];               // the tile of the rest
  __shared__ int wrows[kPT / 64], wfull[kPT / 64];
  __shared__ uint64_t wcls[kPT / 64];
  const int G = a.E + a.S, TR = a.tile_rows;
  const int TK = a.T * a.K;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // A small call is bound by the instructions (16 waves on one CU: one takes each SIMD
  // 16 clocks), so a wave leaves out what it has no ids and no groups for: d 512, E 8 or
  // 64, T = 4 .. 16 3.5 us a launch (5.3 with every wave going through all of it).
  auto any_id = [&](int base, int j) { return base + kPT * j + 64 * wave < TK; };  // (uniform)
  int ev[kIds];
  auto load_ids = [&](int base) {
#pragma unroll
    for (int j = 0; j < kIds; ++j) {
      ev[j] = -1;
      if (!any_id(base, j)) continue;
      const int i = base + tid + kPT * j;
      if (i < TK) ev[j] = a.idx[i];
    }
  };
  for (int g = tid; g < G; g += kPT) cnt[g] = g >= a.E ? a.T : 0;
  load_ids(0);
  __syncthreads();
#pragma unroll 1
  for (int base = 0; base < TK; base += kPT * kIds) {
    if (base) load_ids(base);
#pragma unroll
    for (int j = 0; j < kIds; ++j) {
      if (!any_id(base, j)) break;
      if (ev[j] >= 0 && ev[j] < a.E) atomicAdd(&cnt[ev[j]], 1);
    }
  }
  __syncthreads();
  // thread t owns groups 2t and 2t+1: their rows, full tiles, and the size class
  // 1 .. 4 of their last tile (one 16-bit counter per class)
  const int nw = (G + 127) >> 7;                 // waves that own groups
  const bool owner = wave < nw;
  const int g0 = 2 * tid, g1 = g0 + 1;
  int c0 = 0, c1 = 0, f0 = 0, f1 = 0, k0 = 0, k1 = 0, sr = 0, sf = 0;
  uint64_t p0 = 0, p1 = 0, sc = 0;
  if (owner) {
    const int sh = __builtin_ctz(TR);            // (a power of two)
    c0 = g0 < G ? cnt[g0] : 0;
    c1 = g1 < G ? cnt[g1] : 0;
    f0 = c0 >> sh;
    f1 = c1 >> sh;
    k0 = (4 * (c0 - f0 * TR) + TR - 1) >> sh;
    k1 = (4 * (c1 - f1 * TR) + TR - 1) >> sh;
    p0 = k0 ? 1ull << (16 * (k0 - 1)) : 0;
    p1 = k1 ? 1ull << (16 * (k1 - 1)) : 0;
    sr = c0 + c1;
    sf = f0 + f1;
    sc = p0 + p1;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int r = __shfl_up(sr, o, 64), f = __shfl_up(sf, o, 64);
      const uint64_t c = (uint64_t)__shfl_up((unsigned long long)sc, o, 64);
      if (lane >= o) {
        sr += r;
        sf += f;
        sc += c;
      }
    }
    if (lane == 63) {
      wrows[wave] = sr;
      wfull[wave] = sf;
      wcls[wave] = sc;
    }
  }
  __syncthreads();
  int off0 = 0, off1 = 0, t0 = 0, t1 = 0, r0 = 0, r1 = 0;  // first rows, first full tiles, last tiles
  if (owner) {
    int full_all = 0;
    uint64_t cls_all = 0;
    for (int w = 0; w < nw; ++w) {
      const int r = wrows[w], f = wfull[w];
      const uint64_t c = wcls[w];
      full_all += f;
      cls_all += c;
      sr += w < wave ? r : 0;
      sf += w < wave ? f : 0;
      sc += w < wave ? c : 0;
    }
    off0 = sr - c0 - c1;
    off1 = sr - c1;
    t0 = sf - f0 - f1;
    t1 = sf - f1;
    const uint64_t b0 = sc - p0 - p1, b1 = sc - p1;            // last tiles of each class before
    int cbase[5];                                              // first tile of class k
    cbase[4] = full_all;
#pragma unroll
    for (int k = 3; k >= 1; --k) cbase[k] = cbase[k + 1] + (int)((cls_all >> (16 * k)) & 0xffff);
    auto rem_tile = [&](int k, uint64_t before) {
      int t = 0;
#pragma unroll
      for (int q = 1; q <= 4; ++q)
        if (k == q) t = cbase[q] + (int)((before >> (16 * (q - 1))) & 0xffff);
      return t;
    };
    r0 = rem_tile(k0, b0);
    r1 = rem_tile(k1, b1);
    if (tid == 0 && blockIdx.x == 0) *a.n_tiles = cbase[1] + (int)(cls_all & 0xffff);
    // the slots and bundles of both groups requested together (one dependent
    // pair of loads for the thread); a group that is not resident copies slot 0's
    // bundle (a table has at least one slot), which no kernel reads. The bundle
    // moves as 12 pointer words (held in registers).
    constexpr int kBW = (int)(sizeof(moe_bundle) / 8);
    static_assert(sizeof(moe_bundle) == 8 * kBW && sizeof(GroupTile) == 16 + sizeof(moe_bundle), "record layout");
    if ((tid & (np - 1)) == (int)blockIdx.x) {
      const int s0 = g0 < G && c0 ? a.slot_of[g0] : -1, s1 = g1 < G && c1 ? a.slot_of[g1] : -1;
      uint64_t w0[kBW], w1[kBW];
      const uint64_t* q0 = reinterpret_cast<const uint64_t*>(a.bundles + (s0 > 0 ? s0 : 0));
      const uint64_t* q1 = reinterpret_cast<const uint64_t*>(a.bundles + (s1 > 0 ? s1 : 0));
#pragma unroll
      for (int q = 0; q < kBW; ++q) {
        w0[q] = q0[q];
        w1[q] = q1[q];
      }
      auto emit = [&](int g, int c, int off, int nfull, int full, int rem, int slot, const uint64_t (&w)[kBW]) {
        if (g >= G || c == 0) return;
        if (slot < 0 && a.status) atomicOr(a.status, MOE_STATUS_SLOT_MISS);
        for (int j = 0; j * TR < c; ++j) {
          GroupTile* o = a.tiles + (j < nfull ? full + j : rem);
          o->g = g;
          o->row0 = off + TR * j;
          o->nrows = min(TR, c - TR * j);
          o->slot = slot;
          uint64_t* ob = reinterpret_cast<uint64_t*>(&o->b);
#pragma unroll
          for (int q = 0; q < kBW; ++q) ob[q] = w[q];
        }
      };
      emit(g0, c0, off0, f0, t0, r0, s0, w0);
      emit(g1, c1, off1, f1, t1, r1, s1, w1);
    }
    // each thread read its own two counts only: they become the insertion cursors
    if (g0 < G) {
      cnt[g0] = off0;
      goff[g0] = off0;
      gfull[g0] = t0;
      gnf[g0] = f0 * TR;
      grem[g0] = r0;
    }
    if (g1 < G) {
      cnt[g1] = off1;
      goff[g1] = off1;
      gfull[g1] = t1;
      gnf[g1] = f1 * TR;
      grem[g1] = r1;
    }
  }
  __syncthreads();
  auto place = [&](int g, int pos, int row, int t) {
    const int rel = pos - goff[g];
    a.perm[pos] = row;
    if (rel < gnf[g])
      a.tile_tok[(size_t)gfull[g] * TR + rel] = t;  // (a group's full tiles are consecutive)
    else
      a.tile_tok[(size_t)grem[g] * TR + rel - gnf[g]] = t;
  };
#pragma unroll 1
  for (int base = 0; base < TK; base += kPT * kIds) {
    if (TK > kPT * kIds) load_ids(base);         // (else they are still in registers)
#pragma unroll
    for (int j = 0; j < kIds; ++j) {
      if (!any_id(base, j)) break;
      const int i = base + tid + kPT * j, e = ev[j];
      if (i >= TK) continue;
      const int t = i / a.K, row = t * a.n_list + i - t * a.K;
      if (e >= 0 && e < a.E) {
        if (((e >> 1) & (np - 1)) == (int)blockIdx.x) place(e, atomicAdd(&cnt[e], 1), row, t);
      } else if ((j & (np - 1)) == (int)blockIdx.x) {  // an id outside [0, E) contributes zeros and is reported
        if (a.status) atomicOr(a.status, MOE_STATUS_BAD_INDEX);
        float* y = a.y_experts + (size_t)row * a.d;
        for (int q = 0; q < a.d; ++q) y[q] = 0.f;
      }
    }
  }
  for (int i = blockIdx.x * kPT + tid; i < a.T * a.S; i += np * kPT) {
    const int s = i / a.T, t = i - s * a.T, g = a.E + s;
    place(g, goff[g] + t, t * a.n_list + a.K + s, t);
  }
}

// ---------------------------------------------------------------------------
// prep: A_g x and A_u x of 64 rows of a tile over one of `splits` parts of d, with
// MFMA (ranks as the 16 columns): eight waves take an eighth of the part each, for
// both projections, the loads of two or four k steps in flight; their sums add up
// in LDS as a tree, the parts' in gate/up.
constexpr int kPrepRows = 64;
constexpr int kPrepSplits = 4;                   // parts of d, at most
__global__ void __launch_bounds__(kGT, 4) grouped_prep_kernel(GroupedArgs a) {
  __shared__ float part[kGW][2][4][4][64];
  const int tid = threadIdx.x;
  // (the first parts of all tiles, then the second: neighbours in a launch go to
  // different XCDs, and second parts are often empty)
  const int per = a.max_tiles * a.splits, second = (int)blockIdx.x >= per;
  const int b = blockIdx.x - second * per;
  const int ti = b >> __builtin_ctz(a.splits), Q = b & (a.splits - 1), r0 = second * kPrepRows;
  const int wave = tid >> 6, lane = tid & 63, col = lane & 15, kq = lane >> 4;
  // the tokens of this lane's rows (the tile's token list, read beside the record)
  int tok[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) tok[m] = a.tile_tok[(size_t)ti * a.tile_rows + r0 + 16 * m + col];
  if (ti >= *a.n_tiles) return;
  const GroupTile tl = a.tiles[ti];
  const int nrows = min(kPrepRows, tl.nrows - r0);
  if (tl.slot < 0 || nrows <= 0) return;
  const moe_bundle& bd = tl.b;
  const int d = a.d, r = a.r;
  const int mb = (nrows + 15) >> 4;
  const bool on[2] = {bd.gate.lora_a && bd.gate.lora_b, bd.up.lora_a && bd.up.lora_b};
  const int kw = d / (kGW * a.splits), k0 = (Q * kGW + wave) * kw + kq * 8;
  // (rows past the tile take its first token's, ranks past r rank 0's: their
  // sums are not stored, or multiply zero rows of B)
  const _Float16* arow[2];
  arow[0] = reinterpret_cast<const _Float16*>(on[0] ? bd.gate.lora_a : a.x) + (size_t)(on[0] && col < r ? col : 0) * d + k0;
  arow[1] = reinterpret_cast<const _Float16*>(on[1] ? bd.up.lora_a : a.x) + (size_t)(on[1] && col < r ? col : 0) * d + k0;
  const int tok0 = __shfl(tok[0], 0, 64);
  const _Float16* xrow[4];
#pragma unroll
  for (int m = 0; m < 4; ++m)
    xrow[m] = reinterpret_cast<const _Float16*>(a.x) + (size_t)(16 * m + col < nrows ? tok[m] : tok0) * d + k0;
  f4 acc[2][4];
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int m = 0; m < 4; ++m) acc[c][m] = f4{0.f, 0.f, 0.f, 0.f};
  auto run = [&](auto count) {
    constexpr int MB = decltype(count)::value, KS = MB == 4 ? 2 : 4;
    for (int k = 0; k < kw; k += 32 * KS) {
      h8 b[KS][2], av[KS][MB];
#pragma unroll
      for (int u = 0; u < KS; ++u) {
        const bool in = k + 32 * u < kw;         // uniform
#pragma unroll
        for (int c = 0; c < 2; ++c) b[u][c] = in ? as_h8(ld16(arow[c] + k + 32 * u)) : h8{};
#pragma unroll
        for (int m = 0; m < MB; ++m) av[u][m] = in ? as_h8(ld16(xrow[m] + k + 32 * u)) : h8{};
      }
#pragma unroll
      for (int u = 0; u < KS; ++u)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int m = 0; m < MB; ++m) acc[c][m] = mfma(av[u][m], b[u][c], acc[c][m]);
    }
  };
  if (mb == 1)
    run(std::integral_constant<int, 1>());
  else if (mb == 2)
    run(std::integral_constant<int, 2>());
  else
    run(std::integral_constant<int, 4>());
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (m < mb) part[wave][c][m][e][lane] = acc[c][m][e];
  __syncthreads();
  // lane (col, kq) of block m holds rows 16 m + 4 kq + e, rank col
  for (int p = tid; p < 2 * mb * 256; p += kGT) {
    const int c = p / (mb * 256), m = (p >> 8) % mb, e = (p >> 6) & 3, l = p & 63;
    const int row = 16 * m + 4 * (l >> 4) + e, k = l & 15;
    float v[kGW];
#pragma unroll
    for (int q = 0; q < kGW; ++q) v[q] = part[q][c][m][e][l];
    const float s = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
    if (row < nrows) a.ax[(((size_t)(tl.row0 + r0 + row) * a.splits + Q) * 2 + c) * 16 + k] = s;
  }
}

// ---------------------------------------------------------------------------
// Block b of a GEMM grid -> (token tile, column tile). The dispatcher deals
// blocks to the 8 XCDs in turn, so blocks b and b + 8 share an XCD: every
// column tile of token tile x gets a block that is congruent to x mod 8, the
// ny of them 8 apart. The tile's activations (and its row list) then go
// through one XCD's L2, fetched once instead of once per column tile. The
// grid is the tile count rounded up to a multiple of 8, times ny.
__device__ __forceinline__ void tile_of_block(int b, int ny, int& x, int& y) {
  const int grp = b / (8 * ny), r = b - grp * 8 * ny;
  x = grp * 8 + (r & 7);
  y = r >> 3;
}

// gate/up: workgroup (tile, y) takes the gate and up rows of columns
// [GATE y, GATE y + GATE). Narrow: wave w < 4 the gate rows of columns 16 w ..,
// wave w + 4 the up rows of the same columns, handed over through LDS. Wide: wave
// w the gate and the up rows of columns 16 w .., so silu(g) u stays in registers.
template <class V>
__global__ void __launch_bounds__(kGT, V::EU) grouped_gateup_kernel(GroupedArgs a) {
  constexpr int NBW = V::NBW, TRB = V::TRB, TR = Shape<V>::TR, GATE = Shape<V>::GATE;
  extern __shared__ __attribute__((aligned(16))) char ring[];
  char* const szl = ring + V::RING;
  // after the k loop the ring holds the up accumulators (Narrow), h of the tile
  // (rows padded by 16 bytes: the 16 rows of an operand on different banks) and
  // lora_scale * (A x) of the tile's rows
  constexpr int kU = NBW == 1 ? 4 * TRB * 4 * 64 * 4 : 0;
  constexpr int HP = GATE + 8;
  float* const uacc = reinterpret_cast<float*>(ring);  // [4 waves][m][4 e][64 lanes]
  _Float16(*hs)[HP] = reinterpret_cast<_Float16(*)[HP]>(ring + kU);
  _Float16(*la)[TR][16] = reinterpret_cast<_Float16(*)[TR][16]>(ring + kU + TR * HP * 2);
  static_assert(kU + TR * HP * 2 + 2 * TR * 16 * 2 <= V::RING, "epilogue fits in the ring");
  int bx, by;
  tile_of_block(blockIdx.x, a.I / GATE, bx, by);
  const int tix = bx < a.max_tiles ? bx : 0;
  // (the record and the token list are read beside the count; one past the
  // count is never used)
  const GroupTile tl = a.tiles[tix];
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  // the tokens of the rows this lane copies (unset past the tile's rows)
  const int32_t* tt = a.tile_tok + (size_t)tix * TR;
  constexpr int XJ = Shape<V>::XJ;
  auto copy_row = [&](int j) { return 4 * (wave + kGW * j) + (lane >> 4); };
  const int tr0 = tt[0];
  int tk[XJ];
#pragma unroll
  for (int j = 0; j < XJ; ++j) tk[j] = tt[copy_row(j)];
  if (bx >= *a.n_tiles) return;
  if (tl.slot < 0) return;  // not resident: the down kernel writes zero rows
  const moe_bundle& bd = tl.b;
  const int col = lane & 15, kq = lane >> 4;
  const int d = a.d, I = a.I, r = a.r;
  const int mb = (tl.nrows + 15) >> 4;
  const int c0 = by * GATE;                      // first column of this workgroup
  const int cc = NBW == 1 ? wave >> 2 : 0;       // projection of block 0 (0 gate, 1 up)
  const int wb = NBW == 1 ? wave & 3 : wave;     // column block
  const int i = c0 + wb * 16 + col;              // this lane's gate/up column
  const bool lg = r > 0 && bd.gate.lora_a && bd.gate.lora_b;
  const bool lu = r > 0 && bd.up.lora_a && bd.up.lora_b;
  const bool ld = r > 0 && bd.down.lora_a && bd.down.lora_b;

  // The epilogue's operands, requested now and consumed after the k loop:
  // A x of the tile's rows, the LoRA-B operands and the A_d rows of this
  // workgroup's columns.
  constexpr int NAX = 2 * TR * 16 / kGT;
  float axv[NAX][kPrepSplits];
#pragma unroll
  for (int q = 0; q < NAX; ++q) {
    const int p = tid + q * kGT, pc = p / (TR * 16), row = (p >> 4) % TR, k = p & 15;
    const bool on = row < tl.nrows && k < r && (pc == 0 ? lg : lu);
    const float* src = a.ax + ((size_t)(tl.row0 + row) * a.splits * 2 + pc) * 16 + k;
#pragma unroll
    for (int h = 0; h < kPrepSplits; ++h) axv[q][h] = on && h < a.splits ? src[h * 32] : 0.f;
  }
  h8 bop[NBW];
#pragma unroll
  for (int b = 0; b < NBW; ++b) {
    const bool gate = NBW == 1 ? cc == 0 : b == 0;
    bop[b] = (gate ? lg : lu) ? lora_b_operand(static_cast<const __half*>(gate ? bd.gate.lora_b : bd.up.lora_b), i, r, kq)
                              : h8{};
  }
  h8 adv[GATE / 32];
#pragma unroll
  for (int q = 0; q < GATE / 32; ++q)
    adv[q] = ld && col < r
                 ? as_h8(ld16(static_cast<const __half*>(bd.down.lora_a) + (size_t)col * I + c0 + 32 * q + 8 * kq))
                 : h8{};

  // weight row w_row: its projection and column (the projection pointers are in
  // registers: a pointer loaded inside the copy loop would be a vector load
  // behind the chunks in flight, and its wait would drain them)
  const uint8_t* const gq = static_cast<const uint8_t*>(bd.gate.q);
  const uint8_t* const uq = static_cast<const uint8_t*>(bd.up.q);
  const uint8_t* const gs = static_cast<const uint8_t*>(bd.gate.sz);
  const uint8_t* const us = static_cast<const uint8_t*>(bd.up.sz);
  auto is_gate = [](int w_row) { return NBW == 1 ? w_row < GATE : !(w_row & 16); };
  auto wcol = [=](int w_row) { return c0 + (NBW == 1 ? w_row % GATE : (w_row >> 5) * 16 + (w_row & 15)); };
  auto wrow = [=](int w_row) -> const uint8_t* { return (is_gate(w_row) ? gq : uq) + (size_t)wcol(w_row) * (d / 2); };
  auto srow = [=](int w_row) -> const uint8_t* { return (is_gate(w_row) ? gs : us) + (size_t)wcol(w_row) * (d / 16); };
  // Each lane's source rows are fixed for the tile, and resolved here: a load
  // inside the copy loop would wait for the copies in flight. (Rows past nrows
  // hold no token: they take row 0's, and are never stored.)
  const char* xr[XJ];
#pragma unroll
  for (int j = 0; j < XJ; ++j)
    xr[j] = reinterpret_cast<const char*>(a.xp) + (size_t)(copy_row(j) < tl.nrows ? tk[j] : tr0) * d * 2;
  auto xsrc = [&](int j, int k) -> const void* {
    const char* p = xr[0];
#pragma unroll
    for (int q = 1; q < XJ; ++q)
      if (j == q) p = xr[q];
    return p + (size_t)k * 2;
  };

  f4 acc[NBW][TRB];
#pragma unroll
  for (int b = 0; b < NBW; ++b)
#pragma unroll
    for (int m = 0; m < TRB; ++m) acc[b][m] = f4{0.f, 0.f, 0.f, 0.f};
  tile_gemm<V>(ring, szl, d, mb, wrow, srow, xsrc, acc);

  // lora_scale * (A x) of the tile's rows, fp16 (rank past r: zero)
#pragma unroll
  for (int q = 0; q < NAX; ++q) {
    const int p = tid + q * kGT, pc = p / (TR * 16), row = (p >> 4) % TR, k = p & 15;
    const float v = (axv[q][0] + axv[q][1]) + (axv[q][2] + axv[q][3]);
    la[pc][row][k] = (_Float16)(a.lora_scale * v);
  }
  __syncthreads();
  // LoRA delta: one MFMA step of K = rank against lora_scale * (A x)
#pragma unroll
  for (int b = 0; b < NBW; ++b) {
    const int pc = NBW == 1 ? cc : b;
    if (pc == 0 ? lg : lu) {
#pragma unroll
      for (int m = 0; m < TRB; ++m) {
        if (m >= mb) continue;
        h8 aop = {};
        if (kq < 2) aop = *reinterpret_cast<const h8*>(&la[pc][16 * m + col][kq * 8]);
        acc[b][m] = mfma(aop, bop[b], acc[b][m]);
      }
    }
  }
  if constexpr (NBW == 1) {
    // the up waves hand their sums to the gate waves of the same columns (same lane)
    if (cc == 1) {
#pragma unroll
      for (int m = 0; m < TRB; ++m) {
        if (m >= mb) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e) uacc[((wb * TRB + m) * 4 + e) * 64 + lane] = acc[0][m][e];
      }
    }
    __syncthreads();
  }
  // h = silu(g) u, rounded to fp16, into LDS
  if (cc == 0) {
#pragma unroll
    for (int m = 0; m < TRB; ++m) {
      if (m >= mb) continue;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float g = acc[0][m][e];
        const float u = NBW == 1 ? uacc[((wb * TRB + m) * 4 + e) * 64 + lane] : acc[NBW - 1][m][e];
        hs[16 * m + 4 * kq + e][wb * 16 + col] = (_Float16)(g / (1.0f + expf(-g)) * u);
      }
    }
  }
  __syncthreads();
  // h to memory in pair order, whole 16-byte pieces
  for (int p = tid; p < tl.nrows * (GATE / 8); p += kGT) {
    const int row = p / (GATE / 8), q = p % (GATE / 8);
    const U4 v = *reinterpret_cast<const U4*>(&hs[row][8 * q]);
    *reinterpret_cast<U4*>(a.h + (size_t)(tl.row0 + row) * I + c0 + 8 * q) = perm8(v);
  }
  // the slab's partial A_d h, row x rank over this workgroup's columns: one row
  // block per wave, on the matrix cores
  if (ld) {
    for (int m = wave; m < mb; m += kGW) {
      f4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q < GATE / 32; ++q)
        s = mfma(*reinterpret_cast<const h8*>(&hs[16 * m + col][32 * q + 8 * kq]), adv[q], s);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = 16 * m + 4 * kq + e;
        if (row < tl.nrows) a.adp[((size_t)(tl.row0 + row) * (I / GATE) + by) * 16 + col] = s[e];
      }
    }
  }
}

// down: workgroup (64-row part of a tile, y) takes columns [DOWN y, DOWN y + DOWN).
template <class V>
__global__ void __launch_bounds__(kGT, V::EU) grouped_down_kernel(GroupedArgs a, int nsl) {
  constexpr int NBW = V::NBW, TRB = V::TRB, TR = Shape<V>::TR, DOWN = Shape<V>::DOWN;
  extern __shared__ __attribute__((aligned(16))) char ring[];
  // after the k loop the ring holds lora_scale * (A_d h) of the tile's rows and
  // their y_experts rows
  _Float16(*la)[16] = reinterpret_cast<_Float16(*)[16]>(ring);
  int* ydst = reinterpret_cast<int*>(ring + TR * 16 * 2);
  int bx, by;
  tile_of_block(blockIdx.x, a.d / DOWN, bx, by);
  // (the first parts of all tiles, then the second, as in prep)
  const int second = bx >= a.max_tiles;          // (a tile is one or two parts)
  const int tix = bx - second * a.max_tiles, first = second * TR;
  if (first >= a.tile_rows || tix >= a.max_tiles) return;  // the grid is rounded up
  const GroupTile tl = a.tiles[tix];             // (read beside the count, as in gate/up)
  if (tix >= *a.n_tiles) return;
  const int nrows = min(TR, tl.nrows - first), row0 = tl.row0 + first;
  if (nrows <= 0) return;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int col = lane & 15, kq = lane >> 4;
  const int d = a.d, I = a.I, r = a.r;
  const int mb = (nrows + 15) >> 4;
  const int n0 = by * DOWN + wave * NBW * 16 + col;  // this lane's first output column
  if (tl.slot < 0) {  // not resident: the pair contributes zeros (the miss is reported)
    for (int p = tid; p < nrows * DOWN; p += kGT) {
      const int row = p / DOWN, c = p % DOWN;
      a.y_experts[(size_t)a.perm[row0 + row] * d + by * DOWN + c] = 0.f;
    }
    return;
  }
  const moe_bundle& bd = tl.b;
  const bool ld = r > 0 && bd.down.lora_a && bd.down.lora_b;
  // The epilogue's operands, requested now and consumed after the k loop: the
  // output rows, the LoRA-B operands, and the slab partials of A_d h (thread p
  // holds (row, rank) = ((p + 512 q) / 16, p % 16); the first slabs here, any
  // further ones after the loop).
  constexpr int NLA = TR * 16 / kGT;
  constexpr int kPreSl = 16 / NBW;
  const int ydv = tid < nrows ? a.perm[row0 + tid] : -1;
  h8 bop[NBW];
#pragma unroll
  for (int b = 0; b < NBW; ++b)
    bop[b] = ld ? lora_b_operand(static_cast<const __half*>(bd.down.lora_b), n0 + 16 * b, r, kq) : h8{};
  float adv[NLA][kPreSl];
#pragma unroll
  for (int q = 0; q < NLA; ++q) {
    const int p = tid + q * kGT, row = p >> 4, k = p & 15;
    const bool on = ld && row < nrows && k < r;
    const float* src = a.adp + (size_t)(row0 + row) * nsl * 16 + k;
#pragma unroll
    for (int sl = 0; sl < kPreSl; ++sl) adv[q][sl] = on && sl < nsl ? src[sl * 16] : 0.f;
  }
  // weight row w_row: output column by * DOWN + w_row (the pointers in registers,
  // as in gate/up)
  const size_t nbase = (size_t)by * DOWN;
  const uint8_t* const dq = static_cast<const uint8_t*>(bd.down.q);
  const uint8_t* const dsz = static_cast<const uint8_t*>(bd.down.sz);
  auto wrow = [=](int w_row) -> const uint8_t* { return dq + (nbase + w_row) * (I / 2); };
  auto srow = [=](int w_row) -> const uint8_t* { return dsz + (nbase + w_row) * (I / 16); };
  const char* hbase = reinterpret_cast<const char*>(a.h);
  auto xsrc = [&](int j, int k) -> const void* {
    const int row = 4 * (wave + kGW * j) + (lane >> 4);
    return hbase + ((size_t)(row0 + (row < nrows ? row : 0)) * I + k) * 2;
  };

  f4 acc[NBW][TRB];
#pragma unroll
  for (int b = 0; b < NBW; ++b)
#pragma unroll
    for (int m = 0; m < TRB; ++m) acc[b][m] = f4{0.f, 0.f, 0.f, 0.f};
  tile_gemm<V>(ring, ring + V::RING, I, mb, wrow, srow, xsrc, acc);

  // lora_scale * (A_d h): the slab partials summed in slab order
#pragma unroll
  for (int q = 0; q < NLA; ++q) {
    const int p = tid + q * kGT, row = p >> 4, k = p & 15;
    float v = 0.f;
#pragma unroll
    for (int sl = 0; sl < kPreSl; ++sl) v += adv[q][sl];
    if (ld && row < nrows && k < r) {
      const float* src = a.adp + (size_t)(row0 + row) * nsl * 16 + k;
      // (eight loads at once, added in slab order: d 512, I 1024, T = 8 9.5 us a launch, 10.1
      // one after the other)
      for (int s0 = kPreSl; s0 < nsl; s0 += 8) {
        float w[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) w[u] = s0 + u < nsl ? src[(s0 + u) * 16] : 0.f;
#pragma unroll
        for (int u = 0; u < 8; ++u) v += w[u];
      }
    }
    la[row][k] = (_Float16)(v * a.lora_scale);
  }
  if (tid < TR) ydst[tid] = ydv;
  __syncthreads();
  if (ld) {
#pragma unroll
    for (int m = 0; m < TRB; ++m) {
      if (m >= mb) continue;
      h8 aop = {};
      if (kq < 2) aop = *reinterpret_cast<const h8*>(&la[16 * m + col][kq * 8]);
#pragma unroll
      for (int b = 0; b < NBW; ++b) acc[b][m] = mfma(aop, bop[b], acc[b][m]);
    }
  }
#pragma unroll
  for (int m = 0; m < TRB; ++m) {
    if (m >= mb) continue;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = 16 * m + 4 * kq + e;
      if (row < nrows) {
        float* y = a.y_experts + (size_t)ydst[row] * d + n0;
#pragma unroll
        for (int b = 0; b < NBW; ++b) y[16 * b] = acc[b][m][e];
      }
    }
  }
}

hipError_t allow_lds(const void* kernel) {
  return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsMax);
}

template <class V>
void launch_gateup(const GroupedArgs& a, hipStream_t st) {
  const int tiles8 = (a.max_tiles + 7) / 8 * 8;
  hipLaunchKernelGGL(grouped_gateup_kernel<V>, dim3(tiles8 * (a.I / Shape<V>::GATE)), dim3(kGT), lds_bytes<V>(a.d), st,
                     a);
}

template <class V>
void launch_down(const GroupedArgs& a, hipStream_t st) {
  const int parts8 = (a.max_tiles * (a.tile_rows / Shape<V>::TR) + 7) / 8 * 8;
  const int nsl = a.I / (a.wide ? Shape<GateWide>::GATE : Shape<GateNarrow>::GATE);
  hipLaunchKernelGGL(grouped_down_kernel<V>, dim3(parts8 * (a.d / Shape<V>::DOWN)), dim3(kGT), lds_bytes<V>(a.I), st, a,
                     nsl);
}

}  // namespace

bool grouped_shape_supported(int d, int I, int r, int groups) {
  return d % Shape<DownWide>::DOWN == 0 && I % Shape<GateNarrow>::GATE == 0 && d % 128 == 0 && I % 128 == 0 && r >= 0 &&
         r <= kGroupMaxR && groups <= kGroupMaxG && lds_bytes<GateNarrow>(d) <= kLdsMax && lds_bytes<DownNarrow>(I) <= kLdsMax;
}

// The wide shape from 64 rows a routed group on, if its workgroups fill the chip.
// Whole calls, narrow / wide: d 2048, E 256, K 8: T = 777 184.5 / 186.7 us, 1500 260 /
// 261, 3100 429 / 412; d 4096, E 64, K 4: T = 777 215 / 218, 1000 240 / 242, 1500 328 /
// 301, 3100 570 / 510; d 512, E 16, K 2 (50 to 100 wide workgroups): T = 3100 41 / 45.
constexpr int kWideRows = 64, kWideFill = 256;

GroupedPlan grouped_plan(int T, int d, int I, int E, int K, int S) {
  const long long fill = (long long)T * (K + S) / Shape<GateWide>::TR * (I / Shape<GateWide>::GATE);
  const bool wide = (long long)T * K >= (long long)kWideRows * E && fill >= kWideFill &&
                    I % Shape<GateWide>::GATE == 0 && lds_bytes<GateWide>(d) <= kLdsMax;
  // (a wave's part of d in prep is at least one k step of 32)
  const int splits = d / 256 < kPrepSplits ? d / 256 : kPrepSplits;
  return wide ? GroupedPlan{1, Shape<GateWide>::TR, splits} : GroupedPlan{0, Shape<GateNarrow>::TR, splits};
}

// Beyond d_expert 512 a 256-column down workgroup is a long one (8 chunks, and half of
// the slab partials fetched after them): while the columns of all tiles are no more
// workgroups than CUs, 128 columns are faster, as there are CUs for twice as many. Whole
// calls, 256 / 128 columns, d_expert 1024: d 512, E 64, T = 8 25.7 / 24.0 us; d 2048,
// E 16, K 2, T = 16 34.4 / 32.2; from about 300 workgroups on the other way (d 2048, E 64,
// T = 64 68.0 / 70.9; d 4096, T = 8 62.9 / 65.9). Up to 512 they differ by less than the
// empty workgroups of twice the grid (d 2048, I 512, E 256, T = 1 30.1 / 30.7). The tiles
// are estimated as if the routing were even.
constexpr int kDownNarrowFill = 256;
static bool down_narrow(const GroupedArgs& a) {
  const long long tiles = std::min((long long)a.T * a.K, (long long)a.E) + a.S + (long long)a.T * a.n_list / kGroupMinRows;
  return a.I > 512 && tiles * (a.d / Shape<DownWide>::DOWN) <= kDownNarrowFill;
}

hipError_t launch_grouped_ffn(const GroupedArgs& a, hipStream_t st) {
  // Workgroups of the permutation (a power of two): up to 2,000 ids any number does; whole
  // calls with 1 / 8 / 32: E 256, K 8, T = 1024 197 / 192 / 191 us, T = 3100 390 / 373 / 373;
  // E 1024, K 32, T = 8000 1070 / 869 / 860.
  constexpr int np = 32;
  const size_t xw = (size_t)kPT * kXPieces * 8;   // elements of x per workgroup
  const int xb = (int)(((size_t)a.T * a.d + xw - 1) / xw);
  hipLaunchKernelGGL(grouped_permute_kernel, dim3(np + xb), dim3(kPT), 0, st, a, np);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (a.r > 0) {
    hipLaunchKernelGGL(grouped_prep_kernel, dim3(a.max_tiles * (a.tile_rows / kPrepRows) * a.splits), dim3(kGT), 0, st, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  static bool attr_set = false;
  if (!attr_set) {
    e = allow_lds((const void*)grouped_gateup_kernel<GateNarrow>);
    if (e == hipSuccess) e = allow_lds((const void*)grouped_gateup_kernel<GateWide>);
    if (e == hipSuccess) e = allow_lds((const void*)grouped_down_kernel<DownWide>);
    if (e == hipSuccess) e = allow_lds((const void*)grouped_down_kernel<DownNarrow>);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  if (a.wide)
    launch_gateup<GateWide>(a, st);
  else
    launch_gateup<GateNarrow>(a, st);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (2 * lds_bytes<DownWide>(a.I) <= kLdsMax && !down_narrow(a))
    launch_down<DownWide>(a, st);
  else
    launch_down<DownNarrow>(a, st);
  return hipGetLastError();
}

}  // namespace moe
