// Prefill phase with sequence-level exit (River-LLM method section, "Inference with Seamless
// Exit", list of phases): the whole prompt is processed at one unified depth e_p, blocks
// 1..e_p with the backbone matrices, blocks e_p+1..L with their 4-bit river twins, every
// block writing K/V of every prompt position into the shared cache slot.  Unlike a decode
// step this is dense matrix-matrix work, so it runs on the matrix cores: the prompt is cut
// into chunks of up to kChunk tokens and each block is a sequence of MFMA GEMMs over the
// chunk (fp16 operands, fp32 accumulation) with small element-wise kernels between them:
//
//   [ (embed | h += Wd's sums) + rmsnorm -> GEMM(Wq;Wk;Wv) -> rope + cache store -> causal attention
//     -> GEMM(Wo) -> h += its sums, rmsnorm -> GEMM(Wg;Wu) with swiglu -> GEMM(Wd) ] x L
//
// Operand types: activations are rounded to half precision (fp16) when they enter a GEMM or
// the attention; backbone weights (bf16) are converted to fp16 while a tile is staged in LDS
// (exact but for magnitudes below 2^-14); river weights are dequantised, (code - zero) * scale
// in fp32, and rounded to fp16 while staged; cached K/V (bf16) are converted the same way.
// The residual stream stays fp32 in HBM.  Only bf16 models take this path.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "river_device.h"

namespace river {
namespace pf {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kChunk = 4096;          // most prompt tokens per pass (rows of the activation buffers)
constexpr int TK = 64;
constexpr int LDK = TK + 8;           // LDS row stride in halfs: 144 B, rows 4 banks apart

// v_mfma_f32_32x32x16_f16: D[32x32] += A[32x16] B[16x32].  Lane l supplies row l % 32 of A and
// column l % 32 of B, eight K values each (those of lane group l / 32; which eight is the same
// for A and B, so any fixed assignment gives the right sum).  D: register r of lane l is
// row (r / 4) * 8 + (l / 32) * 4 + r % 4, column l % 32.
__device__ __forceinline__ f32x16 mfma16(half8 a, half8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ f32x16 mfma16_bf16(half8 a, half8 b, f32x16 c) {     // (the registers hold bf16 values)
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ int c_row(int r, int lane) { return (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3); }

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
// eight bf16 values (16 bytes) -> eight fp16 values
__device__ __forceinline__ half8 bf16x8_to_half8(const uint4 &w) {
  half8 h;
  h[0] = (_Float16)bf16_lo(w.x); h[1] = (_Float16)bf16_hi(w.x);
  h[2] = (_Float16)bf16_lo(w.y); h[3] = (_Float16)bf16_hi(w.y);
  h[4] = (_Float16)bf16_lo(w.z); h[5] = (_Float16)bf16_hi(w.z);
  h[6] = (_Float16)bf16_lo(w.w); h[7] = (_Float16)bf16_hi(w.w);
  return h;
}

// Eight 4-bit codes of a row-major word (nibble i = column i) -> fp16 of (code - zero) * scale, taken in
// fp32 as the decode kernels and the oracle take it.  A nibble in bits 6..9 of an fp16 word is the
// subnormal number code * 2^-18, which the mixed-precision fma reads exactly; the product of the zero point
// and the scale, bf16 both, is exact in fp32, so code * scale - zero * scale is rounded once and one
// instruction a weight makes it (the difference first, then its product: three).
__device__ __forceinline__ half8 dequant8(uint32_t w, float s, float zero) {
  const float s18 = s * 0x1p18f, zs = -zero * s;
  half8 h;
#pragma unroll
  for (int k = 0; k < 4; ++k) {                // nibbles k and k + 4
    const uint32_t sh = k < 2 ? w << (6 - 4 * k) : w >> (4 * k - 6);
    const half2v q = __builtin_bit_cast(half2v, sh & 0x03c003c0u);
    h[k] = (_Float16)fmaf((float)q[0], s18, zs);
    h[k + 4] = (_Float16)fmaf((float)q[1], s18, zs);
  }
  return h;
}

// The eight codes themselves: a nibble in the low bits of 1024.0 is 1024 + code.
__device__ __forceinline__ half8 codes8(uint32_t w) {
  half8 h;
#pragma unroll
  for (int k = 0; k < 4; ++k) {                // nibbles k and k + 4
    const half2v q = __builtin_bit_cast(half2v, ((w >> (4 * k)) & 0x000f000fu) | 0x64006400u) - (_Float16)1024.f;
    h[k] = q[0];
    h[k + 4] = q[1];
  }
  return h;
}
// x as a sum of three bf16 numbers (24 bits, exact but for what lies below the smallest of them).  An infinity or NaN
// is the first one, the others 0; a finite x that rounds to an infinity is cut off instead.
__device__ __forceinline__ void split3(float x, uint16_t (&p)[3]) {
  const bool finite = __builtin_isfinite(x);
  p[0] = Store<1>::rne(x);
  if (finite && (p[0] & 0x7fffu) == 0x7f80u) p[0] -= 1;
  x = finite ? x - __uint_as_float((uint32_t)p[0] << 16) : 0.f;
#pragma unroll
  for (int i = 1; i < 3; ++i) {
    p[i] = Store<1>::rne(x);
    x -= __uint_as_float((uint32_t)p[i] << 16);
  }
}
__device__ __forceinline__ void store_split3(uint16_t *dst, size_t plane, const float (&x)[8]) {
  uint32_t w[3][4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    uint16_t a[3], b[3];
    split3(x[2 * e], a);
    split3(x[2 * e + 1], b);
#pragma unroll
    for (int i = 0; i < 3; ++i) w[i][e] = a[i] | (uint32_t)b[i] << 16;
  }
#pragma unroll
  for (int i = 0; i < 3; ++i) *(uint4 *)(dst + i * plane) = make_uint4(w[i][0], w[i][1], w[i][2], w[i][3]);
}

// A 16-bit KV cache holds bf16 values, or IEEE half values when the context keeps its cache in
// FP16 (kv_f16): store one element / fetch eight as fp16 / fetch one as fp32.
__device__ __forceinline__ void cache_store(void *cache, size_t i, float v, int kv_f16) {
  if (kv_f16) ((_Float16 *)cache)[i] = (_Float16)v;
  else Store<1>::st(cache, i, v);
}
__device__ __forceinline__ half8 cache_half8(const uint4 &w, int kv_f16) {
  return kv_f16 ? __builtin_bit_cast(half8, w) : bf16x8_to_half8(w);
}
__device__ __forceinline__ float cache_lo(uint32_t w, int kv_f16) {
  return kv_f16 ? (float)__builtin_bit_cast(half2v, w)[0] : bf16_lo(w);
}
__device__ __forceinline__ float cache_hi(uint32_t w, int kv_f16) {
  return kv_f16 ? (float)__builtin_bit_cast(half2v, w)[1] : bf16_hi(w);
}

// ------------------------------------------------------------------ GEMM
//
// C[M, N] = op(A[M, K] B^T), B = up to three matrices stacked along N (rows of W_q, W_k, W_v;
// of W_gate, W_up), each [rows, K] row-major: dense bf16, or 4-bit codes with one packed
// (scale, zero) pair per (row, group of `group` columns; ceil(K / group) pairs a row).  K % 64 == 0,
// group % 64 == 0, rows of every matrix % 64 == 0; M and N are guarded (rows of A beyond M - 1 read row M - 1).
// op: store fp32, slice ks of K into its own [M, N] plane for the consumer to add up in order, or
// SwiGLU of a gate and an up matrix stored as fp16 [M, ffn] (k_split = 1).
struct GemmB {
  const void *w[3];
  const void *sz[3];
  int rows[3];
};

__device__ __forceinline__ void gemm_b_row(const GemmB &B, int n, int N, int &mat, int &row) {
  n = min(n, N - 1);
  mat = 0;
  if (n >= B.rows[0]) { n -= B.rows[0]; mat = 1; }
  if (mat == 1 && n >= B.rows[1]) { n -= B.rows[1]; mat = 2; }
  row = n;
}

// What bounds it: many rows -- the matrix cores (at the clock the power limit leaves: 68 % of the
// cycles issue MFMAs at 4096 x 28672 x 4096, 1.05 PFLOP/s, where the 128 x 128 tile with one K tile in
// flight reached 0.85); a few hundred rows -- the chain of K tiles of the few workgroups there are (512 x 4096 x
// 14336: 209 us without slices and one tile in flight, 63 now); up to 128 rows: k_pf_gemm_rows.  A 256 x 256 tile halves the LDS reads per MFMA of a 128 x 128 one.  B goes through registers
// because it is converted on the way (bf16 -> fp16, codes -> fp16); one conversion serves all
// wavefronts of the tile.
//
// Tile of C per workgroup (TM x TN), its WM x WN wavefronts, K tiles in flight in registers (PF) and
// workgroups per CU (OCC, bounds the registers).
template <int TM_, int TN_, int WM_, int WN_, int PF_, int OCC_> struct GemmTile {
  static constexpr int TM = TM_, TN = TN_, WM = WM_, WN = WN_, PF = PF_, OCC = OCC_;
  static constexpr int NT = WM * WN * 64;                      // threads
  static constexpr int MW = TM / WM, NW = TN / WN;             // a wavefront's part of the tile
  static constexpr int MB = MW / 32, NB = NW / 32;             // ... in MFMA blocks
  static constexpr int GR = NT / 8;                            // rows a staging round of the workgroup covers
  static constexpr int RA = TM / GR, RB = TN / GR;             // staging rounds per K tile
  static constexpr int LDS_BYTES = 2 * (TM + TN) * LDK * 2;    // two buffers each of A and B
  static_assert((RA == 2 || RA == 4) && (RB == 2 || RB == 4) && RA >= RB && RA * GR == TM && RB * GR == TN,
                "two or four staging rounds");
};
typedef GemmTile<128, 128, 4, 2, 2, 2> TileM;
typedef GemmTile<256, 128, 4, 2, 2, 1> TileN;
typedef GemmTile<256, 256, 4, 2, 1, 1> TileL;
enum { PF_STORE = 0, PF_SWIGLU = 1 };

// Row r of B's tile (a multiple of 8: the matrices' row counts are multiples of 64, so eight rows
// never straddle two of them) -> matrix and row.  SwiGLU: the rows alternate between gate and up
// every NW / 2 rows, so that a wavefront holds both factors of an output.
template <class T, int EPI>
__device__ __forceinline__ void gemm_b_row8(const GemmB &B, int n_tile, int r, int N, int &mat, int &row) {
  if constexpr (EPI == PF_SWIGLU) {
    constexpr int G = T::NW / 2;
    mat = (r / G) & 1;
    row = min(n_tile * (T::TN / 2) + r / (2 * G) * G + r % G, B.rows[0] - 8);
  } else {
    gemm_b_row(B, min(n_tile * T::TN + r, N - 8), N, mat, row);
  }
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t gemm_rsrc(const void *p) {
  return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, 0x7ffffff0, 0x00020000);
}

template <class T, bool W4, int EPI>
__global__ __launch_bounds__(T::NT, T::OCC) void k_pf_gemm(const _Float16 *__restrict__ A, int lda, GemmB B, int N,
                                                           int K, int group, void *C, int ldc, int M, int m_tiles,
                                                           int k_split) {
  extern __shared__ __attribute__((aligned(16))) _Float16 pf_lds[];
  constexpr int TM = T::TM, TN = T::TN, PF = T::PF, GR = T::GR;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wv / T::WN, wn = wv % T::WN;
  // Workgroup -> (tile of C, slice of K).  Consecutive workgroup ids go round the 8 XCDs; the
  // workgroups of one XCD take all M tiles of a (column of N tiles, slice of K) before the next, so
  // that a B tile is fetched from HBM once (its XCD's L2 serves the other M tiles).
  // (one-dimensional grid of 8 * ceil(N tiles * k_split / 8) * m_tiles workgroups)
  const int n_tiles = (N + TN - 1) / TN;
  const int col = ((blockIdx.x >> 3) / m_tiles) * 8 + (blockIdx.x & 7), m_tile = (blockIdx.x >> 3) % m_tiles;
  if (col >= n_tiles * k_split) return;
  const int n_tile = col / k_split, ks_i = col % k_split;
  const int m0 = m_tile * TM;
  const int nk_all = K / TK, kt0 = (int)((long long)nk_all * ks_i / k_split);
  const int nk = (int)((long long)nk_all * (ks_i + 1) / k_split) - kt0;

  // what this thread stages per K tile: a 16-byte segment of A per round; of B one per round (dense)
  // or as many words of 8 codes, consecutive, with the (scale, zero) pair of their row (river)
  constexpr int RA = T::RA, RB = T::RB;
  const int srow = tid >> 3, sk = tid & 7;
  unsigned a_off[RA];
#pragma unroll
  for (int i = 0; i < RA; ++i) a_off[i] = (unsigned)min(m0 + i * GR + srow, M - 1) * (unsigned)lda * 2u + sk * 16u;
  const __amdgpu_buffer_rsrc_t a_rsrc = gemm_rsrc((const char *)A + (size_t)kt0 * TK * 2);
  const int s_dst = srow * LDK + sk * 8;                       // + i * GR * LDK
  __amdgpu_buffer_rsrc_t b_rsrc[W4 ? 1 : RB];
  unsigned b_off = 0;
  const char *b_src = nullptr, *b_sz = nullptr;                // (W4: a thread's row may be of any of the matrices)
  int b_dst = 0;
  if constexpr (W4) {
    const int row_l = tid / (8 / RB), q = tid % (8 / RB);
    int mat, row;
    gemm_b_row8<T, EPI>(B, n_tile, row_l & ~7, N, mat, row);
    row += row_l & 7;
    b_src = (const char *)B.w[mat] + (size_t)row * (K >> 1) + q * RB * 4 + kt0 * (TK / 2);
    b_sz = (const char *)B.sz[mat] + (size_t)row * ((K + group - 1) / group) * 4;   // (the last group may be shorter)
    b_dst = row_l * LDK + q * RB * 8;
  } else {
    b_off = (unsigned)(lane >> 3) * (unsigned)K * 2u + sk * 16u;
#pragma unroll
    for (int i = 0; i < RB; ++i) {                             // the eight rows of this wavefront
      int mat, row;
      gemm_b_row8<T, EPI>(B, n_tile, i * GR + wv * 8, N, mat, row);
      b_rsrc[i] = gemm_rsrc((const char *)B.w[mat] + ((size_t)row * K + kt0 * TK) * 2);
    }
  }

  // K tiles on their way from global memory to LDS: a ring of PF register sets
  u32x4 fa[PF][RA], fb[PF][W4 ? 1 : RB];        // (native vectors: as structs they are kept in scratch memory)
  uint32_t fsz[PF];
  // (tiles are loaded one after the other: the group of the next one by counting, no division per tile)
  const int tiles_per_group = group / TK;
  int g_at = W4 ? kt0 / tiles_per_group : 0, g_left = W4 ? tiles_per_group - kt0 % tiles_per_group : 0;
  auto load_part = [&](int kt, int u, int i) {   // part i of tile kt into set u
    fa[u][i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(a_rsrc, a_off[i], kt * (TK * 2), 0));
    if constexpr (W4) {
      if (i == RA - 1) {                          // (all parts of the set have been staged)
        if constexpr (RB == 4) {
          fb[u][0] = *RIVER_GLOBAL(u32x4, b_src + kt * (TK / 2));
        } else {
          const u32x2 v = *RIVER_GLOBAL(u32x2, b_src + kt * (TK / 2));
          fb[u][0] = u32x4{v.x, v.y, 0u, 0u};
        }
        fsz[u] = *RIVER_GLOBAL(uint32_t, b_sz + (size_t)g_at * 4);
        if (--g_left == 0) { g_left = tiles_per_group; ++g_at; }
      }
    } else if (i < RB) {
      constexpr int n = RB - 1;
      fb[u][i & n] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(b_rsrc[i & n], b_off, kt * (TK * 2), 0));
    }
  };
  auto stage_part = [&](int u, int i, int buf) {  // part i of set u into LDS buffer buf
    _Float16 *const As = pf_lds + buf * TM * LDK, *const Bs = pf_lds + 2 * TM * LDK + buf * TN * LDK;
    *(u32x4 *)(As + s_dst + i * GR * LDK) = fa[u][i];
    if (i >= RB) return;
    if constexpr (W4) {
      const uint32_t w = i == 0 ? fb[u][0].x : i == 1 ? fb[u][0].y : i == 2 ? fb[u][0].z : fb[u][0].w;
      *(half8 *)(Bs + b_dst + i * 8) = dequant8(w, bf16_lo(fsz[u]), bf16_hi(fsz[u]));
    } else {
      const u32x4 w = fb[u][i & (RB - 1)];
      *(half8 *)(Bs + s_dst + i * GR * LDK) = bf16x8_to_half8(make_uint4(w.x, w.y, w.z, w.w));
    }
  };

  f32x16 acc[T::MB][T::NB];
#pragma unroll
  for (int i = 0; i < T::MB; ++i)
#pragma unroll
    for (int j = 0; j < T::NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int r32 = lane & 31, g8 = (lane >> 5) * 8;
  const int ra = (wm * T::MW + r32) * LDK + g8, rb = (wn * T::NW + r32) * LDK + g8;
  // Tile kt is multiplied from LDS buffer kt % 2 while tile kt + 1 goes from its register set into the
  // other buffer and tile kt + 1 + PF into that set.  The operands of MFMA step ks + 1 are read from
  // LDS in front of the products of step ks; those of the next tile's first step in front of the last
  // one's, behind the only workgroup barrier of the tile (by then every wavefront has read all of the
  // tile and written its part of the next), which does not wait for the global loads in flight.
  half8 xa[2][T::MB], xb[2][T::NB];
  auto frags = [&](int buf, int ks, int f) {
    const _Float16 *const Ac = pf_lds + buf * TM * LDK, *const Bc = pf_lds + 2 * TM * LDK + buf * TN * LDK;
#pragma unroll
    for (int i = 0; i < T::MB; ++i) xa[f][i] = *(const half8 *)(Ac + ra + i * 32 * LDK + ks * 16);
#pragma unroll
    for (int j = 0; j < T::NB; ++j) xb[f][j] = *(const half8 *)(Bc + rb + j * 32 * LDK + ks * 16);
  };
  auto body = [&](int kt, int u1, bool stage, bool load) {     // u1: the set of tile kt + 1
    const int cur = kt & 1;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      if (ks == 3) lds_barrier();
      if (ks < 3 || stage) frags(ks < 3 ? cur : cur ^ 1, (ks + 1) & 3, (ks + 1) & 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < RA; ++i) {                           // parts 0, 1 | 2 | 3, or 0 | 1
        if (ks != (RA == 2 ? i : i < 1 ? 0 : i - 1)) continue;
        if (stage) stage_part(u1, i, cur ^ 1);
        if (load) load_part(kt + 1 + PF, u1, i);
      }
#pragma unroll
      for (int i = 0; i < T::MB; ++i)
#pragma unroll
        for (int j = 0; j < T::NB; ++j) {
          const half8 &a = xa[ks & 1][i], &b = xb[ks & 1][j];
          acc[i][j] = mfma16(a, b, acc[i][j]);
        }
      // the step's conversions, LDS writes and loads go between its MFMAs, not in front of them
#pragma unroll
      for (int q = 0; q < T::MB * T::NB; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      // one MFMA
        __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);      // VALU
        __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);      // LDS write
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);      // global load
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
#pragma unroll
  for (int u = 0; u < PF; ++u)
    if (u < nk) {
#pragma unroll
      for (int i = 0; i < RA; ++i) load_part(u, u, i);
    }
#pragma unroll
  for (int i = 0; i < RA; ++i) stage_part(0, i, 0);
  if (PF < nk) {
#pragma unroll
    for (int i = 0; i < RA; ++i) load_part(PF, 0, i);
  }
  lds_barrier();
  frags(0, 0, 0);
  int kt = 0;
  for (; kt + 2 * PF < nk; kt += PF) {            // every load of the round exists
#pragma unroll
    for (int u = 0; u < PF; ++u) body(kt + u, (u + 1) % PF, true, true);
  }
#pragma unroll
  for (int u = 0; u < 2 * PF; ++u) {
    if (kt + u >= nk) goto done;
    body(kt + u, (u + 1) % PF, kt + u + 1 < nk, kt + u + 1 + PF < nk);
  }
done:
  if constexpr (EPI == PF_SWIGLU) {
    constexpr int HB = T::NB / 2;
#pragma unroll
    for (int i = 0; i < T::MB; ++i)
#pragma unroll
      for (int j = 0; j < HB; ++j) {
        const int cc = n_tile * (TN / 2) + wn * (T::NW / 2) + j * 32 + r32;
        if (cc < ldc) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int row = m0 + wm * T::MW + i * 32 + c_row(r, lane);
            const float g = acc[i][j][r], v = acc[i][j + HB][r];
            if (row < M) ((_Float16 *)C)[(size_t)row * ldc + cc] = (_Float16)(g / (1.0f + expf(-g)) * v);
          }
        }
      }
  } else {
    float *const out = (float *)C + (size_t)ks_i * M * ldc;
#pragma unroll
    for (int i = 0; i < T::MB; ++i)
#pragma unroll
      for (int j = 0; j < T::NB; ++j) {
        const int cc = n_tile * TN + wn * T::NW + j * 32 + r32;
        if (cc < N) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int row = m0 + wm * T::MW + i * 32 + c_row(r, lane);
            if (row < M) out[(size_t)row * ldc + cc] = acc[i][j][r];
          }
        }
      }
  }
}

// ---- GEMM of few rows
//
// The same product for up to 128 rows.  k_pf_gemm's 128 x 128 tile is bound there by neither the stream nor the
// matrix cores but by the way of a K tile through the registers: load, convert, write to LDS, barrier, read
// (1500 cycles for 128 x 128 x 64, of which 510 with the matrix cores at work, bf16 or codes alike).  Here
//  * A and B go from global memory to LDS directly (buffer loads with the LDS as their destination), without a register:
//    behind the stage at work up to four more are in flight per CU, of bf16 64 KB of weights,
//    of codes 40, 40, 30 and 20 KB with up to 32, 64, 96 and 128 rows;
//  * a tile is 32 MB rows of A (no products for padding rows beyond 31; rows that do not exist are not
//    loaded) x 128 rows of B; each of the eight wavefronts owns 32 rows of B and half of a stage's columns, so
//    that B is converted once, in the registers its product reads it from;
//  * the operands of a stage are read from LDS during the products of the one before; one barrier a stage.
// A stage is 64 columns of bf16, or 128 of codes with their (scale, zero) pairs.  LDS rows are 128 bytes
// of 16-byte pieces (codes: 64), the piece c of row r in place c ^ (r / 2) % 8 (codes: c ^ (r / 4) % 4): the
// 16 lanes that a 16-byte read serves together then touch every bank once (conflicts: 2 % of the LDS cycles with bf16,
// 5 % with codes, whose pairs are read four bytes a lane).
// Measured (us in a prefill of 77 tokens at the 8B shape, 128 x 128 tile and now; bf16 / codes): QKV 18.2 / 16.6 and 15.7 /
// 17.0, O 12.6 / 14.4 and 11.6 / 14.4, gate/up 49.0 / 47.8 and 45.3 / 39.2, down 28.2 / 25.5 and 23.8 / 22.4.  What bounds it now: bf16
// -- the stream at the clock that is left beside the products (1.7 GHz: 5.2 TB/s in gate/up; of 1200 cycles a stage the matrix
// cores work in 380); codes -- nothing alone: of 2200 cycles a stage (counters of a whole launch, its ends taken off) the
// conversions take 820 of a SIMD, the products 770, the loads 1200 of the
// CU's way to the L2 (30 bytes a cycle, also with 8 workgroups on the chip: a workgroup reads all of A).  A launch that
// is short costs 3 us from its start to the first stage and 1 us behind the last one.  Tried: beginning at different
// stages in different workgroups (no change), A kept in tiles of 64 columns (no
// change).
//
// EXACT (short prompts, whose activations stay in 32 bits): dense -- A holds bf16 rows, the three parts of the
// activations one under the other (see split3), multiplied with the bf16 weights as they are, every product exact; codes
// -- A holds fp16 rows, as the decode kernels round them, multiplied with the codes as they are; a K tile's
// sums S and the sum X of its inputs (a product with ones) go into the result as scale (S - zero X) in fp32,
// the form in which the decode kernels take the scale and the zero point.  (The weights as two fp16 numbers, the
// K tiles taken twice, lost bits of weights below 2e-3 and turned those beyond 65504 into NaN; four 8B river
// blocks and 3 tokens took 900 us that way, 379 now.)
//
template <int MB_, bool W4> struct RowsTile {
  static constexpr int MB = MB_, TM = 32 * MB, TN = 128, NT = 512;
  static constexpr int COLS = W4 ? 128 : 64;                     // columns of a stage
  static constexpr int A_BYTES = TM * COLS * 2, CODES = TN * COLS / 2, PAIRS = 2048;
  static constexpr int STAGE = A_BYTES + (W4 ? CODES + PAIRS : TN * COLS * 2);
  static constexpr int S = STAGE * 5 <= 160 * 1024 ? 5 : STAGE * 4 <= 160 * 1024 ? 4 : 3;
  static constexpr int LDR = 136;                                // floats of a row of sums: rows 4 apart, half a wavefront each, do not meet in a bank
  static constexpr int SUMS = 2 * TM * LDR * 4;
  static constexpr int LDS_BYTES = S * STAGE > SUMS ? S * STAGE : SUMS;
  static constexpr int A_ITEMS = A_BYTES / 1024;                 // loads of a wavefront that a stage of A is
  static constexpr int ITEMS = A_ITEMS + 16;                     // ... and B's (codes: 8, their pairs: 8)
  static_assert(LDS_BYTES <= 160 * 1024, "LDS of a CU");
};

// 64 lanes x 16 (4) bytes from rsrc + voff + soff to LDS at lds + 16 (4) * lane.  In assembly, because the
// compiler makes every LDS read wait for all such loads in flight; rows_wait counts them instead.  (m0, which the compiler warns of
// as a reserved register, is written in front of each load and read by nothing else in these kernels.)
template <bool STREAM>
__device__ __forceinline__ void load_lds16(unsigned lds, unsigned voff, const u32x4 &rsrc, unsigned soff) {
  if constexpr (STREAM)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds"
                 :: "s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory", "m0");
}
__device__ __forceinline__ void load_lds4(unsigned lds, unsigned voff, const u32x4 &rsrc, unsigned soff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, %3 offen lds"
               :: "s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory", "m0");
}
// All but this wavefront's N last loads have landed and its LDS operations are done; then the workgroup.
template <int N>
__device__ __forceinline__ void rows_wait() {
  static_assert(N < 64, "six bits");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(N) : "memory");
}
// ... the loads of `later` stages, N of them each (at most MOST stages)
template <int N, int MOST>
__device__ __forceinline__ void rows_wait_stages(int later) {
  if constexpr (MOST > 0) {
    if (later >= MOST) rows_wait<N * MOST>();
    else rows_wait_stages<N, MOST - 1>(later);
  } else {
    rows_wait<0>();
  }
}
__device__ __forceinline__ u32x4 uniform_rsrc(const void *p) {
  const uint64_t a = (uint64_t)p;
  return u32x4{(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a),
               (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xffffu)), 0x7ffffff0u, 0x00020000u};
}

// Row r of B's tile -> matrix and row, for `run` rows that start at r (8, or 16 of codes).  SwiGLU: 16 rows of the
// gate and 16 of the up matrix in turn, so that lanes l and l + 16 of a wavefront hold the factors of an output.
template <int EPI>
__device__ __forceinline__ void rows_b_row(const GemmB &B, int n_tile, int r, int run, int N, int &mat, int &row) {
  if constexpr (EPI == PF_SWIGLU) {
    mat = (r >> 4) & 1;
    row = min(n_tile * 64 + (r >> 5) * 16 + (r & 15), B.rows[0] - run);
  } else {
    gemm_b_row(B, min(n_tile * 128 + r, N - run), N, mat, row);
  }
}

// How the host deals a product out (no division in front of the first load): one workgroup per (tile of N, slice of K).
constexpr int kRowsMost = 128;  // rows of A that one tile takes
struct RowsDeal {
  int rows32;                 // rows that exist of every 32 (short prompts; else 32)
  int n_tiles, k_split;
  uint32_t split_inv;         // ceil(2^32 / k_split) (k_split = 1: not used): workgroup / k_split is a high product
  int st_base, st_rem;        // stages of a slice: st_base, and one more for the first st_rem
};
template <int MB, bool W4, int EPI, bool EXACT>
__global__ __launch_bounds__(512, 1) void k_pf_gemm_rows(const _Float16 *__restrict__ A, int lda, GemmB B, int N, int K,
                                                         int group, void *C, int ldc, int M, RowsDeal deal) {
  typedef RowsTile<MB, W4> T;
  constexpr bool FOLD = EXACT && W4;
  constexpr int S = T::S, KS = W4 ? 4 : 2;                      // MFMA steps of a wavefront per stage
  constexpr int NJ = (T::ITEMS + 7) / 8, ODD = T::ITEMS % 8;    // loads per wavefront and stage (ODD: the first ODD wavefronts')
  extern __shared__ __attribute__((aligned(16))) char rows_lds[];
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char *)rows_lds;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nb = wv & 3, half = wv >> 2;                        // its rows of B, its half of a stage's columns
  const int col = blockIdx.x;
  if (col >= deal.n_tiles * deal.k_split) return;
  const int n_tile = deal.k_split == 1 ? col : (int)__umulhi((uint32_t)col, deal.split_inv), ks_i = col - n_tile * deal.k_split;
  const int st0 = ks_i * deal.st_base + min(ks_i, deal.st_rem), ns = deal.st_base + (ks_i < deal.st_rem ? 1 : 0);

  // what this wavefront loads per stage: item wv + 8 j = 1 KB of the stage (A's rows, B's rows; the pairs last)
  u32x4 rs[NJ];
  unsigned vo[NJ];
  const int gpr = W4 ? (K + group - 1) / group : 0;
  int g_at = 0, g_left = 0;                                     // this lane's (scale, zero) pair of the next stage
  const int tpg = W4 ? group / 64 : 1, pair_half = lane & 1;
  if constexpr (W4) {                                           // (counted on from there, no division per stage)
    g_at = st0 ? (2 * st0 + pair_half) / tpg : tpg == 1 ? pair_half : 0;
    g_left = tpg - (2 * st0 + pair_half - g_at * tpg);
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int it = wv + 8 * j;
    if (it < T::A_ITEMS) {
      const int sub = it / (4 * MB), r = (it % (4 * MB)) * 8 + (lane >> 3);         // W4: two tiles of 64 columns
      const int piece = (lane & 7) ^ ((r >> 1) & 7);
      rs[j] = uniform_rsrc((const char *)A + (size_t)st0 * T::COLS * 2);
      // (rows that do not exist lie beyond the descriptor's range: zero, without an access)
      vo[j] = r < M && (!EXACT || (r & 31) < deal.rows32) ? (unsigned)r * (unsigned)lda * 2u + sub * 128 + piece * 16 : 0xc0000000u;
    } else if (!W4) {
      const int r0 = (it - T::A_ITEMS) * 8, r = r0 + (lane >> 3), piece = (lane & 7) ^ ((r >> 1) & 7);
      int mat, row;
      rows_b_row<EPI>(B, n_tile, min(r0, 120), 8, N, mat, row);
      rs[j] = uniform_rsrc((const char *)B.w[mat] + ((size_t)row * K + (size_t)st0 * 64) * 2);
      vo[j] = (unsigned)(lane >> 3) * (unsigned)K * 2u + piece * 16;
    } else {
      const int q = (it - T::A_ITEMS) & 7;
      int mat, row;
      rows_b_row<EPI>(B, n_tile, q * 16, 16, N, mat, row);
      if (it < T::A_ITEMS + 8) {                                // 16 rows x 64 bytes of codes
        const int r = lane >> 2, piece = (lane & 3) ^ ((r >> 2) & 3);
        rs[j] = uniform_rsrc((const char *)B.w[mat] + (size_t)row * (K >> 1) + (size_t)st0 * 64);
        vo[j] = (unsigned)r * (unsigned)(K >> 1) + piece * 16;
      } else {                                                  // their pairs: lane -> row lane / 2 % 16, 64 columns lane % 2
        rs[j] = uniform_rsrc((const char *)B.sz[mat] + (size_t)row * gpr * 4);
        vo[j] = (unsigned)((lane >> 1) & 15) * (unsigned)gpr * 4u;
      }
    }
  }
  int at = 0;                                                   // the next stage to load
  // the slice's last stage has 64 columns only
  const bool ragged = W4 && (K & 64) && ks_i == deal.k_split - 1;
  auto issue_as = [&](int buf, auto last) {                     // last: of a ragged row (codes)
    constexpr bool CUT = decltype(last)::value;
    const unsigned dst = lds0 + (unsigned)buf * T::STAGE;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int it = wv + 8 * j;
      if (ODD && j == NJ - 1 && wv >= ODD) continue;
      if (W4 && j == NJ - 1) {                                  // (codes: whole rounds of eight; the last one is the pairs)
        load_lds4(dst + T::A_BYTES + T::CODES + wv * 256, vo[j] + (unsigned)min(g_at, gpr - 1) * 4u, rs[j], 0);
        continue;
      }
      unsigned v = vo[j];
      if constexpr (CUT) {                                      // pieces beyond the row: its last 64 columns again
        if (j < MB) v -= it >= 4 * MB ? 128u : 0u;
        else v -= (v - (unsigned)(lane >> 2) * (unsigned)(K >> 1)) & 32u;
      }
      const unsigned along = (unsigned)at * (W4 && j >= MB ? 64u : T::COLS * 2u);          // columns, of codes or 16 bits
      // (streamed past the caches where all of a round is B's: this workgroup is the only reader of its rows)
      if (8 * j >= T::A_ITEMS) load_lds16<true>(dst + it * 1024u, v, rs[j], along);
      else load_lds16<false>(dst + it * 1024u, v, rs[j], along);
    }
  };
  auto issue = [&](int buf) {                                   // the next stage of the slice into LDS buffer buf
    if (W4 && ragged && at == ns - 1) issue_as(buf, IC<1>{});
    else issue_as(buf, IC<0>{});
    if constexpr (W4) {                                         // (two steps of 64 columns)
      g_left -= 2;
      if (g_left <= 0) { g_left += tpg; ++g_at; }
      if (g_left <= 0) { g_left += tpg; ++g_at; }
    }
    ++at;
  };
  // all loads of stage s have landed, everybody's reads of stage s - 1 are done (`later` stages are in flight behind it)
  auto landed = [&](int later) {
    if constexpr (ODD) {
      if (wv < ODD) rows_wait_stages<NJ, S - 1>(later);
      else rows_wait_stages<NJ - 1, S - 1>(later);
    } else {
      rows_wait_stages<NJ, S - 1>(later);
    }
  };

  f32x16 acc[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;

  // Operands: lane (r32, g) of step ks reads piece ks * 2 + g of a 64-column row, ks = 2 half, 2 half + 1; codes:
  // columns 32 g + 8 ks .. + 7 of this half's 64, piece 4 g + ks of A, word ks of its 16-byte piece of codes.
  const int r32 = lane & 31, g = lane >> 5, sx = (r32 >> 1) & 7;
  unsigned pa[KS];
#pragma unroll
  for (int k = 0; k < KS; ++k)
    pa[k] = r32 * 128u + (((W4 ? 4 * g + k : (2 * half + k) * 2 + g) ^ sx) * 16u) + (W4 ? half * (MB * 4096u) : 0u);
  const unsigned pc = T::A_BYTES + (nb * 32 + r32) * 64u + (((2 * half + g) ^ ((r32 >> 2) & 3)) * 16u);
  const unsigned pz = T::A_BYTES + T::CODES + (2 * nb + (r32 >> 4)) * 256u + (r32 & 15) * 8u + half * 4u;
  half8 xa[2][KS][MB], xb[2][W4 ? 1 : KS];
  uint32_t sz[2];
  auto frags = [&](unsigned at, int f) {
    const char *const b = rows_lds + at;
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      if constexpr (!W4) xb[f][k] = *(const half8 *)(b + T::A_BYTES + nb * 4096 + pa[k]);
      else if (k == 0) { xb[f][0] = *(const half8 *)(b + pc); sz[f] = *(const uint32_t *)(b + pz); }
#pragma unroll
      for (int i = 0; i < MB; ++i) xa[f][k][i] = *(const half8 *)(b + pa[k] + i * 4096);
    }
  };
  // step k of stage set f: B's operand as the product wants it
  auto operand = [&](int f, int k) -> half8 {
    if constexpr (W4) {
      const u32x4 w4 = __builtin_bit_cast(u32x4, xb[f][0]);
      const uint32_t w = k == 0 ? w4.x : k == 1 ? w4.y : k == 2 ? w4.z : w4.w;
      return FOLD ? codes8(w) : dequant8(w, bf16_lo(sz[f]), bf16_hi(sz[f]));
    } else {
      const u32x4 v = __builtin_bit_cast(u32x4, xb[f][k]);
      return EXACT ? xb[f][k] : bf16x8_to_half8(make_uint4(v.x, v.y, v.z, v.w));
    }
  };
  // The products of set f, beside each step's the conversion of the next one's operand (the last step: of set f ^ 1's
  // first): two wavefronts share a SIMD and come out of the same barrier, so that one's conversions do not by
  // themselves fall into the other's products.
  half8 b;
  auto products = [&](int f, bool more) {
    f32x16 part[FOLD ? MB : 1], xsum[FOLD ? MB : 1];
    const half8 ones = (half8)(_Float16)1.f;
    const float s = bf16_lo(sz[f]), z = bf16_hi(sz[f]);
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      half8 nx = b;
      if (k + 1 < KS) nx = operand(f, k + 1);
      else if (more) nx = operand(f ^ 1, 0);
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        if constexpr (FOLD) {
          part[i] = mfma16(xa[f][k][i], b, k ? part[i] : f32x16{});
          xsum[i] = mfma16(xa[f][k][i], ones, k ? xsum[i] : f32x16{});
        } else {
          acc[i] = EXACT ? mfma16_bf16(xa[f][k][i], b, acc[i]) : mfma16(xa[f][k][i], b, acc[i]);
        }
      }
      if constexpr (!EXACT) {
#pragma unroll
        for (int q = 0; q < MB; ++q) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                    // one MFMA
          __builtin_amdgcn_sched_group_barrier(0x002, (20 + MB - 1) / MB, 0);   // VALU
        }
      }
      b = nx;
    }
    if constexpr (FOLD) {
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = fmaf(s, fmaf(-z, xsum[i][r], part[i][r]), acc[i][r]);
    }
  };

#pragma unroll
  for (int s = 0; s < S; ++s)
    if (s < ns) issue(s);
  landed(min(ns - 1, S - 1));
  frags(0, 0);
  int buf = 0;                                                   // buffer of the stage at work
  auto body = [&](int s, int f) {                                // (s + 1 < ns: no LDS read behind a branch, whose end would wait for all)
    const int next = buf + 1 == S ? 0 : buf + 1;
    if (s + S <= ns) landed(S - 2);
    else landed(ns - 2 - s);
    frags(next * T::STAGE, f ^ 1);
    __builtin_amdgcn_sched_barrier(0);
    if (s + S < ns) issue(buf);
    __builtin_amdgcn_sched_barrier(0);
    products(f, true);
    __builtin_amdgcn_sched_barrier(0);
    buf = next;
  };
  b = operand(0, 0);
  const bool live = !(ragged && half);                           // (of the last stage: its second half does not exist)
  int s = 0;
  for (; s + 2 < ns; s += 2) { body(s, 0); body(s + 1, 1); }
  if (s + 1 < ns) {
    body(s, 0);
    if (live) products(1, false);
  } else if (live) {
    products(0, false);
  }

  // The halves' sums meet in LDS, row-major, and leave in 16-byte stores.  (A loop, not unrolled: a launch fetches its
  // code from the caches anew, and the sums of every register in their own instructions were most of it.)
  constexpr int LDR = T::LDR;
  rows_wait<0>();
  {
    float *const mine = (float *)rows_lds + (half * T::TM + (lane >> 5) * 4) * LDR + nb * 32 + r32;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) mine[(i * 32 + (r >> 2) * 8 + (r & 3)) * LDR] = acc[i][r];
  }
  lds_barrier();
  const float *const sums = (const float *)rows_lds;
  auto sum4 = [&](int row, int c) {
    const f32x4 p = *(const f32x4 *)(sums + row * LDR + c), q = *(const f32x4 *)(sums + (T::TM + row) * LDR + c);
    return p + q;
  };
  if constexpr (EPI == PF_SWIGLU) {
#pragma unroll 1
    for (int e = tid; e < T::TM * 16; e += 512) {                // four outputs: 16 columns of gate, then of up, per wavefront's 32
      const int row = e >> 4, c = (e & 15) * 4, at = (c >> 4) * 32 + (c & 15), cc = n_tile * 64 + c;
      if (row >= M || cc >= ldc) continue;
      const f32x4 gt = sum4(row, at), up = sum4(row, at + 16);
      half4 o;
#pragma unroll
      for (int q = 0; q < 4; ++q) o[q] = (_Float16)(gt[q] / (1.0f + expf(-gt[q])) * up[q]);
      *(half4 *)((_Float16 *)C + (size_t)row * ldc + cc) = o;
    }
  } else {
    float *const out = (float *)C + (size_t)ks_i * M * ldc;
#pragma unroll 1
    for (int e = tid; e < T::TM * 32; e += 512) {
      const int row = e >> 5, c = (e & 31) * 4, cc = n_tile * 128 + c;
      if (row < M && cc < N) *(f32x4 *)(out + (size_t)row * ldc + cc) = sum4(row, c);
    }
  }
}

// ------------------------------------------------------- element-wise kernels
//
// Bound by the stream of their operands; one workgroup of 256 per token, 16 bytes and more per lane
// and load.  Partial sums of a K-sliced GEMM (planes of [m, columns], see k_pf_gemm) are added here,
// in slice order, by the kernel that consumes the sum anyway.

struct Run8 { float v[8]; };
__device__ __forceinline__ Run8 ld_run8(const float *p) {
  const float4 a = *(const float4 *)p, b = *(const float4 *)(p + 4);
  return Run8{{a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w}};
}
__device__ __forceinline__ void st_run8(float *p, const Run8 &x) {
  *(float4 *)p = make_float4(x.v[0], x.v[1], x.v[2], x.v[3]);
  *(float4 *)(p + 4) = make_float4(x.v[4], x.v[5], x.v[6], x.v[7]);
}
__device__ __forceinline__ Run8 ld_run8_16(const void *p, size_t i) {       // eight bf16 values
  float f[8];
  const u32x4 w = *RIVER_GLOBAL(u32x4, (const char *)p + i * 2);
  Store<1>::unpack(w, f);
  return Run8{{f[0], f[1], f[2], f[3], f[4], f[5], f[6], f[7]}};
}

// eight norm gains; wide: the pointer is 16-byte aligned (the final norm's need not be)
__device__ __forceinline__ Run8 ld_gain8(const void *gain, int k, bool wide) {
  if (wide) return ld_run8_16(gain, k);
  Run8 x;
  for (int e = 0; e < 8; ++e) x.v[e] = Store<1>::ld(gain, k + e);
  return x;
}
// f(element, exists) for every one of n planes, in order, the loads of up to MOST together (one, four or eight
// by what is left: an element beyond the last plane is plane 0's again, for f to leave out)
template <int U, class F>
__device__ __forceinline__ void add_some_planes(const float *p, size_t stride, int j, int n, F f) {
#pragma unroll
  for (int u = 0; u < U; ++u) f(p + (j + u < n ? (size_t)(j + u) * stride : 0), j + u < n);
}
template <int MOST = 8, class F>
__device__ __forceinline__ void add_planes(const float *p, size_t stride, int n, F f) {
  if (n == 1) {
    add_some_planes<1>(p, stride, 0, n, f);
  } else if constexpr (MOST == 4) {                            // (no choice in the loop: the 24 planes of a short prompt's norm 7.6 us, with it 9.4)
    for (int j = 0; j < n; j += 4) add_some_planes<4>(p, stride, j, n, f);
  } else {
    for (int j = 0; j < n; j += 8) {
      if (n - j > 4) add_some_planes<8>(p, stride, j, n, f);
      else add_some_planes<4>(p, stride, j, n, f);
    }
  }
}

// The residual stream in front of a norm, and the norm: h[t, :] = E[token[t], :] (tokens given: block
// 1's first norm) or h[t, :] += the n_part partial sums of the GEMM in front; x16[t, :] =
// fp16(h[t, :] * rsqrt(mean(h[t, :]^2) + eps) * gain) (x16 null: no norm, the last block's sums only).
// One workgroup per row, rows t0 .. t0 + gridDim.x - 1, which the planes hold from their row 0 on.
// row_out: the row of the last prompt position (t == row_t) is also kept there, the debug view of
// h(0..L) and the head's input.  d % 8 == 0, rows 16-byte aligned.  A row of up to 8192 columns is
// read once and kept in registers between the reduction and the scaling.  256 threads, or 512 for few
// rows, which then leave CUs idle (the host chooses).  plane_rows: rows of a plane.  SPLIT (short prompts): the
// norm is stored as its three bf16 parts, kShort rows below each other (see split3).
constexpr int kNormKeep = 4;
constexpr int kShort = 32;             // rows of a pass over a short prompt
template <bool SPLIT>
__global__ __launch_bounds__(512) void k_pf_norm(float *__restrict__ h, const int *__restrict__ tokens,
                                                 const void *tok_emb, const float *__restrict__ part, int n_part,
                                                 int plane_rows, const void *gain, int d, float eps, _Float16 *x16,
                                                 float *row_out, int row_t, int t0) {
  __shared__ float red[16];
  const int t = t0 + blockIdx.x;
  float *const row = h + (size_t)t * d;
  float *const keep_row = t == row_t ? row_out : nullptr;
  const size_t emb = tokens ? (size_t)tokens[t] * d : 0;
  const bool emb_wide = ((uintptr_t)tok_emb & 15) == 0;        // (the embedding may have any alignment)
  float ss = 0.f;
  auto take = [&](int k) {
    Run8 x;
    if (tokens && emb_wide) {
      x = ld_run8_16(tok_emb, emb + k);
    } else if (tokens) {
      for (int e = 0; e < 8; ++e) x.v[e] = Store<1>::ld(tok_emb, emb + k + e);
    } else {
      x = ld_run8(row + k);
      add_planes<4>(part + (size_t)blockIdx.x * d + k, (size_t)plane_rows * d, n_part, [&](const float *p, bool ok) {
        const Run8 q = ld_run8(p);
#pragma unroll
        for (int e = 0; e < 8; ++e) x.v[e] += ok ? q.v[e] : 0.f;
      });
    }
    if (tokens || n_part) st_run8(row + k, x);
    if (keep_row) st_run8(keep_row + k, x);
#pragma unroll
    for (int e = 0; e < 8; ++e) ss = fmaf(x.v[e], x.v[e], ss);
    return x;
  };
  // (the gains are fetched with the row: behind the reduction they are one more round trip)
  Run8 keep[kNormKeep], kg[kNormKeep];
#pragma unroll
  for (int i = 0; i < kNormKeep; ++i) {
    const int k = threadIdx.x * 8 + i * (int)blockDim.x * 8;
    if (k < d && x16) kg[i] = ld_run8_16(gain, k);
    if (k < d) keep[i] = take(k);
  }
  for (int k = threadIdx.x * 8 + kNormKeep * (int)blockDim.x * 8; k < d; k += (int)blockDim.x * 8) (void)take(k);
  if (!x16) return;
  const float r = 1.0f / sqrtf(block_sum(ss, red) / (float)d + eps);
  auto put = [&](int k, const Run8 &x, const Run8 &g) {
    float v[8];
    half8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = x.v[e] * r * g.v[e];
    if constexpr (SPLIT) {
      store_split3((uint16_t *)x16 + (size_t)t * d + k, (size_t)kShort * d, v);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = (_Float16)v[e];
      *(half8 *)(x16 + (size_t)t * d + k) = o;
    }
  };
#pragma unroll
  for (int i = 0; i < kNormKeep; ++i) {
    const int k = threadIdx.x * 8 + i * (int)blockDim.x * 8;
    if (k < d) put(k, keep[i], kg[i]);
  }
  for (int k = threadIdx.x * 8 + kNormKeep * (int)blockDim.x * 8; k < d; k += (int)blockDim.x * 8) put(k, ld_run8(row + k), ld_run8_16(gain, k));   // (this thread's own)
}

// RoPE on q and k at position pos0 + t; q scaled by log2(e) / sqrt(hd) and stored as fp16 for
// the attention kernel; k (rotated) and v rounded to the cache dtype and written to slot
// (l, pos0 + t) of the shared cache.  qkv: n_part fp32 planes [m, qd + 2 kvd] of the QKV GEMM, added
// in order.  A thread has one item of a token: four rotation pairs (i, i + hd/2) of one head, or four columns of
// v; grid (m, items / 256).  (One workgroup of 512 per token, two or three items a thread one after the
// other: 7.1 us for 77 tokens of the 8B shape with five planes and 30 for 4096 with one, now 4.8 and 25.)
// m: rows of a plane.  Q32: q in fp32 (short prompts).
template <bool Q32>
__global__ __launch_bounds__(256) void k_pf_rope_store(const float *__restrict__ qkv, int n_part, int m,
                                                       const float2 *__restrict__ rope, int nq, int nkv, int hd, int pos0,
                                                       int l, int max_seq, void *kcache, void *vcache, int kv_f16,
                                                       _Float16 *q16) {
  const int t = blockIdx.x, p = pos0 + t, half = hd >> 1, per = half >> 2;
  const int qd = nq * hd, kvd = nkv * hd, ld = qd + 2 * kvd;
  const float qs = 1.4426950408889634f / sqrtf((float)hd);
  auto get = [&](int c) {
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
    add_planes(qkv + (size_t)t * ld + c, (size_t)m * ld, n_part, [&](const float *p, bool ok) {
      const float4 b = *(const float4 *)p;
      a.x += ok ? b.x : 0.f; a.y += ok ? b.y : 0.f; a.z += ok ? b.z : 0.f; a.w += ok ? b.w : 0.f;
    });
    return a;
  };
  auto to_cache = [&](void *cache, size_t i, float x, float y, float z, float w) {
    u32x2 v;
    if (kv_f16) {
      v.x = __builtin_bit_cast(uint32_t, half2v{(_Float16)x, (_Float16)y});
      v.y = __builtin_bit_cast(uint32_t, half2v{(_Float16)z, (_Float16)w});
    } else {
      v.x = (uint32_t)Store<1>::rne(x) | (uint32_t)Store<1>::rne(y) << 16;
      v.y = (uint32_t)Store<1>::rne(z) | (uint32_t)Store<1>::rne(w) << 16;
    }
    *(u32x2 *)((char *)cache + i * 2) = v;
  };
  const int i = blockIdx.y * 256 + threadIdx.x, pairs = (nq + nkv) * per;
  if (i < pairs) {
    const int head = i / per, e = (i % per) * 4;
    const float4 c01 = *(const float4 *)(rope + (size_t)p * half + e), c23 = *(const float4 *)(rope + (size_t)p * half + e + 2);
    const float4 a = get(head * hd + e), b = get(head * hd + e + half);     // q heads, then k heads: contiguous in qkv
    const float lo[4] = {a.x * c01.x - b.x * c01.y, a.y * c01.z - b.y * c01.w, a.z * c23.x - b.z * c23.y, a.w * c23.z - b.w * c23.w};
    const float hi[4] = {a.x * c01.y + b.x * c01.x, a.y * c01.w + b.y * c01.z, a.z * c23.y + b.z * c23.x, a.w * c23.w + b.w * c23.z};
    if (Q32 && head < nq) {
      float *const q = (float *)q16 + (size_t)t * qd + head * hd + e;
      *(float4 *)q = make_float4(lo[0] * qs, lo[1] * qs, lo[2] * qs, lo[3] * qs);
      *(float4 *)(q + half) = make_float4(hi[0] * qs, hi[1] * qs, hi[2] * qs, hi[3] * qs);
    } else if (head < nq) {
      half4 ql, qh;
#pragma unroll
      for (int j = 0; j < 4; ++j) { ql[j] = (_Float16)(lo[j] * qs); qh[j] = (_Float16)(hi[j] * qs); }
      _Float16 *const q = q16 + (size_t)t * qd + head * hd + e;
      *(half4 *)q = ql;
      *(half4 *)(q + half) = qh;
    } else {
      const size_t o = ((size_t)l * max_seq + p) * kvd + (size_t)(head - nq) * hd + e;
      to_cache(kcache, o, lo[0], lo[1], lo[2], lo[3]);
      to_cache(kcache, o + half, hi[0], hi[1], hi[2], hi[3]);
    }
  }
  const int c = (i - pairs) * 4;
  if (c >= 0 && c < kvd) {
    const float4 v = get(qd + kvd + c);
    to_cache(vcache, ((size_t)l * max_seq + p) * kvd + c, v.x, v.y, v.z, v.w);
  }
}

// ------------------------------------------------------------- attention
//
// Causal attention of the chunk's queries (positions pos0 .. pos0 + m - 1) over cache
// positions 0 .. their own.  One workgroup of eight wavefronts per (kv head, HG of its query heads,
// QT = 256 / HG queries), 32 queries of one head per wavefront: the heads that share K and V share
// their staging, which for a bf16 cache is a conversion (HG = 4: half as much of it per product as
// with one head and 128 queries).  Keys in tiles of 64 through two LDS buffers: the next tile's rows
// are fetched while a tile is multiplied and written to the other buffer behind it, one barrier per
// tile.  Transposed products, so that the softmax over keys runs along a lane's registers and the
// probabilities feed the second product from the registers they are in:
//   S^T[key, q] = K[key, :] . Q[q, :]        A = K tile rows (LDS), B = Q (registers, whole loop)
//   O^T[d, q]  += V^T[d, key] P^T[key, q]    A = V tile stored transposed (LDS), B = P^T (registers)
// In S^T's register layout lane l holds, for query l % 32, keys (r/4)*8 + (l/32)*4 + r%4: the
// eight keys of registers 0..7 (8..15) are the K slots of that lane group in the first
// (second) MFMA of a 32-key block; V^T keeps the keys of a lane group next to each other (the middle
// two quadruples of every 16 keys swapped), so that its operand is one 16-byte read.
// The scores carry log2(e)/sqrt(hd) (folded into q16): base-2 online softmax.  Bound by the matrix
// cores and, per tile about as long, the vector units (32 exponentials per lane beside the 32 MFMAs).
// Key 0 is visible to every query, so the running maximum is a real score after the first tile.
// KS = 2 (few workgroups): a step is two tiles of 64 keys, and two wavefronts share 32 queries, one tile of a step
// each; half as many queries per workgroup, twice the workgroups, half as many steps one after the other.  Their two
// softmaxes meet in LDS behind the loop (figures and the line between the two: launch_attn_t).
template <int HD, int HG, int KS>
__global__ __launch_bounds__(512, 1) void k_pf_attn(const _Float16 *__restrict__ q16, const void *kcache,
                                                    const void *vcache, int kv_f16, int nq, int nkv, int l, int max_seq,
                                                    int pos0, int m, _Float16 *o16) {
  constexpr int LDH = HD + 8;                 // K tile row stride (halfs)
  constexpr int LDV = 64 + 8;                 // V^T tile row stride (halfs)
  constexpr int QT = 256 / HG / KS, KT = 64 * KS;               // queries per workgroup, keys of a step
  constexpr int NK = KT * HD / 8 / 512;       // 16-byte K segments per thread
  constexpr int NV = (KT / 2 * HD / 8 + 511) / 512;             // ... pairs of V segments
  extern __shared__ __attribute__((aligned(16))) _Float16 attn_lds[];
  auto Ks = [&](int buf, int tile) { return attn_lds + (buf * KS + tile) * (64 * LDH); };
  auto Vt = [&](int buf, int tile) { return attn_lds + 2 * KS * 64 * LDH + (buf * KS + tile) * (HD * LDV); };
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  // (the kv head changes fastest: with eight of them every XCD's L2 sees the K and V of one)
  const int kvh = blockIdx.x % nkv, h = kvh * (nq / nkv) + (blockIdx.x / nkv) * HG + wv % HG;
  const int qt = (int)(gridDim.y - 1 - blockIdx.y) * QT;    // the longest rows first
  const int q0 = qt + (wv / HG / KS) * 32;                  // first query (chunk-relative) of this wavefront
  const int part = KS == 1 ? 0 : wv / HG % KS;              // its tile of a step
  const int r32 = lane & 31, g = lane >> 5;
  const int qd = nq * HD, kvd = nkv * HD;
  const int tq = min(q0 + r32, m - 1);                      // this lane's query row (clamped: rows >= m are don't-care)
  const int my_pos = pos0 + q0 + r32;                       // its position (unclamped: masks keys beyond it)

  // Q of this wavefront as the B operand of S^T: for K step ks lane group g holds
  // d = ks*16 + g*8 .. +7 of query l % 32
  half8 qb[HD / 16];
#pragma unroll
  for (int ks = 0; ks < HD / 16; ++ks)
    qb[ks] = *(const half8 *)(q16 + (size_t)tq * qd + h * HD + ks * 16 + g * 8);

  f32x16 oacc[HD / 32];
#pragma unroll
  for (int b = 0; b < HD / 32; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[b][r] = 0.f;
  float mrun = -1.0e30f, lrun = 0.f;                        // lrun: this lane group's keys only

  const int last_pos = min(pos0 + qt + QT - 1, pos0 + m - 1);   // last key any query here attends
  const size_t cbase = (size_t)l * max_seq * kvd + (size_t)kvh * HD;
  // A key tile on its way: K rows as 16-byte segments along d; of V two neighbouring keys' segments
  // per thread, which leave as eight 4-byte writes into the transposed tile.
  constexpr int VP = 32 * HD / 8;                           // ... of a tile of 64 keys
  const int v_key = 2 * (tid & 31);
  const int v_at = (v_key & ~15) + (((v_key >> 2) & 1) << 3) + (((v_key >> 3) & 1) << 2) + (v_key & 3);
  u32x4 fk[NK], fv[NV][2];
  auto fetch = [&](int kt) {
#pragma unroll
    for (int i = 0; i < NK; ++i) {
      const int seg = tid + 512 * i, key = seg / (HD / 8), ds = seg % (HD / 8);
      fk[i] = *RIVER_GLOBAL(u32x4, (const char *)kcache + (cbase + (size_t)min(kt + key, last_pos) * kvd + ds * 8) * 2);
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int idx = tid + 512 * i, tile = idx / VP, ds = idx % VP / 32;         // (uniform per wavefront)
      if (tile < KS) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
          fv[i][j] = *RIVER_GLOBAL(u32x4, (const char *)vcache + (cbase + (size_t)min(kt + tile * 64 + v_key + j, last_pos) * kvd + ds * 8) * 2);
      }
    }
  };
  auto stage = [&](int buf) {
#pragma unroll
    for (int i = 0; i < NK; ++i) {
      const int seg = tid + 512 * i, key = seg / (HD / 8), ds = seg % (HD / 8);
      const u32x4 w = fk[i];
      *(half8 *)(Ks(buf, key >> 6) + (key & 63) * LDH + ds * 8) = cache_half8(make_uint4(w.x, w.y, w.z, w.w), kv_f16);
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int idx = tid + 512 * i, tile = idx / VP, ds = idx % VP / 32;
      if (tile < KS) {
        const u32x4 w0 = fv[i][0], w1 = fv[i][1];
        const half8 a = cache_half8(make_uint4(w0.x, w0.y, w0.z, w0.w), kv_f16), b = cache_half8(make_uint4(w1.x, w1.y, w1.z, w1.w), kv_f16);
        _Float16 *const dst = Vt(buf, tile) + ds * 8 * LDV + v_at;
#pragma unroll
        for (int e = 0; e < 8; ++e) *(half2v *)(dst + e * LDV) = half2v{a[e], b[e]};
      }
    }
  };
  fetch(0);
  stage(0);
  lds_barrier();
  int buf = 0;
  for (int kt0 = 0; kt0 <= last_pos; kt0 += KT, buf ^= 1) {
    const bool more = kt0 + KT <= last_pos;
    if (more) fetch(kt0 + KT);
    const int kt = kt0 + part * 64;                          // this wavefront's tile
    const _Float16 *const Kt = Ks(buf, part), *const Vp = Vt(buf, part);
    // wavefronts without queries, and those whose queries all lie before this tile, have nothing to add
    if (q0 < m && kt <= pos0 + q0 + 31) {
      // S^T for the two 32-key blocks of the tile
      f32x16 s[2];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[kb][r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < HD / 16; ++ks)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
          const half8 ka = *(const half8 *)(Kt + (kb * 32 + r32) * LDH + ks * 16 + g * 8);
          s[kb] = mfma16(ka, qb[ks], s[kb]);
        }
      if (kt + 63 > pos0 + q0) {                             // the tile reaches beyond the first query: mask
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (kt + kb * 32 + c_row(r, lane) > my_pos) s[kb][r] = -1.0e30f;
      }
      // running maximum over the lane's 32 keys and the other lane group's 32
      float mx = s[0][0];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kb][r]);
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      if (__any(mx > mrun)) {                                // (lanes whose maximum stays multiply by one)
        mx = fmaxf(mx, mrun);
        const float corr = __builtin_amdgcn_exp2f(mrun - mx);
        mrun = mx;
        lrun *= corr;
#pragma unroll
        for (int b = 0; b < HD / 32; ++b)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[b][r] *= corr;
      }
      half8 pb[2][2];                                        // [key block][MFMA of the block]: B operands
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
          const half2v p = {(_Float16)__builtin_amdgcn_exp2f(s[kb][r] - mrun), (_Float16)__builtin_amdgcn_exp2f(s[kb][r + 1] - mrun)};
          pb[kb][r >> 3][r & 7] = p[0];
          pb[kb][r >> 3][(r & 7) + 1] = p[1];
          // the sum of what is actually multiplied, in fp32
          lrun = __builtin_amdgcn_fdot2(p, half2v{(_Float16)1.f, (_Float16)1.f}, lrun, false);
        }
      // O^T += V^T P^T: per 32-key block two MFMAs
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int b = 0; b < HD / 32; ++b) {
            const half8 va = *(const half8 *)(Vp + (b * 32 + r32) * LDV + kb * 32 + j * 16 + g * 8);
            oacc[b] = mfma16(va, pb[kb][j], oacc[b]);
          }
    }
    if (more) stage(buf ^ 1);
    lds_barrier();
  }
  // O^T[d, q] / l -> o16[q, h*HD + d]; registers 4i .. 4i+3 are four consecutive d
  lrun += __shfl_xor(lrun, 32);
  constexpr int NB = HD / 32 / KS;                          // blocks of 32 d that this wavefront finishes: part * NB on
  if constexpr (KS == 2) {
    // (the other wavefront of these queries: HG wavefronts on or back.  Keys a query does not see at all
    // leave a maximum of -1e30, whose weight is 0 beside the first tile's.)
    f32x4 *const box = (f32x4 *)attn_lds;
    float *const ml = (float *)(box + 8 * NB * 4 * 64);
    const int other = part ? wv - HG : wv + HG;
    auto give = [&](auto O) {                               // the other's blocks
      constexpr int b0 = decltype(O)::value * NB;
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          box[((wv * NB + b) * 4 + i) * 64 + lane] = f32x4{oacc[b0 + b][4 * i], oacc[b0 + b][4 * i + 1], oacc[b0 + b][4 * i + 2], oacc[b0 + b][4 * i + 3]};
    };
    if (part) give(IC<0>{});
    else give(IC<1>{});
    ml[wv * 128 + lane] = mrun;
    ml[wv * 128 + 64 + lane] = lrun;
    lds_barrier();
    const float m2 = ml[other * 128 + lane], l2 = ml[other * 128 + 64 + lane], mx = fmaxf(mrun, m2);
    const float c1 = __builtin_amdgcn_exp2f(mrun - mx), c2 = __builtin_amdgcn_exp2f(m2 - mx);
    lrun = lrun * c1 + l2 * c2;
    auto take = [&](auto P) {
      constexpr int b0 = decltype(P)::value * NB;
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const f32x4 p = box[((other * NB + b) * 4 + i) * 64 + lane];
          oacc[b][4 * i] = oacc[b0 + b][4 * i] * c1 + p.x * c2;
          oacc[b][4 * i + 1] = oacc[b0 + b][4 * i + 1] * c1 + p.y * c2;
          oacc[b][4 * i + 2] = oacc[b0 + b][4 * i + 2] * c1 + p.z * c2;
          oacc[b][4 * i + 3] = oacc[b0 + b][4 * i + 3] * c1 + p.w * c2;
        }
    };
    if (part) take(IC<1>{});
    else take(IC<0>{});
  }
  if (q0 + r32 < m) {
    const float inv = 1.0f / lrun;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        half4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (_Float16)(oacc[b][4 * i + e] * inv);
        *(half4 *)(o16 + (size_t)(q0 + r32) * qd + h * HD + (part * NB + b) * 32 + c_row(4 * i, lane)) = o;
      }
  }
}
constexpr int attn_lds_bytes(int hd, int ks) { return 2 * ks * (64 * (hd + 8) + hd * 72) * 2; }

// The last prompt position alone (behind the last block's keys and values only it goes on) over positions 0 .. P: one
// workgroup per (kv head, group of REP of its query heads, split of the positions), 16 lanes per cached
// position, a running softmax (base 2) per lane group and head, everything but q in fp32.  The splits' results
// meet in the last workgroup to arrive of a head group, in split order.  Bound by latency: 26 us at 4096 positions of the 8B shape, 12 at
// 512, 8 at 255 of the 1B shape; the tiles above, one row of 32 at work, took 139, 26 and 11.7.  A head per
// wavefront: with all heads of a kv head in every lane (each row fetched once) it took 46 and 16, the vector
// instructions of one wavefront per SIMD in a chain.
// part_o, part_ml: as the decode attention leaves them; word 2 of a head's first part_ml entry counts arrivals (zero
// between launches).
template <int HD, int REP>
__global__ __launch_bounds__(256 * REP) void k_pf_attn_last(const _Float16 *__restrict__ q16, const void *kcache, const void *vcache,
                                                            int kv_f16, int nq, int nkv, int l, int max_seq, int P, int n_splits,
                                                            float *part_o, float *part_ml, _Float16 *o16) {
  constexpr int EL = HD / 16, NW = EL / 2, RB = 4;             // elements and words of a lane's slice of a row; rows in a batch
  __shared__ float part[4][REP][HD], wml[4][REP][2];
  __shared__ int flag;
  const int tid = threadIdx.x, dl = tid & 15, wv = tid >> 6, r = wv % REP, quarter = wv / REP;
  const int hgs = nq / nkv / REP, kvh = blockIdx.x / hgs, h0 = kvh * (nq / nkv) + blockIdx.x % hgs * REP;
  const int sp = blockIdx.y, chunk = (P + n_splits) / n_splits, p0 = sp * chunk, p1 = min(P + 1, p0 + chunk);
  const int kvd = nkv * HD;
  const size_t base = (size_t)l * max_seq * kvd + (size_t)kvh * HD + dl * EL;
  float q[EL], o[EL], m = -1.0e30f, ls = 0.f;
#pragma unroll
  for (int e = 0; e < EL; ++e) { q[e] = (float)q16[(h0 + r) * HD + dl * EL + e]; o[e] = 0.f; }
  struct Batch { uint32_t k[RB][NW], v[RB][NW]; };
  auto load = [&](int j0, Batch &t) {                          // (rows beyond the last read it again, masked below)
#pragma unroll
    for (int u = 0; u < RB; ++u) {
      const size_t off = (base + (size_t)min(j0 + 16 * u, p1 - 1) * kvd) * 2;
#pragma unroll
      for (int w = 0; w < NW; w += 2) {
        const u32x2 a = *RIVER_GLOBAL(u32x2, (const char *)kcache + off + w * 4), c = *RIVER_GLOBAL(u32x2, (const char *)vcache + off + w * 4);
        t.k[u][w] = a.x; t.k[u][w + 1] = a.y; t.v[u][w] = c.x; t.v[u][w + 1] = c.y;
      }
    }
  };
  auto consume = [&](int j0, const Batch &t) {
    float sc[RB], mn = m;
#pragma unroll
    for (int u = 0; u < RB; ++u) {
      float dot = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) dot = fmaf(cache_hi(t.k[u][w], kv_f16), q[2 * w + 1], fmaf(cache_lo(t.k[u][w], kv_f16), q[2 * w], dot));
      sc[u] = row16_sum(dot);
      if (j0 + 16 * u >= p1) sc[u] = -1.0e30f;
      mn = fmaxf(mn, sc[u]);
    }
    const float cg = __builtin_amdgcn_exp2f(m - mn);
    m = mn;
    ls *= cg;
#pragma unroll
    for (int e = 0; e < EL; ++e) o[e] *= cg;
#pragma unroll
    for (int u = 0; u < RB; ++u) {
      // (left out by its position, not by its value: a score that is NaN is one, as in the tiles)
      const float pg = j0 + 16 * u < p1 ? __builtin_amdgcn_exp2f(sc[u] - mn) : 0.f;
      ls += pg;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        o[2 * w] = fmaf(pg, cache_lo(t.v[u][w], kv_f16), o[2 * w]);
        o[2 * w + 1] = fmaf(pg, cache_hi(t.v[u][w], kv_f16), o[2 * w + 1]);
      }
    }
  };
  Batch ba, bb;
  constexpr int step = 16 * RB;                                // (16 lane groups of a head: four wavefronts)
  int j0 = p0 + quarter * 4 + ((tid & 63) >> 4);
  if (j0 < p1) load(j0, ba);
  for (; j0 < p1; j0 += 2 * step) {
    load(j0 + step, bb);
    consume(j0, ba);
    load(j0 + 2 * step, ba);
    if (j0 + step < p1) consume(j0 + step, bb);
  }
  // the four lane groups of a wavefront by lane exchange, a head's wavefronts through LDS
#pragma unroll
  for (int off = 16; off <= 32; off <<= 1) {
    const float m2 = __shfl_xor(m, off), l2 = __shfl_xor(ls, off), mn = fmaxf(m, m2);
    const float c1 = __builtin_amdgcn_exp2f(m - mn), c2 = __builtin_amdgcn_exp2f(m2 - mn);
    ls = ls * c1 + l2 * c2;
#pragma unroll
    for (int e = 0; e < EL; ++e) o[e] = o[e] * c1 + __shfl_xor(o[e], off) * c2;
    m = mn;
  }
  if ((tid & 63) < 16) {
#pragma unroll
    for (int e = 0; e < EL; ++e) part[quarter][r][dl * EL + e] = o[e];
    if (dl == 0) { wml[quarter][r][0] = m; wml[quarter][r][1] = ls; }
  }
  __syncthreads();
  const size_t pb = (size_t)h0 * kMaxSplits;
  const int hr = tid / HD, he = tid % HD;                      // (a thread per element of the heads: 256 REP >= REP HD)
  if (hr < REP) {
    float M = -1.0e30f, Ls = 0.f, O = 0.f;
    for (int w = 0; w < 4; ++w) M = fmaxf(M, wml[w][hr][0]);
    for (int w = 0; w < 4; ++w) {
      const float c = __builtin_amdgcn_exp2f(wml[w][hr][0] - M);
      Ls = fmaf(wml[w][hr][1], c, Ls);
      O = fmaf(part[w][hr][he], c, O);
    }
    if (n_splits == 1) {
      o16[(h0 + hr) * HD + he] = (_Float16)(O / Ls);
    } else {
      const size_t pi = pb + hr * kMaxSplits + sp;
      pub(part_o + pi * HD + he, O);
      if (he == 0) { pub(part_ml + pi * 4, M); pub(part_ml + pi * 4 + 1, Ls); }
    }
  }
  if (n_splits == 1 || !last_arriver((unsigned int *)part_ml + pb * 4 + 2, (unsigned)n_splits, &flag)) return;
  if (hr < REP) {
    float mj[kMaxSplits], lj[kMaxSplits], oj[kMaxSplits], M = -1.0e30f, Ls = 0.f, O = 0.f;
#pragma unroll
    for (int j = 0; j < kMaxSplits; ++j) {                     // (all of them fetched before the first is used)
      const size_t pi = pb + hr * kMaxSplits + j;
      mj[j] = j < n_splits ? sub(part_ml + pi * 4) : -1.0e30f;
      lj[j] = j < n_splits ? sub(part_ml + pi * 4 + 1) : 0.f;
      oj[j] = j < n_splits ? sub(part_o + pi * HD + he) : 0.f;
      M = fmaxf(M, mj[j]);
    }
#pragma unroll
    for (int j = 0; j < kMaxSplits; ++j) {
      const float c = __builtin_amdgcn_exp2f(mj[j] - M);       // (an empty split has sum 0)
      Ls = fmaf(lj[j], c, Ls);
      O = fmaf(oj[j], c, O);
    }
    o16[(h0 + hr) * HD + he] = (_Float16)(O / Ls);
  }
}

// ------------------------------------------------------------- short prompts
//
// Prompts below the GEMM prefill's smallest keep the decode kernels' precision: 32-bit activations in backbone
// blocks, fp16 inputs and exact codes in river blocks, fp32 queries, scores and probabilities.  They
// went through the decode kernels one position at a time, a stream of all weights each (section of four
// 8B blocks: 31 tokens 10.5 ms); now up to kShort positions share a pass of the GEMMs above in their
// EXACT form, with the two kernels below between them (31 tokens: 0.63 ms).

// Causal attention of a few rows over the cache (which holds their own keys and values already): one
// wavefront per (row, query head), 16 lanes per cached position, four positions at a time, a running
// softmax (base 2) per lane group.  Bound by latency: a few hundred wavefronts, a few positions each.
// q32: [m][nq hd] fp32, scaled; out: rows of nq hd, three bf16 parts (split) or fp16.
template <int HD>
__global__ __launch_bounds__(256) void k_pf_attn_rows(const float *__restrict__ q32, const void *kcache, const void *vcache,
                                                      int kv_f16, int nq, int nkv, int l, int max_seq, int pos0, bool split,
                                                      void *out) {
  constexpr int EL = HD / 16, NW = EL / 2;
  const int lane = threadIdx.x & 63, slot = lane >> 4, dl = lane & 15;
  const int t = blockIdx.y, h = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (h >= nq) return;
  const int P = pos0 + t, qd = nq * HD, kvd = nkv * HD;
  const size_t base = (size_t)l * max_seq * kvd + (size_t)(h / (nq / nkv)) * HD + dl * EL;
  float q[EL], o[EL], m = -1.0e30f, ls = 0.f;
#pragma unroll
  for (int e = 0; e < EL; ++e) { q[e] = q32[(size_t)t * qd + h * HD + dl * EL + e]; o[e] = 0.f; }
  for (int p0 = 0; p0 <= P; p0 += 16) {
    uint32_t kw[4][NW], vw[4][NW];
#pragma unroll
    for (int u = 0; u < 4; ++u) {                            // (positions beyond the last read it again, masked below)
      const size_t off = (base + (size_t)min(p0 + u * 4 + slot, P) * kvd) * 2;
#pragma unroll
      for (int w = 0; w < NW; w += 2) {
        const u32x2 a = *RIVER_GLOBAL(u32x2, (const char *)kcache + off + w * 4), b = *RIVER_GLOBAL(u32x2, (const char *)vcache + off + w * 4);
        kw[u][w] = a.x; kw[u][w + 1] = a.y; vw[u][w] = b.x; vw[u][w + 1] = b.y;
      }
    }
    float sc[4], mn = m;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float d = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) d = fmaf(cache_hi(kw[u][w], kv_f16), q[2 * w + 1], fmaf(cache_lo(kw[u][w], kv_f16), q[2 * w], d));
      sc[u] = row16_sum(d);
      if (p0 + u * 4 + slot > P) sc[u] = -1.0e30f;
      mn = fmaxf(mn, sc[u]);
    }
    const float cg = __builtin_amdgcn_exp2f(m - mn);
    m = mn;
    ls *= cg;
#pragma unroll
    for (int e = 0; e < EL; ++e) o[e] *= cg;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float pg = sc[u] > -0.5e30f ? __builtin_amdgcn_exp2f(sc[u] - mn) : 0.f;
      ls += pg;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        o[2 * w] = fmaf(pg, cache_lo(vw[u][w], kv_f16), o[2 * w]);
        o[2 * w + 1] = fmaf(pg, cache_hi(vw[u][w], kv_f16), o[2 * w + 1]);
      }
    }
  }
#pragma unroll
  for (int off = 16; off <= 32; off <<= 1) {
    const float m2 = __shfl_xor(m, off), l2 = __shfl_xor(ls, off), mn = fmaxf(m, m2);
    const float c1 = __builtin_amdgcn_exp2f(m - mn), c2 = __builtin_amdgcn_exp2f(m2 - mn);
    ls = ls * c1 + l2 * c2;
#pragma unroll
    for (int e = 0; e < EL; ++e) o[e] = o[e] * c1 + __shfl_xor(o[e], off) * c2;
    m = mn;
  }
  if (slot != 0) return;
  const size_t at = (size_t)t * qd + h * HD + dl * EL;
#pragma unroll
  for (int e = 0; e < EL; ++e) {
    const float v = o[e] / ls;
    if (split) {
      uint16_t p[3];
      split3(v, p);
#pragma unroll
      for (int i = 0; i < 3; ++i) ((uint16_t *)out)[i * (size_t)kShort * qd + at + e] = p[i];
    } else {
      ((_Float16 *)out)[at + e] = (_Float16)v;
    }
  }
}

// a = silu(gate) * up from the planes [n_part][kShort][2 ffn] of the gate/up GEMM, added in order; out: rows of
// ffn, three bf16 parts (split) or fp16.  One thread per eight columns (ffn % 8 == 0).
__global__ __launch_bounds__(256) void k_pf_swiglu_rows(const float *__restrict__ part, int n_part, int ffn, bool split, void *out) {
  const int t = blockIdx.y, k = (blockIdx.x * 256 + (int)threadIdx.x) * 8;
  if (k >= ffn) return;
  const size_t stride = (size_t)kShort * 2 * ffn, row = (size_t)t * 2 * ffn;
  Run8 g{}, u{};
  add_planes(part + row + k, stride, n_part, [&](const float *p, bool ok) {
    const Run8 a = ld_run8(p), b = ld_run8(p + ffn);
#pragma unroll
    for (int e = 0; e < 8; ++e) { g.v[e] += ok ? a.v[e] : 0.f; u.v[e] += ok ? b.v[e] : 0.f; }
  });
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = g.v[e] / (1.0f + expf(-g.v[e])) * u.v[e];
  if (split) {
    store_split3((uint16_t *)out + (size_t)t * ffn + k, (size_t)kShort * ffn, v);
  } else {
    half8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (_Float16)v[e];
    *(half8 *)((_Float16 *)out + (size_t)t * ffn + k) = o;
  }
}

}  // namespace pf

// =====================================================================================
// Batched decode step (several sequences, each at its own position and exit depth)
// =====================================================================================
//
// One decode step for n sequences, six launches per block: QKV GEMM, attention (with RoPE and
// the KV write), O-proj GEMM, gate/up GEMM (the norm in front of it rides on these two, see BdNorm;
// SwiGLU in its epilogue), down GEMM, block end (similarity, exit decision, next norm).  Every GEMM runs the bf16 backbone matrices for the
// rows (sequences) still in the backbone and the 4-bit river twins for the rows that have left
// it, over the same activation tile, each side touching only its own rows and not read at all
// when it has none (so a block whose rows all sit on one side reads one weight set).  With
// depths drawn independently per sequence most blocks read both sets: the reason Eq. 1 takes the
// minimum over the batch.  Which side a row is on is decided on the device after every backbone
// block (k_bd_block_end per sequence, k_bd_decide for Eq. 1's batch rule); the host never waits
// inside a step.
namespace bd {

using namespace pf;

constexpr int kRows = 32;             // most sequences per step (rows of the activation tile)
constexpr int kRecordsB = 1024;       // ring of per-step records of a batched context

struct SeqState {                     // device-side state of the sequences, [max_batch] each
  int *pos;                           // position the token of the current step is written to
  int *token;                         // token to consume next (produced by the last step / prefill)
  int *river;                         // 1: the sequence has left the backbone in the current step
  int *exit_pos;                      // exit position of the current step
  int *forced;                        // forced exit position of the current step (< 0: Eq. 1 decides)
};

// v_mfma_f32_16x16x32_f16: D[16x16] += A[16x32] B[32x16].  Lane l supplies row l % 16 of A and
// column l % 16 of B, the eight K values of lane group l / 16 each; D: register r of lane l is
// row (l / 16) * 4 + r, column l % 16.
typedef float f32x4v __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f32x4v mfma16x16(half8 a, half8 b, f32x4v c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// Eight 4-bit codes of one 32-bit word of the stream-order copy (see BdB: nibble j holds column 2j,
// nibble 4 + j column 2j + 1) -> the eight fp16 values 16 + code in column order: a nibble placed
// in bits 6..9 of the mantissa of 16.0 adds exactly its value, and pair j of the word needs one
// shift and one and-or.  Scale and zero point are applied to the products of a whole quantisation
// group (see bd_gemm_pass), not to the weights, so nothing is rounded here.
__device__ __forceinline__ half8 raw8(uint32_t w) {
  half8 out;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t sh = j < 2 ? w << (6 - 4 * j) : w >> (4 * j - 6);
    const half2v q = __builtin_bit_cast(half2v, (sh & 0x03c003c0u) | 0x4c004c00u);
    out[2 * j] = q[0];
    out[2 * j + 1] = q[1];
  }
  return out;
}

// The activations of a batched step (up to 32 sequence rows x K) are kept in the order the
// matrix-core operands are fetched in, so that a wavefront's A fragment of one MFMA step is one
// contiguous 1 KiB load: [step of 32 columns][row block of 16][lane group g][row % 16][8 columns
// 32 step + 8 g .. + 7]; 32 x K halfs (K % 32 == 0).
__host__ __device__ inline size_t frag_index(int m, int k) {
  return ((((size_t)(k >> 5)) * 2 + (m >> 4)) * 64 + ((k >> 3) & 3) * 16 + (m & 15)) * 8 + (k & 7);
}
__device__ __forceinline__ void frag_store(_Float16 *xf, int m, int k, _Float16 v) { xf[frag_index(m, k)] = v; }
// eight consecutive elements (m, k .. k+7), k % 8 == 0: one 16-byte store
__device__ __forceinline__ void frag_store8(_Float16 *xf, int m, int k, half8 v) { *(half8 *)(xf + frag_index(m, k)) = v; }

// The weights of a batched GEMM are kept a second time in **stream order**: the rows of the GEMM
// (matrices stacked along N, or the gate/up pair interleaved row by row) in units of 8 rows, and per
// unit and K tile the 16-byte pieces in the order the lanes of a wavefront fetch them ([lane group
// g][row % 8]).  A load instruction of a wavefront then reads two runs of 512 contiguous bytes (the
// two 8-row halves of its MFMA block) instead of 64 bytes from each of 16 rows, and the K tiles of
// a unit follow each other in memory.
//   bf16:   [unit][K tile of 64][step s][g][row % 8][columns k0 + 32 s + 8 g .. + 7]
//   codes:  [unit][K tile of 128][g][row % 8][4 words: word s = columns k0 + 32 s + 8 g .. + 7, column
//           2j in nibble j and column 2j + 1 in nibble 4 + j] -- a word is the B operand of one MFMA step
//   pairs:  [unit][K tile of 128][row % 8][64-column half] -- (scale, zero) as one packed word
// Rows beyond N and columns beyond K are zero (pairs: the row's last group).
struct BdB { const void *w, *sz; };
__host__ __device__ inline size_t bd_units(int N) { return (size_t)(N + 7) / 8; }
__host__ __device__ inline size_t bd_dense_bytes(int N, int K) { return bd_units(N) * (size_t)((K + 63) / 64) * 1024; }
__host__ __device__ inline size_t bd_codes_bytes(int N, int K) { return bd_units(N) * (size_t)((K + 127) / 128) * 512; }
__host__ __device__ inline size_t bd_pairs_bytes(int N, int K) { return bd_units(N) * (size_t)((K + 127) / 128) * 64; }

// row n of the GEMM -> (matrix, row) of the row-major source
__device__ __forceinline__ void bd_src_row(const GemmB &B, int interleaved, int n, int N, int &mat, int &row) {
  if (interleaved) { mat = n & 1; row = n >> 1; }
  else gemm_b_row(B, n, N, mat, row);
}
// one thread per 16-byte piece; K % 64 == 0, rows 16-byte aligned
__global__ void k_bd_pack_dense(GemmB B, int interleaved, int N, int K, uint4 *out) {
  const int nkt = (K + 63) / 64;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= bd_units(N) * nkt * 64) return;
  const int r8 = (int)(i & 7), g = (int)((i >> 3) & 3), st = (int)((i >> 5) & 1);
  const size_t t = i >> 6;
  const int kt = (int)(t % nkt), n = (int)(t / nkt) * 8 + r8, k = kt * 64 + st * 32 + g * 8;
  uint4 v = make_uint4(0, 0, 0, 0);
  if (n < N && k + 8 <= K) {
    int mat, row;
    bd_src_row(B, interleaved, n, N, mat, row);
    v = *(const uint4 *)((const char *)B.w[mat] + ((size_t)row * K + k) * 2);
  }
  out[i] = v;
}
__global__ void k_bd_pack_codes(GemmB B, int interleaved, int N, int K, uint4 *out) {
  const int nkt = (K + 127) / 128;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= bd_units(N) * nkt * 32) return;
  const int r8 = (int)(i & 7), g = (int)((i >> 3) & 3);
  const size_t t = i >> 5;
  const int kt = (int)(t % nkt), n = (int)(t / nkt) * 8 + r8;
  uint32_t w[4] = {0u, 0u, 0u, 0u};
  if (n < N) {
    int mat, row;
    bd_src_row(B, interleaved, n, N, mat, row);
    const char *src = (const char *)B.w[mat] + (size_t)row * (K >> 1);
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      const int k = kt * 128 + st * 32 + g * 8;
      if (k + 8 > K) continue;
      // row-major: byte j = column k + 2j in the low nibble, k + 2j + 1 in the high nibble
      const uint32_t v = *(const uint32_t *)(src + (k >> 1));
#pragma unroll
      for (int j = 0; j < 4; ++j)
        w[st] |= (((v >> (8 * j)) & 0xfu) << (4 * j)) | (((v >> (8 * j + 4)) & 0xfu) << (16 + 4 * j));
    }
  }
  out[i] = make_uint4(w[0], w[1], w[2], w[3]);
}
// S.w[m] / S.sz[m]: the scales / zero points of matrix m, [rows][ceil(K / group)] bf16
__global__ void k_bd_pack_pairs(GemmB S, int interleaved, int N, int K, int group, uint32_t *out) {
  const int nkt = (K + 127) / 128, gpr = (K + group - 1) / group;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= bd_units(N) * nkt * 16) return;
  const int j = (int)(i & 1), r8 = (int)((i >> 1) & 7);
  const size_t t = i >> 4;
  const int kt = (int)(t % nkt), n = (int)(t / nkt) * 8 + r8, k = kt * 128 + j * 64;
  uint32_t v = 0;
  if (n < N) {
    int mat, row;
    bd_src_row(S, interleaved, n, N, mat, row);
    const size_t src = (size_t)row * gpr + min(k / group, gpr - 1);
    v = Store<1>::pack(Store<1>::ld(S.w[mat], src), Store<1>::ld(S.sz[mat], src));
  }
  out[i] = v;
}

// The row-wise kernels of a batched step (one workgroup per sequence row: 256 threads at its start,
// 512 at a block's end, where a thread's loads are a chain of latencies) read their row once: thread t
// of T owns columns 8 t + 8 T i .. + 7 and keeps up to kRowKeep such runs in registers between the
// reduction and the second use (longer rows are read again).  n_part > 0: the partial sums [n_part][32][d] of the K-sliced GEMM that adds into h are
// added first, in order, and h is updated.
constexpr int kRowKeep = 4;
__device__ __forceinline__ Run8 load_run8(float *row, const float *part, int n_part, int t, int d, int k) {
  float4 a = *(const float4 *)(row + k), b = *(const float4 *)(row + k + 4);
  if (n_part > 0) {
    // (not add_planes: with its branch for one plane, which a batched step never has, k_bd_block_end takes 142 registers instead of
    // 124, and 5.9 us instead of 5.7 for 32 rows of the 8B shape)
    for (int j = 0; j < n_part; j += 4)
      add_some_planes<4>(part + (size_t)t * d + k, (size_t)kRows * d, j, n_part, [&](const float *p, bool ok) {
        const float4 pa = *(const float4 *)p, pb = *(const float4 *)(p + 4);
        a.x += ok ? pa.x : 0.f; a.y += ok ? pa.y : 0.f; a.z += ok ? pa.z : 0.f; a.w += ok ? pa.w : 0.f;
        b.x += ok ? pb.x : 0.f; b.y += ok ? pb.y : 0.f; b.z += ok ? pb.z : 0.f; b.w += ok ? pb.w : 0.f;
      });
    *(float4 *)(row + k) = a;
    *(float4 *)(row + k + 4) = b;
  }
  return Run8{{a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w}};
}
__device__ __forceinline__ void norm_store_run8(const Run8 &x, float r, const Run8 &g, _Float16 *xf, int t, int k) {
  half8 o;
#pragma unroll
  for (int j = 0; j < 8; ++j) o[j] = (_Float16)(x.v[j] * r * g.v[j]);
  frag_store8(xf, t, k, o);
}

// What a step is told about its sequences, by value: nothing to copy to the device in front of it.
struct StepIn {
  int pos[kRows];             // position the token is written to (the host's count)
  int token[kRows];           // token to consume, or < 0: the one the last step / prefill left
  int forced[kRows];          // forced exit position (< 0: Eq. 1 decides)
};

// Start of a step, one workgroup per sequence: its state (forced exit position 0 puts it into the
// river from the first block on), h[b, :] = E[token[b], :] (also h_prev and the debug view of h(0)),
// sims[b, :] = NaN (blocks that run as river twins keep it), and block 1's attention norm:
// xf[b, :] = fp16(h[b, :] * rsqrt(mean(h[b, :]^2) + eps) * gain) in fragment order; d % 8 == 0.
__global__ __launch_bounds__(256) void k_bd_begin(StepIn in, SeqState st, const void *tok_emb, int d, int vocab, int L,
                                                  float *h, float *h_prev, float *hist, float *sims, const void *gain,
                                                  float eps, _Float16 *xf) {
  __shared__ float red[16];
  const int b = blockIdx.x;
  const int given = in.token[b], tok = min(max(given >= 0 ? given : st.token[b], 0), vocab - 1);
  const bool wide = ((uintptr_t)tok_emb & 15) == 0;            // (the embedding may have any alignment)
  float ss = 0.f;
  auto take = [&](int k) {
    const size_t i = (size_t)tok * d + k, o = (size_t)b * d + k;
    Run8 x;
    if (wide) x = ld_run8_16(tok_emb, i);
    else for (int j = 0; j < 8; ++j) x.v[j] = Store<1>::ld(tok_emb, i + j);
    st_run8(h + o, x);
    st_run8(h_prev + o, x);
    st_run8(hist + o, x);
#pragma unroll
    for (int j = 0; j < 8; ++j) ss = fmaf(x.v[j], x.v[j], ss);
    return x;
  };
  const bool gain_wide = ((uintptr_t)gain & 15) == 0;
  Run8 keep[kRowKeep], kg[kRowKeep];                           // (gains with the row: one round trip)
#pragma unroll
  for (int i = 0; i < kRowKeep; ++i) {
    const int k = threadIdx.x * 8 + i * 2048;
    if (k < d) kg[i] = ld_gain8(gain, k, gain_wide);
    if (k < d) keep[i] = take(k);
  }
  for (int k = threadIdx.x * 8 + kRowKeep * 2048; k < d; k += 2048) (void)take(k);
  for (int i = threadIdx.x; i < L; i += 256) sims[(size_t)b * L + i] = __uint_as_float(0x7fc00000u);
  if (threadIdx.x == 0) {
    const bool r0 = in.forced[b] == 0;
    st.pos[b] = in.pos[b];
    st.forced[b] = in.forced[b];
    st.river[b] = r0 ? 1 : 0;
    st.exit_pos[b] = r0 ? 0 : L;
  }
  const float r = 1.0f / sqrtf(block_sum(ss, red) / (float)d + eps);
#pragma unroll
  for (int i = 0; i < kRowKeep; ++i) {
    const int k = threadIdx.x * 8 + i * 2048;
    if (k < d) norm_store_run8(keep[i], r, kg[i], xf, b, k);
  }
  for (int k = threadIdx.x * 8 + kRowKeep * 2048; k < d; k += 2048)    // stored by this thread itself above
    norm_store_run8(ld_run8(h + (size_t)b * d + k), r, ld_gain8(gain, k, gain_wide), xf, b, k);
}

// C[rows, N] (op)= A[rows, K] B^T for the rows r < n_rows with river[r] == want (want < 0: all
// rows); nothing is read if there is none.  MB = 1: up to 16 rows, MB = 2: up to 32.
//
// The weights are read once, so the kernel is a weight stream with the matrix cores doing the
// arithmetic.  Workgroup = eight wavefronts on `rows_per_wg` consecutive rows of B (a multiple
// of 8, chosen by the host so that the rows divide evenly over the CUs), taken in passes of
// RBW blocks of 16 rows; rows of a block beyond the workgroup's range are not loaded.  The
// wavefronts split K: wavefront w takes every eighth K tile (64 columns dense, 128 columns of
// 4-bit codes).  A lane loads its MFMA operands directly in the layout the instruction wants --
// no LDS on the way: for B, lane (n = lane % 16, g = lane / 16) fetches 16 bytes of row n (dense:
// columns k0 + 32 s + 8 g .. + 7 for the tile's two steps s; codes: the 32 columns
// k0 + 32 g .. + 31, one step per code word, which lie in one quantisation group) from the
// stream-order copy of the weights (see BdB), where they are the lane's piece of a contiguous run, for A the
// same columns of sequence row n (fp16, kept in fragment order: one contiguous 1 KiB per
// wavefront and step, from the L2; every workgroup reads the whole tile once, shared by its RBW
// row blocks).  P tiles are in flight per wavefront in registers.  The partial tiles of the
// wavefronts are summed in wavefront order through LDS.
// op (epi): store fp32, add into fp32, or -- with B's rows interleaved as (gate i, up i) --
// silu(gate) * up stored as fp16 in fragment order (the activation of the down projection; ldc is
// then its column count).
enum { EPI_STORE = 0, EPI_ADD = 1, EPI_SWIGLU = 2, EPI_ADD_NORM = 3 };
// The RMSNorm between a GEMM that completes h and the GEMM that consumes norm(h) costs no pass of
// its own: the producer (EPI_ADD_NORM: h += A B^T) also stores fp16(h * gain) in fragment order
// and, per workgroup and sequence row, the sum of squares of the h values it completed
// (ssq_out[workgroup][32]); the consumer adds those partial sums in workgroup order and applies
// the row's rsqrt(mean(h^2) + eps) to its product tile, which is the same product up to rounding.
constexpr int kSsqLoads = 16;                               // partial sums per lane: producers of up to 256 workgroups
struct BdRowScale {                                         // consumer side, per thread (see k_bd_gemm)
  float *rscale;                                            // LDS [32], or null: no fused norm
  float part[kSsqLoads];
  int d;
  float eps;
  __device__ __forceinline__ void finish() const {          // by every thread of the workgroup, before a workgroup barrier
    float v = 0.f;
#pragma unroll
    for (int u = 0; u < kSsqLoads; ++u) v += part[u];
    v = row16_sum(v);
    if ((threadIdx.x & 15) == 0 && (threadIdx.x >> 4) < kRows) rscale[threadIdx.x >> 4] = 1.0f / sqrtf(v / (float)d + eps);
  }
};
struct BdNorm {
  const void *gain;          // producer: gain of the norm in front of the consumer
  _Float16 *xnext;           // producer: fp16(h * gain), fragment order
  float *ssq_out;            // producer: [gridDim.x][32]
  const float *ssq_in;       // consumer: the producer's partial sums, or null
  int ssq_wgs;               // consumer: workgroups of the producer
  int d;                     // consumer: length of a row of h
  float eps;
};
constexpr int kBdWaves = 8;
constexpr int kBdKSplit = 4;                                // K slices of the narrow GEMMs (see k_bd_gemm)
template <int RBW, int MB> struct BdDepth {                 // K tiles in flight per wavefront (register budget)
  static constexpr int dense = MB == 1 ? (RBW == 1 ? 8 : RBW == 2 ? 5 : RBW == 4 ? 3 : 2) : (RBW == 1 ? 4 : RBW == 2 ? 3 : 2);
  static constexpr int w4 = MB == 1 ? (RBW == 1 ? 6 : RBW == 2 ? 4 : RBW == 4 ? 3 : 2) : (RBW <= 2 ? 3 : 2);
};
__host__ __device__ inline size_t bd_gemm_lds_bytes(int rbw, int mb) { return (size_t)kBdWaves * rbw * mb * 256 * 4; }

template <bool W4, int MB, int RBW>
__device__ __forceinline__ void bd_gemm_pass(const _Float16 *__restrict__ Af, const BdB &B, int N,
                                             int K, void *C, int ldc, int epi,
                                             const int (&flag)[MB + 1], int want, int n_rows, int rows_per_wg,
                                             int k_split, int w0, int nw,
                                             float *red /* [kBdWaves][RBW][MB][256] */, const BdNorm &nrm,
                                             const BdRowScale &rsc) {
  const float *rscale = rsc.rscale;
  constexpr int P = W4 ? BdDepth<RBW, MB>::w4 : BdDepth<RBW, MB>::dense;
  constexpr int TILE = W4 ? 128 : 64;                         // columns per K tile
  constexpr int NA = W4 ? 4 : 2;                              // MFMA steps (16-byte A fragments) per tile
  // the pass is run by wavefronts w0 .. w0 + nw - 1 of the workgroup (all eight, or four when the
  // other four run the other weight format beside it); every wavefront of the workgroup executes the
  // same number of workgroup barriers in either case
  const int tid = threadIdx.x - w0 * 64, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);   // (a scalar: K tiles are addressed by scalar offsets)
  const int r16 = lane & 15, kg = lane >> 4;
  red += (size_t)w0 * RBW * MB * 256;
  // workgroup -> (group of rows, slice of K): with k_split > 1 the output is a partial sum, stored
  // as rows 32 ks .. of C for the consumer to add up (see load_run8)
  const int ks = blockIdx.x % k_split;
  const int wg_r0 = (blockIdx.x / k_split) * rows_per_wg, wg_r1 = min(N, wg_r0 + rows_per_wg);
  const int nkt_all = (K + TILE - 1) / TILE;
  const int kt0 = (int)((long long)nkt_all * ks / k_split), nkt = (int)((long long)nkt_all * (ks + 1) / k_split);
  struct Stage { uint4 a[MB * NA], b[RBW * (W4 ? 1 : 2)]; uint2 sz[W4 ? RBW : 1]; };
  float ssq[MB];                                              // EPI_ADD_NORM: this thread's sum of h^2, row i * 16 + (tid % 256) / 16
#pragma unroll
  for (int i = 0; i < MB; ++i) ssq[i] = 0.f;
  // EPI_ADD_NORM with one row block per pass (d_model of up to 16 rows per CU): h and the gains of this thread's
  // elements of the first pass, at most two, are fetched here, their latency is the K loop's
  constexpr bool kPre = RBW == 1;
  float pre_h[2] = {0.f, 0.f}, pre_g[2] = {0.f, 0.f};
  if (kPre && epi == EPI_ADD_NORM) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int e = tid + q * nw * 64, row = (e / 256) * 16 + ((e & 255) >> 4), n = wg_r0 + (e & 15);
      if (e < MB * 256 && row < n_rows && n < wg_r1) {
        pre_h[q] = ((const float *)C)[(size_t)row * ldc + n];
        pre_g[q] = Store<1>::ld(nrm.gain, n);
      }
    }
  }
  for (int p0 = wg_r0; p0 < wg_r1; p0 += RBW * 16) {
    // Stream order (see BdB): this lane's 16-byte piece of K tile 0 of row block 0 lies in unit p0 / 8
    // or the next one, at [g][row % 8]; a row block further is 2 units, a K tile further one tile.
    // Buffer loads: the pass's base in a descriptor, the lane's part of the address in one 32-bit
    // register, everything that is the same for all lanes in the scalar offset.
    constexpr unsigned UB = W4 ? 512u : 1024u;                // bytes of one unit's K tile
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        (void *)((const char *)B.w + (size_t)(p0 >> 3) * nkt_all * UB), 0, 0x7ffffff0, 0x00020000);
    const __amdgpu_buffer_rsrc_t rz = __builtin_amdgcn_make_buffer_rsrc(
        (void *)((const char *)(W4 ? B.sz : B.w) + (W4 ? (size_t)(p0 >> 3) * nkt_all * 64 : 0)), 0, 0x7ffffff0, 0x00020000);
    const unsigned vw = (unsigned)(r16 >> 3) * nkt_all * UB + (kg * 8 + (r16 & 7)) * 16;
    const unsigned vz = (unsigned)(r16 >> 3) * nkt_all * 64u + (r16 & 7) * 8;      // both halves' pairs
    const unsigned bstride = (unsigned)nkt_all * 2u * UB, sstride = (unsigned)nkt_all * 128u;
    // Rows beyond the workgroup's range, columns beyond K (and K tiles beyond the slice, where such
    // a load is issued at all) get an offset beyond the descriptor's range: a buffer load then
    // returns zero without touching memory, and no load sits behind a branch.
    constexpr unsigned kOut = 0x80000000u;
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc((void *)Af, 0, 0x7ffffff0, 0x00020000);
    auto row_ok = [&](int rb) { return p0 + rb * 16 + r16 < wg_r1; };
    auto ld16 = [&](const __amdgpu_buffer_rsrc_t &r, unsigned voff, unsigned soff, auto stream) {
      constexpr int aux = decltype(stream)::value ? 2 : 0;    // 2: streaming (read once)
      const u32x4 v = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, aux));
      return make_uint4(v.x, v.y, v.z, v.w);
    };
    auto load = [&](int kt, Stage &t) {
      const bool tile = kt < nkt;                             // (the same for all lanes)
      // step kt * NA + s of the activations; K % 64 == 0, so a 128-column tile may end after two steps
      // (columns of A beyond K are not defined; B's are zero)
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int s = 0; s < NA; ++s)
          t.a[i * NA + s] = ld16(ra, tile && (kt * NA + s) * 32 < K ? lane * 16u : kOut,
                                 (unsigned)((kt * NA + s) * 2 + i) * 1024u, IC<0>{});
#pragma unroll
      for (int rb = 0; rb < RBW; ++rb) {
        const unsigned vo = tile && row_ok(rb) ? vw : kOut;
        if constexpr (W4) {
          t.b[rb] = ld16(rw, vo, rb * bstride + (unsigned)kt * UB, IC<1>{});
          const u32x2 q = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(
                                                        rz, tile && row_ok(rb) ? vz : kOut,
                                                        rb * sstride + (unsigned)kt * 64u, 0));
          t.sz[rb] = make_uint2(q.x, q.y);
        } else {
#pragma unroll
          for (int s = 0; s < 2; ++s) t.b[rb * 2 + s] = ld16(rw, vo, rb * bstride + (unsigned)kt * UB + s * 512u, IC<1>{});
        }
      }
    };
    f32x4v acc[RBW][MB];
#pragma unroll
    for (int rb = 0; rb < RBW; ++rb)
#pragma unroll
      for (int i = 0; i < MB; ++i) acc[rb][i] = f32x4v{0.f, 0.f, 0.f, 0.f};
    auto compute = [&](const Stage &t) {
      if constexpr (W4) {
        // The codes go into the matrix cores as they are (16 + code, see raw8).  Per 64-column half of
        // the tile, which lies in one quantisation group: (W x)[m][n] = scale_n * sum_k a_mk (16 +
        // code_nk) - scale_n * (16 + zero_n) * sum_k a_mk; the last sum (rs) comes in the layout of
        // the product tile from a product with a matrix of ones, shared by the row blocks.
        const half8 ones = {(_Float16)1.f, (_Float16)1.f, (_Float16)1.f, (_Float16)1.f,
                            (_Float16)1.f, (_Float16)1.f, (_Float16)1.f, (_Float16)1.f};
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          f32x4v rs[MB];
#pragma unroll
          for (int i = 0; i < MB; ++i) {
            rs[i] = mfma16x16(__builtin_bit_cast(half8, t.a[i * NA + 2 * hf]), ones, f32x4v{0.f, 0.f, 0.f, 0.f});
            rs[i] = mfma16x16(__builtin_bit_cast(half8, t.a[i * NA + 2 * hf + 1]), ones, rs[i]);
          }
#pragma unroll
          for (int rb = 0; rb < RBW; ++rb) {
            const uint32_t w0 = hf ? t.b[rb].z : t.b[rb].x, w1 = hf ? t.b[rb].w : t.b[rb].y;
            const uint32_t pr = hf ? t.sz[rb].y : t.sz[rb].x;
            const half8 b0 = raw8(w0), b1 = raw8(w1);
            const float sc = bf16_lo(pr), nz = -sc * (16.0f + bf16_hi(pr));
#pragma unroll
            for (int i = 0; i < MB; ++i) {
              f32x4v tmp = mfma16x16(__builtin_bit_cast(half8, t.a[i * NA + 2 * hf]), b0, f32x4v{0.f, 0.f, 0.f, 0.f});
              tmp = mfma16x16(__builtin_bit_cast(half8, t.a[i * NA + 2 * hf + 1]), b1, tmp);
#pragma unroll
              for (int r = 0; r < 4; ++r) acc[rb][i][r] += sc * tmp[r] + nz * rs[i][r];
            }
          }
        }
      } else {
#pragma unroll
        for (int rb = 0; rb < RBW; ++rb)
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            const half8 b = bf16x8_to_half8(t.b[rb * 2 + s]);
#pragma unroll
            for (int i = 0; i < MB; ++i)
              acc[rb][i] = mfma16x16(__builtin_bit_cast(half8, t.a[i * NA + s]), b, acc[rb][i]);
          }
      }
    };
    // P stages in flight per wavefront; a round consumes each stage and refills it with the tile P
    // rounds of wavefronts further.  Refills beyond the slice are skipped -- except in the widest
    // 4-bit pass, which issues them all the same (beyond the range: no memory access), because the
    // compiler then needs fewer registers and that pass has none to spare.
    constexpr bool kAlways = W4 && RBW >= 8;
    Stage st[P];
#pragma unroll
    for (int u = 0; u < P; ++u)
      if (kAlways || kt0 + wv + nw * u < nkt) load(kt0 + wv + nw * u, st[u]);
    for (int kt = kt0 + wv; kt < nkt; kt += nw * P) {
#pragma unroll
      for (int u = 0; u < P; ++u) {
        const int k = kt + nw * u;
        if (k < nkt) compute(st[u]);
        if (kAlways || k + nw * P < nkt) load(k + nw * P, st[u]);
      }
    }
    // the partial tiles of the nw wavefronts -> one, in wavefront order; D: register r of lane l is sequence row
    // (l / 16) * 4 + r, B row l % 16
    if (rscale && p0 == wg_r0) rsc.finish();                  // (visible after the barriers below)
    __syncthreads();                                          // the previous pass has been read
#pragma unroll
    for (int rb = 0; rb < RBW; ++rb)
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          red[((wv * RBW + rb) * MB + i) * 256 + (kg * 4 + r) * 16 + r16] = acc[rb][i][r];
    __syncthreads();
    constexpr int TILE_F = RBW * MB * 256;
    int ord = kPre && p0 == wg_r0 ? 0 : 2;                            // which of this thread's elements
    for (int e = tid; e < TILE_F; e += nw * 64, ++ord) {
      const int rb = e / (MB * 256), i = (e / 256) % MB, row = i * 16 + ((e & 255) >> 4), n = p0 + rb * 16 + (e & 15);
      int f = flag[0];                                        // (rows i * 16 + (tid % 256) / 16: see k_bd_gemm)
#pragma unroll
      for (int i2 = 1; i2 < MB; ++i2) f = i2 == i ? flag[i2] : f;
      if (row >= n_rows || n >= wg_r1 || !(want < 0 || f == want)) continue;
      const float rs_row = rscale ? rscale[row] : 1.0f;
      auto total = [&](int idx) {
        float v = red[idx];
#pragma unroll
        for (int w = 1; w < nw; ++w) v += red[w * TILE_F + idx];
        return v * rs_row;
      };
      if (epi == EPI_SWIGLU) {
        if (n & 1) continue;
        const float g = total(e), u = total(e + 1);
        frag_store((_Float16 *)C, row, n >> 1, (_Float16)(g / (1.0f + expf(-g)) * u));
      } else {
        float *p = (float *)C + (size_t)(k_split > 1 ? ks * kRows + row : row) * ldc + n;
        const float v = total(e);
        if (epi == EPI_ADD_NORM) {
          const float hv = (ord == 0 ? pre_h[0] : ord == 1 ? pre_h[1] : *p) + v;
          *p = hv;
          frag_store(nrm.xnext, row, n, (_Float16)(hv * (ord == 0 ? pre_g[0] : ord == 1 ? pre_g[1] : Store<1>::ld(nrm.gain, n))));
#pragma unroll
          for (int i2 = 0; i2 < MB; ++i2)
            if (i2 == i) ssq[i2] = fmaf(hv, hv, ssq[i2]);
        } else if (epi == EPI_ADD) *p += v;
        else *p = v;
      }
    }
  }
  if (epi == EPI_ADD_NORM) {
    // this workgroup's sums of squares per sequence row: the 16 lanes of a row, then the thread
    // groups 256 apart (the same rows), in a fixed order
    __syncthreads();                                          // the last pass has been read
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const float sr = row16_sum(ssq[i]);
      if ((tid & 15) == 0) red[(tid >> 8) * kRows + i * 16 + ((tid & 255) >> 4)] = sr;
    }
    __syncthreads();
    if (tid < MB * 16 && tid < n_rows && (want < 0 || flag[MB] == want)) {
      float v = red[tid];
      if (nw * 64 > 256) v += red[kRows + tid];
      nrm.ssq_out[(size_t)blockIdx.x * kRows + tid] = v;
    }
  }
}

// One launch per GEMM of a step: the bf16 matrices for the rows still in the backbone, the 4-bit
// twins for the rows that have left it (sides: which of the two have rows, 0 if only the device
// knows; kSideDense alone: the bf16 matrices for all rows, as the LM head needs).  A side without rows is not read.  Af: the activations in fragment
// order (see frag_index).  k_split > 1: narrow matrices (16 rows per CU would leave every
// workgroup reading all of A for one row block) are dealt out as k_split K slices of four times
// the rows; C is then the partial-sum buffer [k_split][32][ldc].
enum { kSideDense = 1, kSideTwin = 2 };
template <int MB, int RBW>
__global__ __launch_bounds__(512) void k_bd_gemm(const _Float16 *__restrict__ Af, BdB Bd, BdB Bq,
                                                 int N, int K, void *C, int ldc, int epi,
                                                 const int *__restrict__ river, int sides, int n_rows,
                                                 int rows_per_wg, int k_split, BdNorm nrm) {
  extern __shared__ float red[];
  __shared__ float rscale[kRows];
  // Which sides have rows: told by the host where it is known before the step, else every wavefront
  // looks at the rows' flags for itself (no workgroup barrier in front of the first weight load).
  // Only when both have does a row's flag matter beyond that; this thread's are fetched here, their
  // latency is the K loop's: rows i * 16 + (tid % 256) / 16 of the epilogue and row tid of the sums
  // of squares, tid counted from the first wavefront of its side.
  if (sides == 0) {
    const int l64 = threadIdx.x & 63, f = l64 < n_rows ? river[l64] : -1;
    sides = (__any(f == 0) ? kSideDense : 0) | (__any(f > 0) ? kSideTwin : 0);
  }
  sides = __builtin_amdgcn_readfirstlane(sides);
  const bool dense = sides & kSideDense, twin = sides & kSideTwin;
  int flag[MB + 1] = {};
  if (dense && twin) {
    const int tid = threadIdx.x & (kBdWaves / 2 * 64 - 1);
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const int row = i * 16 + ((tid & 255) >> 4);
      flag[i] = row < n_rows ? river[row] : -1;
    }
    flag[MB] = tid < n_rows ? river[tid] : -1;
  }
  // consumer of a fused norm: the producer's partial sums of squares of row threadIdx.x / 16 are
  // fetched here (16 lanes per row, up to kSsqLoads each) and added up, in a fixed order, where the
  // first product tile is complete (BdRowScale::finish) -- their latency is the K loop's
  BdRowScale rsc{nrm.ssq_in ? rscale : nullptr, {}, nrm.d, nrm.eps};
  if (nrm.ssq_in) {
    const int row = threadIdx.x >> 4, j0 = threadIdx.x & 15;
#pragma unroll
    for (int u = 0; u < kSsqLoads; ++u) {
      const int j = j0 + 16 * u;
      rsc.part[u] = row < n_rows && j < nrm.ssq_wgs ? nrm.ssq_in[(size_t)j * kRows + row] : 0.f;
    }
  }
  // Both sides: four wavefronts each, side by side -- the 4-bit side's dequantisation runs in the
  // shadow of the bf16 side's memory waits, and there is one ramp-up and one tail instead of two.
  constexpr int ND = kBdWaves / 2;                              // wavefronts of the bf16 side when both run (3 .. 4 measured best)
  const bool second = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) >= ND;   // (a scalar branch)
  if (dense && (!twin || !second))
    bd_gemm_pass<false, MB, RBW>(Af, Bd, N, K, C, ldc, epi, flag, twin ? 0 : -1, n_rows,
                                 rows_per_wg, k_split, 0, twin ? ND : kBdWaves, red, nrm, rsc);
  if (twin && (!dense || second))
    bd_gemm_pass<true, MB, RBW>(Af, Bq, N, K, C, ldc, epi, flag, dense ? 1 : -1, n_rows,
                                rows_per_wg, k_split, dense ? ND : 0, dense ? kBdWaves - ND : kBdWaves, red, nrm, rsc);
}

// Single-query attention of a batched step with RoPE and the KV write in front of it.  One
// workgroup per (sequence b, kv head, group of REP query heads of that kv head, split of the
// positions 0 .. pos[b]): the K/V rows of the kv head are read once for the REP heads.
//
// Prologue (from the raw QKV rows the GEMM left): the REP query vectors rotated at position
// pos[b] and scaled by log2(e)/sqrt(hd), this token's k (rotated) and v rounded to the cache
// dtype, all into LDS; the workgroup whose split holds position pos[b] (the first head group)
// also writes them to slot (b, l, pos[b]) of the shared cache -- the same slot for backbone and
// river rows -- and nobody reads that slot from the cache in this launch.
// Sixteen lanes share a cached row (HD/16 elements each, one 16- or 8-byte load), the 16 lane
// groups stride over the split's positions in batches of four K rows and their V rows, the next
// batch in flight while one is consumed.  Every lane group keeps a running softmax per head
// (base 2, rescaled once per batch; DPP row sums for the scores); lane groups, wavefronts and --
// with several splits -- workgroups are merged in a fixed order: every workgroup publishes (max,
// sum, unnormalised output) per head and the last one to arrive of the group merges them in
// split order (device-coherent stores and loads, no fences).  The result goes to o16 in fragment
// order (frag_store), the output projection's input.
constexpr int kBdAttnMaxSplits = 8;
__host__ __device__ inline size_t bd_attn_lds_bytes(int rep, int hd) {
  return ((size_t)rep * hd + 2 * hd + 64 + 4 * rep * hd) * 4;
}
template <int HD, bool KV_F16, int REP>
__global__ __launch_bounds__(256) void k_bd_attn(const float *__restrict__ qkv, const float2 *__restrict__ rope,
                                                 void *kcache, void *vcache, int nq, int nkv, int n_seq, int l,
                                                 int max_seq, size_t seq_stride, const int *__restrict__ pos,
                                                 int n_splits, float *part_o, float *part_ml,
                                                 unsigned int *tickets, _Float16 *o16) {
  constexpr int EL = HD / 16, HALF = HD / 2;                   // EL: elements per lane of a cached row
  extern __shared__ float sm[];
  float *qs = sm;                                              // [REP][HD]
  float *kc = qs + REP * HD, *vc = kc + HD;                    // this token's k, v (cache-rounded values)
  float *red = vc + HD;                                        // [64]
  float *part = red + 64;                                      // [4 wavefronts][REP][HD]
  const int tid = threadIdx.x, grp = tid >> 4, dl = tid & 15, wv = tid >> 6;
  const int rep = nq / nkv, hgs = rep / REP;
  // Workgroup index -> (data group g = (sequence, kv head, split), head group hg) such that the head
  // groups that read the same K/V rows run on the same XCD (consecutive workgroup ids go round the
  // 8 XCDs) and meet in that XCD's L2.
  const int bi = blockIdx.x, g = (bi / (8 * hgs)) * 8 + (bi & 7), hg = (bi % (8 * hgs)) >> 3;
  if (g >= n_seq * nkv * n_splits) return;
  const int sp = g % n_splits, kvh = (g / n_splits) % nkv, b = g / (n_splits * nkv);
  const int h0 = kvh * rep + hg * REP;
  const int P = pos[b], T = P + 1, qd = nq * HD, kvd = nkv * HD, ld = qd + 2 * kvd;
  const int chunk = (T + n_splits - 1) / n_splits, p0 = sp * chunk, p1 = min(T, p0 + chunk);
  const bool owner = P >= p0 && P < p1;                        // this split holds the current position
  const float *row_in = qkv + (size_t)b * ld;
  const size_t base = (size_t)b * seq_stride + (size_t)l * max_seq * kvd + (size_t)kvh * HD;
  // The cached rows p0 .. pc - 1 (the current position, the last one, is not read from the cache:
  // it seeds the first lane group's state from LDS).  Lane group grp takes rows p0 + grp + 16 t in
  // batches of RB, K and V rows together, the next batch in flight while one is consumed.
  const int pc = owner ? P : p1;
  constexpr int RB = 4;
  constexpr int NW = EL / 2;                                   // 32-bit words of a lane's row slice
  struct Batch { uint32_t k[RB][NW], v[RB][NW]; };
  auto load = [&](int j0, Batch &t) {
#pragma unroll
    for (int u = 0; u < RB; ++u) {
      const int j = min(j0 + 16 * u, pc - 1);                  // rows beyond the last read it again (masked below)
      const size_t off = (base + (size_t)j * kvd + dl * EL) * 2;
      if constexpr (NW == 4) {
        const uint4 a = *(const uint4 *)((const char *)kcache + off), c = *(const uint4 *)((const char *)vcache + off);
        t.k[u][0] = a.x; t.k[u][1] = a.y; t.k[u][2] = a.z; t.k[u][3] = a.w;
        t.v[u][0] = c.x; t.v[u][1] = c.y; t.v[u][2] = c.z; t.v[u][3] = c.w;
      } else {
        const uint2 a = *(const uint2 *)((const char *)kcache + off), c = *(const uint2 *)((const char *)vcache + off);
        t.k[u][0] = a.x; t.k[u][1] = a.y;
        t.v[u][0] = c.x; t.v[u][1] = c.y;
      }
    }
  };
  // the first batch does not depend on this step's q, k, v: it is in flight during the prologue
  Batch ba, bb;
  const int step = 16 * RB;
  int j0 = p0 + grp;
  if (j0 < pc) load(j0, ba);
  // ---- prologue: RoPE, rounding, KV write
  {
    const float qscale = 1.4426950408889634f / sqrtf((float)HD);
    for (int t = tid; t < REP * HALF; t += 256) {
      const int r = t / HALF, e = t % HALF;
      const float2 cs = rope[(size_t)P * HALF + e];
      const float *src = row_in + (h0 + r) * HD;
      const float a = src[e], c = src[e + HALF];
      qs[r * HD + e] = (a * cs.x - c * cs.y) * qscale;
      qs[r * HD + e + HALF] = (a * cs.y + c * cs.x) * qscale;
    }
    if (owner) {
      auto rnd = [](float v) { return KV_F16 ? (float)(_Float16)v : Store<1>::rnd(v); };
      const bool writer = hg == 0;
      const size_t slot = base + (size_t)P * kvd;
      if (tid < HALF) {
        const int e = tid;
        const float2 cs = rope[(size_t)P * HALF + e];
        const float *src = row_in + qd + kvh * HD;
        const float a = src[e], c = src[e + HALF];
        const float lo = a * cs.x - c * cs.y, hi = a * cs.y + c * cs.x;
        kc[e] = rnd(lo); kc[e + HALF] = rnd(hi);
        if (writer) { cache_store(kcache, slot + e, lo, KV_F16); cache_store(kcache, slot + e + HALF, hi, KV_F16); }
      } else if (tid >= 128 && tid < 128 + HD) {
        const int e = tid - 128;
        const float v = row_in[qd + kvd + kvh * HD + e];
        vc[e] = rnd(v);
        if (writer) cache_store(vcache, slot + e, v, KV_F16);
      }
    }
  }
  __syncthreads();
  float q[REP][EL];
#pragma unroll
  for (int r = 0; r < REP; ++r)
#pragma unroll
    for (int e = 0; e < EL; ++e) q[r][e] = qs[r * HD + dl * EL + e];
  // running softmax per head (base 2: the scores carry log2 e): maximum, sum, weighted values
  float m[REP], ls[REP], o[REP][EL];
#pragma unroll
  for (int r = 0; r < REP; ++r) {
    m[r] = -1.0e30f; ls[r] = 0.f;
#pragma unroll
    for (int e = 0; e < EL; ++e) o[r][e] = 0.f;
  }
  if (owner && grp == 0) {
#pragma unroll
    for (int r = 0; r < REP; ++r) {
      float dot = 0.f;
#pragma unroll
      for (int e = 0; e < EL; ++e) dot = fmaf(kc[dl * EL + e], q[r][e], dot);
      m[r] = row16_sum(dot);
      ls[r] = 1.f;
#pragma unroll
      for (int e = 0; e < EL; ++e) o[r][e] = vc[dl * EL + e];
    }
  }
  auto consume = [&](int j0, const Batch &t) {
    float sc[RB][REP];
#pragma unroll
    for (int u = 0; u < RB; ++u) {
      float kf[EL];
#pragma unroll
      for (int w = 0; w < NW; ++w) { kf[2 * w] = cache_lo(t.k[u][w], KV_F16); kf[2 * w + 1] = cache_hi(t.k[u][w], KV_F16); }
      const bool ok = j0 + 16 * u < pc;
#pragma unroll
      for (int r = 0; r < REP; ++r) {
        float dot = 0.f;
#pragma unroll
        for (int e = 0; e < EL; ++e) dot = fmaf(kf[e], q[r][e], dot);
        sc[u][r] = ok ? row16_sum(dot) : -1.0e30f;
      }
    }
#pragma unroll
    for (int r = 0; r < REP; ++r) {
      float mn = m[r];
#pragma unroll
      for (int u = 0; u < RB; ++u) mn = fmaxf(mn, sc[u][r]);
      const float cg = __builtin_amdgcn_exp2f(m[r] - mn);      // <= 1; 1 while nothing has been seen
      m[r] = mn;
      ls[r] *= cg;
#pragma unroll
      for (int e = 0; e < EL; ++e) o[r][e] *= cg;
#pragma unroll
      for (int u = 0; u < RB; ++u) sc[u][r] = sc[u][r] > -0.5e30f ? __builtin_amdgcn_exp2f(sc[u][r] - mn) : 0.f;
    }
#pragma unroll
    for (int u = 0; u < RB; ++u) {
      float vf[EL];
#pragma unroll
      for (int w = 0; w < NW; ++w) { vf[2 * w] = cache_lo(t.v[u][w], KV_F16); vf[2 * w + 1] = cache_hi(t.v[u][w], KV_F16); }
#pragma unroll
      for (int r = 0; r < REP; ++r) {
        ls[r] += sc[u][r];
#pragma unroll
        for (int e = 0; e < EL; ++e) o[r][e] = fmaf(sc[u][r], vf[e], o[r][e]);
      }
    }
  };
  // (the loads of the loop are issued whether or not their rows exist -- beyond the last row they
  // fetch it again -- so that none sits behind a branch and a batch's wait leaves the next one alone)
  for (; j0 < pc; j0 += 2 * step) {
    load(j0 + step, bb);
    consume(j0, ba);
    load(j0 + 2 * step, ba);
    if (j0 + step < pc) consume(j0 + step, bb);
  }
  // merge: the four lane groups of a wavefront by lane exchange (lanes 16 and 32 apart hold the
  // same elements), then the four wavefronts through LDS, both in a fixed order
#pragma unroll
  for (int r = 0; r < REP; ++r) {
#pragma unroll
    for (int off = 16; off <= 32; off <<= 1) {
      const float m2 = __shfl_xor(m[r], off), l2 = __shfl_xor(ls[r], off);
      const float mn = fmaxf(m[r], m2);
      const float c1 = __builtin_amdgcn_exp2f(m[r] - mn), c2 = __builtin_amdgcn_exp2f(m2 - mn);
      ls[r] = ls[r] * c1 + l2 * c2;
#pragma unroll
      for (int e = 0; e < EL; ++e) o[r][e] = o[r][e] * c1 + __shfl_xor(o[r][e], off) * c2;
      m[r] = mn;
    }
  }
  float *wml = red;                                            // [4 wavefronts][REP][2]
  if ((tid & 63) < 16) {
#pragma unroll
    for (int r = 0; r < REP; ++r) {
#pragma unroll
      for (int e = 0; e < EL; ++e) part[(wv * REP + r) * HD + dl * EL + e] = o[r][e];
      if (dl == 0) { wml[(wv * REP + r) * 2] = m[r]; wml[(wv * REP + r) * 2 + 1] = ls[r]; }
    }
  }
  __syncthreads();
  // element e of head r over the four wavefronts -> (M, L, O) of this split
  auto split_result = [&](int r, int e, float &M, float &Ls, float &O) {
    M = -1.0e30f; Ls = 0.f; O = 0.f;
    for (int w = 0; w < 4; ++w) M = fmaxf(M, wml[(w * REP + r) * 2]);
    for (int w = 0; w < 4; ++w) {
      const float cw = __builtin_amdgcn_exp2f(wml[(w * REP + r) * 2] - M);   // a wavefront that saw nothing has sum 0
      Ls = fmaf(wml[(w * REP + r) * 2 + 1], cw, Ls);
      O = fmaf(part[(w * REP + r) * HD + e], cw, O);
    }
  };
  if (n_splits == 1) {
    for (int t = tid; t < REP * HD; t += 256) {
      float M, Ls, O;
      split_result(t / HD, t % HD, M, Ls, O);
      frag_store(o16, b, (h0 + t / HD) * HD + t % HD, (_Float16)(O / Ls));
    }
    return;
  }
  // ---- several splits: publish the partial result, the last workgroup of the group merges
  for (int t = tid; t < REP * HD; t += 256) {
    const int r = t / HD, e = t % HD;
    float M, Ls, O;
    split_result(r, e, M, Ls, O);
    const size_t pi = ((size_t)b * nq + h0 + r) * kBdAttnMaxSplits + sp;
    pub(part_o + pi * HD + e, O);
    if (e == 0) { pub(part_ml + pi * 2, M); pub(part_ml + pi * 2 + 1, Ls); }
  }
  if (!last_arriver(tickets + ((size_t)b * nkv + kvh) * hgs + hg, (unsigned)n_splits, (int *)(red + 60))) return;
  for (int t = tid; t < REP * HD; t += 256) {
    const int r = t / HD, e = t % HD;
    const size_t pb = ((size_t)b * nq + h0 + r) * kBdAttnMaxSplits;
    // every split's numbers are fetched before the first is used (in a loop over the splits each one was a
    // round trip, twice: 4 us of 22 with four splits)
    float mj[kBdAttnMaxSplits], lj[kBdAttnMaxSplits], oj[kBdAttnMaxSplits];
#pragma unroll
    for (int j = 0; j < kBdAttnMaxSplits; ++j) {
      mj[j] = -1.0e30f; lj[j] = oj[j] = 0.f;
      if (j < n_splits) {                                      // (uniform)
        mj[j] = sub(part_ml + (pb + j) * 2);
        lj[j] = sub(part_ml + (pb + j) * 2 + 1);
        oj[j] = sub(part_o + (pb + j) * HD + e);
      }
    }
    float Mg = -1.0e30f;
#pragma unroll
    for (int j = 0; j < kBdAttnMaxSplits; ++j) Mg = fmaxf(Mg, mj[j]);
    float Lg = 0.f, Og = 0.f;
#pragma unroll
    for (int j = 0; j < kBdAttnMaxSplits; ++j) {
      const float cj = __builtin_amdgcn_exp2f(mj[j] - Mg);     // an empty split has sum 0
      Lg = fmaf(lj[j], cj, Lg);
      Og = fmaf(oj[j], cj, Og);
    }
    frag_store(o16, b, (h0 + r) * HD + e, (_Float16)(Og / Lg));
  }
}

// After block l1 (1-based), one workgroup per sequence b: s_b = cos(h_prev[b], h[b]) if the row
// is still in the backbone (recorded, and kept in s_of for k_bd_decide); h(l1) of the row is
// kept (hist, the debug view) and becomes the next block's h_prev; with decide != 0 the row's own
// exit decision (forced position, else s_b > tau; first hit at or above L_s, never at L -- the
// caller passes decide = 0 outside that range and when Eq. 1's batch rule decides); then the
// RMSNorm in front of the next GEMM (the next block's attention norm, or the final norm) into
// xf in fragment order -- its sum of squares is the similarity's <h, h>.
__global__ __launch_bounds__(512) void k_bd_block_end(float *h_prev, float *__restrict__ h, int d, int l1, int L,
                                                      SeqState st, float *s_of, float *sims /* [n][L] of this step */,
                                                      float *hist /* [n][d] */, int decide, float tau,
                                                      const void *next_gain, float eps, _Float16 *xf,
                                                      const float *__restrict__ part, int n_part) {
  __shared__ float red[32];
  const int b = blockIdx.x;
  const bool live = st.river[b] == 0;
  float *row = h + (size_t)b * d;
  float p3[3] = {0.f, 0.f, 0.f};
  // one run: the sums of Eq. 1's similarity, h(l1) into h_prev and the debug view
  auto take = [&](int k) {
    const float4 a0 = *(const float4 *)(h_prev + (size_t)b * d + k), a1 = *(const float4 *)(h_prev + (size_t)b * d + k + 4);
    const Run8 c = load_run8(row, part, n_part, b, d, k);      // (adds the down projection's partial sums)
    const float a[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      p3[0] = fmaf(a[j], c.v[j], p3[0]); p3[1] = fmaf(a[j], a[j], p3[1]); p3[2] = fmaf(c.v[j], c.v[j], p3[2]);
    }
    const float4 c0 = make_float4(c.v[0], c.v[1], c.v[2], c.v[3]), c1 = make_float4(c.v[4], c.v[5], c.v[6], c.v[7]);
    *(float4 *)(h_prev + (size_t)b * d + k) = c0; *(float4 *)(h_prev + (size_t)b * d + k + 4) = c1;
    *(float4 *)(hist + (size_t)b * d + k) = c0; *(float4 *)(hist + (size_t)b * d + k + 4) = c1;
    return c;
  };
  const bool gain_wide = ((uintptr_t)next_gain & 15) == 0;
  Run8 keep[kRowKeep], kg[kRowKeep];                           // (gains with the row: one round trip)
#pragma unroll
  for (int i = 0; i < kRowKeep; ++i) {
    const int k = threadIdx.x * 8 + i * (int)blockDim.x * 8;
    if (k < d) kg[i] = ld_gain8(next_gain, k, gain_wide);
    if (k < d) keep[i] = take(k);
  }
  for (int k = threadIdx.x * 8 + kRowKeep * (int)blockDim.x * 8; k < d; k += (int)blockDim.x * 8) (void)take(k);
  block_sum_k<3>(p3, red);
  if (live && threadIdx.x == 0) {
    float s = 0.f;
    if (p3[1] > 0.f && p3[2] > 0.f) s = fminf(1.0f, fmaxf(-1.0f, p3[0] / (sqrtf(p3[1]) * sqrtf(p3[2]))));
    s_of[b] = s;
    sims[(size_t)b * L + (l1 - 1)] = s;
    if (decide) {
      const int f = st.forced[b];
      if (f >= 0 ? f == l1 : s > tau) { st.river[b] = 1; st.exit_pos[b] = l1; }
    }
  }
  const float r = 1.0f / sqrtf(p3[2] / (float)d + eps);
#pragma unroll
  for (int i = 0; i < kRowKeep; ++i) {
    const int k = threadIdx.x * 8 + i * (int)blockDim.x * 8;
    if (k < d) norm_store_run8(keep[i], r, kg[i], xf, b, k);
  }
  for (int k = threadIdx.x * 8 + kRowKeep * (int)blockDim.x * 8; k < d; k += (int)blockDim.x * 8)    // updated by this thread itself above
    norm_store_run8(load_run8(row, nullptr, 0, b, d, k), r, ld_gain8(next_gain, k, gain_wide), xf, b, k);
}

// The exit decision after backbone block l1 from the similarities k_bd_block_end left (launched
// when Eq. 1's batch rule is in force).  rule 0: every
// sequence for itself (s_b > tau); rule 1: Eq. 1 as printed, the whole batch leaves together
// once min_b s_b > tau.  A forced exit position overrides the threshold for its sequence.
// First hit at or above L_s, never at L, strict '>'.  One wavefront.
__global__ void k_bd_decide(int n, int l1, int L, int min_exit, float tau, int rule, SeqState st,
                            const float *__restrict__ s_of) {
  if (threadIdx.x != 0 || l1 < min_exit || l1 >= L) return;
  bool all_pass = true;                                       // Eq. 1's minimum over the batch
  for (int b = 0; b < n; ++b)
    if (!st.river[b] && !(s_of[b] > tau)) all_pass = false;
  for (int b = 0; b < n; ++b) {
    if (st.river[b]) continue;
    const int f = st.forced[b];
    const bool go = f >= 0 ? f == l1 : (rule == 1 ? all_pass : s_of[b] > tau);
    if (go) { st.river[b] = 1; st.exit_pos[b] = l1; }
  }
}

// Greedy token of every sequence (lowest index on ties) and its record.  kBdArgmaxChunks workgroups per sequence scan a chunk of the
// row each and publish (value, index); the last one to arrive takes the best of them in chunk
// order (part: [n][chunks][2], tickets: [n], zero between launches).
constexpr int kBdArgmaxChunks = 16;
// host_row (pinned; null: nobody waits): [max_batch] tokens, [max_batch] exits, [n][L] similarities
__global__ __launch_bounds__(256) void k_bd_argmax(const float *__restrict__ logits, int vocab, SeqState st,
                                                   int *rec_token, int *rec_exit, float *part, unsigned int *tickets,
                                                   int *host_row, int max_batch, const float *sims, int L) {
  __shared__ float red[64];
  __shared__ int flag;
  const int b = blockIdx.x / kBdArgmaxChunks, c = blockIdx.x % kBdArgmaxChunks;
  const int per = ((vocab + kBdArgmaxChunks - 1) / kBdArgmaxChunks + 3) / 4 * 4;
  const int i_begin = c * per, i_end = min(vocab, i_begin + per);
  float best = -INFINITY;
  int besti = 0x7fffffff;
  const float *row = logits + (size_t)b * vocab;
  // eight loads in flight per thread (the scan is a chain of load latencies otherwise)
  for (int i0 = i_begin + threadIdx.x; i0 < i_end; i0 += 8 * blockDim.x) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = i0 + u * blockDim.x;
      v[u] = i < i_end ? row[i] : -INFINITY;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = i0 + u * (int)blockDim.x;
      argmax_take(best, besti, v[u], i < i_end ? i : 0x7fffffff);
    }
  }
  block_argmax(best, besti, red);
  float *mine = part + ((size_t)b * kBdArgmaxChunks + c) * 2;
  if (threadIdx.x == 0) { pub(mine, best); pub(mine + 1, __int_as_float(besti)); }
  if (!last_arriver(tickets + b, kBdArgmaxChunks, &flag)) return;
  // the chunks' maxima, a lane each (one thread after the other's round trip: 16 of them)
  best = -INFINITY;
  besti = 0x7fffffff;
  if (threadIdx.x < 64) {
    if (threadIdx.x < kBdArgmaxChunks) {
      const float *pj = part + ((size_t)b * kBdArgmaxChunks + threadIdx.x) * 2;
      argmax_take(best, besti, sub(pj), __float_as_int(sub(pj + 1)));
    }
#pragma unroll
    for (int o = kBdArgmaxChunks / 2; o > 0; o >>= 1) {
      const float v2 = __shfl_xor(best, o);
      const int i2 = __shfl_xor(besti, o);
      argmax_take(best, besti, v2, i2);
    }
  }
  if (threadIdx.x == 0) {
    st.token[b] = besti;
    rec_token[b] = besti;
    rec_exit[b] = st.exit_pos[b];
    if (host_row) { host_store(host_row + b, besti); host_store(host_row + max_batch + b, st.exit_pos[b]); }
  }
  if (host_row)
    for (int i = threadIdx.x; i < L; i += blockDim.x)
      host_store(host_row + 2 * max_batch + b * L + i, __float_as_int(sims[(size_t)b * L + i]));
}

}  // namespace bd
}  // namespace river
