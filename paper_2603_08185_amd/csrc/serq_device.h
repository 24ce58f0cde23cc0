// Device-side helpers shared by the SERQ kernels (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/serq.h"

namespace serq {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
// native vectors for anything staged in registers (aggregate vector structs
// would be kept in memory and moved around with memcpy)
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------------------
// Private packed layouts (all produced by the library itself).
//
// Weight blob Wq: [N/32][K/64] fragments of 1 KiB.  Fragment (nb,kb) holds the
// 32 output channels n = 32*nb + (lane & 31) and the 64 input channels
// 64*kb .. 64*kb+63.  Lane `lane` owns 16 bytes = 4 dwords; dword d covers the
// 8 channels k0 = 64*kb + 32*(lane>>5) + 8*d .. k0+7, and byte j of that dword
// holds channel k0+j in its low nibble and channel k0+4+j in its high nibble
// (two's complement).  One wave-wide 16-byte load therefore brings in exactly
// the A operands of two 32x32x32 int8 MFMAs, and
//      lo = (w << 4) & 0xF0F0F0F0,   hi = w & 0xF0F0F0F0
// are operand dwords holding 16*q for channels k0..k0+3 and k0+4..k0+7.
//
// Activations Xq, 8-bit: int8 [M][K], natural order.
// Activations Xq, 4-bit: [M][K/2] bytes; each dword covers 8 consecutive
// channels with the same nibble interleave as the weights.
//
// Low-rank blob Rp: [N/32][r/16] fragments of 1 KiB; lane owns 8 consecutive
// 16-bit elements R[16*jb + 8*(lane>>5) + p][32*nb + (lane & 31)], p = 0..7:
// the A operand of one 32x32x16 f16/bf16 MFMA.
// ---------------------------------------------------------------------------

constexpr uint32_t kNibMask = 0xF0F0F0F0u;

// 16x the signed nibbles of w, as two int8x4 operand dwords.
__device__ __forceinline__ void unpack16(uint32_t w, int& lo, int& hi) {
  lo = (int)((w << 4) & kNibMask);
  hi = (int)(w & kNibMask);
}

// One 16-byte packed fragment piece -> the operands of two K=32 MFMA steps.
__device__ __forceinline__ void unpack_frag(const u4& p, v4i& t0, v4i& t1) {
  int a, b;
  unpack16(p.x, a, b); t0.x = a; t0.y = b;
  unpack16(p.y, a, b); t0.z = a; t0.w = b;
  unpack16(p.z, a, b); t1.x = a; t1.y = b;
  unpack16(p.w, a, b); t1.z = a; t1.w = b;
}

__device__ __forceinline__ v4i as_v4i(const u4& p) { return __builtin_bit_cast(v4i, p); }

// storage-type helpers -------------------------------------------------------
__device__ __forceinline__ float bf16_to_f32(uint16_t u) { return __uint_as_float(((uint32_t)u) << 16); }
__device__ __forceinline__ float f16_to_f32(uint16_t u) { return (float)__builtin_bit_cast(_Float16, u); }
// silu(g) * u in fp32 with the hardware's exp2 and reciprocal (an ulp each, so the product is good to
// a few ulps; the correctly rounded expf and an IEEE division made the fused quantisers VALU-bound);
// g -> -inf gives g * 0 = -0, g -> +inf gives g * 1
__device__ __forceinline__ float silu_mul(float g, float u) {
  return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u;
}

// ---- helpers shared by several kernels -------------------------------------------------------------
// LDS byte address of a pointer into shared memory
__device__ __forceinline__ uint32_t lds_addr(const void* ptr) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)ptr;
}
// Direct global -> LDS load, 16 bytes per lane, no staging registers: global (sbase + voff) lands at
// LDS (lds_base_uniform + 16 * lane).  Counted by hand with vmcnt by the callers.
__device__ __forceinline__ void dma16(const void* sbase, uint32_t voff, uint32_t lds_base_uniform) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(lds_base_uniform), "v"(voff), "s"(sbase) : "memory", "m0");
}
// The same from an address of every lane's own.
__device__ __forceinline__ void dma16_at(const void* src, uint32_t lds_base_uniform) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(lds_base_uniform), "v"(src) : "memory", "m0");
}
// dma16 with 4 bytes per lane.
__device__ __forceinline__ void dma4(const void* sbase, uint32_t voff, uint32_t lds_base_uniform) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
               :: "s"(lds_base_uniform), "v"(voff), "s"(sbase) : "memory", "m0");
}
// dma16 by the active ones of the first four lanes (a test of the lane would be a branch).
__device__ __forceinline__ void dma64(const void* sbase, uint32_t voff, uint32_t lds_base_uniform) {
  uint64_t lanes;
  asm volatile("s_mov_b32 m0, %1\n\ts_and_saveexec_b64 %0, 15\n\tglobal_load_lds_dwordx4 %2, %3\n\ts_mov_b64 exec, %0"
               : "=&s"(lanes) : "s"(lds_base_uniform), "v"(voff), "s"(sbase) : "memory", "m0", "scc");
}
// 16 bytes of E2M1 codes as an operand of the block-scaled MFMA (its FP4 forms read the first 16 bytes only)
__device__ __forceinline__ v8i fp4_operand(const u4& v) {
  const v4i q = as_v4i(v);
  return __builtin_shufflevector(q, q, 0, 1, 2, 3, -1, -1, -1, -1);
}
// 8 consecutive channels (piece `chunk`) of a row stored as XDT: as loaded, and as fp32.  In two steps, so that a thread can have all
// its pieces under way before it looks at the first one.
template <int XDT> struct Raw8 { u4 a; };
template <> struct Raw8<SERQ_F32> { u4 a, b; };
template <int XDT>
__device__ __forceinline__ Raw8<XDT> fetch8(const void* row, int chunk) {
  Raw8<XDT> r;
  if constexpr (XDT == SERQ_F32) {
    r.a = ((const u4*)row)[2 * (size_t)chunk];
    r.b = ((const u4*)row)[2 * (size_t)chunk + 1];
  } else {
    r.a = ((const u4*)row)[chunk];
  }
  return r;
}
template <int XDT>
__device__ __forceinline__ void values8(const Raw8<XDT>& r, float v[8]) {
  if constexpr (XDT == SERQ_F32) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[i] = __uint_as_float(r.a[i]);
      v[4 + i] = __uint_as_float(r.b[i]);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t w = r.a[i];
      if constexpr (XDT == SERQ_BF16) {
        v[2 * i] = __uint_as_float(w << 16);
        v[2 * i + 1] = __uint_as_float(w & 0xffff0000u);
      } else {
        v[2 * i] = f16_to_f32((uint16_t)(w & 0xffffu));
        v[2 * i + 1] = f16_to_f32((uint16_t)(w >> 16));
      }
    }
  }
}
// Threads per row of a quantiser that needs the whole row before its first code (integer, asymmetric), for M rows of nchunk pieces.
// Few rows are bound by a row's own latency and want its pieces side by side; many short ones by the rate at which waves start and
// want fewer threads with two or three pieces each.  In between the arithmetic counts, most of all the gated product's, and a thread
// whose last piece lies past the row does it for nothing: up to 896 pieces the workgroup is little larger than the row needs.
// The gated product and the asymmetric quantiser have more to do per piece, so that their short rows are few for longer.  Without
// flattening factors more codes of 16-bit input take the long way (an exact division), and waves that share a SIMD evenly count for few
// rows.  Measured (us, 8-bit codes, with the factors unless stated; threads x pieces; int: integer, glu: its gated product, asym):
//   up to 128 pieces, 64 x 2 / 128 / 256: int K = 1024 M = 1 2.0 / 2.0 / 2.1, M = 1000 3.05 / 3.28 / 3.68, M = 4096 5.1 / 6.8 / 7.9
//   129 .. 256, 128 x 2 / 256 x 1: K = 2048 int M = 200 2.44 / 2.39, M = 549 2.67 / 3.04, M = 4096 6.3 / 9.5; glu M = 400 3.10 / 2.94,
//   M = 549 3.20 / 3.44; asym M = 400 2.87 / 2.59, M = 1000 3.15 / 3.31
//   257 .. 384, 128 x 3 / 192 x 2 / 256 x 2: K = 3072 int M = 1 2.13 / 1.94 / 1.99, M = 1000 3.47 / 3.37 / 3.55, M = 4096 8.16 / 7.76 /
//   8.14; glu M = 549 3.89 / 3.72 / 3.75, M = 1000 4.12 / 4.11 / 4.53; asym M = 1000 3.82 / 3.72 / 3.98
//   385 .. 512, 128 / 192 x 3 / 256 x 2: K = 4096 int M = 300 3.21 / 3.08 / 2.74, M = 4096 9.9 / 9.7 / 9.4; glu M = 549 4.60 / 4.63 / 3.93
//   513 .. 640, 256 x 3 / 320 x 2 / 512 x 2: K = 4352 int M = 300 3.06 / 2.88 / 3.15, M = 549 3.53 / 3.32 / 3.62, M = 4096 10.3 / 10.4 /
//   12.0; glu M = 549 4.61 / 4.20 / 4.97, M = 1649 8.5 / 8.0 / 9.6, M = 4096 15.8 / 15.1 / 18.3; asym M = 1000 5.20 / 4.97 / 5.54; without
//   factors, 320 x 2 / 512 x 2: K = 5120 asym M = 24 3.57 / 2.85, M = 200 3.45 / 3.02, int M = 200 3.16 / 2.91
//   641 .. 768, 256 x 3 / 384 x 2 / 512 x 2: K = 6144 int M = 64 2.75 / 2.62 / 2.62, M = 549 3.85 / 3.80 / 3.89, M = 4096 13.0 / 13.4 / 13.8; glu
//   M = 400 4.16 / 4.34 / 4.29, M = 549 4.99 / 5.00 / 5.24, M = 1649 9.4 / 9.8 / 10.4; asym M = 400 3.68 / 3.84 / 3.75, M = 4096 13.9 / 15.4 / 16.0;
//   without factors, 384 x 2 / 512 x 2: asym M = 200 3.47 / 3.08, int M = 24 3.11 / 2.76
//   769 .. 896, 448 x 2 / 512 x 2: K = 6656 glu M = 1000 7.04 / 7.39, M = 4096 20.1 / 20.6
//   897 .. 1024, 256 / 512 x 2 / 768: K = 8192 int M = 64 3.01 / 2.67 / 2.77, M = 1000 6.9 / 6.5 / 7.4; glu M = 1000 8.3 / 7.9 / 9.3
//   1025 .. 1152, 384 x 3 / 512 x 3 / 768 x 2: K = 9216 glu M = 400 5.53 / 5.41 / 5.37, M = 549 6.83 / 7.15 / 7.06, M = 4096 30.2 / 30.9 / 33.3;
//   without factors, 384 x 3 / 512 x 3: int M = 700 7.61 / 7.14, asym 8.80 / 7.96
//   1153 .. 1536, 512 x 3 / 768 x 2: int K = 10240 M = 1 2.82 / 2.70, M = 512 5.91 / 5.70, M = 700 6.71 / 6.85; glu K = 12288 M = 400 6.10 /
//   6.05, M = 4096 38.2 / 39.6; asym K = 12288 M = 200 4.56 / 4.33
//   1537 .. 2048, 512 x 4 / 1024 x 2: int K = 14336 M = 16 3.58 / 3.34, M = 512 6.77 / 6.56, M = 1000 10.8 / 11.2; glu M = 16 4.55 / 4.20;
//   asym M = 200 4.89 / 4.64, M = 400 7.02 / 7.10
//   2049 .. 4096, walked twice by 256 / kept by 1024 x 3 or 4: int K = 20480 M = 1 6.4 / 3.8, M = 1000 20.7 / 14.5, M = 4096 79.7 /
//   49.9; glu K = 28672 M = 400 23.7 / 16.5; asym K = 16448 M = 2000 33.2 / 24.3
//   more, walked by 256 / 512: int K = 32832 M = 1 8.8 / 6.3, M = 2000 65.2 / 61.4; K = 65536 M = 400 29.0 / 29.4, M = 4096 260 / 246
enum class Quantizer { kPlain, kGated, kAsym };
inline int quantizer_threads(Quantizer q, int nchunk, int64_t M) {
  if (nchunk <= 128) return 64;
  if (nchunk <= 256) return M <= (q == Quantizer::kPlain ? 256 : 512) ? 256 : 128;
  if (nchunk <= 384) return 192;
  if (nchunk <= 512) return 256;
  if (nchunk <= 768) return M <= 384 ? 512 : nchunk <= 640 ? 320 : 256;
  if (nchunk <= 896) return 448;
  if (nchunk <= 1024) return 512;
  if (nchunk <= 2048) {
    if (M <= (q == Quantizer::kAsym ? 256 : 512)) return nchunk <= 1536 ? 768 : 1024;
    return q == Quantizer::kGated && nchunk <= 1152 ? 384 : 512;
  }
  return nchunk <= 4096 ? 1024 : 512;
}
// Its launch: LAUNCH(threads, pieces), 0 pieces for a row that is walked twice.
#define SERQ_QUANTIZER_LAUNCH(threads, per, LAUNCH)        \
  do {                                                     \
    if ((threads) == 64) LAUNCH(64, 2);                    \
    else if ((threads) == 128) LAUNCH(128, 2);             \
    else if ((threads) == 192) LAUNCH(192, 2);             \
    else if ((threads) == 256 && (per) == 1) LAUNCH(256, 1); \
    else if ((threads) == 256 && (per) == 2) LAUNCH(256, 2); \
    else if ((threads) == 256) LAUNCH(256, 3);             \
    else if ((threads) == 320) LAUNCH(320, 2);             \
    else if ((threads) == 384) LAUNCH(384, 3);             \
    else if ((threads) == 448) LAUNCH(448, 2);             \
    else if ((threads) == 768) LAUNCH(768, 2);             \
    else if ((threads) == 1024 && (per) == 2) LAUNCH(1024, 2); \
    else if ((threads) == 1024 && (per) == 3) LAUNCH(1024, 3); \
    else if ((threads) == 1024) LAUNCH(1024, 4);           \
    else if ((per) <= 2) LAUNCH(512, 2);                   \
    else if ((per) == 3) LAUNCH(512, 3);                   \
    else if ((per) == 4) LAUNCH(512, 4);                   \
    else LAUNCH(512, 0);                                   \
  } while (0)
// Rows of one launch: the threads along a grid are counted in 32 bits, without an error where that wraps round, and a row takes up to
// 1024.
constexpr int64_t kLaunchRows = 1 << 21;
// The rows of a quantiser: pieces `chunk`, chunk + KT, ... (NC of them) of a row of nchunk, flattened: x * s_inv, or silu(x) * u * s_inv.
// All loads -- the row, the second row, the flattening factors -- are requested before the first value is used, piece by piece: the first
// one's arithmetic runs while the others are on their way (gated product K = 4096 M = 4096, all of the row first 14.0, piece by piece 13.8;
// K = 12288 M = 1000 10.99 / 10.50; K = 14336 M = 1000 12.9 / 12.4).  Behind a test of each piece, as they were, every piece waited for
// its own loads, one after the other, and the factors for the row.  (Pieces past the row: its last one again.)  With 1024 threads, where a
// good part of the last round lies past the row, and with one piece each, the arithmetic is left out for pieces that no lane of the wave
// has: a wave has `pieces_of` them, and the values of the others are not set.  (Elsewhere the tests cost more than they spare: gated
// product, K = 11008 M = 1024, 512 threads 10.9 / 11.4 us without / with them; 1024 threads, where they pay, M = 256 5.3 / 5.0.)
template <int KT, int NC>
__device__ __forceinline__ int pieces_of(int chunk, int nchunk) {
  if (KT < 1024 && NC > 1) return NC;
  const int left = nchunk - __builtin_amdgcn_readfirstlane(chunk);
  return left <= 0 ? 0 : (left + KT - 1) / KT;
}
// FORM: with the factors (1), without (0), or by a test of s_inv (2)
template <int XDT, int KT, int NC, bool GLU, int FORM>
__device__ __forceinline__ void fetch_rows_form(const void* row, const void* urow, const float* s_inv, int chunk, int nchunk, float (&v)[NC][8]) {
  const bool flat = FORM == 2 ? s_inv != nullptr : FORM == 1;
  Raw8<XDT> x[NC], u[NC];
  int at[NC];
  const int nc = pieces_of<KT, NC>(chunk, nchunk);
#pragma unroll
  for (int c = 0; c < NC; ++c) at[c] = min(chunk + c * KT, nchunk - 1);
  v4f sa[NC], sb[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    x[c] = fetch8<XDT>(row, at[c]);
    if constexpr (GLU) u[c] = fetch8<XDT>(urow, at[c]);
    if (flat) {
      sa[c] = ((const v4f*)s_inv)[2 * (size_t)at[c]];
      sb[c] = ((const v4f*)s_inv)[2 * (size_t)at[c] + 1];
    }
  }
  __builtin_amdgcn_sched_barrier(0);                    // (else the compiler requests some of them behind the arithmetic of others)
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    if (c >= nc) continue;                              // uniform
    values8<XDT>(x[c], v[c]);
    if constexpr (GLU) {
      float t[8];
      values8<XDT>(u[c], t);
#pragma unroll
      for (int i = 0; i < 8; ++i) v[c][i] = silu_mul(v[c][i], t[i]);
    }
    if (flat) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[c][i] *= sa[c][i];
        v[c][4 + i] *= sb[c][i];
      }
    }
  }
}
// Behind a test of s_inv the waits count as if the factors were not under way, and the first piece waits for most of the second.  The
// gated product, whose arithmetic is worth starting early, takes a path of its own with them and without (us, one path / two: K = 2560
// M = 549 3.60 / 3.45, K = 4096 M = 549 3.90 / 3.79; MXFP4 K = 3200 M = 4096 11.60 / 11.05); with more than two pieces a thread the
// registers that takes cost more (K = 10240 M = 549 7.3 / 7.6 with three), as without the product (K = 14336 M = 4096 8 % slower).
template <int XDT, int KT, int NC, bool GLU>
__device__ __forceinline__ void fetch_rows(const void* row, const void* urow, const float* s_inv, int chunk, int nchunk, float (&v)[NC][8]) {
  if constexpr (GLU && NC <= 2) {
    if (s_inv) fetch_rows_form<XDT, KT, NC, GLU, 1>(row, urow, s_inv, chunk, nchunk, v);
    else fetch_rows_form<XDT, KT, NC, GLU, 0>(row, urow, s_inv, chunk, nchunk, v);
  } else {
    fetch_rows_form<XDT, KT, NC, GLU, 2>(row, urow, s_inv, chunk, nchunk, v);
  }
}

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
  v2f x = {f, 0.0f};
  v2bf y = __builtin_convertvector(x, v2bf);
  return (uint16_t)(__builtin_bit_cast(uint32_t, y) & 0xffffu);
}
__device__ __forceinline__ uint32_t f32x2_to_bf16x2(float a, float b) {
  v2f x = {a, b};
  v2bf y = __builtin_convertvector(x, v2bf);
  return __builtin_bit_cast(uint32_t, y);
}
__device__ __forceinline__ uint32_t f32x2_to_f16x2(float a, float b) {
  v2f x = {a, b};
  v2h y = __builtin_convertvector(x, v2h);
  return __builtin_bit_cast(uint32_t, y);
}
__device__ __forceinline__ uint16_t f32_to_f16_rne(float f) {
  return __builtin_bit_cast(uint16_t, (_Float16)f);
}

template <int DT> struct Elem;
template <> struct Elem<SERQ_F32> {
  typedef float T;
  static __device__ __forceinline__ float ld(const void* p, size_t i) { return ((const float*)p)[i]; }
};
template <> struct Elem<SERQ_F16> {
  typedef uint16_t T;
  static __device__ __forceinline__ float ld(const void* p, size_t i) { return f16_to_f32(((const uint16_t*)p)[i]); }
};
template <> struct Elem<SERQ_BF16> {
  typedef uint16_t T;
  static __device__ __forceinline__ float ld(const void* p, size_t i) { return bf16_to_f32(((const uint16_t*)p)[i]); }
};

__device__ __forceinline__ float ld_any(const void* p, int dt, size_t i) {
  if (dt == SERQ_F32) return ((const float*)p)[i];
  if (dt == SERQ_F16) return f16_to_f32(((const uint16_t*)p)[i]);
  return bf16_to_f32(((const uint16_t*)p)[i]);
}

// 8 signed codes -> 8 exact 16-bit floats (|code| <= 128 is exact in both formats).
// `lo`,`hi` hold the codes as bytes c0..c3 / c4..c7.
__device__ __forceinline__ u4 codes8_to_16bit(int c[8], bool bf16) {
  u4 o;
  if (bf16) {
    o.x = f32x2_to_bf16x2((float)c[0], (float)c[1]);
    o.y = f32x2_to_bf16x2((float)c[2], (float)c[3]);
    o.z = f32x2_to_bf16x2((float)c[4], (float)c[5]);
    o.w = f32x2_to_bf16x2((float)c[6], (float)c[7]);
  } else {
    o.x = f32x2_to_f16x2((float)c[0], (float)c[1]);
    o.y = f32x2_to_f16x2((float)c[2], (float)c[3]);
    o.z = f32x2_to_f16x2((float)c[4], (float)c[5]);
    o.w = f32x2_to_f16x2((float)c[6], (float)c[7]);
  }
  return o;
}

// the 8 codes of channels k0..k0+7 from an 8-bit row (two dwords) ...
__device__ __forceinline__ void codes_from_a8(uint32_t d0, uint32_t d1, int c[8]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    c[j] = __builtin_amdgcn_sbfe((int)d0, 8 * j, 8);
    c[4 + j] = __builtin_amdgcn_sbfe((int)d1, 8 * j, 8);
  }
}
// ... and from one interleaved 4-bit dword.
__device__ __forceinline__ void codes_from_a4(uint32_t d, int c[8]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    c[j] = __builtin_amdgcn_sbfe((int)d, 8 * j, 4);
    c[4 + j] = __builtin_amdgcn_sbfe((int)d, 8 * j + 4, 4);
  }
}

// Exchanges within a wave without going through LDS, as a shuffle does (quantisers, us, shuffles / these: K = 4096 M = 1 2.44 / 2.26,
// M = 4096 11.5 / 11.2, K = 14336 M = 64 4.00 / 3.82; asymmetric K = 14336 M = 1 3.63 / 3.40).
// lanes 1, 2 apart, then the mirror images of 8 and of 16 lanes: after all four, every lane of 16 has met all the others
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  const int i = __float_as_int(v);
  return __int_as_float(__builtin_amdgcn_update_dpp(i, i, CTRL, 0xf, 0xf, false));
}
constexpr int kDpp1 = 0xB1, kDpp2 = 0x4E, kDppMirror8 = 0x141, kDppMirror16 = 0x140;
// op over the 64 lanes of a wave, the result in all of them (op: commutative and associative)
template <class Op>
__device__ __forceinline__ float wave_reduce(float v, const Op& op) {
  v = op(v, dpp<kDpp1>(v));
  v = op(v, dpp<kDpp2>(v));
  v = op(v, dpp<kDppMirror8>(v));
  v = op(v, dpp<kDppMirror16>(v));
  uint32_t i = __float_as_uint(v);
  const auto a = __builtin_amdgcn_permlane16_swap(i, i, false, false);   // rows of 16 lanes: 0 1 2 3 -> 0 0 2 2 and 1 1 3 3
  v = op(__uint_as_float(a[0]), __uint_as_float(a[1]));
  i = __float_as_uint(v);
  const auto b = __builtin_amdgcn_permlane32_swap(i, i, false, false);   // halves: 0 1 -> 0 0 and 1 1
  return op(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float wave_max(float v) {
  return wave_reduce(v, [](float a, float b) { return fmaxf(a, b); });
}

// Number of compute units of the current device, asked on every call;
// 256 if the runtime cannot say.
inline int device_cu_count() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
    n = 256;
  return n;
}

// ---------------------------------------------------------------------------
// host-side launchers implemented in the individual .hip files
// ---------------------------------------------------------------------------
struct LinearArgs {
  const uint8_t* Xq; const float* scale; int abits;
  const u4* Wq; const float* wscale;
  int s_begin; int r; const u4* Rp; int r_dtype;
  const float* rscale;                  // r_dtype == SERQ_I4: the per-channel scales inside the blob Rp
  int M, N, K;
  void* Y; int y_dtype; int64_t ldy;
  int32_t* acc_out; int64_t ldacc;      // non-NULL: store raw accumulators instead of Y
  void* workspace; size_t workspace_bytes;
  int splitk; int groupm; int coltiles; int skinny_waves;
};

size_t skinny_workspace_bytes(int N);
int launch_skinny(const LinearArgs& a, hipStream_t st);
int launch_mfma(const LinearArgs& a, hipStream_t st);
bool mid_wanted(const LinearArgs& a);
int launch_mid(const LinearArgs& a, hipStream_t st);
size_t mfma_split_workspace_bytes(int M, int N, int K, int abits, int forced);
int launch_quantize_act(const void* X, const void* U, int x_dtype, const float* s_inv, int64_t M, int K, int64_t ldx,
                        int64_t ldu, int abits, void* Xq, float* scale, hipStream_t st);

int launch_mfma_peak(const void* operands, int iters, int workgroups, void* sink, hipStream_t st);
int launch_mfma_fp4_peak(const void* operands, int iters, int workgroups, int scale_a, int scale_b, void* sink,
                         hipStream_t st);
int launch_read_peak(const void* src, size_t bytes, int workgroups, void* sink, hipStream_t st);

// the layer with group-128 weight scales (grouped.hip, grouped_mid.hip)
struct G128Args {
  const uint8_t* Xq; const float* scale; const int32_t* zero;
  const u4* Wq; const uint16_t* gsc; const float* wsum;
  const u4* Rp; int r_dtype; int s_begin; int r;
  int M, N, K;
  void* Y; int y_dtype; int64_t ldy;
};
bool g128_mid_wanted(const G128Args& a, int abits);
int launch_g128_mid(const G128Args& a, int abits, hipStream_t st);
// MXFP4 path (mx.hip, gemm_mx.hip)
struct MxLinearArgs {
  const uint8_t* Xq; const uint8_t* xsc;
  const u4* Wq; const uint8_t* wsc;
  int s_begin; int r; const u4* Rq; const uint8_t* rsc;
  int M, N, K;
  void* Y; int y_dtype; int64_t ldy;
  int coltiles;
  int splitk;                       // K slices: per channel block (decode kernel) or per tile (0 = choose, 1 = none)
  void* workspace; size_t workspace_bytes;
};
size_t mx_split_workspace_bytes(int M, int N, int K, int forced);
int launch_mx_quantize_act(const void* X, const void* U, int x_dtype, const float* s_inv, int64_t M, int K, int64_t ldx,
                           int64_t ldu, void* Xq, uint8_t* xsc, hipStream_t st);
int mx_pack_weights_impl(const void* W, int w_dtype, const float* s, const int32_t* perm, int N, int K, int r,
                         void* Wq, uint8_t* wsc, void* Rq, uint8_t* rsc, hipStream_t st);
int mx_unpack_weights_impl(const void* Wq, const uint8_t* wsc, int N, int K, uint8_t* codes, uint8_t* E, hipStream_t st);
int mx_unpack_act_impl(const void* Xq, const uint8_t* xsc, int64_t M, int K, uint8_t* codes, uint8_t* E, hipStream_t st);
int launch_mx_linear(const MxLinearArgs& a, hipStream_t st);
int launch_skinny_mx(const MxLinearArgs& a, hipStream_t st);
bool mx_mid_wanted(const MxLinearArgs& a);
int launch_mx_mid(const MxLinearArgs& a, hipStream_t st);
size_t skinny_mx_workspace_bytes(int N);

int pack_weights_impl(const void* W, int w_dtype, const float* s, const int32_t* perm_in, int N, int K, int r,
                      void* Wq_out, float* wscale_out, int32_t* perm_out, float* s_inv_out, void* R_out,
                      int r_dtype, void* Rp_out, hipStream_t st);
int prepare_perm_impl(const void* W, int w_dtype, const float* s, const int32_t* perm_in, int N, int K,
                      int32_t* perm_out, float* s_inv_out, hipStream_t st);
int pack_lowrank_impl(void* R, int N, int r, void* Rp, bool unpack, hipStream_t st);
size_t lowrank_q4_frag_bytes(int N, int r);
int pack_lowrank_q4_impl(const void* R, int r_dtype, int N, int r, void* Rq, hipStream_t st);
int unpack_lowrank_q4_impl(const void* Rq, int N, int r, int8_t* codes, float* rscale, hipStream_t st);
int unpack_weights_impl(const void* Wq, int N, int K, int8_t* out, hipStream_t st);
int unpack_act_impl(const void* Xq, int abits, int64_t M, int K, int8_t* out, hipStream_t st);

}  // namespace serq
