// The layer in the paper's accuracy-table setting (Sec. 4.1, implementation details): weights quantised
// in groups of 128 input channels (round-to-nearest, symmetric INT4, one 16-bit scale per output channel
// and group), activations per token with round-to-nearest ASYMMETRIC integer quantisation:
//
//   x^[m,k] = scale[m] (Xq[m,k] - zero[m]),      w^[n,k] = gscale[n, k/128] Wq[n,k],
//   Y[m,n]  = sum_k x^[m,k] w^[n,k] + sum_{j<r} x^[m,S_j] R[j,n]                      (Eq. 2 + Eq. 7, first line)
//           = scale[m] ( sum_g gscale[n,g] acc_g[m,n] - zero[m] wsum[n] + sum_j (Xq[m,S_j] - zero[m]) R[j,n] ),
//   acc_g[m,n] = sum_{k in group g} Xq[m,k] Wq[n,k]  (exact, INT32),   wsum[n] = sum_k w^[n,k]  (offline).
//
// The integer sums run on the int8 MFMA exactly as in the per-channel path; what changes is that the
// INT32 tile is folded into an fp32 tile after every group of 128 channels (one convert and one fused
// multiply-add per element and group -- the vector unit works about as long as the matrix unit), and the
// zero point becomes a rank-one term of the epilogue.  The rank-r term takes the re-centred codes
// (Xq - zero, at most 255 in magnitude: exact in bf16 and fp16).
//
// This file holds the whole variant: the asymmetric quantiser, the offline preparation, a
// weight-streaming kernel for M <= 32 and an LDS-tiled kernel above, and their C entry points.
// Weight codes use the fragment layout of the per-channel path (serq_unpack_weights reads them back);
// group scales: [N/32][K/128][32 channels] fp16.
#include <type_traits>

#include "gemm_tile.h"
#include "serq_device.h"

namespace serq {
namespace {

constexpr int kGroup = 128;

__device__ __forceinline__ float f16bits_to_f32(uint16_t u) { return (float)__builtin_bit_cast(_Float16, u); }

// ---------------------------------------------------------------------------------------------------
// asymmetric per-token quantiser: lo = min(0, min v), hi = max(0, max v), scale = (hi - lo) / (2^n - 1),
// z = rne(-lo / scale), code = clip(rne(v / scale) + z, 0, 2^n - 1); stored re-centred by 2^(n-1).
// Every decision is IEEE fp32, as in the oracle.  One workgroup per token, the row kept in registers.
// ---------------------------------------------------------------------------------------------------
template <int KT>
__device__ __forceinline__ void block_minmax(float& lo, float& hi, float* red) {
  lo = wave_reduce(lo, [](float a, float b) { return fminf(a, b); });
  hi = wave_max(hi);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { red[2 * w] = lo; red[2 * w + 1] = hi; }
  __syncthreads();
  lo = red[0]; hi = red[1];
#pragma unroll
  for (int i = 1; i < KT / 64; ++i) { lo = fminf(lo, red[2 * i]); hi = fmaxf(hi, red[2 * i + 1]); }
}

// codes of 8 values: rne(v / sc) + z, clamped to [0, top], re-centred.  t = v * rcp(sc) decides unless it
// lies within 1.25 * 2^-22 max(|t|, 1) of a half-integer (then, and for tiny scales, the divisions are done).
template <int ABITS>
__device__ __forceinline__ void asym_codes8(const float v[8], float sc, float rsc, float z, int c[8]) {
  constexpr float top = (float)((1 << ABITS) - 1);
  constexpr float kMagic = 12582912.0f;
  float r[8], maxd = 0.0f, maxt = 1.0f;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float t = v[i] * rsc;
    r[i] = (t + kMagic) - kMagic;                       // round-half-to-even for |t| < 2^22
    maxd = fmaxf(maxd, fabsf(t - r[i]));
    maxt = fmaxf(maxt, fabsf(t));
  }
  if (sc < 1e-30f || !(maxt < 4194304.0f) || 0.5f - maxd < 2.98023223876953125e-07f * maxt) {
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = rintf(v[i] / sc);
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) c[i] = (int)fminf(fmaxf(r[i] + z, 0.0f), top) - (1 << (ABITS - 1));
}

template <int ABITS>
__device__ __forceinline__ void store_codes8(const int c[8], void* xq_row, int chunk) {
  if constexpr (ABITS == 8) {
    const uint32_t d0 = (c[0] & 0xff) | ((c[1] & 0xff) << 8) | ((c[2] & 0xff) << 16) | ((uint32_t)(c[3] & 0xff) << 24);
    const uint32_t d1 = (c[4] & 0xff) | ((c[5] & 0xff) << 8) | ((c[6] & 0xff) << 16) | ((uint32_t)(c[7] & 0xff) << 24);
    ((uint2*)xq_row)[chunk] = make_uint2(d0, d1);
  } else {
    uint32_t o = 0;                                     // byte j: code j (low nibble), code 4+j (high nibble)
#pragma unroll
    for (int j = 0; j < 4; ++j) o |= ((uint32_t)(c[j] & 0xf) | ((uint32_t)(c[4 + j] & 0xf) << 4)) << (8 * j);
    ((uint32_t*)xq_row)[chunk] = o;
  }
}

// KT = threads per row, NC = 16-byte pieces a thread keeps in registers (0: any K, the row is read twice)
template <int XDT, int ABITS, int KT, int NC>
__global__ __launch_bounds__(KT) void quantize_act_asym_kernel(const void* __restrict__ X, const float* __restrict__ s_inv,
                                                                 int K, int64_t ldx, void* __restrict__ Xq,
                                                                 float* __restrict__ scale, int32_t* __restrict__ zero) {
  __shared__ float red[2 * KT / 64];
  const int64_t m = blockIdx.x;
  const int nchunk = K >> 3;
  constexpr size_t esz = (XDT == SERQ_F32) ? 4 : 2;
  const char* row = (const char*)X + (size_t)m * (size_t)ldx * esz;
  char* xq_row = (char*)Xq + (size_t)m * ((size_t)K * ABITS / 8);
  constexpr float top = (float)((1 << ABITS) - 1);
  float lo = 0.0f, hi = 0.0f;                           // the range always contains 0
  constexpr int NB = NC > 0 ? NC : 4;                   // pieces under way at a time
  float v[NB][8];
  auto fetch = [&](int chunk) { fetch_rows<XDT, KT, NB, false>(row, nullptr, s_inv, chunk, nchunk, v); };
  auto range = [&](int chunk) {
    const int nc = pieces_of<KT, NB>(chunk, nchunk);
#pragma unroll
    for (int c = 0; c < NB; ++c)
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (c < nc) { lo = fminf(lo, v[c][i]); hi = fmaxf(hi, v[c][i]); }
  };
  if constexpr (NC > 0) {
    fetch(threadIdx.x);
    range(threadIdx.x);
  } else {
    for (int chunk = threadIdx.x; chunk < nchunk; chunk += NB * KT) {
      fetch(chunk);
      range(chunk);
    }
  }
  block_minmax<KT>(lo, hi, red);
  const float span = hi - lo;
  const float sc = span > 0.0f ? span / top : 1.0f;
  const float z = rintf(-lo / sc);
  if (threadIdx.x == 0) {
    scale[m] = sc;
    zero[m] = (int)z - (1 << (ABITS - 1));
  }
  const float rsc = __builtin_amdgcn_rcpf(sc);
  auto store = [&](int chunk0) {
#pragma unroll
    for (int c = 0; c < NB; ++c) {
      const int chunk = chunk0 + c * KT;
      if (chunk < nchunk) {
        int c8[8];
        asym_codes8<ABITS>(v[c], sc, rsc, z, c8);
        store_codes8<ABITS>(c8, xq_row, chunk);
      }
    }
  };
  if constexpr (NC > 0) {
    store(threadIdx.x);
  } else {
    for (int chunk = threadIdx.x; chunk < nchunk; chunk += NB * KT) {
      fetch(chunk);
      store(chunk);
    }
  }
}

template <int XDT, int ABITS>
int launch_asym_t(const void* X, const float* s_inv, int64_t M, int K, int64_t ldx, void* Xq, float* scale,
                  int32_t* zero, hipStream_t st) {
  const int nchunk = K >> 3;
  const int threads = quantizer_threads(Quantizer::kAsym, nchunk, M);
  const int per = (nchunk + threads - 1) / threads;
  dim3 grid((unsigned)M), block((unsigned)threads);
#define SERQ_QAA(KT, NC) \
  hipLaunchKernelGGL((quantize_act_asym_kernel<XDT, ABITS, KT, NC>), grid, block, 0, st, X, s_inv, K, ldx, Xq, scale, zero)
  SERQ_QUANTIZER_LAUNCH(threads, per, SERQ_QAA);
#undef SERQ_QAA
  return hipGetLastError() == hipSuccess ? SERQ_OK : SERQ_EHIP;
}

// ---------------------------------------------------------------------------------------------------
// offline preparation (not timed; written for clarity)
// ---------------------------------------------------------------------------------------------------
constexpr int kT = 256;

__device__ __forceinline__ float folded_w(const void* W, int w_dtype, const float* s, size_t n, int K, int k_orig) {
  float w = ld_any(W, w_dtype, n * (size_t)K + k_orig);
  if (s) w = w * s[k_orig];
  return w;
}
__device__ __forceinline__ int quant7(float w, float gs) {
  float t = rintf(w / gs);
  t = fminf(fmaxf(t, -7.0f), 7.0f);
  return (int)t;
}
__device__ __forceinline__ size_t gscale_index(size_t n, int g, int G) { return ((n >> 5) * G + g) * 32 + (n & 31); }

// one wave per (output channel, group): gscale = fp16(max |w| / 7) kept inside fp16's positive range; 1 for a zero group
__global__ __launch_bounds__(kT) void group_scale_kernel(const void* __restrict__ W, int w_dtype, const float* __restrict__ s,
                                                         const int32_t* __restrict__ perm, int N, int K,
                                                         uint16_t* __restrict__ gsc) {
  const int G = K / kGroup;
  const size_t gw = (size_t)blockIdx.x * (kT / 64) + (threadIdx.x >> 6);
  if (gw >= (size_t)N * G) return;
  const size_t n = gw / G;
  const int g = (int)(gw % G);
  const int l = threadIdx.x & 63;
  float m = fmaxf(fabsf(folded_w(W, w_dtype, s, n, K, perm[g * kGroup + l])),
                  fabsf(folded_w(W, w_dtype, s, n, K, perm[g * kGroup + 64 + l])));
  m = wave_max(m);
  if (l == 0) {
    float f = 1.0f;
    if (m > 0.0f) {
      f = (float)(_Float16)(m / 7.0f);
      f = fminf(fmaxf(f, 5.9604644775390625e-08f), 65504.0f);
    }
    gsc[gscale_index(n, g, G)] = __builtin_bit_cast(uint16_t, (_Float16)f);
  }
}

// one thread per packed dword of the weight blob (the fragment layout of the per-channel path)
__global__ __launch_bounds__(kT) void quant_pack_grouped_kernel(const void* __restrict__ W, int w_dtype,
                                                                const float* __restrict__ s, const int32_t* __restrict__ perm,
                                                                const uint16_t* __restrict__ gsc, int N, int K,
                                                                uint32_t* __restrict__ blob) {
  const size_t idx = (size_t)blockIdx.x * kT + threadIdx.x;
  if (idx >= (size_t)N * K / 8) return;
  const int d = idx & 3;
  const int lane = (idx >> 2) & 63;
  const size_t frag = idx >> 8;
  const int KB = K >> 6;
  const int kb = frag % KB;
  const size_t n = (frag / KB) * 32 + (lane & 31);
  const int k0 = kb * 64 + (lane >> 5) * 32 + d * 8;
  const float gs = f16bits_to_f32(gsc[gscale_index(n, k0 / kGroup, K / kGroup)]);
  uint32_t out = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int lo = quant7(folded_w(W, w_dtype, s, n, K, perm[k0 + j]), gs);
    const int hi = quant7(folded_w(W, w_dtype, s, n, K, perm[k0 + 4 + j]), gs);
    out |= ((uint32_t)(lo & 0xf) | ((uint32_t)(hi & 0xf) << 4)) << (8 * j);
  }
  blob[idx] = out;
}

// wsum[n] = sum_k gscale[n, k/128] * Wq[n,k], accumulated in fp64 (one workgroup per output channel)
__global__ __launch_bounds__(kT) void wsum_kernel(const void* __restrict__ W, int w_dtype, const float* __restrict__ s,
                                                  const int32_t* __restrict__ perm, const uint16_t* __restrict__ gsc,
                                                  int K, float* __restrict__ wsum) {
  __shared__ double red[kT];
  const size_t n = blockIdx.x;
  const int G = K / kGroup;
  double a = 0.0;
  for (int k = threadIdx.x; k < K; k += kT) {
    const float gs = f16bits_to_f32(gsc[gscale_index(n, k / kGroup, G)]);
    a += (double)gs * (double)quant7(folded_w(W, w_dtype, s, n, K, perm[k]), gs);
  }
  red[threadIdx.x] = a;
  __syncthreads();
  for (int o = kT / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) wsum[n] = (float)red[0];
}

// R[j,n] = W^[n,j] - gscale[n, j/128] * Wq[n,j] for the r leading channels (canonical and/or packed)
__global__ __launch_bounds__(kT) void residual_grouped_kernel(const void* __restrict__ W, int w_dtype, const float* __restrict__ s,
                                                              const int32_t* __restrict__ perm, const uint16_t* __restrict__ gsc,
                                                              int N, int K, int r, void* __restrict__ R_out, int r_dtype,
                                                              uint16_t* __restrict__ Rp_out) {
  const size_t idx = (size_t)blockIdx.x * kT + threadIdx.x;
  if (idx >= (size_t)r * N) return;
  const int j = idx / N;
  const size_t n = idx % N;
  const float gs = f16bits_to_f32(gsc[gscale_index(n, j / kGroup, K / kGroup)]);
  const float w = folded_w(W, w_dtype, s, n, K, perm[j]);
  const float res = __fmaf_rn(-gs, (float)quant7(w, gs), w);
  uint16_t h = 0;
  if (r_dtype == SERQ_BF16) h = f32_to_bf16_rne(res);
  else if (r_dtype == SERQ_F16) h = f32_to_f16_rne(res);
  if (R_out) {
    if (r_dtype == SERQ_F32) ((float*)R_out)[idx] = res;
    else ((uint16_t*)R_out)[idx] = h;
  }
  if (Rp_out) {
    const int JB = r >> 4;
    const int jb = j >> 4, g = (j >> 3) & 1, p = j & 7;
    Rp_out[(((n >> 5) * JB + jb) * 64 + (int)(n & 31) + 32 * g) * 8 + p] = h;
  }
}

__global__ __launch_bounds__(kT) void unpack_gscale_kernel(const uint16_t* __restrict__ gsc, int N, int G, float* __restrict__ out) {
  const size_t idx = (size_t)blockIdx.x * kT + threadIdx.x;
  if (idx >= (size_t)N * G) return;
  out[idx] = f16bits_to_f32(gsc[gscale_index(idx / G, (int)(idx % G), G)]);
}

inline unsigned blocks_for(size_t n) { return (unsigned)((n + kT - 1) / kT); }

// ---------------------------------------------------------------------------------------------------
// the layer
// ---------------------------------------------------------------------------------------------------
using GParams = G128Args;

// 8 re-centred codes (code - zero) of one lane as exact 16-bit floats; all zero for a lane without a token
// (in two steps, so that a loop can have the loads of several fragments in flight before it converts the first)
template <int ABITS>
__device__ __forceinline__ u2 lr_load(const uint8_t* xrow, int col) {
  if constexpr (ABITS == 8) return *(const u2*)(xrow + col);
  else return u2{*(const uint32_t*)(xrow + (col >> 1)), 0u};
}
template <int ABITS>
__device__ __forceinline__ u4 lr_convert(const u2& x, int zm, bool valid, bool bf) {
  int c[8];
  if constexpr (ABITS == 8) codes_from_a8(x.x, x.y, c);
  else codes_from_a4(x.x, c);
#pragma unroll
  for (int i = 0; i < 8; ++i) c[i] = valid ? c[i] - zm : 0;
  return codes8_to_16bit(c, bf);
}
// The same for a lane that always has a token (or a duplicate of one whose results are never stored: the columns
// of the MFMA are independent), in fewer vector operations: the codes are turned into unsigned bytes by flipping
// their sign bit, converted straight from the packed bytes, and re-centred by one subtraction (zero + the flipped
// bit's worth).  |code - zero| <= 255, so the fp32 values are whole numbers that both 16-bit formats hold exactly.
template <int ABITS>
__device__ __forceinline__ u4 lr_convert_packed(const u2& x, int zm, bool bf) {
  float f[8];
  if constexpr (ABITS == 8) {
    const uint32_t t0 = x.x ^ 0x80808080u, t1 = x.y ^ 0x80808080u;
    const float off = (float)(128 + zm);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      f[k] = (float)((t0 >> (8 * k)) & 0xffu) - off;
      f[4 + k] = (float)((t1 >> (8 * k)) & 0xffu) - off;
    }
  } else {
    // byte j of the dword: code j in the low nibble, code 4 + j in the high nibble
    const uint32_t t = x.x ^ 0x88888888u;
    const uint32_t lo = t & 0x0f0f0f0fu, hi = (t >> 4) & 0x0f0f0f0fu;
    const float off = (float)(8 + zm);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      f[k] = (float)((lo >> (8 * k)) & 0xffu) - off;
      f[4 + k] = (float)((hi >> (8 * k)) & 0xffu) - off;
    }
  }
  u4 o;
  if (bf) {
    o.x = f32x2_to_bf16x2(f[0], f[1]); o.y = f32x2_to_bf16x2(f[2], f[3]);
    o.z = f32x2_to_bf16x2(f[4], f[5]); o.w = f32x2_to_bf16x2(f[6], f[7]);
  } else {
    o.x = f32x2_to_f16x2(f[0], f[1]); o.y = f32x2_to_f16x2(f[2], f[3]);
    o.z = f32x2_to_f16x2(f[4], f[5]); o.w = f32x2_to_f16x2(f[6], f[7]);
  }
  return o;
}
__device__ __forceinline__ v16f mfma_lr16(const u4& r, const u4& x, v16f acc, bool bf) {
  if (bf) return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, r), __builtin_bit_cast(v8bf, x), acc, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, r), __builtin_bit_cast(v8h, x), acc, 0, 0, 0);
}

// ---- M <= 32: one workgroup of 8 waves per block of 32 output channels, weights streamed once ----------
// Wave w takes the groups w, w+8, ... NG at a time: the 1-KiB weight fragments, the groups' scales and
// the token codes are all requested before the first is used.  The tokens are the MFMA's row operand
// and the weights its column operand, so a lane holds ONE output channel (one group scale per lane) and
// its registers are tokens: register e of lane (c, g) is token 8*(e/4) + 4g + e%4 of channel c.  With M <= 8
// tokens only registers 0..3 carry anything, with M <= 16 registers 0..7, ...: the fold of a group's INT32
// tile into the fp32 tile touches 4*MQ registers (MQ = ceil(M/8)), not 16.
// The token codes come as whole lines, straight into the wave's own LDS region (16-byte pieces xor-swizzled per row), and
// are read back as operands: per lane from L2 they touch 32 lines an instruction.  They are requested before
// the weights, because loads retire in order, and one hand-counted wait on "all but the weights" covers them.
// What the end needs -- a fragment of the rank-r term per wave, scales, zero points, wsum -- is requested before the loop.
// The eight waves are added through LDS in a fixed order (run-to-run identical).
//
// Bound by the weight stream and, with many tokens, by staging the token rows in every workgroup.  Measured (us, token
// codes per lane from L2 and end operands requested late / this form, r = 128, W4A8, N x K, weights out of cache): 11008 x
// 4096 M = 1 8.8 / 7.2, M = 16 11.0 / 8.4, M = 32 14.9 / 10.4; 28672 x 8192 M = 1 29.5 / 22.4, M = 32 47.6 / 33.4.
constexpr int kPitch = 33;
constexpr int kSkinnyWaves = 8;
template <int ABITS, int MQ, int NG>
struct GSkinny {
  static constexpr int XROW = 128 * ABITS / 8;              // bytes of a token's codes of one group: 128 or 64
  static constexpr int RPI = 1024 / XROW;                   // token rows one direct load covers: 8 or 16
  static constexpr int NX = (8 * MQ + RPI - 1) / RPI;       // direct loads per group
  static constexpr int XG = NX * 1024;
  static constexpr int RED = 8 * MQ * kPitch * 4;           // a wave's partial sums, later in the same place
  static constexpr int REGION = NG * XG > RED ? NG * XG : (RED + 15) / 16 * 16;
  static __device__ __forceinline__ int swz(int row) { return ABITS == 8 ? ((row >> 1) & 7) : ((row >> 2) & 3); }
};
template <int ABITS, int MQ, int NG>
__global__ __launch_bounds__(64 * kSkinnyWaves) void serq_g128_skinny_kernel(const GParams p) {
  using T = GSkinny<ABITS, MQ, NG>;
  constexpr int SH = ABITS == 8 ? 4 : 8;
  constexpr float kInv = 1.0f / (float)(1 << SH);
  constexpr int NE = 4 * MQ;                                // live accumulator registers
  __shared__ __align__(16) uint8_t lds[kSkinnyWaves * T::REGION];
  const int tid = threadIdx.x, l = tid & 63, m = l & 31, g = l >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nb = blockIdx.x;
  const int KB = p.K >> 6, G = p.K >> 7;
  const uint32_t rowbytes = (uint32_t)p.K * ABITS / 8;
  const bool mv = m < p.M;
  const uint8_t* xrow = p.Xq + (size_t)(mv ? m : 0) * rowbytes;
  const u4* wfr = p.Wq + (size_t)nb * KB * 64 + l;
  const uint16_t* gsl = p.gsc + (size_t)nb * G * 32 + m;    // this lane's channel (lane & 31)
  uint8_t* my = lds + w * T::REGION;
  const uint32_t my_lds = __builtin_amdgcn_readfirstlane(lds_addr(my));
  const v16i kZero16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};

  // ---- what the end needs, requested first -----------------------------------------------------------
  const bool has_lr = p.r > 0 && p.Rp != nullptr;
  const bool bf = p.r_dtype == SERQ_BF16;
  const int JB = has_lr ? p.r >> 4 : 0;
  const u4* rfr = p.Rp + (size_t)nb * JB * 64 + l;
  const int zm = (p.zero && mv) ? p.zero[m] : 0;
  u4 rf = {0u, 0u, 0u, 0u};
  u2 xr = {0u, 0u};
  if (w < JB) {
    rf = rfr[(size_t)w * 64];
    xr = lr_load<ABITS>(xrow, p.s_begin + 16 * w + 8 * g);
  }
  constexpr int NQ = (256 * MQ + 64 * kSkinnyWaves - 1) / (64 * kSkinnyWaves);
  float sc_m[NQ];
  int z_m[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int mt = (tid >> 5) + q * 2 * kSkinnyWaves;
    sc_m[q] = mt < p.M ? p.scale[mt] : 0.0f;
    z_m[q] = (p.zero && mt < p.M) ? p.zero[mt] : 0;
  }
  const float wsum = p.wsum[nb * 32 + (tid & 31)];

  float accf[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) accf[e] = 0.0f;
  // this lane's piece of a direct load: row l / pieces-per-row of it, slot l % pieces-per-row
  constexpr int P = T::XROW / 16;
  const int xr0 = l / P;
  uint32_t xv[T::NX];
#pragma unroll
  for (int i = 0; i < T::NX; ++i) {
    const int row = xr0 + T::RPI * i;
    xv[i] = (uint32_t)(row < p.M ? row : p.M - 1) * rowbytes + 16u * ((l % P) ^ T::swz(row));   // rows past M: duplicates
  }
  // operand rows of this lane (rows that are not staged: any, their results are not used)
  const int mr = m < T::NX * T::RPI ? m : T::NX * T::RPI - 1;
  const uint8_t* xop = my + mr * T::XROW;
  const int xsw = T::swz(mr);
  auto group_mfma = [&](const u4& wa, const u4& wb, const uint8_t* xs, float gs) {
    v16i acc;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      v4i a0, a1, b0, b1;
      unpack_frag(u ? wb : wa, a0, a1);
      if constexpr (ABITS == 8) {
        b0 = *(const v4i*)(xs + 16 * ((4 * u + 2 * g) ^ xsw));
        b1 = *(const v4i*)(xs + 16 * ((4 * u + 2 * g + 1) ^ xsw));
      } else {
        unpack_frag(*(const u4*)(xs + 16 * ((2 * u + g) ^ xsw)), b0, b1);
      }
      // tokens first: rows of the result are tokens, columns (lanes) are channels; the group starts from zero
      if (u == 0) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(b0, a0, kZero16, 0, 0, 0);
      else acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(b0, a0, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(b1, a1, acc, 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < NE; ++e) accf[e] = __builtin_fmaf(gs, (float)acc[e], accf[e]);
  };
#pragma unroll 1
  for (int grp = w; grp < G; grp += NG * kSkinnyWaves) {
    u4 wv[NG][2];
    uint16_t gsv[NG];                                       // (converted where they are used: nothing waits for them here)
    int gq[NG];                                             // a wave without a q-th group repeats the first (unused)
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      gq[q] = grp + q * kSkinnyWaves < G ? grp + q * kSkinnyWaves : grp;
      gsv[q] = gsl[(size_t)gq[q] * 32];
    }
#pragma unroll
    for (int q = 0; q < NG; ++q)
#pragma unroll
      for (int i = 0; i < T::NX; ++i) dma16(p.Xq + (size_t)gq[q] * T::XROW, xv[i], my_lds + (uint32_t)(q * T::XG + 1024 * i));
#pragma unroll
    for (int q = 0; q < NG; ++q)
#pragma unroll
      for (int f = 0; f < 2; ++f) wv[q][f] = __builtin_nontemporal_load(&wfr[(size_t)(2 * gq[q] + f) * 64]);
    // the weight loads are the only vector-memory operations younger than the token rows
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * NG) : "memory");
#pragma unroll
    for (int q = 0; q < NG; ++q)
      if (grp + q * kSkinnyWaves < G) group_mfma(wv[q][0], wv[q][1], xop + q * T::XG, f16bits_to_f32(gsv[q]));   // uniform over the wave
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the operands have been read: the region may be refilled
  }
  // rank-r term on the re-centred codes, added to the wave's tile
  if (has_lr) {
    v16f accl;
#pragma unroll
    for (int e = 0; e < 16; ++e) accl[e] = 0.0f;
    for (int jb = w; jb < JB; jb += kSkinnyWaves) {
      if (jb != w) {                                        // ranks beyond the first block of each wave
        rf = rfr[(size_t)jb * 64];
        xr = lr_load<ABITS>(xrow, p.s_begin + 16 * jb + 8 * g);
      }
      accl = mfma_lr16(lr_convert<ABITS>(xr, zm, mv, bf), rf, accl, bf);
    }
#pragma unroll
    for (int e = 0; e < NE; ++e) accf[e] = __builtin_fmaf(accf[e], kInv, accl[e]);   // 2^-SH: exact
  } else {
#pragma unroll
    for (int e = 0; e < NE; ++e) accf[e] *= kInv;
  }
  // combine: register 4i+e of lane (c,g) is token 8i + 4g + e of channel c
  float* red = reinterpret_cast<float*>(my);
#pragma unroll
  for (int e = 0; e < NE; ++e) red[(8 * (e >> 2) + 4 * g + (e & 3)) * kPitch + m] = accf[e];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int nl = tid & 31, mt = (tid >> 5) + q * 2 * kSkinnyWaves;
    if (mt >= p.M) continue;
    float tot = 0.0f;
#pragma unroll
    for (int ww = 0; ww < kSkinnyWaves; ++ww) tot += *reinterpret_cast<const float*>(lds + ww * T::REGION + 4 * (mt * kPitch + nl));
    const int n = nb * 32 + nl;
    const float y = sc_m[q] * (tot - (float)z_m[q] * wsum);
    const size_t o = (size_t)mt * p.ldy + n;
    if (p.y_dtype == SERQ_F32) ((float*)p.Y)[o] = y;
    else if (p.y_dtype == SERQ_BF16) ((uint16_t*)p.Y)[o] = f32_to_bf16_rne(y);
    else ((uint16_t*)p.Y)[o] = f32_to_f16_rne(y);
  }
}

// ---- larger M: LDS-tiled kernel, 128 tokens x 128 channels per workgroup of 4 waves (2 x 2) ---------------
// One stage = one group of 128 input channels: 4 blocks x 2 weight fragments (8 KiB), 128 token rows
// (16 KiB at 8 bits, 8 KiB at 4 bits; 16-byte pieces xor-swizzled per row so that the operand reads are
// free of bank conflicts) and the group's 128 scales (256 B).  The stages form a ring (3 deep at 8 bits,
// 4 at 4 bits) filled by direct global -> LDS loads (no staging registers) that run two or three groups
// ahead of the arithmetic and are counted by hand with vmcnt; one barrier per group.  Two workgroups
// share a compute unit, so the barrier of one is covered by the other.
// Each wave owns 2 x 2 MFMA tiles of fp32 accumulators.  Tokens are the MFMA's row operand and weights its column
// operand: a lane holds one channel of each block, so a group's scales are one register per block.  The operands of
// the next group are copied from LDS to registers while this group is multiplied (the registers for that come from
// the scales and from keeping two INT32 tiles, not four): the products never wait for an LDS read.  The four MFMAs
// of a group run tile by tile, and the convert-and-FMA pairs that fold the tile before are issued between them, so
// that the vector unit works in the shadow of the matrix unit.  The first group stands outside the loop and does not wait
// for the second one to land.
//
// The loads of a group are spread over the products of the group whose slot they take: requested in one go behind the barrier, as
// they were, they queue at the address unit and a wave whose load waits there issues nothing else (us, in one go / spread, r = 0,
// 6144 x 4096 M = 4096 131.6 / 126.6).  R comes through the ring as well, in stages of its own with the token codes it meets, and its
// type is a compile-time choice: chosen at run time, the two products made the compiler copy a whole tile after each of them, and
// the fragments had come straight from L2, waited for four at a time (us, with both steps, r = 128 unless stated, N x K: W4A8
// 6144 x 4096 M = 3000 110.4 / 102.6, 11008 x 4096 M = 4096 254.5 / 240.9, 4096 x 11008 234.1 / 221.9, r = 256 6144 x 4096
// 159.5 / 145.1; W4A4 11008 x 4096 242.7 / 233.2;
// the type alone, at run time / compile time: W4A8 6144 x 4096 M = 3000 107.0 / 104.2, r = 256 M = 4096 146.8 / 142.9, 2912 x 1024 M = 1649
// r = 64 17.6 / 17.3, W4A4 11008 x 4096 235.7 / 232.3, W4A8 11008 x 4096 and 4096 x 11008 level).
// What bounds it now (counters, W4A8 6144 x 4096 M = 3000): vector issue slots 71 % taken, matrix unit 40 %, LDS 20 %; 190 vector
// instructions per wave and group, 128 of them folds.
//
// With a short K the end of the tile counts: everything it takes from LDS is read in one go, before anything is written
// there, and 16-bit results go through LDS by channel (below).  Measured (us, end as it was with results exchanged between
// lanes and reads behind tests / this form, W4A8 r = 0, N x K): 2048 x 256 M = 4096 11.1 / 9.8; 11008 x 1024 M = 1024
// 25.6 / 23.7, fp32 output 31.3 / 28.3; 6144 x 4096 M = 3000 99.5 / 97.9.
template <int ABITS>
struct GTile {
  static constexpr int XROW = 128 * ABITS / 8;       // bytes of a token's 128 codes
  static constexpr int P = XROW / 16;                // 16-byte pieces per token row: 8 or 4
  static constexpr int WB = 4 * 2 * 1024;
  static constexpr int XB = 128 * XROW;
  static constexpr int SC_OFF = WB + XB;             // 4 blocks x 32 fp16 scales
  static constexpr int STAGE = SC_OFF + 256;
  static constexpr int NS = ABITS == 8 ? 3 : 4;      // ring depth
  static constexpr int NLX = 128 * P / 256;          // token loads per thread and group: 4 or 2
  static constexpr int nl(int ni) { return ni + NLX + 1; }   // direct loads per wave and stage
  // a stage of the rank-r term: the R fragments of RK ranks where the weights lie, behind them the 128 token rows
  static constexpr int RK = ABITS == 8 ? 64 : 32;    // 64 / 16 bytes of a token row
  static constexpr int RF = RK / 16;                 // fragments per channel block
  static constexpr int RP = RK * ABITS / 128;        // 16-byte pieces per row: 4 or 1
  static constexpr int RX_OFF = 4 * RF * 1024;
  static constexpr int NLR = (2 * RP + 3) / 4;       // token loads per wave: 2 or 1
  static __device__ __forceinline__ int swz_r(int row) { return ABITS == 8 ? (row >> 2) & 3 : 0; }
  static constexpr int TS_OFF = NS * STAGE;          // for the epilogue: 128 token scales, zero points and wsum of the tile
  static constexpr int LDS = TS_OFF + 3 * 128 * 4;
  static __device__ __forceinline__ int swz(int row) { return ABITS == 8 ? ((row >> 1) & 7) : ((row >> 2) & 3); }
  static_assert(2 * LDS <= 160 * 1024, "two workgroups per compute unit");
  static_assert(RX_OFF + 128 * 16 * RP <= STAGE, "the rank-r operands fit a stage");
};

template <int ABITS, int NI>
struct GOp { u4 w[NI][2], x[2][ABITS == 8 ? 4 : 2]; float gs[NI]; };   // raw operands and scales of one group

// LR: the type of R, or kNoRank for a layer without the rank-r term, whose code is in the way of short layers (us, with it / without,
// r = 0, N x K: W4A8 1856 x 512 M = 931 6.65 / 6.38, 6144 x 640 M = 2048 19.0 / 18.75, 1856 x 1024 8.28 / 8.02; W4A4 8800 x 1024 M = 1384
// 23.8 / 23.1).
constexpr int kNoRank = -1;
template <int ABITS, bool HALVES, int LR>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void serq_g128_tiled_kernel(const GParams p, int full) {
  using T = GTile<ABITS>;
  constexpr int SH = ABITS == 8 ? 4 : 8;
  constexpr float kInv = 1.0f / (float)(1 << SH);
  constexpr int NS = T::NS;
  __shared__ __align__(16) uint8_t lds[T::LDS];
  const int tid = threadIdx.x, l = tid & 63, lm = l & 31, g = l >> 5;
  const int wu = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = wu & 1, wm = wu >> 1;
  const int NB = p.N >> 5, KB = p.K >> 6, G = p.K >> 7;
  // workgroup id -> tile: one contiguous range of tiles per XCD, in bands of 8 token tiles, so that the
  // tiles in flight on one XCD share their weight and token panels in its L2.  HALVES: workgroups from `full` on
  // (a multiple of 8) take half a tile each, the 64-channel halves of the tiles that are left on their XCD.
  const int tm = (p.M + 127) >> 7, tn = (NB + 3) >> 2;
  const bool halved = HALVES && (int)blockIdx.x >= full;
  const int bid = halved ? blockIdx.x - full : blockIdx.x;
  const int logical = xcd_first(bid & 7, tm * tn) + (halved ? (full >> 3) + (bid >> 4) : bid >> 3);
  if (halved && logical >= xcd_first((bid & 7) + 1, tm * tn)) return;   // (an XCD with a tile less than others)
  int tile_m, tile_n;
  band_tile(logical, tm, tn, 8, tile_m, tile_n);
  const int nb0 = tile_n * 4 + (halved ? 2 * ((bid >> 3) & 1) : 0);
  if (nb0 >= NB) return;                              // the second half of a last, narrow tile
  const int nbt = NB - nb0 < (halved ? 2 : 4) ? NB - nb0 : (halved ? 2 : 4);
  const int m0 = tile_m * 128;
  const int mrows = p.M - m0 < 128 ? p.M - m0 : 128;
  const size_t rowbytes = (size_t)p.K * ABITS / 8;

  // ---- what this wave sends from global memory into a stage ---------------------------------------
  // A direct load puts the 16 bytes of lane l at (wave-uniform LDS base) + 16 l, so the swizzle of the
  // token pieces is applied on the source side.  Per group and wave: 2 weight fragments, NLX x 64 token
  // pieces, and (4 lanes) the 64 bytes of scales of block w.
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_addr(lds));
  // (few registers, every one is taken in the main loop: the weight and scale offsets are wave-uniform but for the lane, and
  // the token rows of the NLX loads lie 1024 / XROW * 4 rows apart, with the same swizzle)
  constexpr int XSTEP = 256 / T::P;                   // rows from one token load of a thread to its next
  static_assert((XSTEP & 15) == 0, "the same swizzle");
  const int xrow0 = tid / T::P;
  const int xc = (tid % T::P) ^ T::swz(xrow0);        // the global piece that lives in this lane's slot
  const uint32_t xv0 = (uint32_t)xrow0 * (uint32_t)rowbytes + 16u * xc;
  const uint32_t xlast = (uint32_t)(mrows - 1) * (uint32_t)rowbytes + 16u * xc;   // rows past M: duplicates of the last, never stored
  const uint8_t* wbase = (const uint8_t*)p.Wq + (size_t)nb0 * KB * 1024;
  const uint8_t* xbase = p.Xq + (size_t)m0 * rowbytes;
  const uint8_t* sbase = (const uint8_t*)p.gsc + (size_t)nb0 * G * 64;
  // The sequence of stages: the G groups of the layer, then LG stages of RK ranks each for the rank-r term.
  constexpr bool has_lr = LR != kNoRank, BF = LR != SERQ_F16;
  const int JB = has_lr ? p.r >> 4 : 0;
  const int LG = (JB + T::RF - 1) / T::RF;
  const int GT = G + LG;
  // Everything from here on is specialised on the channel blocks per wave: 2, or 1 in half a tile.
  auto body = [&](auto ni_c) {
  constexpr int NI = decltype(ni_c)::value;
  using Op = GOp<ABITS, NI>;
  // direct load d (of nl(NI)) of group gi into slot st
  auto fill = [&](int gi, int st, int d) {
    const uint32_t sb = lds0 + (uint32_t)st * T::STAGE;
    if (d < NI) {
      int b = 2 * d + (wu >> 1);                      // blocks past the tile: duplicates, never stored
      b = b < nbt ? b : nbt - 1;
      dma16(wbase + (size_t)gi * 2048 + (size_t)(b * KB + (wu & 1)) * 1024, (uint32_t)l * 16u, sb + 1024 * wu + 4096 * d);
    } else if (d < NI + T::NLX) {
      const int i = d - NI;
      uint32_t step = (uint32_t)rowbytes;
      asm volatile("" : "+s"(step));                  // added here: left alone, the compiler keeps all the sums
      const uint32_t xv = xv0 + (uint32_t)(i * XSTEP) * step;
      dma16(xbase + (size_t)gi * T::XROW, xv < xlast ? xv : xlast, sb + T::WB + 1024 * wu + 4096 * i);
    } else {
      dma64(sbase + (size_t)gi * 64 + (size_t)(wu < nbt ? wu : nbt - 1) * G * 64, (uint32_t)l * 16u, sb + T::SC_OFF + 64 * wu);
    }
  };
  // The loads of stage lg of the rank-r term: fragment f of block b at (b * RF + f) KiB, then the token rows.  Fragments past r,
  // rows past M: duplicates, not used.  The count is that of a group, with repetitions: the waits count all stages alike.
  auto fill_lr = [&](int lg, int st) {
    const uint32_t sb = lds0 + (uint32_t)st * T::STAGE;
    constexpr int NR = NI * T::RF / 2;                // fragments per wave
    constexpr int NT = T::nl(NI) - NR;                // the other loads
    static_assert(NT >= T::NLR, "a stage of the rank-r term takes no more loads than a group");
    auto fragment = [&](int i) {
      const int n = wu + 4 * i, b = n / T::RF, jb = lg * T::RF + n % T::RF;
      dma16((const uint8_t*)p.Rp + ((size_t)(nb0 + (b < nbt ? b : nbt - 1)) * JB + (jb < JB ? jb : JB - 1)) * 1024,
            (uint32_t)l * 16u, sb + 1024 * n);
    };
#pragma unroll
    for (int i = 0; i < NR; ++i) fragment(i);
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      if (i < T::NLR) {
        int n = 64 * (wu + 4 * i) + l;                // piece of the stage
        if (T::RP == 1) n &= 127;                     // 4-bit tokens: waves 2 and 3 repeat the loads of 0 and 1
        const int row = n / T::RP;
        int pc = (n % T::RP) ^ T::swz_r(row);
        const int have = (p.r - lg * T::RK + 15) / 16;   // pieces of 16 channels the rows have (4-bit: one piece holds 32)
        if (ABITS == 8 && pc >= have) pc = have - 1;
        dma16(p.Xq + (size_t)m0 * rowbytes + (size_t)(p.s_begin + lg * T::RK) * ABITS / 8,
              (uint32_t)(row < mrows ? row : mrows - 1) * (uint32_t)rowbytes + 16u * pc,
              sb + T::RX_OFF + 1024 * (T::RP == 1 ? wu & 1 : wu + 4 * i));
      } else {
        fragment(0);
      }
    }
  };
  auto issue = [&](int q, int st) {
    if (!has_lr || q < G) {
#pragma unroll
      for (int d = 0; d < T::nl(NI); ++d) fill(q, st, d);
    } else {
      fill_lr(q - G, st);
    }
  };

  // what the epilogue needs of the tile's tokens and channels, requested before the ring (older loads do not disturb its
  // counting) and straight into LDS: waves 0, 1 bring scales and zero points, waves 2, 3 wsum
  {
    const int i = 64 * (wu & 1) + l;
    const uint32_t ts = lds0 + T::TS_OFF + 256 * (wu & 1);
    if (wu < 2) {
      const uint32_t row = 4u * (uint32_t)(i < mrows ? i : mrows - 1);
      dma4(p.scale + m0, row, ts);
      if (p.zero) dma4(p.zero + m0, row, ts + 512);
    } else {
      dma4(p.wsum + 32 * nb0, 4u * (uint32_t)(i < 32 * nbt ? i : 0), ts + 1024);
    }
  }

  // this wave's blocks NI*wn + i and token rows 32*(2*wm + j) + lm
  const int xrow = 64 * wm + lm;                      // (row 32 further: the same swizzle)
  const int xoff = T::WB + xrow * T::XROW, xsw = T::swz(xrow);
  // piece c ^ xsw of that row for c = (piece of this half-wave) ^ k: one address and an xor of 16 * k, because the row and
  // stage offsets leave those bits free
  const int xbase_off = xoff + 16 * ((ABITS == 8 ? 2 * g : g) ^ xsw);
  static_assert(T::STAGE % 128 == 0 && T::WB % 128 == 0, "stage offsets keep the low address bits free for the xor");
  auto read_w = [&](int st, Op& o) {
    const uint8_t* s = lds + st * T::STAGE;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
#pragma unroll
      for (int f = 0; f < 2; ++f) o.w[i][f] = *(const u4*)(s + (((NI * wn + i) * 2 + f) * 64 + l) * 16);
      o.gs[i] = (float)*(const _Float16*)(s + T::SC_OFF + 64 * (NI * wn + i) + 2 * lm);
    }
  };
  auto read_x = [&](int st, Op& o) {
    const int xa = st * T::STAGE + xbase_off;
#pragma unroll
    for (int h = 0; h < (ABITS == 8 ? 4 : 2); ++h) {
      const int k = ABITS == 8 ? 4 * (h >> 1) + (h & 1) : 2 * h;   // 8-bit: fragment h/2, K half h%2; 4-bit: fragment h
#pragma unroll
      for (int j = 0; j < 2; ++j) o.x[j][h] = *(const u4*)(lds + (xa ^ (16 * k)) + 32 * j * T::XROW);
    }
  };

  v16i acc[2];                                        // INT32 tiles: the one being multiplied, the one being folded
  v16f accf[NI][2];
  const v16i kZero16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    acc[j] = kZero16;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) accf[i][j][e] = 0.0f;
  }
  float gprev = 0.0f;                                 // scale of the tile whose fold is still owed: the last one of the group before

  // the tiles of a group; the MFMAs of tile u = 2*i + j shadow the fold of the tile before.  The next group's weights
  // are read once the registers of this group's first block are free.
  // FILL: group `gf` is requested into slot `sf`, its loads spread over the products.  Requested in one go behind the barrier,
  // the loads of all waves queue at the address unit, and a wave whose load waits there issues nothing else.
  auto multiply = [&](auto ahead, auto fill_c, const Op& o, int nst, Op& nxt, int gf, int sf) {
    constexpr int NLF = decltype(fill_c)::value ? T::nl(NI) : 0, NPOS = 8 * NI;
#pragma unroll
    for (int u = 0; u < 2 * NI; ++u) {
      if (decltype(ahead)::value && u == NI) {
        read_w(nst, nxt);
        fence();
      }
      const int i = u >> 1, j = u & 1;
      const int pu = (u + 2 * NI - 1) % (2 * NI), pi = pu >> 1, pj = pu & 1;
      const float gs = u == 0 ? gprev : o.gs[pi];
      v4i a[4], b[4];
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        unpack_frag(o.w[i][f], a[2 * f], a[2 * f + 1]);
        if constexpr (ABITS == 8) {
          b[2 * f] = as_v4i(o.x[j][2 * f]);
          b[2 * f + 1] = as_v4i(o.x[j][2 * f + 1]);
        } else {
          unpack_frag(o.x[j][f], b[2 * f], b[2 * f + 1]);
        }
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        // the first product of a group starts from zero (a constant operand, no registers to clear)
        if (t == 0) acc[u & 1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(b[t], a[t], kZero16, 0, 0, 0);
        else acc[u & 1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(b[t], a[t], acc[u & 1], 0, 0, 0);
        // (nothing behind the first: the last product of the tile before has not come out yet)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (t > 0 && e * 3 / 16 == t - 1)
            accf[pi][pj][e] = __builtin_fmaf(gs, (float)acc[(u & 1) ^ 1][e], accf[pi][pj][e]);
#pragma unroll
        for (int d = 0; d < NLF; ++d)
          if (d * NPOS / T::nl(NI) == 4 * u + t) fill(gf, sf, d);
        fence();
      }
    }
    gprev = o.gs[NI - 1];
  };

  // the first `younger` stages behind the one waited for may still be in flight
  auto wait_stage = [&](int younger) {
    if (younger >= NS - 1) wait_dma_barrier<(NS - 1) * T::nl(NI)>();
    else if (younger == NS - 2) wait_dma_barrier<(NS - 2) * T::nl(NI)>();
    else wait_dma_barrier<0>();
  };
  auto behind = [&](int q) { return (q + NS - 1 < GT - 1 ? q + NS - 1 : GT - 1) - q; };
#pragma unroll
  for (int s = 0; s < NS; ++s)
    if (s < GT) issue(s, s);
  Op A, B;
  wait_stage(behind(0));
  read_w(0, A);
  read_x(0, A);
  int st = 0;                                         // slot of the current group
  auto group = [&](auto first_c, auto steady_c, int gi, const Op& cur, Op& nxt) {
    constexpr bool FIRST = decltype(first_c)::value, STEADY = decltype(steady_c)::value;
    if (FIRST) multiply(std::false_type{}, std::false_type{}, cur, 0, nxt, 0, 0);
    const int free = st;
    const int next = st + 1 == NS ? 0 : st + 1;
    const int last = gi + NS - 1 < GT - 1 ? gi + NS - 1 : GT - 1;
    if (STEADY || last - gi == NS - 1) wait_dma_barrier<(NS - 2) * T::nl(NI)>();
    else wait_dma_barrier<0>();
    if (!STEADY && gi + NS < GT) issue(gi + NS, free);
    st = next;
    read_x(st, nxt);                                  // (behind the last group: bytes that are never used)
    if (FIRST) read_w(st, nxt);
    fence();
    if (!FIRST) multiply(std::true_type{}, steady_c, cur, st, nxt, gi + NS, free);
  };
  using Yes = std::true_type;
  using No = std::false_type;
  group(Yes{}, No{}, 0, A, B);
  int gi = 1;
#pragma unroll 1
  for (; gi + 1 + NS < G; gi += 2) {
    group(No{}, Yes{}, gi, B, A);
    group(No{}, Yes{}, gi + 1, A, B);
  }
#pragma unroll 1
  for (; gi + 1 < G; gi += 2) {
    group(No{}, No{}, gi, B, A);
    group(No{}, No{}, gi + 1, A, B);
  }
  if (gi < G) group(No{}, No{}, gi, B, A);

  // ---- epilogue: zero point, rank-r term on the re-centred codes, token scale, one store ----------------
  // register e of lane (lm, g) in tile (i, j): token 32*(2*wm + j) + 8*(e/4) + 4*g + e%4, channel
  // 32*(nb0 + NI*wn + i) + lm; blocks from nbt on are not stored
  // (lane indices taken anew: every register that lives through the main loop for the sake of the end is one too many)
  int te = tid;
  asm volatile("" : "+v"(te));
  const int l = te & 63, lm = l & 31, g = l >> 5;
  fence();
#pragma unroll
  for (int e = 0; e < 16; ++e) accf[NI - 1][1][e] = __builtin_fmaf(gprev, (float)acc[1][e], accf[NI - 1][1][e]);
  const float* tsc = reinterpret_cast<const float*>(lds + T::TS_OFF);       // (in LDS since the first stage was waited for)
  const int* tzr = reinterpret_cast<const int*>(lds + T::TS_OFF + 512);
  const float* tws = reinterpret_cast<const float*>(lds + T::TS_OFF + 1024);
  v4i z[2][4];                                          // (read in one go: behind a test each they would be waited for one by one)
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) z[j][q4] = v4i{0, 0, 0, 0};
  if (p.zero) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) z[j][q4] = *(const v4i*)(tzr + 32 * (2 * wm + j) + 8 * q4 + 4 * g);
  }
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const float ws = tws[32 * (NI * wn + i) + lm];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e)
        accf[i][j][e] = __builtin_fmaf(accf[i][j][e], kInv, -(float)z[j][e >> 2][e & 3] * ws);   // 2^-SH: exact
  }
  if constexpr (has_lr) {
    // R fragments and token codes come through the ring, RK ranks at a time (they ran ahead of the last main groups, like any
    // stage), and are read in one go.
    int zm[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) zm[j] = p.zero ? tzr[32 * (2 * wm + j) + lm] : 0;
#pragma unroll 1
    for (int lg = 0; lg < LG; ++lg) {
      const int q = G + lg;
      // stage q has landed, and every wave has read the one before, whose slot is refilled
      wait_stage(lg == 0 ? behind(q) : (q + NS - 2 < GT - 1 ? q + NS - 2 : GT - 1) - q);
      if (lg > 0) {
        if (q - 1 + NS < GT) issue(q - 1 + NS, st);
        st = st + 1 == NS ? 0 : st + 1;
      }
      const uint8_t* s = lds + st * T::STAGE;
      u4 rr[T::RF][NI];
      u2 xr[T::RF][2];
#pragma unroll
      for (int f = 0; f < T::RF; ++f) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int row = 64 * wm + 32 * j + lm;
          const uint8_t* xs = s + T::RX_OFF + 16 * T::RP * row;
          if constexpr (ABITS == 8) xr[f][j] = *(const u2*)(xs + 16 * (f ^ T::swz_r(row)) + 8 * g);
          else xr[f][j] = u2{*(const uint32_t*)(xs + 8 * f + 4 * g), 0u};
        }
#pragma unroll
        for (int i = 0; i < NI; ++i) rr[f][i] = *(const u4*)(s + ((NI * wn + i) * T::RF + f) * 1024 + l * 16);
      }
      fence();
#pragma unroll
      for (int f = 0; f < T::RF; ++f) {
        if (lg * T::RF + f < JB) {                        // uniform
          u4 xf[2];
#pragma unroll
          for (int j = 0; j < 2; ++j) xf[j] = lr_convert_packed<ABITS>(xr[f][j], zm[j], BF);   // rows past M: duplicates, never stored
#pragma unroll
          for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) accf[i][j] = mfma_lr16(xf[j], rr[f][i], accf[i][j], BF);
        }
      }
    }
  }
  v4f sm[2][4];                                         // (all of them before anything is written to LDS, which would hold up the reads)
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) sm[j][q4] = *(const v4f*)(tsc + 32 * (2 * wm + j) + 8 * q4 + 4 * g);
  if (p.y_dtype == SERQ_F32) {
    // fp32 output: 32 lanes write 128 contiguous bytes straight from the accumulators
    const int mw = 64 * wm;                             // this wave's first row
    float* yw = (float*)p.Y + (size_t)(m0 + mw) * p.ldy + 32 * nb0;
    const size_t lane = (size_t)(4 * g) * p.ldy + lm;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int b = NI * wn + i;
      if (b >= nbt) break;
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int r = 32 * j + 8 * (e >> 2) + (e & 3);
          if (mw + r + 4 * g < mrows) yw[(size_t)r * p.ldy + 32 * b + lane] = sm[j][e >> 2][e & 3] * accf[i][j][e];
        }
    }
    return;
  }
  // 16-bit output: cast and transposed through LDS (the ring is free now).  A lane holds four consecutive tokens of one
  // channel: LDS holds a row of 256 B per channel (128 tokens), the 16-byte piece pt of channel c at piece pt ^ swz_y(c).
  // A thread reads the same four tokens of eight channels, pairs the channels up and stores 16 bytes per token: 16 lanes
  // write 256 contiguous bytes.  (Neighbouring lanes exchanging halves before LDS instead: twice the LDS writes and four
  // times the register moves.)
  __syncthreads();                                      // every wave is done with the ring
  const bool ybf = p.y_dtype == SERQ_BF16;
  auto swz_y = [](int c) { return (c & 15) ^ ((c >> 3) & 15); };   // distinct over 16 neighbours and over 16 steps of 8
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const int pt = 4 * (2 * wm + j) + q4;             // tokens 8*pt + 4*g + 0..3
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const v4f f = sm[j][q4];
        const float y0 = f.x * accf[i][j][4 * q4], y1 = f.y * accf[i][j][4 * q4 + 1];
        const float y2 = f.z * accf[i][j][4 * q4 + 2], y3 = f.w * accf[i][j][4 * q4 + 3];
        u2 o;
        if (ybf) o = u2{f32x2_to_bf16x2(y0, y1), f32x2_to_bf16x2(y2, y3)};
        else o = u2{f32x2_to_f16x2(y0, y1), f32x2_to_f16x2(y2, y3)};
        const int c = 32 * (NI * wn + i) + lm;
        *(u2*)(lds + c * 256 + 16 * (pt ^ swz_y(c)) + 8 * g) = o;
      }
    }
  __syncthreads();
  const int c8 = te & 15;                              // channels 8*c8 + 0..7
  if (c8 < 4 * nbt) {
    u2 v[2][8];
#pragma unroll
    for (int it = 0; it < 2; ++it) {
      const int tq = 16 * it + (te >> 4);               // tokens 4*tq + 0..3
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int c = 8 * c8 + k;
        v[it][k] = *(const u2*)(lds + c * 256 + 16 * ((tq >> 1) ^ swz_y(c)) + 8 * (tq & 1));
      }
    }
    uint16_t* yt = (uint16_t*)p.Y + (size_t)(m0 + 4 * (te >> 4)) * p.ldy + nb0 * 32 + 8 * c8;
#pragma unroll
    for (int it = 0; it < 2; ++it)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const uint32_t sel = t & 1 ? 0x07060302u : 0x05040100u;   // the upper / lower halves of two channels
        auto two = [&](int k) {
          return __builtin_amdgcn_perm(t < 2 ? v[it][k + 1].x : v[it][k + 1].y, t < 2 ? v[it][k].x : v[it][k].y, sel);
        };
        const int r = 64 * it + t;
        if (4 * (te >> 4) + r < mrows) *(u4*)(yt + (size_t)r * p.ldy) = u4{two(0), two(2), two(4), two(6)};
      }
  }
  };
  if constexpr (HALVES) {
    if (halved) {
      body(std::integral_constant<int, 1>{});
      return;
    }
  }
  body(std::integral_constant<int, 2>{});
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline bool dtype_ok(int dt) { return dt == SERQ_F32 || dt == SERQ_F16 || dt == SERQ_BF16; }
inline int check_nk128(int64_t N, int64_t K) {
  if (K < 128 || K > 131072 || (K % 128) != 0) return SERQ_ESHAPE;
  if (N < 32 || (N % 32) != 0 || N > (1 << 24)) return SERQ_ESHAPE;
  return SERQ_OK;
}
inline int hip_ok() { return hipGetLastError() == hipSuccess ? SERQ_OK : SERQ_EHIP; }

}  // namespace
}  // namespace serq

using namespace serq;

extern "C" {

size_t serq_g128_scale_bytes(int64_t N, int64_t K) {
  if (check_nk128(N, K) != SERQ_OK) return 0;
  return (size_t)N * (size_t)(K / kGroup) * 2;
}

int serq_quantize_act_asym(const void* X, int x_dtype, const float* s_inv, int64_t M, int64_t K, int64_t ldx, int abits,
                           void* Xq_out, float* scale_out, int32_t* zero_out, void* stream) {
  if (abits != 4 && abits != 8) return SERQ_EDTYPE;
  if (!dtype_ok(x_dtype)) return SERQ_EDTYPE;
  if (M < 0 || M > (1 << 30) || K < 64 || K > 131072 || (K % 64) != 0) return SERQ_ESHAPE;
  if (ldx < K) return SERQ_ESHAPE;
  if ((ldx % 8) != 0) return SERQ_EALIGN;
  if (M == 0) return SERQ_OK;
  if (!X || !Xq_out || !scale_out || !zero_out) return SERQ_ENULL;
  if (!aligned16(X) || !aligned16(Xq_out) || !aligned16(s_inv) || (reinterpret_cast<uintptr_t>(scale_out) & 3u) ||
      (reinterpret_cast<uintptr_t>(zero_out) & 3u))
    return SERQ_EALIGN;
  hipStream_t st = (hipStream_t)stream;
  for (int64_t m0 = 0; m0 < M; m0 += kLaunchRows) {
    const int64_t mc = M - m0 < kLaunchRows ? M - m0 : kLaunchRows;
    const void* Xs = (const char*)X + (size_t)m0 * (size_t)ldx * (x_dtype == SERQ_F32 ? 4 : 2);
    void* Xqs = (char*)Xq_out + (size_t)m0 * ((size_t)K * abits / 8);
#define SERQ_QAA_DT(DT)                                                                                              \
  (abits == 4 ? launch_asym_t<DT, 4>(Xs, s_inv, mc, (int)K, ldx, Xqs, scale_out + m0, zero_out + m0, st)             \
              : launch_asym_t<DT, 8>(Xs, s_inv, mc, (int)K, ldx, Xqs, scale_out + m0, zero_out + m0, st))
    const int rc = x_dtype == SERQ_F32 ? SERQ_QAA_DT(SERQ_F32) : x_dtype == SERQ_F16 ? SERQ_QAA_DT(SERQ_F16) : SERQ_QAA_DT(SERQ_BF16);
#undef SERQ_QAA_DT
    if (rc != SERQ_OK) return rc;
  }
  return SERQ_OK;
}

int serq_g128_pack_weights(const void* W, int w_dtype, const float* s, const int32_t* perm_in, int64_t N, int64_t K, int r,
                           void* Wq_out, void* gscale_out, float* wsum_out, int32_t* perm_out, float* s_inv_out,
                           void* R_out, int r_dtype, void* Rp_out, void* stream) {
  if (!W || !Wq_out || !gscale_out || !wsum_out || !perm_out || !s_inv_out) return SERQ_ENULL;
  if (!dtype_ok(w_dtype)) return SERQ_EDTYPE;
  int rc = check_nk128(N, K);
  if (rc != SERQ_OK) return rc;
  if (r < 0 || (r % 16) != 0 || r > K) return SERQ_ESHAPE;
  if (r > 0 && (R_out || Rp_out)) {
    if (!dtype_ok(r_dtype)) return SERQ_EDTYPE;
    if (Rp_out && r_dtype != SERQ_F16 && r_dtype != SERQ_BF16) return SERQ_EDTYPE;
  }
  if (!aligned16(W) || !aligned16(Wq_out) || !aligned16(gscale_out) || !aligned16(wsum_out) || !aligned16(perm_out) ||
      !aligned16(s_inv_out) || !aligned16(R_out) || !aligned16(Rp_out) || !aligned16(s) || !aligned16(perm_in))
    return SERQ_EALIGN;
  hipStream_t st = (hipStream_t)stream;
  rc = prepare_perm_impl(W, w_dtype, s, perm_in, (int)N, (int)K, perm_out, s_inv_out, st);
  if (rc != SERQ_OK) return rc;
  const int G = (int)(K / kGroup);
  uint16_t* gsc = (uint16_t*)gscale_out;
  hipLaunchKernelGGL(group_scale_kernel, dim3(blocks_for((size_t)N * G * 64)), dim3(kT), 0, st, W, w_dtype, s, perm_out,
                     (int)N, (int)K, gsc);
  hipLaunchKernelGGL(quant_pack_grouped_kernel, dim3(blocks_for((size_t)N * K / 8)), dim3(kT), 0, st, W, w_dtype, s,
                     perm_out, gsc, (int)N, (int)K, (uint32_t*)Wq_out);
  hipLaunchKernelGGL(wsum_kernel, dim3((unsigned)N), dim3(kT), 0, st, W, w_dtype, s, perm_out, gsc, (int)K, wsum_out);
  if (r > 0 && (R_out || Rp_out))
    hipLaunchKernelGGL(residual_grouped_kernel, dim3(blocks_for((size_t)r * N)), dim3(kT), 0, st, W, w_dtype, s, perm_out,
                       gsc, (int)N, (int)K, r, R_out, r_dtype, (uint16_t*)Rp_out);
  return hip_ok();
}

int serq_g128_unpack_scales(const void* gscale, int64_t N, int64_t K, float* out, void* stream) {
  if (!gscale || !out) return SERQ_ENULL;
  const int rc = check_nk128(N, K);
  if (rc != SERQ_OK) return rc;
  const int G = (int)(K / kGroup);
  hipLaunchKernelGGL(unpack_gscale_kernel, dim3(blocks_for((size_t)N * G)), dim3(kT), 0, (hipStream_t)stream,
                     (const uint16_t*)gscale, (int)N, G, out);
  return hip_ok();
}

int serq_g128_linear(const void* Xq, const float* scale, const int32_t* zero, int abits,
                     const void* Wq, const void* gscale, const float* wsum,
                     int s_begin, int r, const void* Rp, int r_dtype,
                     int64_t M, int64_t N, int64_t K, void* Y, int y_dtype, int64_t ldy, int flags, void* stream) {
  if (abits != 4 && abits != 8) return SERQ_EDTYPE;
  if (!dtype_ok(y_dtype)) return SERQ_EDTYPE;
  int rc = check_nk128(N, K);
  if (rc != SERQ_OK) return rc;
  if (M < 0 || M > (1 << 22)) return SERQ_ESHAPE;
  if (r < 0 || (r % 16) != 0 || s_begin < 0 || (s_begin % 32) != 0 || (int64_t)s_begin + r > K) return SERQ_ESHAPE;
  if (r > 0 && Rp && r_dtype != SERQ_F16 && r_dtype != SERQ_BF16) return SERQ_EDTYPE;
  if (ldy < N) return SERQ_ESHAPE;
  if (M == 0) return SERQ_OK;
  if (!Xq || !scale || !Wq || !gscale || !wsum || !Y) return SERQ_ENULL;
  if ((ldy % 8) != 0 || !aligned16(Y) || !aligned16(Xq) || !aligned16(Wq) || !aligned16(gscale) || !aligned16(wsum) ||
      !aligned16(Rp) || (reinterpret_cast<uintptr_t>(scale) & 3u) || (reinterpret_cast<uintptr_t>(zero) & 3u))
    return SERQ_EALIGN;
  const int path = flags & 0xff;
  if (path != SERQ_PATH_AUTO && path != SERQ_PATH_SKINNY && path != SERQ_PATH_MFMA) return SERQ_EUNSUPPORTED;
  if (path == SERQ_PATH_SKINNY && M > 32) return SERQ_ESHAPE;
  GParams p;
  p.Xq = (const uint8_t*)Xq; p.scale = scale; p.zero = zero;
  p.Wq = (const u4*)Wq; p.gsc = (const uint16_t*)gscale; p.wsum = wsum;
  p.Rp = (r > 0 ? (const u4*)Rp : nullptr); p.r_dtype = r_dtype; p.s_begin = s_begin; p.r = Rp ? r : 0;
  p.M = (int)M; p.N = (int)N; p.K = (int)K;
  p.Y = Y; p.y_dtype = y_dtype; p.ldy = ldy;
  hipStream_t st = (hipStream_t)stream;
  const bool skinny = path == SERQ_PATH_SKINNY || (path == SERQ_PATH_AUTO && M <= 32);
  if (path == SERQ_PATH_AUTO && !skinny && flags == 0 && g128_mid_wanted(p, abits)) return launch_g128_mid(p, abits, st);
  if (skinny) {
    dim3 grid((unsigned)(N / 32));
    // specialised on ceil(M / 8): the number of accumulator register quads that hold tokens.  Four groups in flight per
    // wave pay once it has two rounds of them and few tokens to stage (us, 2 / 4 in flight, r = 128, W4A8, N x K):
    // 4096 x 11008 M = 1 9.2 / 8.3, M = 8 8.5 / 8.5, M = 16 9.9 / 10.2; 11008 x 4096 M = 1 7.2 / 7.1, M = 16 8.4 / 8.5.
#define SERQ_G128_SKINNY(AB, MQ, NG) \
  hipLaunchKernelGGL((serq_g128_skinny_kernel<AB, MQ, NG>), grid, dim3(64 * kSkinnyWaves), 0, st, p)
    const int mq = (int)((M + 7) / 8);
    const bool deep = mq == 1 && K / kGroup >= 64;
    if (abits == 8) {
      if (deep) SERQ_G128_SKINNY(8, 1, 4);
      else if (mq == 1) SERQ_G128_SKINNY(8, 1, 2);
      else if (mq == 2) SERQ_G128_SKINNY(8, 2, 2);
      else if (mq == 3) SERQ_G128_SKINNY(8, 3, 2);
      else SERQ_G128_SKINNY(8, 4, 2);
    } else {
      if (deep) SERQ_G128_SKINNY(4, 1, 4);
      else if (mq == 1) SERQ_G128_SKINNY(4, 1, 2);
      else if (mq == 2) SERQ_G128_SKINNY(4, 2, 2);
      else if (mq == 3) SERQ_G128_SKINNY(4, 3, 2);
      else SERQ_G128_SKINNY(4, 4, 2);
    }
#undef SERQ_G128_SKINNY
  } else {
    const long long tiles = (long long)((N / 32 + 3) / 4) * ((M + 127) / 128);
    if (tiles > 0x7fffffffLL) return SERQ_ESHAPE;
    // Two workgroups share a compute unit.  What is left after whole rounds is dealt out in halves when that still gives
    // every compute unit at most one workgroup: alone there, a whole tile takes half a round.  Measured (us, whole / halves,
    // W4A8 r = 128, N x K): 64 tiles left 6144 x 4096 M = 1500 74.1 / 66.3; 128 left M = 3000 133 / 126; 160 left
    // 14336 x 4096 M = 700 (W4A4) 71.5 / 75.6; 192 left 11008 x 4096 M = 4096 260 / 264.
    const long long ncu = device_cu_count();
    const long long full = tiles / (2 * ncu) * (2 * ncu), left = tiles - full;
    const bool halves = left > 0 && 2 * left <= ncu && full % 8 == 0;
    const dim3 grid((unsigned)(halves ? full + 16 * ((left + 7) / 8) : tiles));
    const int lr = r > 0 && Rp != nullptr ? r_dtype : kNoRank;
#define SERQ_G128_TILED(AB, HALVES, LR) \
  hipLaunchKernelGGL((serq_g128_tiled_kernel<AB, HALVES, LR>), grid, dim3(256), 0, st, p, HALVES ? (int)full : 0)
#define SERQ_G128_TILED_R(AB, HALVES)                                \
  do {                                                               \
    if (lr == kNoRank) SERQ_G128_TILED(AB, HALVES, kNoRank);         \
    else if (lr == SERQ_F16) SERQ_G128_TILED(AB, HALVES, SERQ_F16);  \
    else SERQ_G128_TILED(AB, HALVES, SERQ_BF16);                     \
  } while (0)
    if (abits == 8) {
      if (halves) SERQ_G128_TILED_R(8, true);
      else SERQ_G128_TILED_R(8, false);
    } else {
      if (halves) SERQ_G128_TILED_R(4, true);
      else SERQ_G128_TILED_R(4, false);
    }
#undef SERQ_G128_TILED_R
#undef SERQ_G128_TILED
  }
  return hip_ok();
}

}  // extern "C"
