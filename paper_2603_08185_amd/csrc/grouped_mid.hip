// The layer with group-128 weight scales for batches between decode and prefill: tiles of 64 tokens x 64 channels, the
// 8 waves of a workgroup sharing K (mid_tile.h says why; the formulas are those of grouped.hip).
//
// A wave takes whole groups of 128 channels: one stage of 4-bit tokens, two of 8-bit ones, each with the group's 64
// scales.  The four products of an MFMA tile start from zero and the INT32 tile is folded into the wave's fp32 tile
// while the next tile's products run.  Tokens are the MFMA's row operand and weights its column operand (as in the decode
// kernel of grouped.hip): a lane holds one channel of each block, so it needs one scale per block and group, not sixteen.
// The waves' fp32 tiles are added through LDS in wave order (run-to-run identical),
// each wave finishing half an MFMA tile: zero point, rank-r term on the re-centred codes, token scale.
//
// What bounds it: the L2 -> LDS stream, as in gemm_mid.hip, and next to it the vector unit (128 fold operations per wave
// and group beside 16 products).  Measured (M = 150, 4096 x 11008, W4A4, r = 64): 18 us; the 128 x 128 tiles of the tiled
// kernel give 64 workgroups there and take 76 us.
#include "mid_tile.h"

namespace serq {
namespace {

template <int ABITS>
struct GMid {
  static constexpr int FR = ABITS == 8 ? 1 : 2;
  static constexpr int SC_OFF = kMidX + 2 * FR * 1024;   // 2 blocks x 32 fp16 scales
  static constexpr int STAGE = SC_OFF + 128;
  static constexpr int NS = ABITS == 8 ? 3 : 2;
  static constexpr int NL = 4 + 2 * FR + 1;
  static constexpr int REGION = NS * STAGE;
  static constexpr int SH = ABITS == 8 ? 4 : 8;
  static constexpr int LDS = kMidWaves * REGION;
  static_assert(REGION >= kMidPart, "a partial tile fits the ring it replaces");
  static_assert(LDS <= 160 * 1024, "LDS budget");
};

template <int FR>
struct GMidOp { u4 w[2][FR], x[2][2]; float gs[2]; };

template <int ABITS, bool BF>
__global__ __launch_bounds__(kMidThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void serq_g128_mid_kernel(const G128Args p, int tiles_m, int tiles_n) {
  using T = GMid<ABITS>;
  constexpr int FR = T::FR, NS = T::NS;
  __shared__ __align__(16) uint8_t lds[T::LDS];
  const int tid = threadIdx.x, l = tid & 63, lm = l & 31, g = l >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tile_m, tile_n;
  map_block(blockIdx.x, tiles_m, tiles_n, tiles_m, tile_m, tile_n);
  const int m0 = tile_m * 64, nb0 = tile_n * 2;
  const int NB = p.N >> 5, G = p.K >> 7;
  const int nbt = NB - nb0 < 2 ? 1 : 2;
  const int mrows = p.M - m0 < 64 ? p.M - m0 : 64;
  const uint32_t rowbytes = (uint32_t)p.K * ABITS / 8;

  MidLoads<FR> ld;
  ld.init(p.Xq, p.Wq, p.K, rowbytes, m0, mrows, nb0, nbt, l);
  const int ng = G > w ? (G - w + kMidWaves - 1) / kMidWaves : 0;   // groups w, w + 8, ... are this wave's
  constexpr int SPG = ABITS == 8 ? 2 : 1;              // stages per group
  const int nst = ng * SPG;
  uint8_t* my = lds + w * T::REGION;
  const uint32_t my_lds = __builtin_amdgcn_readfirstlane(lds_addr(my));
  const uint8_t* sbase = (const uint8_t*)p.gsc + (size_t)nb0 * G * 64;
  const uint32_t sv = (uint32_t)((l >> 2 & 1) && nbt > 1 ? G * 64 : 0) + (l & 3) * 16;   // lanes 0..3: block 0, 4..7: block 1

  // ---- operands of the rank-r term, in chunks of 128 ranks: every wave brings two R fragments and 16 codes of 8 token
  // rows per lane, the first chunk requested before anything else (oldest loads: the ring's counting is not disturbed)
  const int JB = p.r >> 4;
  constexpr int NJ = 8;
  u4 lrr[2], lrx;
  int lzm = 0;
  const int lrow = 8 * w + (l >> 3);
  const int lrm = m0 + (lrow < mrows ? lrow : mrows - 1);
  auto lr_fetch = [&](int jb0) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int f = 2 * w + q, b = f >> 3, jb = jb0 + (f & 7);
      lrr[q] = p.Rp[((size_t)(nb0 + (b < nbt ? b : 0)) * JB + (jb < JB ? jb : JB - 1)) * 64 + l];
    }
    const int have = 16 * (JB - jb0);                  // channels of this chunk
    const int c = 16 * (l & 7) < have ? 16 * (l & 7) : 0;
    const uint8_t* src = p.Xq + (size_t)lrm * rowbytes + (size_t)(p.s_begin + 16 * jb0 + c) * ABITS / 8;
    if constexpr (ABITS == 8) {
      lrx = *(const u4*)src;
    } else {
      const u2 v = *(const u2*)src;
      lrx = u4{v.x, v.y, 0u, 0u};
    }
  };
  constexpr int LRX_OFF = 16 * 1024;                   // R fragments at 0, codes (64 rows x 256 B of 16-bit floats) here
  auto lr_park = [&]() {
#pragma unroll
    for (int q = 0; q < 2; ++q) *(u4*)(lds + (2 * w + q) * 1024 + l * 16) = lrr[q];
    uint8_t* row = lds + LRX_OFF + lrow * 256;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      int k[8];
      if constexpr (ABITS == 8) codes_from_a8(h ? lrx.z : lrx.x, h ? lrx.w : lrx.y, k);
      else codes_from_a4(h ? lrx.y : lrx.x, k);
#pragma unroll
      for (int e = 0; e < 8; ++e) k[e] -= lzm;         // at most 255 in magnitude: exact in both 16-bit formats
      *(u4*)(row + 16 * ((2 * (l & 7) + h) ^ (lrow & 15))) = codes8_to_16bit(k, BF);
    }
  };
  if (JB > 0) {
    lr_fetch(0);
    if (p.zero) lzm = p.zero[lrm];
  }

  // ---- main loop ------------------------------------------------------------------------------------------------
  v16i acc[2][2];
  v16f accf[2][2];
  const v16i kZero16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      acc[i][j] = kZero16;
#pragma unroll
      for (int e = 0; e < 16; ++e) accf[i][j][e] = 0.0f;
    }
  const int xsw = mid_swz(lm);
  auto slot = [&](int t) { return (t % NS) * T::STAGE; };
  auto group = [&](int t) { return w + kMidWaves * (SPG == 2 ? t >> 1 : t); };
  auto fill = [&](int t, int k) {
    const int s = SPG == 2 ? 2 * group(t) + (t & 1) : group(t);
    if (k < T::NL - 1) ld.issue_one(s, my_lds + slot(t), k);
    else if (l < 8) dma16(sbase + (size_t)group(t) * 64, sv, my_lds + slot(t) + T::SC_OFF);
  };
  auto read = [&](auto par, int t, GMidOp<FR>& o) {
    const uint8_t* s = my + slot(t);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
      for (int f = 0; f < FR; ++f) o.w[i][f] = *(const u4*)(s + kMidX + (i * FR + f) * 1024 + l * 16);
      if (SPG == 1 || decltype(par)::value == 1) {       // the scales are used at the end of the group
        o.gs[i] = (float)*(const _Float16*)(s + T::SC_OFF + 64 * i + 2 * lm);
      }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int c = ABITS == 8 ? 2 * g + h : 2 * h + g;
        o.x[j][h] = *(const u4*)(s + (32 * j + lm) * 64 + 16 * (c ^ xsw));
      }
  };
  // MFMA tiles one after another, 2 products a step: tile k / FR (4-bit: fragment k % 2 of it).  In the step after its
  // last product a tile is folded; the last one right behind it (the other wave of the SIMD works meanwhile).
  auto product = [&](auto par, const GMidOp<FR>& o, int k) {
    const int q = k / FR, f = k % FR;
    const int i = q >> 1, j = q & 1;
    const bool first = SPG == 2 ? decltype(par)::value == 0 : f == 0;
    const bool last = SPG == 2 ? decltype(par)::value == 1 : f == FR - 1;
    v4i a0, a1, b0, b1;
    unpack_frag(o.w[i][f], a0, a1);
    if constexpr (ABITS == 8) {
      b0 = as_v4i(o.x[j][0]);
      b1 = as_v4i(o.x[j][1]);
    } else {
      unpack_frag(o.x[j][f], b0, b1);
    }
    if (first) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(b0, a0, kZero16, 0, 0, 0);
    else acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(b0, a0, acc[i][j], 0, 0, 0);
    acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(b1, a1, acc[i][j], 0, 0, 0);
    auto fold = [&](int u) {
      const float gs = o.gs[u >> 1];
#pragma unroll
      for (int e = 0; e < 16; ++e)
        accf[u >> 1][u & 1][e] = __builtin_fmaf(gs, (float)acc[u >> 1][u & 1][e], accf[u >> 1][u & 1][e]);
      // pinned here: left alone, the compiler puts folds off and keeps every INT32 tile alive (99 registers spilled)
      asm volatile("" : "+v"(accf[u >> 1][u & 1]));
    };
    if (last && q > 0) fold(q - 1);
    if (last && q == 3) {
      fence();
      fold(3);
    }
  };
  mid_loop<NS, T::NL, T::NL, 4 * FR, GMidOp<FR>>(
      nst,
      [&](int t) {
#pragma unroll
        for (int k = 0; k < T::NL; ++k) fill(t, k);
      },
      fill, read, product);

  // ---- the waves meet; wave w finishes registers 8*(w%2) .. +7 of MFMA tile (i, j), w/2 = 2*i + j ------------------
  constexpr float kInv = 1.0f / (float)(1 << T::SH);
  const int ti = w >> 2, tj = (w >> 1) & 1, hq = 2 * (w & 1);
  const int blk = nb0 + (ti < nbt ? ti : 0);
  const int n = 32 * blk + lm;                         // this lane's channel
  const int mloc = 32 * tj + 8 * hq + 4 * g;           // registers 4*q + e: token mloc + 8*q + e
  float sm[8], zf[8];
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = mloc + 8 * q + e, m = m0 + (r < mrows ? r : mrows - 1);
      sm[4 * q + e] = p.scale[m];
      zf[4 * q + e] = p.zero ? (float)p.zero[m] : 0.0f;
    }
  const float ws = p.wsum[n];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *(v4f*)(my + ((2 * i + j) * 4 + q) * 1024 + l * 16) =
            v4f{accf[i][j][4 * q], accf[i][j][4 * q + 1], accf[i][j][4 * q + 2], accf[i][j][4 * q + 3]};
  __syncthreads();
  float y[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) y[e] = 0.0f;
#pragma unroll
  for (int ww = 0; ww < kMidWaves; ++ww)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const v4f v = *(const v4f*)(lds + ww * T::REGION + ((w >> 1) * 4 + hq + q) * 1024 + l * 16);
      y[4 * q] += v.x; y[4 * q + 1] += v.y; y[4 * q + 2] += v.z; y[4 * q + 3] += v.w;
    }
#pragma unroll
  for (int e = 0; e < 8; ++e) y[e] = __builtin_fmaf(y[e], kInv, -zf[e] * ws);   // 2^-SH: exact
  if (JB > 0) {
    v16f af;                                           // the tile the matrix unit adds to
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      af[e] = hq ? 0.0f : y[e];
      af[8 + e] = hq ? y[e] : 0.0f;
    }
    for (int jb0 = 0; jb0 < JB; jb0 += NJ) {
      __syncthreads();                                 // the partial tiles (the chunk before) have been read
      lr_park();
      __syncthreads();
      if (jb0 + NJ < JB) lr_fetch(jb0 + NJ);
      const int lr = 32 * tj + lm;                     // the token row this lane multiplies
      const uint8_t* row = lds + LRX_OFF + lr * 256;
#pragma unroll
      for (int q = 0; q < NJ; ++q) {
        if (jb0 + q < JB) {                            // uniform
          const u4 rr = *(const u4*)(lds + (ti * NJ + q) * 1024 + l * 16);
          const u4 xf = *(const u4*)(row + 16 * ((2 * q + g) ^ (lr & 15)));
          if constexpr (BF)
            af = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, xf), __builtin_bit_cast(v8bf, rr), af, 0, 0, 0);
          else
            af = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, xf), __builtin_bit_cast(v8h, rr), af, 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = hq ? af[8 + e] : af[e];
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) y[e] *= sm[e];

  if (p.y_dtype == SERQ_F32) {                         // 32 lanes write 128 contiguous bytes
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int r = mloc + 8 * (e >> 2) + (e & 3);
      if (r < mrows && ti < nbt) ((float*)p.Y)[(size_t)(m0 + r) * p.ldy + n] = y[e];
    }
    return;
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int r = mloc + 8 * (e >> 2) + (e & 3), c = 32 * ti + lm;
    *(uint16_t*)(lds + r * 128 + 16 * ((c >> 3) ^ (r & 7)) + 2 * (c & 7)) =
        p.y_dtype == SERQ_BF16 ? f32_to_bf16_rne(y[e]) : f32_to_f16_rne(y[e]);
  }
  __syncthreads();
  mid_store16<kMidThreads>(lds, tid, (uint16_t*)p.Y, p.ldy, m0, mrows, 32 * nb0, nbt);
}

}  // namespace

// Up to two tiles per compute unit.  Measured (us, tiled kernel / this one, r = 128, W4A8; W4A4 the same or better):
//   1 round:  4096 x 11008 M = 256 73.1 / 28.2;  4096 x 4096 M = 256 32.8 / 14.1;  6144 x 4096 M = 100 33.1 / 13.1
//   2 rounds: 4096 x 11008 M = 512 73.2 / 51.0;  4096 x 4096 M = 512 32.9 / 25.0;  6144 x 4096 M = 256 32.8 / 24.3;
//             28672 x 4096 M = 64 34.5 / 32.3;  1024 x 1024 M = 2048 14.9 / 13.3
//   3 rounds: 6144 x 4096 M = 512 33.6 / 36.0;  11008 x 4096 M = 256 33.4 / 35.5;  4096 x 11008 M = 768 74.0 / 73.4
// (N x K).  From three rounds on the tiled kernel, which moves two thirds of the bytes per product, is as fast or faster.
bool g128_mid_wanted(const G128Args& a) { return mid_rounds(a.M, a.N, device_cu_count()) <= 2; }

int launch_g128_mid(const G128Args& a, int abits, hipStream_t st) {
  const int tm = (a.M + 63) / 64, tn = (a.N + 63) / 64;
  const dim3 grid((unsigned)(tm * tn)), block(kMidThreads);
  const bool bf = a.r_dtype != SERQ_F16;
#define SERQ_GMID_LAUNCH(AB, BF) hipLaunchKernelGGL((serq_g128_mid_kernel<AB, BF>), grid, block, 0, st, a, tm, tn)
  if (abits == 8) {
    if (bf) SERQ_GMID_LAUNCH(8, true); else SERQ_GMID_LAUNCH(8, false);
  } else {
    if (bf) SERQ_GMID_LAUNCH(4, true); else SERQ_GMID_LAUNCH(4, false);
  }
#undef SERQ_GMID_LAUNCH
  return hipGetLastError() == hipSuccess ? SERQ_OK : SERQ_EHIP;
}

}  // namespace serq
