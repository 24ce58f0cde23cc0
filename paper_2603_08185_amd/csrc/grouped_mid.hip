// The layer with group-128 weight scales for batches between decode and prefill: tiles of 64 tokens x 64 channels, the
// 4 or 8 waves of a workgroup sharing K (mid_tile.h says why; the formulas are those of grouped.hip).
//
// A wave takes whole groups of 128 channels, a step of 4-bit tokens or a unit of 8-bit ones, with the group's 64
// scales.  The four products of an MFMA tile start from zero and the INT32 tile is folded into the wave's fp32 tile
// while the next tile's products run.  Tokens are the MFMA's row operand and weights its column operand (as in the decode
// kernel of grouped.hip): a lane holds one channel of each block, so it needs one scale per block and group, not sixteen.
// The waves' fp32 tiles are added through LDS in wave order (run-to-run identical), each of 8 waves finishing half an MFMA
// tile, each of 4 a whole one: zero point, rank-r term on the re-centred codes, token scale.
//
// What bounds it: the load stream, as in gemm_mid.hip, and next to it the vector unit (128 fold operations per wave
// and group beside 16 products).  Measured (M = 150, 4096 x 11008, W4A4, r = 64, graph replay): 20 us; the 128 x 128 tiles of the
// tiled kernel give 64 workgroups there, 128 in halves, and take 48 us.  W4A8, r = 128, 64- / 128-byte token rows: 4096 x 11008
// M = 256 28.1 / 23.3 us, 4096 x 4096 M = 150 12.1 / 11.4, M = 400 19.1 / 17.3.
#include "mid_tile.h"

namespace serq {
namespace {

template <int ABITS>
struct GMid {
  static constexpr int SC_OFF = kMidX + (ABITS == 8 ? 2 : 4) * 1024;   // fp16 scales: 32 of a block (4-bit: of two blocks)
  static constexpr int STAGE = SC_OFF + (ABITS == 8 ? 256 : 128);
  static constexpr int NS = ABITS == 8 ? 3 : 2;
  static constexpr int NL = ABITS == 8 ? 7 : 9;
  static constexpr int REGION = NS * STAGE;
  static constexpr int SH = ABITS == 8 ? 4 : 8;
  static_assert(REGION >= kMidPart, "a partial tile fits the ring it replaces");
  static_assert(8 * REGION <= 160 * 1024, "LDS budget");
};

struct GMidUnitOp { u4 w[2][2], x[2][4]; float gs[2]; };
struct GMidStepOp { u4 w[2][2], x[2][2]; float gs[2]; };

template <int ABITS, bool BF, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 2)))
void serq_g128_mid_kernel(const G128Args p, int tiles_m, int tiles_n, int band) {
  using T = GMid<ABITS>;
  constexpr int NS = T::NS;
  __shared__ __align__(16) uint8_t lds[NW * T::REGION];
  const int tid = threadIdx.x, l = tid & 63, lm = l & 31, g = l >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tile_m, tile_n;
  map_block(blockIdx.x, tiles_m, tiles_n, band, tile_m, tile_n);
  const int m0 = tile_m * 64, nb0 = tile_n * 2;
  const int NB = p.N >> 5, G = p.K >> 7;
  const int nbt = NB - nb0 < 2 ? 1 : 2;
  const int mrows = p.M - m0 < 64 ? p.M - m0 : 64;
  const uint32_t rowbytes = (uint32_t)p.K * ABITS / 8;

  std::conditional_t<ABITS == 8, MidUnits<2, NW, false>, MidLoads> ld;   // a unit, or a step, is a group: a fold needs all of it
  if constexpr (ABITS == 8) ld.init(p.Xq, p.Wq, p.K, rowbytes, m0, mrows, nb0, nbt, w, l);
  else ld.init(p.Xq, p.Wq, p.K, rowbytes, m0, mrows, nb0, nbt, l);
  const int nst = G > w ? (G - w + NW - 1) / NW : 0;   // 4-bit: groups w, w + NW, ... are this wave's
  uint8_t* my = lds + w * T::REGION;
  const uint32_t my_lds = __builtin_amdgcn_readfirstlane(lds_addr(my));
  const uint8_t* sbase = (const uint8_t*)p.gsc + (size_t)nb0 * G * 64;
  const uint32_t sv = (uint32_t)((l >> 2 & 1) && nbt > 1 ? G * 64 : 0) + (l & 3) * 16;   // lanes 0..3: block 0, 4..7: block 1

  // ---- operands of the rank-r term, in chunks of 128 ranks: every wave brings two R fragments and 16 codes of 8 token
  // rows per lane, the first chunk requested before anything else (4-bit: oldest
  // loads, the ring's counting is not disturbed) or in front of the wave's last unit (8-bit: no load of the ring is waited for any more)
  const int JB = p.r >> 4;
  constexpr int NJ = 8;
  constexpr int VH = 8 / NW;                           // (a wave of 4 brings the shares of two of 8)
  u4 lrr[VH][2], lrx[VH];
  int lzm[VH];
  auto lr_row = [&](int v) { return 8 * (VH * w + v) + (l >> 3); };
  auto lr_m = [&](int v) { return m0 + (lr_row(v) < mrows ? lr_row(v) : mrows - 1); };
  auto lr_fetch = [&](int jb0) {
#pragma unroll
    for (int v = 0; v < VH; ++v) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int f = 2 * (VH * w + v) + q, b = f >> 3, jb = jb0 + (f & 7);
      lrr[v][q] = p.Rp[((size_t)(nb0 + (b < nbt ? b : 0)) * JB + (jb < JB ? jb : JB - 1)) * 64 + l];
    }
    const int have = 16 * (JB - jb0);                  // channels of this chunk
    const int c = 16 * (l & 7) < have ? 16 * (l & 7) : 0;
    const uint8_t* src = p.Xq + (size_t)lr_m(v) * rowbytes + (size_t)(p.s_begin + 16 * jb0 + c) * ABITS / 8;
    if constexpr (ABITS == 8) {
      lrx[v] = *(const u4*)src;
    } else {
      const u2 x = *(const u2*)src;
      lrx[v] = u4{x.x, x.y, 0u, 0u};
    }
    }
  };
  constexpr int LRX_OFF = 16 * 1024;                   // R fragments at 0, codes (64 rows x 256 B of 16-bit floats) here
  auto lr_park = [&]() {
#pragma unroll
    for (int v = 0; v < VH; ++v) {
    const int lrow = lr_row(v);
#pragma unroll
    for (int q = 0; q < 2; ++q) *(u4*)(lds + (2 * (VH * w + v) + q) * 1024 + l * 16) = lrr[v][q];
    uint8_t* row = lds + LRX_OFF + lrow * 256;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      int k[8];
      if constexpr (ABITS == 8) codes_from_a8(h ? lrx[v].z : lrx[v].x, h ? lrx[v].w : lrx[v].y, k);
      else codes_from_a4(h ? lrx[v].y : lrx[v].x, k);
#pragma unroll
      for (int e = 0; e < 8; ++e) k[e] -= lzm[v];         // at most 255 in magnitude: exact in both 16-bit formats
      *(u4*)(row + 16 * ((2 * (l & 7) + h) ^ (lrow & 15))) = codes8_to_16bit(k, BF);
    }
    }
  };
  auto lr_first = [&]() {
    if (JB > 0) {
      lr_fetch(0);
#pragma unroll
      for (int v = 0; v < VH; ++v) lzm[v] = p.zero ? p.zero[lr_m(v)] : 0;
    }
  };
  if (ABITS == 4) lr_first();

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
  // MFMA tiles one after another, a fragment a step.  In the step after its last product a tile is folded; the last one of a
  // stage right behind it (the other wave of the SIMD works meanwhile).
  auto fold = [&](int u, float gs) {
#pragma unroll
    for (int e = 0; e < 16; ++e)
      accf[u >> 1][u & 1][e] = __builtin_fmaf(gs, (float)acc[u >> 1][u & 1][e], accf[u >> 1][u & 1][e]);
    // pinned here: left alone, the compiler puts folds off and keeps every INT32 tile alive (99 registers spilled)
    asm volatile("" : "+v"(accf[u >> 1][u & 1]));
  };
  if constexpr (ABITS == 8) {
    const int xsw = mid_swz128(lm);
    auto slot = [&](int h, int u) { return (2 * u + h) % NS * T::STAGE; };
    auto fill = [&](auto whole_c, auto h_c, int u, int k) {
      constexpr int H = decltype(h_c)::value;
      constexpr bool WHOLE = decltype(whole_c)::value;
      if (k < T::NL - 1) {
        ld.template issue_one<WHOLE>(H, u, my_lds + slot(H, u), k);
      } else {
        const int grp = (WHOLE ? (w + NW * u) * 2 : ld.flast) >> 1;
        dma4(sbase + ((size_t)(H && nbt > 1 ? G : 0) + grp) * 64, 4u * (l & 15), my_lds + slot(H, u) + T::SC_OFF);
      }
    };
    auto read = [&](auto, auto h_c, int u, GMidUnitOp& o) {
      constexpr int H = decltype(h_c)::value;
      const uint8_t* s = my + slot(H, u);
#pragma unroll
      for (int f = 0; f < 2; ++f) o.w[H][f] = *(const u4*)(s + kMidX + f * 1024 + l * 16);
      o.gs[H] = (float)*(const _Float16*)(s + T::SC_OFF + 2 * lm);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = 4 * (q >> 1) + 2 * g + (q & 1);
        o.x[H][q] = *(const u4*)(s + lm * 128 + 16 * (c ^ xsw));
      }
    };
    auto product = [&](auto h_c, const GMidUnitOp& o, int k) {   // tile 2*h + k/2, fragment k % 2
      constexpr int H = decltype(h_c)::value;
      const int q = 2 * H + k / 2, f = k % 2;
      const int i = q >> 1, j = q & 1;
      v4i a0, a1, b0, b1;
      unpack_frag(o.w[i][f], a0, a1);
      b0 = as_v4i(o.x[j][2 * f]);
      b1 = as_v4i(o.x[j][2 * f + 1]);
      if (f == 0) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(b0, a0, kZero16, 0, 0, 0);
      else acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(b0, a0, acc[i][j], 0, 0, 0);
      acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(b1, a1, acc[i][j], 0, 0, 0);
      if (k == 3) {
        fold(2 * H, o.gs[H]);
        fence();
        fold(2 * H + 1, o.gs[H]);
      }
    };
    mid_unit_loop<NS, T::NL, T::NL, 4, GMidUnitOp>(ld.nu, ld.nfull, ld.brief(), fill, read, product, lr_first);
  } else {
    const int xsw = mid_swz(lm);
    auto slot = [&](int t) { return (t % NS) * T::STAGE; };
    auto group = [&](int t) { return w + NW * t; };
    auto fill = [&](int t, int k) {
      const int s = group(t);
      if (k < T::NL - 1) ld.issue_one(s, my_lds + slot(t), k);
      else if (l < 8) dma16(sbase + (size_t)group(t) * 64, sv, my_lds + slot(t) + T::SC_OFF);
    };
    auto read = [&](int t, GMidStepOp& o) {
      const uint8_t* s = my + slot(t);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
#pragma unroll
        for (int f = 0; f < 2; ++f) o.w[i][f] = *(const u4*)(s + kMidX + (i * 2 + f) * 1024 + l * 16);
        o.gs[i] = (float)*(const _Float16*)(s + T::SC_OFF + 64 * i + 2 * lm);
      }
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int c = 2 * h + g;
          o.x[j][h] = *(const u4*)(s + (32 * j + lm) * 64 + 16 * (c ^ xsw));
        }
    };
    auto product = [&](const GMidStepOp& o, int k) {   // tile k / 2, fragment k % 2
      const int q = k / 2, f = k % 2;
      const int i = q >> 1, j = q & 1;
      v4i a0, a1, b0, b1;
      unpack_frag(o.w[i][f], a0, a1);
      unpack_frag(o.x[j][f], b0, b1);
      if (f == 0) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(b0, a0, kZero16, 0, 0, 0);
      else acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(b0, a0, acc[i][j], 0, 0, 0);
      acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(b1, a1, acc[i][j], 0, 0, 0);
      if (f == 1 && q > 0) fold(q - 1, o.gs[(q - 1) >> 1]);
      if (f == 1 && q == 3) {
        fence();
        fold(3, o.gs[1]);
      }
    };
    mid_loop<T::NL, 8, GMidStepOp>(
        nst,
        [&](int t) {
#pragma unroll
          for (int k = 0; k < T::NL; ++k) fill(t, k);
        },
        fill, read, product);
  }

  // ---- the waves meet.  8 waves: wave w finishes registers 8*(w%2) .. +7 of MFMA tile (i, j), w/2 = 2*i + j; 4 waves: all
  // of tile w = 2*i + j
  constexpr float kInv = 1.0f / (float)(1 << T::SH);
  constexpr int QN = 16 / NW, NE = 4 * QN;             // register quads, registers
  const int tt = NW == 8 ? w >> 1 : w;
  const int ti = tt >> 1, tj = tt & 1, hq = NW == 8 ? 2 * (w & 1) : 0;
  const int blk = nb0 + (ti < nbt ? ti : 0);
  const int n = 32 * blk + lm;                         // this lane's channel
  const int mloc = 32 * tj + 8 * hq + 4 * g;           // registers 4*q + e: token mloc + 8*q + e
  float sm[NE], zf[NE];
#pragma unroll
  for (int q = 0; q < QN; ++q)
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
  float y[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) y[e] = 0.0f;
#pragma unroll
  for (int ww = 0; ww < NW; ++ww)
#pragma unroll
    for (int q = 0; q < QN; ++q) {
      const v4f v = *(const v4f*)(lds + ww * T::REGION + (tt * 4 + hq + q) * 1024 + l * 16);
      y[4 * q] += v.x; y[4 * q + 1] += v.y; y[4 * q + 2] += v.z; y[4 * q + 3] += v.w;
    }
#pragma unroll
  for (int e = 0; e < NE; ++e) y[e] = __builtin_fmaf(y[e], kInv, -zf[e] * ws);   // 2^-SH: exact
  if (JB > 0) {
    v16f af;                                           // the tile the matrix unit adds to
#pragma unroll
    for (int e = 0; e < 16; ++e) af[e] = NW == 4 ? y[e % NE] : (e >> 3) == (hq >> 1) ? y[e & 7] : 0.0f;
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
    for (int e = 0; e < NE; ++e) y[e] = NW == 4 ? af[e] : hq ? af[(8 + e) & 15] : af[e];
  }
#pragma unroll
  for (int e = 0; e < NE; ++e) y[e] *= sm[e];

  if (p.y_dtype == SERQ_F32) {                         // 32 lanes write 128 contiguous bytes
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const int r = mloc + 8 * (e >> 2) + (e & 3);
      if (r < mrows && ti < nbt) ((float*)p.Y)[(size_t)(m0 + r) * p.ldy + n] = y[e];
    }
    return;
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const int r = mloc + 8 * (e >> 2) + (e & 3), c = 32 * ti + lm;
    *(uint16_t*)(lds + r * 128 + 16 * ((c >> 3) ^ (r & 7)) + 2 * (c & 7)) =
        p.y_dtype == SERQ_BF16 ? f32_to_bf16_rne(y[e]) : f32_to_f16_rne(y[e]);
  }
  __syncthreads();
  mid_store16<64 * NW>(lds, tid, (uint16_t*)p.Y, p.ldy, m0, mrows, 32 * nb0, nbt);
}

}  // namespace

// Up to three tiles per compute unit, as far as that is the cheaper kernel.  One tile: always; two: always with 4-bit tokens.
// Else by prices as in mid_tile.h, which know the rank here, because the tiled kernel pays more for it:
//   small tiles  c0 + c1 R + K/1024 (c2 + c3 R + c4 y) + c5 (MB of weight codes) + r/128 (c6 + c7 R)
//   tiled        d0 + d1 K/1024 (halves of tiles) or d2 K/1024 (whole ones) + d3 (r > 0) + d4 r/128
// fitted to 800 launches with an error of 4 to 5 % (three tiles per compute unit are at most one round of the tiled kernel); 8-bit tokens'
// small-tile price to 367 layers of the kernel with whole-line token rows, 7 % (of 500 other layers of two and three tiles 8 would be more
// than 3 % faster in the other kernel, the worst 6 %; with the price of 64-byte rows 41, the worst 18 %).
// Measured (us, tiled kernel / this one, N x K, weights from HBM; in brackets: tiles of the busiest compute unit):
//   W4A8 r = 128  4096 x 4096 M = 256 (1) 23.1 / 13.4, M = 512 (2) 23.0 / 21.9, M = 768 (3) 33.4 / 28.2;  11008 x 14336 M = 128 (2)
//        59.5 / 53.3;  15968 x 6144 M = 128 (2) 32.6 / 28.7
//   r = 0  4096 x 1024 M = 512 (2) 8.5 / 8.8, M = 768 (3) 11.3 / 13.6 (both to the tiled kernel);  4096 x 4096 M = 768 (3)
//        29.4 / 28.1;  8096 x 5120 M = 192 (2) 23.7 / 21.7
//   W4A4 r = 128  4096 x 14336 M = 512 (2) 62 / 43, M = 768 (3) 96 / 62;  4096 x 768 M = 768 (3) level
bool g128_mid_wanted(const G128Args& a, int abits) {
  const int ncu = device_cu_count();
  const long long rounds = mid_rounds(a.M, a.N, ncu);
  if (rounds > 3) return false;
  if (rounds == 1 || (rounds == 2 && abits == 4)) return true;
  static constexpr MidPrice small8 = {{2.28f, 2.24f, 0.11f, 0.81f, 0.60f, 0.07f}}, small4 = {{2.64f, 2.28f, 0.27f, 0.80f, 0.34f, 0.05f}};
  const long long tiles = ((long long)a.M + 127) / 128 * ((a.N + 127) / 128);
  const float k = a.K / 1024.0f, r = a.r / 128.0f;
  const float small = abits == 8 ? mid_price(small8, a.M, a.N, a.K, ncu) + r * (0.69f + 0.31f * rounds)
                                 : mid_price(small4, a.M, a.N, a.K, ncu) + r * (0.35f + 0.49f * rounds);
  const float tiled = 4.6f + k * (2 * tiles <= ncu ? (abits == 8 ? 3.65f : 3.80f) : (abits == 8 ? 6.1f : 6.4f)) +
                      (a.r > 0 ? 0.31f : 0.0f) + r * 3.45f;
  return 0.97f * small < tiled;
}

int launch_g128_mid(const G128Args& a, int abits, hipStream_t st) {
  const int tm = (a.M + 63) / 64, tn = (a.N + 63) / 64;
  const dim3 grid((unsigned)(tm * tn));
  const bool bf = a.r_dtype != SERQ_F16;
  const int band = mid_band(tm, (long long)a.M * a.K * abits / 8);
  // One tile per compute unit at most: 8 waves, which the folds need to keep the vector units busy.  More tiles: workgroups
  // of 4 waves, two of which share a compute unit, so that one's start and end run beside the other's main loop.
  // Measured (us, 8 / 4 waves, r = 128, N x K): W4A8 4096 x 11008 M = 100 21.9 / 23.3, M = 333 41.2 / 35.4; 6144 x 4096
  // M = 100 12.2 / 13.0, M = 256 22.2 / 18.0; 4096 x 1024 M = 100 7.1 / 8.0, M = 333 12.9 / 9.9; W4A4 4096 x 11008 M = 150 19.4 / 21.3, M = 333 35.8 / 32.0.
  const bool eight = tm * tn <= device_cu_count();
#define SERQ_GMID_LAUNCH(AB, BF)                                                                                       \
  do {                                                                                                                 \
    if (eight) hipLaunchKernelGGL((serq_g128_mid_kernel<AB, BF, 8>), grid, dim3(512), 0, st, a, tm, tn, band);         \
    else hipLaunchKernelGGL((serq_g128_mid_kernel<AB, BF, 4>), grid, dim3(256), 0, st, a, tm, tn, band);               \
  } while (0)
  if (abits == 8) {
    if (bf) SERQ_GMID_LAUNCH(8, true); else SERQ_GMID_LAUNCH(8, false);
  } else {
    if (bf) SERQ_GMID_LAUNCH(4, true); else SERQ_GMID_LAUNCH(4, false);
  }
#undef SERQ_GMID_LAUNCH
  return hipGetLastError() == hipSuccess ? SERQ_OK : SERQ_EHIP;
}

}  // namespace serq
