// SERQ linear layer for batches between decode and prefill: the integer layer of gemm_mfma.hip in tiles of
// 64 tokens x 64 channels, the 4 waves of a workgroup sharing K (mid_tile.h says why).
//   Y[m,n] = scale[m] * ( wscale[n] * sum_k Xq[m,k] Wq[n,k] + sum_j Xq[m,S_j] R[j,n] )
//
// The waves' INT32 partial tiles meet in LDS once: each wave sums one MFMA tile over the waves -- integer addition, the same
// bits as the tiled kernel -- scales it and adds the rank-r term with the matrix unit on top, exactly as the tiled kernel does.
//
// What bounds it: with 8-bit tokens at M = 256, N = 4096, K = 11008 the kernel takes 20.5 us (23.1 with 64-byte token rows); the
// same load stream without products, launch included, 12.6 us (at K = 11264), the matrix unit alone 6.  The rest is the start
// and the end of a tile and what the two do not overlap.  Fixed costs: 4 us at K = 256, r = 0 in a graph, 1 us more for r = 128.
// The tiled kernel with 4 K slices and a second launch takes 32 us there; M = 100, 6144 x 4096: 9.0 against 24.4 us.
// The rank-r operands through LDS, converted once: 2.2 -> 1.0 us at r = 128.  They used to wait for the partial tiles to be added and
// then took their place, two barriers later; beside the partial tiles, of which a wave parks only those it does not finish itself, they
// are there at the same barrier.  us, before / now, r = 128 unless given, N x K, weights from HBM: W4A8 4096 x 1024 M = 100 5.85 / 5.68,
// 4096 x 4096 M = 333 15.3 / 14.9, M = 512 17.6 / 17.3, 6144 x 4096 M = 100 10.21 / 10.04, 4096 x 11008 M = 256 20.7 / 20.5; W4A4 4096 x 4096
// M = 333 r = 64 13.85 / 13.47, M = 900 r = 256 26.6 / 26.1.  Requested before the last products instead of behind them: the same with
// 8-bit tokens, with 4-bit ones 4096 x 11008 M = 200 16.2 -> 16.8; half a unit earlier still 6144 x 4096 M = 100 10.2 -> 10.45.
// Rings of twice the depth where a workgroup has a compute unit to itself: 9.3 -> 10.0 us at M = 100, 6144 x 4096 (the first stage
// lands behind all the others' requests).
//
// Two workgroups share a compute unit: one's start and end run beside the other's main loop.  Workgroups of 8 waves that have one to
// themselves keep more loads in flight, which pays no more since the loads are whole lines: us, 8 / 4 waves, W4A8, r = 128, N x K, one tile
// per compute unit at most: 4096 x 11008 M = 100 18.2 / 18.1, M = 256 20.9 / 20.5; 4096 x 9216 M = 150 14.0 / 13.2; 4096 x 14336 M = 256
// 25.8 / 24.5; 16384 x 11008 M = 64 23.7 / 24.1; 4096 x 4096 M = 100 9.6 / 9.1; the one length where 8 waves are better is K = 2048, whose
// units come out even: 4096 x 2048 M = 100 6.9 / 7.3 (4096 x 1536 7.2 / 6.9, 4096 x 2560 8.5 / 7.9).  More tiles: 4096 x 4096
// M = 333 17.7 / 14.3.
#include "mid_tile.h"

namespace serq {
namespace {

struct MidParams {
  const uint8_t* Xq; const float* scale;
  const u4* Wq; const float* wscale;
  const u4* Rp; int s_begin; int r;
  const float* rscale;
  int M, N, K;
  void* Y; int y_dtype; int64_t ldy;
  int32_t* acc_out; int64_t ldacc;
  int tiles_m, tiles_n, band;
};

constexpr int NW = 4;                                // waves of a workgroup

template <int ABITS>
struct Mid {
  static constexpr int STAGE = kMidX + (ABITS == 8 ? 2 : 4) * 1024;   // 6 KiB: half a unit / 8 KiB: a step
  static constexpr int NS = ABITS == 8 ? 3 : 2;
  static constexpr int NL = ABITS == 8 ? 6 : 8;      // direct loads of a stage
  static constexpr int REGION = NS * STAGE;          // LDS of one wave: 18 KiB / 16 KiB
  static constexpr int SH = ABITS == 8 ? 4 : 8;
  // A wave keeps the MFMA tile that it finishes and parks the other three at the start of its region.  Behind them lies its share
  // of a chunk of the rank-r term, 128 ranks: four R fragments (4-bit R: two, of the first two waves) and the codes of 16 token rows
  // of 256 bytes, the first XIN of them in its region, the others behind all regions.
  static constexpr int LRR_OFF = 3 * kMidPart / 4, LRX_OFF = LRR_OFF + 4 * 1024;
  static constexpr int XIN = REGION - LRX_OFF >= 8 * 256 ? 8 : 0;
  static constexpr int LDS = NW * (REGION + (16 - XIN) * 256);
  static_assert(REGION >= LRX_OFF + XIN * 256, "what a wave parks fits the ring it replaces");
  static_assert(2 * LDS <= 160 * 1024, "LDS budget: two workgroups");
};

struct MidUnitOp { u4 w[2][2], x[2][4]; };           // w: [channel block][fragment], x: [token block][2 * fragment + K half]
struct MidStepOp { u4 w[2][2], x[2][2]; };           // x: [token block][fragment]

template <int ABITS, int LRT>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 2)))
void serq_mid_kernel(const MidParams p) {
  using T = Mid<ABITS>;
  constexpr int NS = T::NS;
  __shared__ __align__(16) uint8_t lds[T::LDS];
  const int tid = threadIdx.x, l = tid & 63, lm = l & 31, g = l >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tile_m, tile_n;
  map_block(blockIdx.x, p.tiles_m, p.tiles_n, p.band, tile_m, tile_n);
  const int m0 = tile_m * 64, nb0 = tile_n * 2;
  const int NB = p.N >> 5;
  const int nbt = NB - nb0 < 2 ? 1 : 2;
  const int mrows = p.M - m0 < 64 ? p.M - m0 : 64;
  const uint32_t rowbytes = (uint32_t)p.K * ABITS / 8;

  std::conditional_t<ABITS == 8, MidUnits<2, NW>, MidLoads> ld;
  if constexpr (ABITS == 8) ld.init(p.Xq, p.Wq, p.K, rowbytes, m0, mrows, nb0, nbt, w, l);
  else ld.init(p.Xq, p.Wq, p.K, rowbytes, m0, mrows, nb0, nbt, l);
  const int steps = (ld.KB + 1) / 2;
  const int nst = steps > w ? (steps - w + NW - 1) / NW : 0;   // 4-bit: steps w, w + NW, ... are this wave's
  uint8_t* my = lds + w * T::REGION;
  const uint32_t my_lds = __builtin_amdgcn_readfirstlane(lds_addr(my));

  v16i acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0;

  if constexpr (ABITS == 8) {
    const int xsw = mid_swz128(lm);
    auto slot = [&](int h, int u) { return (2 * u + h) % NS * T::STAGE; };
    // (the second fragment of a unit that has but one is not multiplied: `brief`)
    auto read = [&](auto, auto h_c, int u, MidUnitOp& o) {
      constexpr int H = decltype(h_c)::value;
      const uint8_t* s = my + slot(H, u);
#pragma unroll
      for (int f = 0; f < 2; ++f) o.w[H][f] = *(const u4*)(s + kMidX + f * 1024 + l * 16);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = 4 * (q >> 1) + 2 * g + (q & 1);
        o.x[H][q] = *(const u4*)(s + lm * 128 + 16 * (c ^ xsw));
      }
    };
    // group k of half h: token block k % 2 and channel block k / 2 of fragment h
    auto product = [&](auto h_c, const MidUnitOp& o, int k) {
      const int j = k & 1, i = (k >> 1) & 1, f = decltype(h_c)::value;
      v4i a0, a1, b0, b1;
      unpack_frag(o.w[i][f], a0, a1);
      b0 = as_v4i(o.x[j][2 * f]);
      b1 = as_v4i(o.x[j][2 * f + 1]);
      acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a0, b0, acc[i][j], 0, 0, 0);
      acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a1, b1, acc[i][j], 0, 0, 0);
    };
    mid_unit_loop<NS, T::NL, T::NL, 4, MidUnitOp>(
        ld.nu, ld.nfull, ld.brief(),
        [&](auto whole_c, auto h_c, int u, int k) {
          constexpr int H = decltype(h_c)::value;
          ld.template issue_one<decltype(whole_c)::value>(H, u, my_lds + slot(H, u), k);
        },
        read, product, []() {});
  } else {
    const int xsw = mid_swz(lm);                       // the same for row lm and row 32 + lm
    auto slot = [&](int t) { return (t % NS) * T::STAGE; };
    auto read = [&](int t, MidStepOp& o) {
      const uint8_t* s = my + slot(t);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int f = 0; f < 2; ++f) o.w[i][f] = *(const u4*)(s + kMidX + (i * 2 + f) * 1024 + l * 16);
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int f = 0; f < 2; ++f) o.x[j][f] = *(const u4*)(s + (32 * j + lm) * 64 + 16 * ((2 * f + g) ^ xsw));
      if (ld.KB - (w + NW * t) * 2 < 2) {               // no second fragment: zero weights
#pragma unroll
        for (int i = 0; i < 2; ++i) o.w[i][1] = u4{0u, 0u, 0u, 0u};
      }
    };
    // group k: token block k % 2, channel block k / 2 % 2 of fragment k / 4
    auto product = [&](const MidStepOp& o, int k) {
      const int j = k & 1, i = (k >> 1) & 1, f = k >> 2;
      v4i a0, a1, b0, b1;
      unpack_frag(o.w[i][f], a0, a1);
      unpack_frag(o.x[j][f], b0, b1);
      acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a0, b0, acc[i][j], 0, 0, 0);
      acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a1, b1, acc[i][j], 0, 0, 0);
    };
    mid_loop<T::NL, 8, MidStepOp>(
        nst, [&](int t) { ld.issue(w + NW * t, my_lds + slot(t)); },
        [&](int t, int k) { ld.issue_one(w + NW * t, my_lds + slot(t), k); }, read, product);
  }

  // ---- what the end of the tile needs from memory, requested before the waves meet ------------------------------
  // Wave w finishes MFMA tile (i, j), w = 2*i + j.
  constexpr int QN = 4, NE = 4 * QN;                  // register quads, registers
  const int ti = w >> 1, tj = w & 1;
  const int blk = nb0 + (ti < nbt ? ti : 0);          // (a block past the layer repeats the first and is not stored)
  const int mloc = 32 * tj + lm;
  const int m = m0 + (mloc < mrows ? mloc : mrows - 1);
  constexpr float kInv = 1.0f / (float)(1 << T::SH);
  constexpr bool lr_int = LRT == SERQ_I4;
  constexpr bool bf = LRT != SERQ_F16;
  const int JB = p.acc_out ? 0 : (lr_int ? (p.r + 63) >> 6 : p.r >> 4);   // fragments of R per channel block
  constexpr int NJ = lr_int ? 2 : 8;                  // of which a chunk holds so many
  // A chunk of the rank-r term is dealt out in 8 shares, two to a wave: 2 of its R fragments (4-bit R: one, shares 0..3) and
  // 16 codes of 8 token rows per lane; 16-bit R takes the codes as exact 16-bit floats, converted once here instead of by
  // every wave that multiplies them.
  constexpr int VH = 8 / NW;
  u4 lrr[VH][2], lrx[VH];
  auto lr_fetch = [&](int jb0) {
#pragma unroll
    for (int v = 0; v < VH; ++v) {
    const int vw = VH * w + v, lrow = 8 * vw + (l >> 3);
#pragma unroll
    for (int q = 0; q < (lr_int ? 1 : 2); ++q) {
      const int f = lr_int ? (vw & 3) : 2 * vw + q;
      const int b = f >> (lr_int ? 1 : 3), jb = jb0 + (f & (NJ - 1));
      lrr[v][q] = p.Rp[((size_t)(nb0 + (b < nbt ? b : 0)) * JB + (jb < JB ? jb : JB - 1)) * 64 + l];
    }
    const int c0 = p.s_begin + (lr_int ? 64 : 16) * jb0;   // first channel of the chunk
    const int have = (JB - jb0) * (lr_int ? 64 : 16);  // channels it has
    const int c = 16 * (l & 7) < have ? 16 * (l & 7) : 0;
    const uint8_t* src = p.Xq + (size_t)(m0 + (lrow < mrows ? lrow : mrows - 1)) * rowbytes + (size_t)(c0 + c) * ABITS / 8;
    if constexpr (ABITS == 8) {
      lrx[v] = *(const u4*)src;
    } else {
      const u2 x = *(const u2*)src;
      lrx[v] = u4{x.x, x.y, 0u, 0u};
    }
    }
  };
  // where fragment f of a chunk lies (brought by wave f / 4, 4-bit R: f / 2), and token row `row` of it (by wave row / 16)
  auto lr_frag = [&](int f) { return lds + (lr_int ? (f >> 1) * T::REGION + (f & 1) * 1024 : (f >> 2) * T::REGION + (f & 3) * 1024) + T::LRR_OFF; };
  auto lr_row = [&](int row) {
    const int ww = row >> 4, k = row & 15;
    return lds + (k < T::XIN ? ww * T::REGION + T::LRX_OFF + k * 256
                             : NW * T::REGION + (ww * (16 - T::XIN) + k - T::XIN) * 256);
  };
  auto lr_park = [&]() {
#pragma unroll
    for (int v = 0; v < VH; ++v) {
    const int vw = VH * w + v, lrow = 8 * vw + (l >> 3);
#pragma unroll
    for (int q = 0; q < (lr_int ? 1 : 2); ++q) {
      const int f = lr_int ? (vw & 3) : 2 * vw + q;
      if (!lr_int || vw < 4) *(u4*)(lr_frag(f) + l * 16) = lrr[v][q];
    }
    uint8_t* row = lr_row(lrow);
    const int c = l & 7;                              // 16 channels
    if constexpr (lr_int) {
      if constexpr (ABITS == 8) *(u4*)(row + 16 * (c ^ (lrow & 15))) = lrx[v];
      else *(u2*)(row + 16 * ((c >> 1) ^ (lrow & 15)) + 8 * (c & 1)) = u2{lrx[v].x, lrx[v].y};
    } else {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        int k[8];
        if constexpr (ABITS == 8) codes_from_a8(h ? lrx[v].z : lrx[v].x, h ? lrx[v].w : lrx[v].y, k);
        else codes_from_a4(h ? lrx[v].y : lrx[v].x, k);
        *(u4*)(row + 16 * ((2 * c + h) ^ (lrow & 15))) = codes8_to_16bit(k, bf);
      }
    }
    }
  };
  if (JB > 0) lr_fetch(0);
  float wsc[NE], rsc[NE], sm = 0.0f;
#pragma unroll
  for (int e = 0; e < NE; ++e) wsc[e] = rsc[e] = 0.0f;
  if (!p.acc_out) {
    sm = p.scale[m];
#pragma unroll
    for (int q = 0; q < QN; ++q) {
      const int n = 32 * blk + 8 * q + 4 * g;
      const float4 v = *(const float4*)(p.wscale + n);
      wsc[4 * q] = v.x * kInv; wsc[4 * q + 1] = v.y * kInv; wsc[4 * q + 2] = v.z * kInv; wsc[4 * q + 3] = v.w * kInv;
      if (lr_int && JB > 0) {
        const float4 u = *(const float4*)(p.rscale + n);
        rsc[4 * q] = u.x * kInv; rsc[4 * q + 1] = u.y * kInv; rsc[4 * q + 2] = u.z * kInv; rsc[4 * q + 3] = u.w * kInv;
      }
    }
  }

  // ---- the waves meet -------------------------------------------------------------------------------------------
  // Tile t goes to slot (t - w - 1) % 4 of this wave's region; its own stays in registers.
  v16i tot;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const v16i& a = acc[t >> 1][t & 1];
    if (t == w) {                                      // uniform
      tot = a;
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *(v4i*)(my + (((t - w - 1) & 3) * 4 + q) * 1024 + l * 16) = v4i{a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]};
    }
  }
  if (JB > 0) lr_park();
  __syncthreads();
#pragma unroll
  for (int d = 1; d < NW; ++d) {                       // wave w + d has this wave's tile in slot 3 - d
    const uint8_t* src = lds + ((w + d) & 3) * T::REGION + (3 - d) * 4096 + l * 16;
#pragma unroll
    for (int q = 0; q < QN; ++q) {
      const v4i v = *(const v4i*)(src + q * 1024);
      tot[4 * q] += v.x; tot[4 * q + 1] += v.y; tot[4 * q + 2] += v.z; tot[4 * q + 3] += v.w;
    }
  }

  const bool live = mloc < mrows && ti < nbt;
  const int n = 32 * blk + 4 * g;                      // registers 4*q + e: channel n + 8*q + e
  if (p.acc_out) {
    if (live) {
#pragma unroll
      for (int q = 0; q < QN; ++q)
        *(v4i*)(p.acc_out + (size_t)m * p.ldacc + n + 8 * q) =
            v4i{tot[4 * q] >> T::SH, tot[4 * q + 1] >> T::SH, tot[4 * q + 2] >> T::SH, tot[4 * q + 3] >> T::SH};
    }
    return;
  }
  float y[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) y[e] = wsc[e] * (float)tot[e];
  v16f af;                                            // 16-bit R: the tile the matrix unit adds to
#pragma unroll
  for (int e = 0; e < 16; ++e) af[e] = y[e];
  for (int jb0 = 0; jb0 < JB; jb0 += NJ) {
    if (jb0 > 0) {                                     // (the loads of this chunk were requested a chunk ago)
      __syncthreads();
      lr_park();
      __syncthreads();
    }
    if (jb0 + NJ < JB) lr_fetch(jb0 + NJ);
    const uint8_t* row = lr_row(mloc);
    auto piece = [&](int c) { return *(const u4*)(row + 16 * (c ^ (mloc & 15))); };
#pragma unroll
    for (int q = 0; q < NJ; ++q) {
      if (jb0 + q < JB) {                              // uniform
        const int f = ti * NJ + q;
        const u4 rr = *(const u4*)(lr_frag(f) + l * 16);
        if constexpr (lr_int) {
          v4i a0, a1, b0, b1;
          unpack_frag(rr, a0, a1);
          if constexpr (ABITS == 8) {
            b0 = as_v4i(piece(4 * q + 2 * g));
            b1 = as_v4i(piece(4 * q + 2 * g + 1));
          } else {
            unpack_frag(piece(2 * q + g), b0, b1);
          }
          v16i tq;
#pragma unroll
          for (int e = 0; e < 16; ++e) tq[e] = 0;
          tq = __builtin_amdgcn_mfma_i32_32x32x32_i8(a0, b0, tq, 0, 0, 0);
          tq = __builtin_amdgcn_mfma_i32_32x32x32_i8(a1, b1, tq, 0, 0, 0);
#pragma unroll
          for (int e = 0; e < NE; ++e) y[e] = __builtin_fmaf(rsc[e], (float)tq[e], y[e]);
        } else {
          const u4 xf = piece(2 * q + g);
          if constexpr (bf)
            af = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, rr), __builtin_bit_cast(v8bf, xf), af, 0, 0, 0);
          else
            af = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, rr), __builtin_bit_cast(v8h, xf), af, 0, 0, 0);
        }
      }
    }
  }
  if constexpr (!lr_int) {
#pragma unroll
    for (int e = 0; e < NE; ++e) y[e] = af[e];
  }
#pragma unroll
  for (int e = 0; e < NE; ++e) y[e] *= sm;

  if (p.y_dtype == SERQ_F32) {
    if (live) {
#pragma unroll
      for (int q = 0; q < QN; ++q)
        *(float4*)((float*)p.Y + (size_t)m * p.ldy + n + 8 * q) = make_float4(y[4 * q], y[4 * q + 1], y[4 * q + 2], y[4 * q + 3]);
    }
    return;
  }
  __syncthreads();                                     // every wave has read the partial tiles: the rows take their place
#pragma unroll
  for (int q = 0; q < QN; ++q) mid_park16(lds, mloc, 4 * ti + q, g, y + 4 * q, p.y_dtype == SERQ_BF16);
  __syncthreads();
  mid_store16<64 * NW>(lds, tid, (uint16_t*)p.Y, p.ldy, m0, mrows, 32 * nb0, nbt);
}

}  // namespace

// Up to three tiles per compute unit, four with 4-bit tokens, as far as that is the cheaper kernel (mid_cheaper): the larger
// tiles of the tiled kernel move half the bytes per product, and with a long K its slices fill the chip too.  Measured
// (us, tiled kernel / this one, r = 128, N x K, weights from HBM; in brackets: tiles of the busiest compute unit):
//   W4A8  4096 x 4096 M = 256 (1) 26.4 / 10.1, M = 512 (2) 25.4 / 16.4, M = 768 (3) 26.9 / 22.7;  4096 x 14336 M = 256 (1) 34.7 / 24.6,
//         M = 512 (2) 49.6 / 45.8, M = 768 (3) 78.6 / 63.7;  11008 x 14336 M = 100 (2) 78 / 43, M = 192 (3) 59.7 / 58.4, from the
//         last-level cache 55.9 / 51.2 (to the tiled kernel);  11008 x 11008 M = 192 (3) 49.0 / 46.2;  4096 x 17408 M = 384 (2) 52.7 / 50.1;
//         4096 x 28672 M = 256 (1) 51.6 / 45.9, M = 512 (2) 74.5 / 82.7 (to the tiled kernel)
//   W4A4  4096 x 4096 M = 1024 (4) 26 / 24;  4096 x 14336 M = 1024 (4) 67 / 63;  11008 x 28672 M = 256 (3) 92 / 102, weights
//         from the last-level cache 93 / 87
// Ranks up to 1024 do not move the line: both kernels pay alike for them.
bool mid_wanted(const LinearArgs& a) {
  static constexpr MidPrice small8 = {{2.82f, 1.58f, 0.17f, 0.73f, 0.50f, 0.05f}}, small4 = {{3.02f, 1.66f, 0.17f, 0.53f, 0.40f, 0.07f}};
  static constexpr TiledPrice tiled8 = {{8.15f, 2.74f, 0.83f, 3.26f, 8.33f, 0.83f}}, tiled4 = {{8.66f, 2.25f, 0.94f, 0.0f, 6.69f, 0.61f}};
  const size_t skip = skinny_workspace_bytes(a.N);
  const size_t have = a.workspace && a.workspace_bytes > skip ? a.workspace_bytes - skip : 0;
  return a.abits == 8 ? mid_cheaper(small8, tiled8, a.M, a.N, a.K, 8, 3, 1.02f, have)
                      : mid_cheaper(small4, tiled4, a.M, a.N, a.K, 4, 4, 0.93f, have);
}

int launch_mid(const LinearArgs& a, hipStream_t st) {
  MidParams p;
  p.Xq = a.Xq; p.scale = a.scale; p.Wq = a.Wq; p.wscale = a.wscale;
  p.Rp = a.Rp; p.s_begin = a.s_begin; p.r = a.Rp ? a.r : 0;
  p.rscale = a.rscale;
  p.M = a.M; p.N = a.N; p.K = a.K;
  p.Y = a.Y; p.y_dtype = a.y_dtype; p.ldy = a.ldy;
  p.acc_out = a.acc_out; p.ldacc = a.ldacc;
  p.tiles_m = (a.M + 63) / 64;
  p.tiles_n = (a.N + 63) / 64;
  p.band = mid_band(p.tiles_m, (long long)a.M * a.K * a.abits / 8);
  const dim3 grid((unsigned)(p.tiles_m * p.tiles_n));
  const bool has_lr = p.r > 0 && p.acc_out == nullptr;
  const int lrt = !has_lr ? SERQ_BF16 : a.r_dtype;
#define SERQ_MID_LAUNCH(AB, LRT) hipLaunchKernelGGL((serq_mid_kernel<AB, LRT>), grid, dim3(64 * NW), 0, st, p)
  if (a.abits == 8) {
    if (lrt == SERQ_I4) SERQ_MID_LAUNCH(8, SERQ_I4);
    else if (lrt == SERQ_F16) SERQ_MID_LAUNCH(8, SERQ_F16);
    else SERQ_MID_LAUNCH(8, SERQ_BF16);
  } else {
    if (lrt == SERQ_I4) SERQ_MID_LAUNCH(4, SERQ_I4);
    else if (lrt == SERQ_F16) SERQ_MID_LAUNCH(4, SERQ_F16);
    else SERQ_MID_LAUNCH(4, SERQ_BF16);
  }
#undef SERQ_MID_LAUNCH
  return hipGetLastError() == hipSuccess ? SERQ_OK : SERQ_EHIP;
}

}  // namespace serq
