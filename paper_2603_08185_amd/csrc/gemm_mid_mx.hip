// The MXFP4 layer for batches between decode and prefill: tiles of 64 tokens x 64 channels, the 4 waves of a workgroup
// sharing K (mid_tile.h says why).
//   Y[m,n] = sum_k X^[m,k] W^[n,k] + sum_{j<r} X^[m,s_begin+j] R^[n,j]
//
// A wave's units are the 256-channel scale tiles (what is left over is dealt in halves of them), the scales of the tile
// with the first half.  A 16-byte piece from LDS is an operand of the block-scaled MFMA as it is.  The
// compensation fragments (64 ranks each) are dealt to the waves one by one after the main loop; the first one's operands
// are requested in front of the last unit.  The waves' fp32 tiles are added through LDS in wave order: the same result
// from run to run.
//
// What bounds it: the load stream and how far the products overlap it, as in gemm_mid.hip.  Measured (M = 200, 4096 x 14336,
// r = 128, graph replay): 16.3 us (17.9 with 64-byte token rows), the tiled kernel with its K slices and second launch 33 us; M = 500,
// 4096 x 4096 11.9 -> 10.5 us, M = 200, K = 1024 4.5 -> 4.6 us.  The rank-r term costs nothing that shows.
#include "mid_tile.h"

namespace serq {
namespace {

struct MxMidParams {
  const uint8_t* Xq; const uint8_t* xsc;
  const u4* Wq; const uint8_t* wsc;
  const u4* Rq; const uint8_t* rsc; int s_begin; int r;
  int M, N, K;
  void* Y; int y_dtype; int64_t ldy;
  int tiles_m, tiles_n, band;
};

constexpr int FU = 4;                                // fragments of a unit: a 256-channel scale tile
constexpr int STAGE = kMidX + FU * 1024;             // 8 KiB
constexpr int NW = 4;                                // waves: two workgroups share a compute unit
constexpr int NS = 2;
constexpr int WS_OFF = NS * STAGE;                   // weight scales of a tile: 2 blocks x 64 dwords
constexpr int XS_OFF = WS_OFF + 512;                 // token scales of a tile: 64 rows x 8 bytes
constexpr int REGION = XS_OFF + 512;
static_assert(REGION >= kMidPart, "a partial tile fits the ring it replaces");

struct MxMidOp { u4 w[2][FU], x[2][FU]; uint32_t ws[2], xs[2]; };   // ws, xs: byte c is the scale of fragment c

__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 2)))
void serq_mx_mid_kernel(const MxMidParams p) {
  __shared__ __align__(16) uint8_t lds[NW * REGION];      // 17 KiB a wave
  const int tid = threadIdx.x, l = tid & 63, lm = l & 31, g = l >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tile_m, tile_n;
  map_block(blockIdx.x, p.tiles_m, p.tiles_n, p.band, tile_m, tile_n);
  const int m0 = tile_m * 64, nb0 = tile_n * 2;
  const int NB = p.N >> 5;
  const int nbt = NB - nb0 < 2 ? 1 : 2;
  const int mrows = p.M - m0 < 64 ? p.M - m0 : 64;
  const uint32_t rowbytes = (uint32_t)p.K >> 1;
  const size_t Mp = (size_t)((p.M + 1) & ~1);          // rows of a tile of the token-scale array

  MidUnits<FU, NW, true, true> ld;
  ld.init(p.Xq, p.Wq, p.K, rowbytes, m0, mrows, nb0, nbt, w, l);
  const int T = (ld.KB + 3) >> 2;                      // scale tiles
  uint8_t* my = lds + w * REGION;
  const uint32_t my_lds = __builtin_amdgcn_readfirstlane(lds_addr(my));
  const uint32_t xsel = g ? 0x07050301u : 0x06040200u;   // bytes g, 2+g, 4+g, 6+g of a token's 8 scales

  // ---- the first compensation fragment of this wave, requested in front of its last unit (when no load of the ring is
  // waited for any more)
  const int LF = (p.r + 63) >> 6, LT = (LF + 3) >> 2;   // fragments and scale tiles of the compensation matrix per block
  u4 rq[2], rx[2];
  uint32_t rs[2], rxs[2];
  auto lr_fetch = [&](int jf) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const size_t b = nb0 + (i < nbt ? i : 0);
      rq[i] = p.Rq[(b * LF + jf) * 64 + l];
      rs[i] = ((const uint32_t*)p.rsc)[(b * LT + (jf >> 2)) * 64 + l] >> (8 * (jf & 3));
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int r0 = 32 * j + lm, m = m0 + (r0 < mrows ? r0 : mrows - 1);
      rx[j] = *(const u4*)(p.Xq + (size_t)m * rowbytes + ((p.s_begin + 64 * jf) >> 1) + 16 * g);
      const u2 e = *(const u2*)(p.xsc + ((size_t)((p.s_begin >> 8) + (jf >> 2)) * Mp + m) * 8);
      rxs[j] = __builtin_amdgcn_perm(e.y, e.x, xsel) >> (8 * (jf & 3));
    }
  };

  // ---- main loop ------------------------------------------------------------------------------------------------
  v16f acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
  const int xsw = mid_swz128(lm);
  // scales of a tile, in one load: lanes 0..15 / 16..31 bring those of weight block 0 / 1, lanes 32..63 those of two token rows
  // each
  const int rp = 2 * (l & 31) < mrows ? l & 31 : (mrows - 1) >> 1;
  const uint8_t* scsrc = l < 32 ? p.wsc + ((size_t)nb0 * T + (l >= 16 && nbt > 1 ? T : 0)) * 256 + (l & 15) * 16
                                : p.xsc + (size_t)m0 * 8 + rp * 16;
  const uint64_t scstep = l < 32 ? 256 : Mp * 8;       // from one tile's to the next one's
  auto fill = [&](auto whole_c, auto h_c, int u, int k) {
    constexpr int H = decltype(h_c)::value;
    if (k < 8) {
      ld.template issue_one<decltype(whole_c)::value>(H, u, my_lds + H * STAGE, k);
    } else {
      const int tile = (decltype(whole_c)::value ? FU * (w + NW * u) : ld.flast) >> 2;
      dma16_at(scsrc + (uint64_t)tile * scstep, my_lds + WS_OFF);   // WS_OFF + 512 = XS_OFF
    }
  };
  auto read = [&](auto whole_c, auto h_c, int u, MxMidOp& o) {
    constexpr int H = decltype(h_c)::value;
    const uint8_t* s = my + H * STAGE;
#pragma unroll
    for (int f = 0; f < FU; ++f) {
      o.w[H][f] = *(const u4*)(s + kMidX + f * 1024 + l * 16);
      o.x[H][f] = *(const u4*)(s + lm * 128 + 16 * ((2 * f + g) ^ xsw));
    }
    if constexpr (H == 0) {
#pragma unroll
      for (int i = 0; i < 2; ++i) o.ws[i] = *(const uint32_t*)(my + WS_OFF + 256 * i + 4 * l);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const u2 e = *(const u2*)(my + XS_OFF + (32 * j + lm) * 8);
        o.xs[j] = __builtin_amdgcn_perm(e.y, e.x, xsel);
      }
      if constexpr (!decltype(whole_c)::value) {       // the bytes of the fragments it has come first, the others'
        const int nf = ld.frags(u), sh = u < ld.nfull ? 0 : 8 * (ld.rest & 3);   // scales become 1 (their codes are zero)
        const uint32_t one = nf < 4 ? 0x7f7f7f7fu << (8 * nf) : 0u, keep = nf < 4 ? ~(~0u << (8 * nf)) : ~0u;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          o.ws[i] = (o.ws[i] >> sh & keep) | one;
          o.xs[i] = (o.xs[i] >> sh & keep) | one;
        }
      }
    }
    if constexpr (!decltype(whole_c)::value) {
#pragma unroll
      for (int f = 1; f < FU; ++f) o.w[H][f] &= f < ld.frags(u) ? ~0u : 0u;
    }
  };
  auto product = [&](auto h_c, const MxMidOp& o, int k) {
    constexpr int H = decltype(h_c)::value;
    const int j = k & 1, i = (k >> 1) & 1;
    if (k < 4)
      acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fp4_operand(o.w[i][2 * H]), fp4_operand(o.x[j][2 * H]), acc[i][j],
                                                                  4, 4, 2 * H, (int)o.ws[i], 2 * H, (int)o.xs[j]);
    else
      acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fp4_operand(o.w[i][2 * H + 1]), fp4_operand(o.x[j][2 * H + 1]),
                                                                  acc[i][j], 4, 4, 2 * H + 1, (int)o.ws[i], 2 * H + 1, (int)o.xs[j]);
  };
  mid_unit_loop<NS, 9, 8, 8, MxMidOp>(ld.nu, ld.nfull, ld.brief(), fill, read, product, [&]() {
    if (w < LF) lr_fetch(w);
  });

  // ---- compensation fragments w, w + NW, ... ---------------------------------------------------------------------------
  for (int jf = w; jf < LF; jf += NW) {
    if (jf != w) lr_fetch(jf);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fp4_operand(rq[i]), fp4_operand(rx[j]), acc[i][j], 4, 4, 0,
                                                                    (int)rs[i], 0, (int)rxs[j]);
  }

  // ---- the waves meet; wave w finishes MFMA tile (i, j), w = 2*i + j ------------------------------------------------
  constexpr int QN = 4, NE = 4 * QN;                   // register quads, registers
  const int ti = w >> 1, tj = w & 1;
  const int blk = nb0 + (ti < nbt ? ti : 0);
  const int mloc = 32 * tj + lm;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *(v4f*)(my + ((2 * i + j) * 4 + q) * 1024 + l * 16) =
            v4f{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
  __syncthreads();
  float y[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) y[e] = 0.0f;
#pragma unroll
  for (int ww = 0; ww < NW; ++ww)
#pragma unroll
    for (int q = 0; q < QN; ++q) {
      const v4f v = *(const v4f*)(lds + ww * REGION + (w * 4 + q) * 1024 + l * 16);
      y[4 * q] += v.x; y[4 * q + 1] += v.y; y[4 * q + 2] += v.z; y[4 * q + 3] += v.w;
    }
  if (p.y_dtype == SERQ_F32) {
    if (mloc < mrows && ti < nbt) {
      const int n = 32 * blk + 4 * g;
#pragma unroll
      for (int q = 0; q < QN; ++q)
        *(float4*)((float*)p.Y + (size_t)(m0 + mloc) * p.ldy + n + 8 * q) =
            make_float4(y[4 * q], y[4 * q + 1], y[4 * q + 2], y[4 * q + 3]);
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

// Up to four tiles per compute unit, as far as that is the cheaper kernel (mid_cheaper).  Measured (us, tiled kernel / this
// one, r = 128, N x K, weights from HBM; in brackets: tiles of the busiest compute unit):
//   4096 x 4096 M = 256 (1) 20.8 / 7.6, M = 512 (2) 20.7 / 12.0, M = 768 (3) 21.2 / 15.2, M = 1024 (4) 22.1 / 19.1;
//   4096 x 14336 M = 256 (1) 35.8 / 20.0, M = 512 (2) 46.5 / 32.7, M = 768 (3) 68 / 46;  11008 x 14336 M = 100 (2) 46 / 34, M = 256
//   (3) 51.5 / 48.6, weights from the last-level cache 46.9 / 36.8;  11008 x 20480 M = 256 (3) 67.4 / 68.8 (to the tiled kernel; from the
//   last-level cache 60.8 / 51.2);  4096 x 28672 M = 256 (1) 47.9 / 35.4, M = 512 (2) 57.9 / 60.4 (to the tiled kernel; 53.4 / 48.7)
// Workgroups of 8 waves, one to a compute unit, with 64-byte token rows: 4096 x 4096 M = 256 8.9 against 8.5, M = 512 15.4 against 12.4;
// 4096 x 11008 M = 768 42.0 against 35.9.
bool mx_mid_wanted(const MxLinearArgs& a) {
  static constexpr MidPrice small = {{2.45f, 1.17f, 0.22f, 0.52f, 0.39f, 0.06f}};
  static constexpr TiledPrice tiled = {{6.65f, 3.09f, 0.42f, 0.83f, 9.38f, 0.37f}};
  const size_t skip = skinny_mx_workspace_bytes(a.N);
  const size_t have = a.workspace && a.workspace_bytes > skip ? a.workspace_bytes - skip : 0;
  return mid_cheaper(small, tiled, a.M, a.N, a.K, 0, 4, 0.95f, have);
}

int launch_mx_mid(const MxLinearArgs& a, hipStream_t st) {
  MxMidParams p;
  p.Xq = a.Xq; p.xsc = a.xsc; p.Wq = a.Wq; p.wsc = a.wsc;
  p.Rq = a.Rq; p.rsc = a.rsc; p.s_begin = a.s_begin; p.r = a.Rq ? a.r : 0;
  p.M = a.M; p.N = a.N; p.K = a.K;
  p.Y = a.Y; p.y_dtype = a.y_dtype; p.ldy = a.ldy;
  p.tiles_m = (a.M + 63) / 64;
  p.tiles_n = (a.N + 63) / 64;
  p.band = mid_band(p.tiles_m, (long long)a.M * a.K / 2);
  const dim3 grid((unsigned)(p.tiles_m * p.tiles_n));
  hipLaunchKernelGGL(serq_mx_mid_kernel, grid, dim3(64 * NW), 0, st, p);
  return hipGetLastError() == hipSuccess ? SERQ_OK : SERQ_EHIP;
}

}  // namespace serq
