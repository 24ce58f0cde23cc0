// Pieces shared by the kernels for batches between decode and prefill (gemm_mid.hip, gemm_mid_mx.hip, grouped_mid.hip):
// 64 tokens x 64 output channels per workgroup, K dealt out to its 4 (group scales: 4 or 8) waves.
//
// Why this shape.  With a few hundred tokens the layer is bound by the bytes that go from L2 to the compute
// units, and by having a workgroup for each of them.  Tiles of 256 tokens leave most of the chip idle (one token
// tile x N/64) unless K is cut across workgroups, whose partial tiles then have to meet in memory in a second
// launch.  Here the partial tiles meet in LDS: every wave owns the whole 64 x 64 tile for its share of K
// (64 accumulator registers), so nothing is shared between waves and the main loop has no barrier -- a wave
// waits for its own loads only, and the other wave of its SIMD works meanwhile.
//
// A wave's loads run through a ring of stages in its own LDS region, filled by direct global -> LDS loads counted
// by hand.  There are two ways to cut them:
//   steps (4-bit integer tokens): a stage holds 64 token rows of 64 bytes and the weight fragments of two channel blocks for
//     the same channels; steps are dealt round-robin, so that the waves read neighbouring pieces of the same rows;
//   units (8-bit tokens, MXFP4): 128 bytes of the token rows, in two stages.  L2 hands out whole 128-byte lines: measured from
//     L2, all compute units at once, pieces of 64 bytes come at 17 TB/s, of 128 bytes at 35 TB/s, which is the address
//     units' 64 B/clk.  Stage h holds the 32 rows of token block h and the fragments of weight block h, so it is no larger
//     than a step, and the operands of a unit are complete once both have been read to registers.
// Units need a whole unit in registers before the first product and the next one behind it: 96 operand registers at the peak,
// and a pipeline that fills later.  Measured (us, steps / units, r = 128, N x K, the layer alone, weights from HBM):
//   W4A8    4096 x 11008 M = 256 23.1 / 20.1;  4096 x 4096 M = 64 9.4 / 8.5, M = 100 8.4 / 8.5, M = 256 9.6 / 9.3, M = 333
//           13.3 / 13.2;  6144 x 4096 M = 100 8.9 / 9.0;  11008 x 4096 M = 200 20.7 / 20.8;  6144 x 1024 M = 100 6.2 / 5.9
//   W4A8, group scales  4096 x 11008 M = 256 28.1 / 23.3;  4096 x 4096 M = 150 12.1 / 11.4, M = 400 19.1 / 17.3
//   MXFP4   4096 x 14336 M = 200 17.9 / 16.3;  4096 x 4096 M = 200 7.7 / 6.9, M = 500 11.9 / 10.5;  4096 x 1024 M = 200 4.5 / 4.6
// Where units lose a little alone, the layer with its quantiser in front does not (6144 x 4096 M = 100 12.7 / 12.3, 11008 x 4096 M = 200
// 25.8 / 25.4, MXFP4 4096 x 1024 M = 200 7.2 / 7.1): there is no second form for short K.
//   W4A4    4096 x 14336 M = 333 31.2 / 30.4, but 4096 x 4096 12.6 / 13.3 (few, large units), and with group scales, whose
//           second accumulators leave too few registers, 4096 x 11008 M = 150 20.1 / 25.2: 4-bit integer tokens keep steps
#ifndef SERQ_MID_TILE_H_
#define SERQ_MID_TILE_H_
#include <type_traits>

#include "gemm_tile.h"

namespace serq {
namespace {

constexpr int kMidX = 64 * 64;                       // token bytes of a stage: 64 rows of 64 bytes or 32 of 128
constexpr int kMidPart = 4 * 4 * 64 * 16;            // a wave's partial tile: [tile 2*i + j][register quad][lane][16 B]

// A 64-byte row is a quarter of the 256 bytes that the 64 banks serve at once: rows r .. r+3 take the quarters in
// turn, and the pieces of rows 4 apart are spread by the xor.
__device__ __forceinline__ int mid_swz(int row) { return (row >> 2) & 3; }
// The same for rows of 128 bytes.
__device__ __forceinline__ int mid_swz128(int row) { return (row >> 1) & 7; }

// Token tiles per band of the tile order (map_block).  All of them, while the token codes fit the 4 MiB of an XCD's L2: then
// every XCD reads its own weight panels and no others.  Beyond that, bands of up to 8: the tiles in flight on an XCD, 32 or
// 64 of them, read a block of about 8 x 8 panels, not every token panel for one or two weight panels.
// Measured (us, one band / bands, r = 128, N x K): W4A8 1024 x 14336 M = 2048 68.7 / 47.6, M = 3000 100 / 69.7;
// 1024 x 4096 M = 3000 31.3 / 22.9; MXFP4 1024 x 4096 M = 4096 26.6 / 20.9; at 4 MiB W4A8 512 x 1024 M = 4096 8.6 / 8.0;
// below, 1024 x 1536 M = 2048 9.2 / 9.4, 512 x 1024 M = 1500 5.7 / 6.0.  Bands of 4, 6 and 12: within 3 % of 8.
inline int mid_band(int tiles_m, long long token_bytes) {
  if (token_bytes < (4LL << 20)) return tiles_m;
  const int bands = (tiles_m + 7) / 8;
  return (tiles_m + bands - 1) / bands;
}

// how many tiles the busiest compute unit gets
inline long long mid_rounds(int M, int N, int ncu) {
  const long long tiles = ((long long)M + 63) / 64 * (((long long)N + 63) / 64);
  return (tiles + ncu - 1) / ncu;
}

// ---- small tiles or large ones (host side) --------------------------------------------------------------------
// Prices in us of this kernel and of the tiled one, compared where neither wins everywhere.  Both are straight-line fits
// to measured launches, 256 <= K <= 28672, N = 256 .. 28672, M from 33 to as many tokens as the rules admit, weights once
// from HBM and once from the last-level cache (the geometric mean of the two times; the cache moves this kernel by up to
// 20 % and the tiled one hardly).  Standard error of the tiled prices and of W4A4's 4 to 6 % at r = 128; other ranks move both alike.  W4A8's
// small-tile price is fitted to its kernel with whole-line token rows (383 layers of one to three tiles, 256 <= K <= 28672, ranks 0 to 256:
// 10 %); of 400 other layers of two and three tiles 6 would be more than 3 % faster in the other kernel (the worst 5 %), with the price of
// 64-byte rows 9 (26 %).  MXFP4's is that of 64-byte rows: at long K the kernel is up to 15 % cheaper, and the tiled one's price 6 % too low
// as well.  The rule chooses right with them all the same: of 400 layers of two to four tiles 12 would be more than 3 % faster in the other
// kernel, and all lose 0.3 % on average; with a small-tile price fitted to whole lines 13 and 0.3 %.
//   small tiles: c0 + c1 R + K/1024 (c2 + c3 R + c4 y) + c5 (MB of weight codes),  R tiles of the busiest compute unit,
//                y = M N / (4096 compute units): duplicated rows of a ragged tile cost less than real ones
//   tiled:       c0 rounds + k (c1 + c2 wide + c3 max(0, wide - 4)), k = rounds K / 1024 / slices;
//                with K slices c4 for the second launch and c5 for 5 MB of parked tiles, written and read
struct MidPrice { float c[6]; };
inline float mid_price(const MidPrice& p, int M, int N, int K, int ncu) {
  const float R = (float)mid_rounds(M, N, ncu), k = K / 1024.0f, y = (float)M * N / (4096.0f * ncu);
  return p.c[0] + p.c[1] * R + k * (p.c[2] + p.c[3] * R + p.c[4] * y) + p.c[5] * ((float)N * K / 2e6f);
}
struct TiledPrice { float c[6]; };
inline float tiled_price(const TiledPrice& p, const SplitPlan& pl, int M, int N, int K, int ncu) {
  const long long wg = (long long)((M + 255) / 256) * pl.C * pl.S;
  const float rounds = (float)((wg + ncu - 1) / ncu), k = rounds * K / (1024.0f * pl.S);
  const float us = p.c[0] * rounds + k * (p.c[1] + p.c[2] * pl.wide + p.c[3] * (pl.wide > 4 ? pl.wide - 4 : 0));
  return pl.S > 1 ? us + p.c[4] + p.c[5] * ((float)pl.S * M * N * 8.0f / 5e6f) : us;
}
// The layers of gemm_mfma.hip and gemm_mx.hip.  One tile per compute unit at most: always small tiles (11 % faster than the tiled
// kernel at K = 28672, below that up to 70 %).  Two: the prices are asked for long K only, up to K = 8192 small tiles
// win by 12 % or more.  Beyond: by the prices, up to `most` tiles and, below K = 512, up to two.  `favour` (5 and 7 %) is what
// a small-tile price may lie above the other: within the error of the prices the small tiles are kept.  W4A8's prices need
// none: with 1.02, 1.00 and 0.97 the 293 fitted layers of two and three tiles lose 0.15, 0.13 and 0.13 % on average (0.25 with its price
// of 64-byte rows), and 1.02 leaves three tiles of long K, level on fresh weights, to the kernel that reads fewer bytes.
//   ws_have: what the caller's workspace has room for behind the decode path's words; without enough the tiled kernel runs
//   unsliced.  Layers with fewer than 16 channels per compute unit (N < 4096) are not given to slices here: their parked tiles
//   would lie where the decode path of a wider layer, which may share the workspace, keeps words that have to stay zero.
inline bool mid_cheaper(const MidPrice& small, const TiledPrice& tiled, int M, int N, int K, int kind, int most, float favour,
                        size_t ws_have) {
  const int ncu = device_cu_count();
  const long long R = mid_rounds(M, N, ncu);
  if (R > most || (K < 512 && R > 2)) return false;
  if (R == 1 || (R == 2 && K <= 8192)) return true;
  SplitPlan pl = plan_split(M, N, K, kind, ncu, 0);
  if (pl.S > 1) {
    if (N < 16 * ncu) return true;
    if (parked_bytes(pl, (M + 255) / 256) > ws_have) pl = plan_split(M, N, K, kind, ncu, 1);
    else if (R > 2 && K > 16384 && kind != 4) return false;   // W4A8 11008 M = 192, small / tiled, us: K = 17408 67 / 68, 20480
                                                              // 80 / 77, 28672 109 / 109, where the prices say 110 / 127
  }
  return favour * mid_price(small, M, N, K, ncu) < tiled_price(tiled, pl, M, N, K, ncu);
}

// ---- steps ----------------------------------------------------------------------------------------------------
// The workgroup's tile and a wave's share of its loads.
// A step is 128 channels of 4-bit tokens: FR fragments of each weight block.
struct MidLoads {
  static constexpr int FR = 2;
  const uint8_t* xbase; const uint8_t* wbase;        // first token row / first weight fragment of the tile
  uint32_t xv[4];                                    // this lane's four token pieces: row offset + piece
  uint32_t back;                                     // what a piece of the second fragment steps back when there is none
  uint32_t wl;
  size_t wstep1;                                     // from the fragments of block 0 to those of block 1 (0: there is none)
  int KB;                                            // fragments per channel block

  __device__ __forceinline__ void init(const uint8_t* Xq, const u4* Wq, int K, uint32_t rowbytes, int m0, int mrows, int nb0,
                                       int nbt, int l) {
    KB = K >> 6;
    xbase = Xq + (size_t)m0 * rowbytes;
    wbase = (const uint8_t*)Wq + (size_t)nb0 * KB * 1024;
    wstep1 = nbt > 1 ? (size_t)KB * 1024 : 0;
    wl = (uint32_t)l * 16u;
    const int c = (l & 3) ^ ((l >> 4) & 3);          // piece 64*i + l is slot l%4 of row 16*i + l/4
    back = c >= 2 ? 32u : 0u;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      int row = 16 * i + (l >> 2);
      row = row < mrows ? row : mrows - 1;           // rows past M: duplicates, never stored
      xv[i] = (uint32_t)row * rowbytes + 16u * c;
    }
  }
  // direct load k (of 4 + 2*FR) of step s into the stage at LDS address `st`
  __device__ __forceinline__ void issue_one(int s, uint32_t st, int k) const {
    const bool half = KB - s * FR < FR;              // the last step of an odd number of fragments
    if (k < 4) {
      dma16(xbase + (size_t)s * 64, half ? xv[k] - back : xv[k], st + 1024u * k);
    } else {
      const int i = (k - 4) / FR, f = (k - 4) % FR;
      dma16(wbase + (size_t)s * FR * 1024 + i * wstep1 + (half ? 0 : f) * 1024, wl, st + 1024u * k);
    }
  }
  __device__ __forceinline__ void issue(int s, uint32_t st) const {
#pragma unroll
    for (int k = 0; k < 4 + 2 * FR; ++k) issue_one(s, st, k);
  }
};

// all but the youngest N vector-memory operations of this wave have completed
template <int N>
__device__ __forceinline__ void mid_landed() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }
// this wave's LDS reads have returned: the stage they came from may be refilled
__device__ __forceinline__ void mid_reads_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// The main loop of a wave over its stages 0 .. nst-1, in a ring of two.  The operands of a stage are copied to registers one
// stage ahead, which frees its slot: the slot is refilled, two stages further, between the products of the stage before.
// (A direct load blocks the wave while the address unit is busy with the other waves' loads; between two products
// that costs nothing.)
//   start(t)              the first loads of stage t (prologue)
//   fill(t, k)            direct load k (of NL) of stage t into its slot
//   read(t, op)           the operands of stage t, from LDS
//   product(op, k)        the k-th of NP groups of products on the operands `op`
// Loads requested before the loop are older than its own, so they do not disturb its counting.
template <int NL, int NP, class Op, class Start, class Fill, class Read, class Product>
__device__ __forceinline__ void mid_loop(int nst, const Start& start, const Fill& fill, const Read& read,
                                         const Product& product) {
  constexpr int NS = 2;
  if (nst == 0) return;
#pragma unroll
  for (int t = 0; t < NS; ++t)
    if (t < nst) start(t);
  Op A, B;
  if (nst > 1) mid_landed<NL>(); else mid_landed<0>();
  read(0, A);
  mid_reads_done();
  if (NS < nst) start(NS);
  int t = 0;
  auto stage = [&](auto steady_c, const Op& cur, Op& nxt) {
    constexpr bool STEADY = decltype(steady_c)::value;
    const bool refill = STEADY || t + 1 + NS < nst;
    if (STEADY) {
      mid_landed<NL>();
      read(t + 1, nxt);
    } else if (t + 1 < nst) {
      if (nst - 2 - t >= 1) mid_landed<NL>(); else mid_landed<0>();
      read(t + 1, nxt);
    }
    fence();
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      product(cur, k);
      if (k == 0) mid_reads_done();
#pragma unroll
      for (int d = 0; d < NL; ++d)
        if (d * (NP - 1) / NL == k && refill) fill(t + 1 + NS, d);
      fence();
    }
    ++t;
  };
  while (t + 2 + NS < nst) {
    stage(std::true_type{}, A, B);
    stage(std::true_type{}, B, A);
  }
  while (t < nst) {
    stage(std::false_type{}, A, B);
    if (t < nst) stage(std::false_type{}, B, A);
  }
}

// ---- units ----------------------------------------------------------------------------------------------------
// The workgroup's tile and a wave's share of its loads.
// FU: fragments of 64 channels per unit (2: 8-bit tokens, 4: 4-bit tokens).
// Units w, w + NW, ... are wave w's, as far as they go round; the fragments left over are dealt out in pieces of half a unit
// if that is enough (SPLIT), else of a unit, one to a wave: its last unit, with nf of FU fragments.
// LEAN: two registers for the token offsets instead of eight, and two vector and one scalar operation more per load.  For the
// MXFP4 kernel, whose operands leave no room for eight: with them 4 registers were spilled on the way into the steady loop, and
// behind their reload the compiler waited for all loads of the ring, every second unit (us, eight / two, r = 128, N x K,
// weights from HBM: 4096 x 14336 M = 200 17.8 / 17.0, 4096 x 4096 M = 100 7.2 / 6.9).  The integer kernels have the registers and are faster with
// eight (4096 x 4096 M = 100 8.6 / 9.1, 4096 x 8192 M = 40 11.4 / 12.2).
template <int FU, int NW, bool SPLIT = true, bool LEAN = false>
struct MidUnits {
  static constexpr int PPF = 8 / FU;                 // 16-byte pieces of a token row per fragment
  const uint8_t* xbase; const uint8_t* wbase;        // first token row / first weight fragment of the tile
  // This lane's token pieces: row offset + piece.  Load k of half h brings the rows of group q = 4*h + k, 8*q .. 8*q + 7.
  // LEAN: those of groups 0 and 1; the pieces of groups 2 apart are the same, their rows lie 2 * xgroup apart.
  uint32_t xv[LEAN ? 2 : 8];
  uint32_t xgroup, xlast;                            // LEAN: bytes of 8 rows; where the tile's last row begins
  uint32_t wl;
  size_t wstep1;                                     // from the fragments of block 0 to those of block 1 (0: there is none)
  int KB;                                            // fragments per channel block
  int w, nfull, nu, nf, rest;                        // whole units, units, fragments of a last one and the first of them
  int flast, hlast;                                  // the last unit, whole or not: its first fragment and how many it has

  __device__ __forceinline__ void init(const uint8_t* Xq, const u4* Wq, int K, uint32_t rowbytes, int m0, int mrows, int nb0,
                                       int nbt, int wave, int l) {
    KB = K >> 6;
    w = wave;
    nfull = KB / (FU * NW);
    const int left = KB - nfull * (FU * NW);
    constexpr int H = FU / 2 * NW;
    const int piece = SPLIT ? FU / 2 * ((left + H - 1) / H) : FU;   // (numbers, not conditions: those would go through vector registers)
    rest = nfull * (FU * NW) + w * piece;
    nf = KB - rest < piece ? KB - rest : piece;
    nf = nf < 0 ? 0 : nf;
    nu = nfull + (nf < 1 ? nf : 1);
    flast = nf > 0 ? rest : (w + NW * (nfull - 1)) * FU;
    hlast = nf > 0 ? nf : FU;
    xbase = Xq + (size_t)m0 * rowbytes;
    wbase = (const uint8_t*)Wq + (size_t)nb0 * KB * 1024;
    wstep1 = nbt > 1 ? (size_t)KB * 1024 : 0;
    wl = (uint32_t)l * 16u;
    xgroup = 8 * rowbytes;
    xlast = (uint32_t)(mrows - 1) * rowbytes;
#pragma unroll
    for (int q = 0; q < (LEAN ? 2 : 8); ++q) {
      int row = 8 * q + (l >> 3);
      if (!LEAN && row >= mrows) row = mrows - 1;    // rows past M: duplicates, never stored
      xv[q] = (uint32_t)row * rowbytes + 16u * xpiece(l, q);
    }
  }
  static __device__ __forceinline__ int xpiece(int l, int k) { return (l & 7) ^ mid_swz128(8 * k + (l >> 3)); }
  __device__ __forceinline__ bool brief() const { return nf > 0 && nf <= FU / 2; }
  __device__ __forceinline__ int frags(int u) const { return u < nfull ? FU : nf; }
  // direct load k (of 4 + FU) of half h of unit u into the stage at LDS address `st`; WHOLE: the unit is one that has all its
  // fragments; else it is the last one, which may lack some.  For pieces that it lacks whatever follows in memory is fetched, but nothing
  // behind its last piece of the tile's last row, and for fragments its last one: both are multiplied by zeros.  The same bound holds for
  // rows past M (LEAN), which are not stored; they begin a row's length or more behind that row.
  template <bool WHOLE>
  __device__ __forceinline__ void issue_one(int h, int u, uint32_t st, int k) const {
    const int f0 = WHOLE ? (w + NW * u) * FU : flast;
    const int have = WHOLE || !SPLIT ? FU : hlast;   // (not SPLIT: every unit is whole)
    if (k < 4) {
      uint32_t v = xv[LEAN ? k & 1 : 4 * h + k];
      if constexpr (LEAN) {
        uint32_t g = xgroup;
        asm volatile("" : "+s"(g));                  // added here: left alone, the compiler keeps all eight sums
        v += (4 * h + (k & 2)) * g;
      }
      if constexpr (LEAN || (SPLIT && !WHOLE)) {
        uint32_t lim = xlast + 16u * (have * PPF - 1);
        if constexpr (!LEAN) asm volatile("" : "+s"(lim));   // bounded here: the same
        v = v < lim ? v : lim;
      }
      dma16(xbase + (size_t)f0 * (16 * PPF), v, st + 1024u * k);
    } else {
      const int f = k - 4 < have ? k - 4 : have - 1;
      dma16(wbase + (size_t)(f0 + f) * 1024 + (h ? wstep1 : 0), wl, st + 1024u * k);
    }
  }
};

// The main loop over a wave's nu units.  Stage t of the ring is half t % 2 of unit t / 2.  The operands of a half
// are copied to registers one unit ahead, which frees its slot: the slot is refilled, NS stages further, between the
// products of the current unit.  (A direct load blocks the wave while the address unit is busy with the other waves'
// loads; between two products that costs nothing.)
//   fill(whole, h, u, k)  direct load k of half h of unit u into its slot (not whole: of the last unit)
//   read(whole, h, u, op) half h of the operands of unit u, from LDS
//   product(h, op, k)     the k-th of NP groups of products of the h-th half of the fragments
//   last()                before the products of the last unit: the place to request what the tile's end needs
// h, whole: compile-time constants; whole: the unit has all its fragments (false: it is the last one and may lack some;
// `brief`: it has none in its second half).  Half h takes NLh direct loads.  The first nfull units are whole.
// Loads requested before the loop are older than its own, so they do not disturb its counting.
//
// Everything that depends on how many units are left is decided at compile time: the units behind the steady state are
// written out one by one.  Control flow between the products lets the compiler sink products and widened codes below it,
// which keeps the operands of several units alive (up to 50 registers more).
template <int NS, int NL0, int NL1, int NP, class Op, class Fill, class Read, class Product, class Last>
__device__ __forceinline__ void mid_unit_loop(int nu, int nfull, bool brief, const Fill& fill, const Read& read, const Product& product,
                                         const Last& last) {
  static_assert(NS == 2 || NS == 3, "waits");
  using H0 = std::integral_constant<int, 0>;
  using H1 = std::integral_constant<int, 1>;
  constexpr int D = (NS + 1) / 2;                    // units between the current one and the one requested, less 1
  if (nu == 0) {
    last();
    return;
  }
  // a stage of half H has landed, BEHIND of the ring's stages are under way behind it
  auto landed = [&](auto h_c, auto behind_c) {
    constexpr int H = decltype(h_c)::value, BEHIND = decltype(behind_c)::value < NS - 1 ? decltype(behind_c)::value : NS - 1;
    mid_landed<BEHIND >= 2 ? NL0 + NL1 : BEHIND == 1 ? (H ? NL0 : NL1) : 0>();
  };
  // All loads of a stage, before the first products.  A unit that is whole is fetched as one here too, which is a choice made at run
  // time: the other form picks the pieces of every lane and fragment, and the first products wait for it.  Instructions up to a
  // W4A8 wave's 12th load 324 -> 264, MXFP4 375 -> 326; us, r = 128, N x K, weights from HBM: W4A8 4096 x 4096 M = 100 8.9 -> 8.6,
  // M = 64 8.8 -> 8.5, 6144 x 4096 M = 100 9.4 -> 9.2 (steps: 8.5, 9.4, 9.0), MXFP4 4096 x 1024 M = 200 4.8 -> 4.6 (4.5).
  auto start = [&](auto h_c, int u) {
    constexpr int NLS = decltype(h_c)::value ? NL1 : NL0;
    if (u < nfull) {
#pragma unroll
      for (int k = 0; k < NLS; ++k) fill(std::true_type{}, h_c, u, k);
    } else {
#pragma unroll
      for (int k = 0; k < NLS; ++k) fill(std::false_type{}, h_c, u, k);
    }
  };
  start(H0{}, 0);
  start(H1{}, 0);
  if (NS == 3 && nu > 1) start(H0{}, 1);
  auto first = [&](Op& op) {
    using Two = std::integral_constant<int, 2>;
    if (nu > 1) landed(H0{}, Two{}); else landed(H0{}, H1{});
    read(std::false_type{}, H0{}, 0, op);
    mid_reads_done();
    if (nu > 1) start(std::integral_constant<int, NS & 1>{}, 1);
    if (nu > 1) landed(H1{}, Two{}); else landed(H1{}, H0{});
    read(std::false_type{}, H1{}, 0, op);
    mid_reads_done();
    if (nu > D) start(std::integral_constant<int, (NS + 1) & 1>{}, D);
  };
  int u = 0;
  // unit u, with LEFT units behind it; LEFT > D + 1 stands for any such number
  auto unit = [&](auto left_c, Op& cur, Op& nxt) {
    constexpr int LEFT = decltype(left_c)::value;
    // two branches that begin with the same products: the compiler would hoist those (and keep their results apart)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
      for (auto& v : cur.w[i]) asm volatile("" : "+v"(v));
#pragma unroll
      for (auto& v : cur.x[i]) asm volatile("" : "+v"(v));
    }
    auto half = [&](auto h_c) {
      constexpr int H = decltype(h_c)::value;
      constexpr int HR = (H + NS) & 1;                // the stage requested here: half HR of unit u + AHEAD
      constexpr int AHEAD = 1 + (H + NS) / 2;
      constexpr int NLR = AHEAD > LEFT ? 0 : HR ? NL1 : NL0;
      using whole_next = std::integral_constant<bool, (LEFT > 1)>;
      using whole_req = std::integral_constant<bool, (LEFT > AHEAD)>;
      if constexpr (LEFT > 0) {
        landed(h_c, std::integral_constant<int, 2 * LEFT - 1 - H>{});
        read(whole_next{}, h_c, u + 1, nxt);
      } else if constexpr (H == 0) {
        last();
      }
      fence();
#pragma unroll
      for (int k = 0; k < NP; ++k) {
        product(h_c, cur, k);
        if (LEFT > 0 && k == 0) mid_reads_done();
#pragma unroll
        for (int d = 0; d < NLR; ++d)
          if (d * (NP - 1) / (NLR > 0 ? NLR : 1) == k) fill(whole_req{}, std::integral_constant<int, HR>{}, u + AHEAD, d);
        fence();
      }
    };
    half(H0{});
    if (LEFT > 0 || !brief) half(H1{});
    ++u;
  };
  using Any = std::integral_constant<int, D + 2>;
  using L3 = std::integral_constant<int, 3>;
  using L2 = std::integral_constant<int, 2>;
  Op A, B;
  if (nu & 1) {                                      // an even number of units behind the first
    first(A);
  } else {
    first(B);
    if (nu == 2) unit(H1{}, B, A);
    else if (NS == 3 && nu == 4) unit(L3{}, B, A);
    else unit(Any{}, B, A);
  }
  while (nu - u > 2 * D + 1) {
    unit(Any{}, A, B);
    unit(Any{}, B, A);
  }
  if (NS == 3 && nu - u > 3) {
    unit(Any{}, A, B);
    unit(L3{}, B, A);
  }
  if (nu - u > 1) {
    unit(L2{}, A, B);
    unit(H1{}, B, A);
  }
  unit(H0{}, A, B);
}

// Rows of 64 16-bit results in LDS (128 bytes), 16-byte piece pc of row r at piece pc ^ (r & 7): four consecutive channels
// of one token per lane in, whole row segments out.
constexpr int kMidOut = 64 * 128;
__device__ __forceinline__ void mid_park16(uint8_t* out, int r, int pc, int g, const float y[4], bool bf) {
  u2 o;
  if (bf) o = u2{f32x2_to_bf16x2(y[0], y[1]), f32x2_to_bf16x2(y[2], y[3])};
  else o = u2{f32x2_to_f16x2(y[0], y[1]), f32x2_to_f16x2(y[2], y[3])};
  *(u2*)(out + r * 128 + 16 * (pc ^ (r & 7)) + 8 * g) = o;
}
template <int THREADS>
__device__ __forceinline__ void mid_store16(const uint8_t* out, int tid, uint16_t* Y, int64_t ldy, int m0, int mrows, int n0,
                                            int nbt) {
  const int pc = tid & 7;
#pragma unroll
  for (int r0 = 0; r0 < 64; r0 += THREADS / 8) {
    const int r = r0 + (tid >> 3);
    if (r < mrows && pc < 4 * nbt)
      *(u4*)(Y + (size_t)(m0 + r) * ldy + n0 + 8 * pc) = *(const u4*)(out + r * 128 + 16 * (pc ^ (r & 7)));
  }
}

}  // namespace
}  // namespace serq
#endif  // SERQ_MID_TILE_H_
