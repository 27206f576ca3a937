// Tile shapes of the tiled GEMMs (gemm_w4.hip), and which one runs with which
// split along K.  Host arithmetic on sizes only: no HIP, so that a plain C++
// program can ask for the choice too.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

namespace sq {
namespace {

constexpr int KT = 128;     // input channels per stage
constexpr int GROUP_M = 8;  // m-tiles per supertile of 128-row tiles (L2 reuse)

// ---- 8-bit activations
// Shape: NWM x NWN waves, each TM x TN tiles of 16 x 16, WGS workgroups per CU.
// Which shape runs is decided by choose16.  Alternatives measured to the
// 128 x 128 tiles' 2 x 2 waves of 64 x 64: 2 x 4 waves of 64 x 32 (four waves
// per SIMD) the same speed without the raised-priority MFMA phase and 1 %
// slower with it, 1 x 4 waves of 128 x 32 1-2 % slower.
template <int NWM_, int NWN_, int TM_, int TN_, int WGS>
struct Shape16 {
  static constexpr int NWM = NWM_, NWN = NWN_, NWAVE = NWM * NWN, NTHREADS = NWAVE * 64;
  static constexpr int TM = TM_, TN = TN_, WROWS = 16 * TM, WCOLS = 16 * TN;
  static constexpr int BM = NWM * WROWS, BN = NWN * WCOLS;
  static constexpr int DIST = 2, STAGES = 3, WGS_PER_CU = WGS;
  static constexpr int GROUP = GROUP_M * 128 / BM;  // m-tiles per supertile: 1024 rows
  static constexpr int LAG = 3;                     // tiles between a tile's MFMAs and its fold
  // one stage in LDS: A codes, packed weights, then each wave's 256-byte
  // area of weight-step pairs (the Layout<8, false> arrangement, except that
  // weight column n holds chunk c at position c ^ ((n >> 1) & 3): the 16
  // columns of a fragment read then fill all 64 banks; with (n >> 2) & 3 the
  // read took twice as long in an LDS probe, and the kernel gained 0.5 %)
  static constexpr int A_BYTES = BM * KT, B_BYTES = BN * KT / 2, W_BYTES = NWAVE * 256;
  static constexpr int STAGE = A_BYTES + B_BYTES + W_BYTES;
  static constexpr int A_DMA = A_BYTES / 1024 / NWAVE, B_DMA = B_BYTES / 1024 / NWAVE;
  static_assert(A_DMA * 1024 * NWAVE == A_BYTES && B_DMA * 1024 * NWAVE == B_BYTES, "whole loads per wave");
  static_assert(A_DMA % 2 == 0, "the swizzle of a load depends on its number's parity");
  static_assert(WGS * STAGES * STAGE <= 160 * 1024, "the workgroups of a CU fit in its LDS");
};
using P16 = Shape16<2, 2, 4, 4, 2>;   // 128 x 128 tiles
using P16H = Shape16<1, 4, 4, 2, 3>;  // 64 x 128
using P16Q = Shape16<2, 2, 2, 2, 4>;  // 64 x 64

// 256 x 128 tiles (gemm_tall16_kernel)
struct T16 {
  static constexpr int NWM = 2, NWN = 2, NWAVE = 4, NTHREADS = 256;
  static constexpr int BM = 256, BN = 128;
  static constexpr int TM = 8, TN = 4, WROWS = 128, WCOLS = 64;
  static constexpr int WGS_PER_CU = 2;
  static constexpr int A_BYTES = BM * KT, B_BYTES = BN * KT / 2, STAGE = A_BYTES + B_BYTES;
  static constexpr int A_DMA = A_BYTES / 1024 / NWAVE, B_DMA = B_BYTES / 1024 / NWAVE;
  static constexpr int GROUP = 4;  // m-tiles per supertile
  static constexpr int LAG = 3;  // tiles between a tile's MFMAs and its fold
};

// ---- 4-bit activations on the fp8 matrix cores
// Shape: 2 x 2 waves, each TM_ x TN_ tiles of 32 x 32, WGS workgroups per CU.
template <int TM_, int TN_, int WGS>
struct Shape8 {
  static constexpr int NWAVE = 4, TM = TM_, TN = TN_, WROWS = 32 * TM, WCOLS = 32 * TN;
  static constexpr int BM = 2 * WROWS, BN = 2 * WCOLS, WGS_PER_CU = WGS;
  static constexpr int GROUP = GROUP_M * 128 / BM;
  static constexpr int A_BYTES = BM * KT;      // fp8 code rows of 128 B, chunk c at c ^ ((r >> 1) & 7)
  static constexpr int B_BYTES = BN * KT / 2;  // packed weight rows of 64 B, chunk c at c ^ ((r >> 2) & 3)
  static constexpr int B_OFF = A_BYTES;
  // fp32 group steps sigma and kc: row 32 w + i, block half b at w * 256 + b * 128 + i * 4
  static constexpr int SROWS = BM / 32;  // waves that load steps
  static constexpr int SG_OFF = B_OFF + B_BYTES;
  static constexpr int KC_OFF = SG_OFF + SROWS * 256;
  static constexpr int W_OFF = KC_OFF + SROWS * 256;  // weight-step pairs: columns 2 i, 2 i + 1 at i * 4
  static constexpr int STAGE = W_OFF + 256;
  static constexpr int STAGES = 2;  // loads run one stage ahead
  static constexpr int A_DMA = A_BYTES / 1024 / NWAVE, B_DMA = B_BYTES / 1024 / NWAVE;
  static_assert(WGS * STAGES * STAGE <= 160 * 1024, "the workgroups of a CU fit in its LDS");
};
using F8 = Shape8<2, 2, 2>;   // 128 x 128 tiles
using F8H = Shape8<1, 2, 2>;  // 64 x 128
using F8Q = Shape8<1, 1, 4>;  // 64 x 64

// ---- split plans
// Split plan of the pipelined kernel (tiles of BM x BN, `slots` workgroups at
// once): the tiles that fill whole rounds run whole; the R left over (all of
// them when there are fewer tiles than slots) are each split into S K ranges
// when that is faster.  In units of one stage of one tile on one workgroup,
// the split tail takes about nkt / S stages plus the partial sums' traffic,
// c * R * S with c = (rows * BN * 8 bytes written and read back) / (about
// 4.4 MB moved per stage time), plus about two for the extra launch;
// S ~ sqrt(nkt / (c R)), with ranges of >= 2 stages, R * S <= slots and R * S
// units of BM * BN floats fitting in `partial_bytes`.  Only the pipelined
// paths split (their blocks never straddle a range boundary).
struct Plan {
  int ntiles, ndp, split;
};
template <int BM, int BN>
Plan plan_split(int32_t M, int32_t N, int32_t K, int slots, size_t partial_bytes) {
  const int ntm = (M + BM - 1) / BM, ntn = (N + BN - 1) / BN;
  const int ntiles = ntm * ntn;
  Plan p{ntiles, ntiles, 1};
  const int nkt = K / KT;
  const int rest = ntiles % slots;
  if (rest == 0 || nkt < 4) return p;
  // rows of a left-over tile: the left-over tiles are the last ones of the
  // logical order, which lie in the last row of tiles when there are few
  const int rows = (ntm == 1 || rest <= ntn) ? M - BM * (ntm - 1) : BM;
  const double c = rows * static_cast<double>(BN) * 8.0 / 4.4e6;
  int split = static_cast<int>(std::lround(std::sqrt(nkt / (c * rest))));
  split = std::min(std::min(split, nkt / 2), slots / rest);
  constexpr size_t unit = static_cast<size_t>(BM) * BN * sizeof(float);
  while (split >= 2 && static_cast<size_t>(rest) * split * unit > partial_bytes) --split;
  if (split < 2) return p;
  const double t_split = static_cast<double>(nkt) / split + c * rest * split + 2.0;
  if (t_split >= nkt) return p;
  p.ndp = ntiles - rest;
  p.split = split;
  return p;
}

// 128 x 128 tiles, two workgroups per CU.
inline Plan pipe_plan(int32_t M, int32_t N, int32_t K, int cus, size_t partial_bytes) {
  return plan_split<128, 128>(M, N, K, cus * 2, partial_bytes);
}

// Bytes of partial sums that the 128 x 128 plan asks for (0 when it does not split).
inline size_t pipe_partial_bytes(int32_t M, int32_t N, int32_t K, int cus) {
  const Plan p = pipe_plan(M, N, K, cus, ~static_cast<size_t>(0));
  return static_cast<size_t>(p.ntiles - p.ndp) * (p.split > 1 ? p.split : 0) * (128 * 128 * sizeof(float));
}

// ---- 8-bit activations on 16 x 16 MFMA tiles: tile shape and split plan
// A launch takes about
//   fixed + rounds x (stages x stage[workgroups per CU] + tile) [+ split tail],
// in us, where a round is one set of resident workgroups, a stage's time
// depends on how many of them share a CU, and a split tail adds its second
// kernel and its partial sums' traffic.  The constants are least-squares fits to
// the measured times of every shape on 195 sizes (130 to 8384 rows, 256 to 13824
// channels), separately for 128-wide weight groups and one step per channel (no
// fold); they predict a launch within 6-7 % (standard deviation; 10-13 % below
// five stages).  On 611 other sizes (129 to 16768 rows, 256 to 14336 channels) the
// choice is 1.24 x (per channel 1.20 x) faster than 128 x 128 tiles everywhere
// (geometric mean), within 2 % of the best plan measured, and more than 2 % slower
// than 128 x 128 tiles on 7 of the 1222 (0.91 x at worst: 312 x 10624 -> 3712 per
// channel).
struct Cost16 {
  double fixed;     // launch, first loads
  double stage[4];  // one 128-channel stage with 1 .. 4 workgroups on the CU
  double tile;      // epilogue
  double split;     // the second kernel of a split
  double traffic;   // per 4.4 MB of partial sums written and read back
};
template <class P, bool PC>
constexpr Cost16 cost16();
template <>
constexpr Cost16 cost16<T16, false>() { return {0.0, {1.31, 1.91}, 7.6, 2.2, 0.55}; }
template <>
constexpr Cost16 cost16<P16, false>() { return {1.2, {0.84, 1.04}, 4.2, 2.9, 0.48}; }
template <>
constexpr Cost16 cost16<P16H, false>() { return {1.9, {0.45, 0.63, 0.955}, 2.4, 3.5, 0.57}; }
template <>
constexpr Cost16 cost16<P16Q, false>() { return {1.7, {0.355, 0.45, 0.665, 0.78}, 1.8, 3.3, 0.56}; }
template <>
constexpr Cost16 cost16<T16, true>() { return {0.1, {0.91, 1.37}, 7.5, 2.1, 0.54}; }
template <>
constexpr Cost16 cost16<P16, true>() { return {0.7, {0.565, 0.745}, 4.8, 2.8, 0.56}; }
template <>
constexpr Cost16 cost16<P16H, true>() { return {1.9, {0.375, 0.49, 0.815}, 2.4, 2.8, 0.69}; }
template <>
constexpr Cost16 cost16<P16Q, true>() { return {2.1, {0.285, 0.37, 0.53, 0.71}, 1.5, 2.5, 0.84}; }

// Estimated time in us of a plan of shape P.
template <class P, bool PC>
double cost_of(const Plan& p, int32_t M, int32_t K, int cus) {
  constexpr Cost16 c = cost16<P, PC>();
  const int nkt = K / KT, slots = cus * P::WGS_PER_CU;
  auto stage = [&](int items) { return c.stage[std::min((items + cus - 1) / cus, P::WGS_PER_CU) - 1]; };
  const int full = p.ndp / slots, whole = p.ndp % slots, r = p.ntiles - p.ndp;
  double t = c.fixed + full * (nkt * c.stage[P::WGS_PER_CU - 1] + c.tile);
  if (r == 0) return whole > 0 ? t + nkt * stage(whole) + c.tile : t;
  const int both = (nkt + p.split - 1) / p.split;  // stages that whole tiles and split ranges run side by side
  t += both * stage(whole + r * p.split) + (whole > 0 ? (nkt - both) * stage(whole) : 0.0) + c.tile + c.split;
  return t + c.traffic * (static_cast<double>(r) * p.split * std::min(M, P::BM) * P::BN * 8.0 / 4.4e6);
}

// The cheapest plan of shape P, its time in `best`.  The tiles past the last
// full round of workgroup slots are either a round of their own or are split
// along K (ranges of at least two stages, partial sums within
// `partial_bytes`); when more than a workgroup per CU is left over, also: one
// whole tile per CU and the rest split beside them.
template <class P, bool PC>
Plan plan16(int32_t M, int32_t N, int32_t K, int cus, size_t partial_bytes, double& best) {
  const int ntm = (M + P::BM - 1) / P::BM, ntn = (N + P::BN - 1) / P::BN;
  if (static_cast<int64_t>(ntm) * ntn > (1 << 30)) {  // tile numbers are int; 128 x 128 tiles always fit
    best = HUGE_VAL;
    return Plan{};
  }
  const int ntiles = ntm * ntn, slots = cus * P::WGS_PER_CU, rest = ntiles % slots;
  Plan p{ntiles, ntiles, 1};
  best = cost_of<P, PC>(p, M, K, cus);
  constexpr size_t unit = static_cast<size_t>(P::BM) * P::BN * sizeof(float);
  for (int whole = 0; whole < rest; whole += cus) {  // whole tiles in the last round
    const int r = rest - whole;
    const int smax = std::min(std::min(K / KT / 2, (slots - whole) / r), 32);
    for (int S = 2; S <= smax && static_cast<size_t>(r) * S * unit <= partial_bytes; ++S) {
      const Plan q{ntiles, ntiles - r, S};
      const double t = cost_of<P, PC>(q, M, K, cus);
      if (t < best) p = q, best = t;
    }
  }
  return p;
}

enum Tile : int { kTile256x128, kTile128x128, kTile64x128, kTile64x64 };
struct Choice {
  Tile tile;
  Plan plan;
};
inline int tile_outputs(Tile t) {
  return t == kTile256x128 ? 256 * 128 : t == kTile128x128 ? 128 * 128 : t == kTile64x128 ? 64 * 128 : 64 * 64;
}
// 128 x 128 tiles with the plan of plan_split, unless another shape or split
// is estimated to be at least 5 % faster (about the model's error).
template <bool PC>
Choice choose16(int32_t M, int32_t N, int32_t K, int cus, size_t partial_bytes) {
  // the partial sums that the workspace query allows for, and no more: the
  // plan, and with it the order of the sums, is the same in a larger buffer
  partial_bytes = std::min(partial_bytes, pipe_partial_bytes(M, N, K, cus));
  Choice c{kTile128x128, pipe_plan(M, N, K, cus, partial_bytes)};
  const double base = cost_of<P16, PC>(c.plan, M, K, cus);
  const bool short_k = K <= 5 * KT && c.plan.ntiles > 2 * cus;
  double best = 0.95 * base, t;
  auto offer = [&](Tile tile, const Plan& p) {
    if (t < best) c = {tile, p}, best = t;
  };
  offer(kTile128x128, plan16<P16, PC>(M, N, K, cus, partial_bytes, t));
  // below 12 stages the tall tiles' epilogues no longer hide behind each other
  // (8384 x 1024 -> 3072: 50.4 us against 46.8, 8384 x 1536 -> 4608: 88.8 against 93.5)
  if (K >= 12 * KT) offer(kTile256x128, plan16<T16, PC>(M, N, K, cus, partial_bytes, t));
  // Two regions where the estimates of the smaller tiles are too low, and so have
  // to promise more.  Up to five stages with more than a round of 128 x 128 tiles,
  // the epilogues that share a CU weigh more (up to 30 % low: 2227 x 384 -> 8576 per
  // channel on 64 x 64 tiles 23.3 us, on 128 x 128 21.2).  One step per channel from 40 stages on,
  // split and 64 x 64 tiles read the operands more often than a stage's time knows
  // (4142 x 12160 -> 960 75.0 us on 64 x 64 tiles, 67.9 on 128 x 128).
  auto offer_small = [&](Tile tile, const Plan& p) {
    const bool long_k = PC && K >= 40 * KT && (tile == kTile64x64 || p.split > 1);
    if (t < (short_k ? 0.85 : long_k ? 0.90 : 0.95) * base) offer(tile, p);
  };
  offer_small(kTile64x128, plan16<P16H, PC>(M, N, K, cus, partial_bytes, t));
  offer_small(kTile64x64, plan16<P16Q, PC>(M, N, K, cus, partial_bytes, t));
  return c;
}

// 4-bit activations on the fp8 matrix cores.  The outputs equal the int8 path's
// (sq_gemm_w4a4) bit for bit, so every output keeps that path's split: where
// its 128 x 128 tiles are all whole or all split, 64 x 128 or 64 x 64 tiles
// with the same split are taken if estimated at least 5 % faster (where only
// its last round is split, 128 x 128 tiles stay).  The constants are fits to
// 99 sizes (136 to 4192 rows, 512 to 13824 channels; standard deviation
// 4-5 %).  On those sizes the choice is 1.23 x faster than 128 x 128 tiles
// everywhere (geometric mean; 0.98 x at worst, within the runs' spread).
template <>
constexpr Cost16 cost16<F8, false>() { return {3.2, {1.29, 1.67}, 2.0, 4.0, 0.47}; }
template <>
constexpr Cost16 cost16<F8H, false>() { return {2.4, {0.727, 0.914}, 2.0, 2.5, 0.88}; }
template <>
constexpr Cost16 cost16<F8Q, false>() { return {3.8, {0.471, 0.624, 0.933, 1.23}, 0.0, 3.3, 0.75}; }

// All tiles of shape P whole, or (S > 1) all split into S ranges: the plan,
// its estimated time in `t`.
template <class P>
Plan plan8(int32_t M, int32_t N, int32_t K, int S, int cus, double& t) {
  constexpr Cost16 c = cost16<P, false>();
  const int ntiles = ((M + P::BM - 1) / P::BM) * ((N + P::BN - 1) / P::BN), slots = cus * P::WGS_PER_CU;
  const int items = ntiles * S, full = items / slots, rest = items % slots, stages = (K / KT + S - 1) / S;
  t = c.fixed + full * (stages * c.stage[P::WGS_PER_CU - 1] + c.tile);
  if (rest > 0) t += stages * c.stage[(rest + cus - 1) / cus - 1] + c.tile;
  if (S > 1) t += c.split + c.traffic * (static_cast<double>(items) * std::min(M, P::BM) * P::BN * 8.0 / 4.4e6);
  return Plan{ntiles, S > 1 ? 0 : ntiles, S};
}

inline Choice choose8(int32_t M, int32_t N, int32_t K, int cus, size_t partial_bytes) {
  Choice c{kTile128x128, pipe_plan(M, N, K, cus, partial_bytes)};
  // (many tiles: 128 x 128 fill the chip, and tile numbers stay far below int)
  if ((c.plan.split > 1 && c.plan.ndp > 0) || c.plan.ntiles > 8 * cus) return c;
  const int S = c.plan.split;
  double best, t;
  plan8<F8>(M, N, K, S, cus, best);
  best *= 0.95;
  // four 64 x 64 tiles hold what a 128 x 128 one does: their partial sums fit where its fit
  const Plan h = plan8<F8H>(M, N, K, S, cus, t);
  if (t < best) c = {kTile64x128, h}, best = t;
  const Plan q = plan8<F8Q>(M, N, K, S, cus, t);
  if (t < best) c = {kTile64x64, q};
  return c;
}

// Sums that the calibration epilogue leaves: one per wave of a whole tile (all
// shapes have four waves), one per workgroup (1024 outputs) of a split tile's
// second kernel.
inline size_t err_parts(const Choice& c) {
  static_assert(P16::NWAVE == 4 && P16H::NWAVE == 4 && P16Q::NWAVE == 4 && T16::NWAVE == 4 && F8::NWAVE == 4, "");
  const Plan& p = c.plan;
  if (p.split == 1) return static_cast<size_t>(p.ntiles) * 4;
  return static_cast<size_t>(p.ndp) * 4 + static_cast<size_t>(p.ntiles - p.ndp) * (tile_outputs(c.tile) / 1024);
}

}  // namespace
}  // namespace sq
