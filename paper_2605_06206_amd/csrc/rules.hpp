// Choices between kernels that depend on sizes alone: plain host code, tested
// without a GPU.
#pragma once

namespace foe {

// Renormalised routing of C > 1 clusters: one pass over x that scores all C*E
// experts in a workgroup per 16 tokens, or a workgroup per cluster and 16 tokens.
// The second reads x once per cluster, but spreads the work where few tokens leave
// most CUs idle, and past 64 score columns, where the one-pass kernel has four waves
// and little in flight.  Both times in us, fitted to 1300 measured sizes (2 to
// 64 clusters, 8 to 256 columns, 1 to 32768 tokens, d 512 to 7168) within about a
// tenth; the second is taken where it comes out a tenth faster.  One-pass workgroups
// beyond a first on each CU (4096 tokens) wait for it (bf16, past 64 columns);
// per-cluster ones run several to a CU and are bound by x, about 1.3 us per CU
// and 1024 columns of it.  Measured, one pass and per cluster:
//   8 x 8, d 2048: 1 token 15.9 and 6.3, 2040 tokens 15.8 and 14.7; d 4096: 2040
//     tokens 24.6 and 26.4; 8 x 4, d 4096: 2040 tokens 16.2 and 23.8
//   8 x 32, d 2048: 1 token 47 and 9, 8192 tokens 96 and 42; d 4096: 32768 tokens
//     635 and 369
//   8 x 16, d 2048: 2048 tokens 28.9 and 17.8; d 4096: 4096 tokens 45 and 59
//   32 x 4, d 4096: 256 tokens 70 and 14, 4096 tokens 70 and 164
//   fp32, d 2048: 4 x 32: 4096 tokens 97 and 48, 32768 tokens 299 and 373
// Up to 64 columns the one-pass kernels of 2048 tokens and more are always taken.
inline bool route_per_cluster(bool bf16, int C, int T, int d, int E) {
  const int Et = C * E;
  if (C < 2 || (Et <= 64 && T >= 2048)) return false;
  const double D = d / 1024.0, wg = T / 4096.0;  // workgroups per CU
  const double sel = Et <= 64 ? 1.0 / 3 : Et <= 128 ? 1.0 : 1.6;  // selection, per cluster
  double one, per;
  if (bf16) {
    one = ((T + 4095) / 4096) * (6 + D * (0.9 + 0.054 * Et) + sel * C);
    per = 3 + D * (1 + 0.04 * E) + 1.3 * D * C * wg;
  } else {
    if (Et <= 64) {
      one = 3 + D * (2 + 0.16 * Et) + sel * C;
    } else {
      const double first = D * (6.5 + 0.29 * Et) + sel * C;
      const double many = wg * (D * (Et <= 128 ? 8.6 + 0.08 * Et : 0.21 * Et) + 0.3 * C);
      one = first > many ? first : many;
    }
    per = 3 + D * (1.5 + 0.04 * E) + D * (2.1 + 0.11 * E) * C * wg;
  }
  return per < 0.9 * one;
}

// Form of the bf16 expert FFN: weight stream (few rows per expert), medium tiles,
// large tiles, large tiles with both GEMMs in one launch (the block's, where F is
// a multiple of 64; elsewhere the same as kLarge).
enum class FfnForm { kStream, kMid, kLarge, kFused };

// The form for E experts (of all clusters) and a mean of rows / E rows each; an
// expert's rows end half a tile into its last tile on average.  us of a block call
// below.
// - Under 32 rows the weights are streamed for 32 rows at a time.  With more, most
//   experts need a second pass over their weights (d 2048, F 1024, 16 experts: 24
//   rows 61 against 62 with the medium tiles, 32 rows 68 against 63, 64 rows 137
//   against 66; but see stream_spreads).
// - The medium tiles read every weight once for up to 128 rows, by four times as
//   many workgroups as the large ones, two to a CU.  They win while the large
//   tiles would leave CUs idle, or would be less than 3/8 full (under 96 rows),
//   until the work (tiles x K steps) is long enough that the large tiles'
//   fewer operand bytes count, or the tiles are too many rounds; unless the
//   medium ones are more than a round where the large ones run at once.  Medium and
//   best of the large forms: d = F = 1024, 40 experts: 96 rows 94 and 104; d 768, F
//   1536, 12 experts: 307 rows 72 and 114; d 2048, F 1024, 24 experts: 128 rows 148
//   and 119; d 2560, F 1536, 16 experts: 250 rows 194 and 151; 64 experts: d 1280,
//   F 768, 64 rows 123 and 139, d 4096, F 1024, 95 rows 420 and 384; d 4096, F 512,
//   32 experts: 160 rows 219 and 193; d 4096, F 256, 48 experts: 450 rows 415 and 295,
//   but 16 experts: 320 rows 111 and 139.
// - The large tiles as one launch of both GEMMs once the tiles of one of them fill
//   the chip: before that the CUs without a gate/up tile take down tiles and wait
//   for their rows, and two launches are faster (d 2048, F 1024, 16 experts: 256 rows
//   119 against 138; but d 4096, F 256, 48 experts, 450 rows 342 against 295).
// The lines are fitted to 520 sizes (4 to 96 experts, 64 to 2000 rows, d 768 to 6144,
// F 256 to 2048, uniform and skewed routers): 1% above the best form on average.
inline FfnForm ffn_form(int E, int d, int F, long long rows, int cus) {
  if (rows < 32LL * E) return FfnForm::kStream;
  auto tiles = [](double m, int n, int bn) { return m * ((n + bn - 1) / bn); };
  const double mid = rows / 128.0 + E / 2.0, large = rows / 256.0 + E / 2.0;  // tiles of rows
  const double work = mid * d * F / cus;
  const double gu = tiles(mid, F, 64) / cus, dn = tiles(mid, d, 128) / cus;
  // tiles of experts with a tenth more rows than the mean
  const double even = (double)E * ((long long)(1.1 * rows / E / 256.0) + 1);
  const bool idle = tiles(large, F, 128) < cus &&
                    (tiles(large, d, 256) < cus || tiles(even, d, 256) <= cus);
  const bool at_once = idle && tiles(even, F, 128) <= cus;
  if ((rows < 96LL * E && work < 560e3) ||
      (work < 312e3 && dn <= 4.5 && gu <= (at_once ? 2.2 : 4.0)) ||
      (work < 352e3 && dn <= 8.3 && gu <= 1.1))
    return FfnForm::kMid;
  return idle ? FfnForm::kLarge : FfnForm::kFused;
}

// fp32 expert FFN through the tiled kernel, whose loads reach a gathered source (of
// gather_rows rows; 0: rows in order), and 64 rows of any operand, through 32-bit
// offsets below 2^31; larger ones take the plain kernels.
inline bool f32_tiled(int d, int F, long long gather_rows) {
  constexpr long long range = (1ll << 31) - 64;
  const long long widest = d > F ? d : F;
  return widest * 256 <= range && gather_rows * d * 4 <= range;
}

// The weight stream from the routing decisions themselves (R pairs per cluster): a
// workgroup takes 64 gate/up or 128 down columns of an expert, 32 rows in a pass.
// From 32 rows per expert on, the passes are dealt to as many workgroups as the
// CUs have room for (a workgroup's LDS fills one), up to 8: one after another, the
// passes of a skewed router's first expert add up.
inline int stream_parts(int R, int E, long long workgroups, int cus) {
  if (R < 32 * E) return 1;
  const long long p = cus / workgroups;
  return p < 1 ? 1 : p > 8 ? 8 : (int)p;
}

// From 32 to 64 rows per expert: the stream instead of the medium tiles, which need an
// index and a combine launch, where both products leave room for two parts, or
// one for every 8 experts (the more experts, the more passes a skewed router's
// first one has).  us a block call, medium tiles and stream: 8 experts of 40 rows,
// d 768, F 256 in 2 clusters 35 and 25; 12 of 48, d 1280, F 512 45 and 32; with a
// router skewed as (rank + 1)^-1.2, 16 of 48, d 512, F 256 35 and 43.  On average
// over 212 drawn sizes with room for two parts 0.71 of the medium tiles' time with
// a uniform router, 0.73 and 0.82 with one skewed as (rank + 1)^-0.5 and ^-1.2;
// with less room 0.99, 1.23 and 1.96 (162 sizes).
inline bool stream_spreads(int C, int E, int R, int d, int F, int cus) {
  if (R < 32 * E || R >= 64 * E) return false;
  const long long gu = (long long)C * E * ((F + 63) / 64), dn = (long long)C * E * ((d + 127) / 128);
  const int parts = E > 16 ? (E + 7) / 8 : 2;
  return parts * (gu > dn ? gu : dn) <= cus;
}

}  // namespace foe
