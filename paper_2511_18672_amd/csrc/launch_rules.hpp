// Host-only rules that choose how a launch is divided: plain C++ on sizes, with
// no HIP types, so that they can be checked without a GPU.
#pragma once

#include <stdint.h>

#include <algorithm>

#include "sphinx.h"

namespace sphinx {

// Waves of a k_attn_temporal_lanes launch: request r has chunks[r] neighbouring
// waves for each of its columns, from wave first[r] on; first[R] is their number.
struct TemporalWaves {
  uint32_t first[SPHINX_MAX_REQUESTS + 1];
  uint32_t chunks[SPHINX_MAX_REQUESTS];
};

// A wave takes four queries of a column at a time.  A column of F frames has at
// most F / 4 such chunks, but in a sparse selection most columns have fewer and
// most of those waves would find nothing, at a cost of about 0.1 us per thousand.
// So a request's columns get their chunks, but together no more than about two
// waves per selected token; a wave then takes every chunks[r]-th chunk.  Per
// layer pair at D 1024, one wave per column / this rule / the longest request's
// F / 4 for every column: 62 frames of 2048 columns, 3 % selected 21 / 19 / 29 us
// (with the latent cache 167 / 147 / 278); 60 frames of 4 columns beside two
// frames of 262144, 1 % 142 / 109 / 911; 64 frames of 512 columns, 30 %
// 248 / 59 / 74.  With one wave per token instead of two, 60 frames of 16 columns
// beside two frames of 16384, 10 %, take 53 us instead of 39; with four, the first
// of these takes 186 us with the cache.
inline TemporalWaves temporal_waves(int R, const int32_t* frames, const int32_t* h, const int32_t* w,
                                    const int32_t* cu_sel) {
  TemporalWaves P = {};
  for (int r = 0; r < R; ++r) {
    const int64_t cols = (int64_t)(h[r] >> 1) * (w[r] >> 1), sel = cu_sel[r + 1] - cu_sel[r];
    P.chunks[r] = (uint32_t)std::clamp<int64_t>((2 * sel + cols - 1) / cols, 1, (frames[r] + 3) / 4);
    P.first[r + 1] = P.first[r] + P.chunks[r] * (uint32_t)cols;
  }
  return P;
}

// Tiles of a bf16 GEMM: one workgroup per CU with a deep ring (rows per tile),
// one tall tile per CU, 192- and 128-row tiles in one launch, or 192- or 128-row
// tiles at two workgroups per CU.
enum GemmTiles { kDeep64, kDeep128, kDeep192, kDeep256, kTall, kMixWide, kMixNarrow, kPair192, kPair128 };

// n1 row tiles of 32 t1 rows, then n2 of 32 t2 rows.
struct TallPlan {
  int t1, n1, t2, n2;
};

struct GemmPlan {
  GemmTiles tiles;
  int bn;         // kTall: columns per tile
  TallPlan tall;  // kTall
  int nb, ns;     // mixes: 192- and 128-row tiles (of an XCD's band of rows when narrow) per column tile
};

// Relative time of `tiles` workgroups at two per CU: whole rounds, plus half a
// round for a last round that leaves every CU at most one tile (a lone tile
// runs about twice as fast), else a whole one; `w` is the tile's cost in
// 128-row-tile rounds.  Measured on the block GEMMs at M from 4.9k to 19.4k,
// this picks the faster of the 128- and 192-row tiles or one within 1 %.
inline double tile_rounds(int64_t tiles, int64_t slots, double w) {
  const int64_t full = tiles / slots, rem = tiles % slots;
  return w * ((double)full + (rem == 0 ? 0.0 : rem * 2 <= slots ? 0.5 : 1.0));
}

// Estimated times (us) of one round of tiles, for choosing between the tile
// families: fitted on 64 block GEMMs of M 400 to 30925 at hidden sizes 512,
// 1024 and 1152 (each in a stream of equal launches, so at power-limited
// clocks); k is K in units of 1024, an h-row tile's cost grows with h.
// Two 192x128 tiles per CU: 24 us at M 3226, N 3072, K 1024.
inline double pair_round(int K) { return 4.0 + 20.6 * (K / 1024.0); }
// One tall tile of h x bn per CU: 18.5, 26.9 and 29.8 us at 128, 224 and 256
// rows of 256 columns, K 1024; gated 64 and 107 us at 128 and 256 rows, K 4096
// (the residual's read and write is not hidden by another workgroup).
inline double tall_round(int h, int bn, int K, bool gated) {
  const double k = K / 1024.0, cols = h * bn / 256.0;
  return (gated ? 4.0 : 1.4) + 5.2 * k + cols * ((gated ? 0.073 : 0.03) + 0.06 * k);
}
// Without a residual these rates decide between the families as well.  In steps
// at 15 hidden sizes from 256 to 2048 and M 1296 to 31680 the choice costs 1 %
// against the faster of the two on average; against two-per-CU tiles three of
// about 250 launches lose more than 2 %, all three rounds of 192x256 (D 2048, M 6080,
// QKV: 144 us, 130; D 1536, M 12096, N 3072: 116, 108), which elsewhere gain 4 to 14 %.
//
// Gated launches of more than one round need more: later rounds take longer than
// the first, by more the smaller the tile (M 10816, D 1536, K 6144: 232 us on two
// rounds of 128x256, 202 on two tiles per CU; but M 31680: 525 on three rounds of
// 256x256, 646).  Times of whole launches, fitted on the out-projection
// and MLP2 of those steps (5 and 7 % rms).  Tiles of 192 columns gain nothing in
// two or three rounds at all (M 27552, D 768, K 3072: 163 us, 149; M 31680,
// D 1152, K 4608: 370, 352), but in five they do (M 31680, D 1920, K 7680: 926,
// 1133).  So over 173 gated launches the choice costs 0.3 % against the faster
// family on average and 2.5 % at most against two tiles per CU (on 42 launches
// measured afterwards, 4 %); the rates of one round alone cost up to 14 %.
inline double gated_tall_time(int bn, double r1, int t1, double r2, int t2, int K) {
  const double k = K / 1024.0;
  auto round = [&](int t) { return 1.6 * k - 5.4 + t * bn / 8.0 * (0.109 + 0.08 * k); };
  auto later = [&](int t) { return round(t) * (2.15 - t * bn / 2048.0); };  // t bn / 2048: the tile in 256x256 ones
  return 9.0 + round(t1) + (r1 - 1.0) * later(t1) + (r2 > 0.0 ? r2 * later(t2) : 0.0);
}
inline double gated_pair_time(double rounds, int K) {
  return 7.8 + rounds * (10.3 + 18.7 * (K / 1024.0)) * (1.0 + 0.345 * std::max(0.0, 1.0 - 1.0 / rounds));
}
// The fastest plan of tall tiles by the rates of one round: equal row tiles, or whole
// rounds of one height and one round of another for the rows left.
struct TallChoice {
  int bn = 0;
  TallPlan p{8, 0, 8, 0};
  double us = 1e30;
};
inline TallChoice choose_tall(bool gated, int qcols, int M, int N, int K, int cus) {
  TallChoice best;
  for (int bn : {256, 192}) {
    if (N % bn != 0 || qcols % bn != 0) continue;
    const int64_t nt = N / bn;
    auto take = [&](const TallPlan& p, double us) {
      if (us < best.us) best = TallChoice{bn, p, us};
    };
    for (int t = 3; t <= 8; ++t) {
      const int64_t n = (M + 32 * t - 1) / (32 * t);
      take(TallPlan{t, (int)n, t, 0}, (double)((n * nt + cus - 1) / cus) * tall_round(32 * t, bn, K, gated));
    }
    const int64_t per = cus / nt;  // row tiles of a round
    if (per == 0) continue;
    for (int t1 = 6; t1 <= 8; ++t1) {
      const int64_t r = M / (32 * t1 * per), n1 = r * per, left = M - n1 * 32 * t1;
      if (r == 0 || left == 0) continue;
      const int64_t t2 = std::max<int64_t>(3, (left + 32 * per - 1) / (32 * per));
      if (t2 > 8) continue;
      take(TallPlan{t1, (int)n1, (int)t2, (int)((left + 32 * t2 - 1) / (32 * t2))},
           r * tall_round(32 * t1, bn, K, gated) + tall_round(32 * (int)t2, bn, K, gated));
    }
  }
  return best;
}

// `pair`: the rounds of two tiles per CU.
inline bool gated_tall_faster(const TallChoice& c, int N, int K, int cus, double pair) {
  const auto rounds = [&](int n) { return (double)(((int64_t)n * (N / c.bn) + cus - 1) / cus); };
  const double r1 = rounds(c.p.n1), r2 = rounds(c.p.n2);
  if (c.bn == 192 && r1 + r2 > 1.0 && r1 + r2 <= 3.0) return false;
  return gated_tall_time(c.bn, r1, c.p.t1, r2, c.p.t2, K) < gated_pair_time(pair, K);
}

// The tiles of an M x N x K bf16 GEMM (N and K multiples of 128) on `cus` CUs;
// gated: the epilogue reads and writes the residual; qcols: leading columns
// that are scaled, whole column tiles of them (0 for none).
inline GemmPlan plan_gemm(bool gated, int qcols, int M, int N, int K, int cus) {
  GemmPlan p = {};
  const int64_t nt = N / 128, slots = 2 * (int64_t)cus;
  const int64_t t128 = nt * ((M + 127) / 128), t192 = nt * ((M + 191) / 192);
  const int64_t t256 = nt * ((M + 255) / 256), t64 = nt * ((M + 63) / 64);
  // few tiles: the smallest row tile (128, 192 or 256 rows) whose tiles
  // all fit on the CUs at once, one per CU with a deeper ring (128, 160
  // or 144 KB of LDS; 64-row tiles 96 KB).  Tall tiles give nothing that a
  // step shows here (MLP1 at M 1613: 18.7 us against 19.1 alone, the step
  // within its noise)
  if (t128 <= cus || t192 <= cus || t256 <= cus) {
    // 64-row tiles where 128-row ones would leave more than half the CUs idle
    if (t64 <= cus && 2 * t128 <= cus) p.tiles = kDeep64;
    else p.tiles = t128 <= cus ? kDeep128 : t192 <= cus ? kDeep192 : kDeep256;
    return p;
  }
  // mixed tiles: narrow N, 192-row tiles filling more than half of one round
  int nb = -1, ns = 0;
  if (nt <= 8 && slots % 16 == 0 && t192 * 2 > slots && t192 <= slots) {
    const int per = (int)(slots / 8 / nt);  // slots per XCD and column tile
    const int need = (M + 7) / 8;           // rows per XCD band
    nb = std::max(0, (need - 128 * per + 63) / 64);
    ns = per - nb;
    if (nb * 2 > per) nb = -1;  // some CU would hold two 192-row tiles
  }
  // tall tiles where they are estimated faster than two 192- or 128-row
  // tiles per CU; the narrow mix below takes three quarters of a round
  // (M 9677: out-projection 27 us against 30 on tall tiles, MLP2 73 against 75)
  const TallChoice tall = choose_tall(gated, qcols, M, N, K, cus);
  const double rounds =
      nb >= 0 ? 0.75 : std::min(tile_rounds(t192, slots, 1.0), tile_rounds(t128, slots, 1.0 / 1.41));
  if (tall.us < 1e30 && (gated ? gated_tall_faster(tall, N, K, cus, rounds) : tall.us < rounds * pair_round(K))) {
    p.tiles = kTall;
    p.bn = tall.bn;
    p.tall = tall.p;
    return p;
  }
  // wide N needing more than three rounds of 192-row tiles: the last round
  // all 128-row tiles (ns per column tile), 192-row tiles before it
  if (nt > 8 && t192 > 3 * slots) {
    p.ns = (int)(slots / nt);
    p.nb = (M - 128 * p.ns + 191) / 192;
    if (p.ns > 0 && p.nb > 0) {
      p.tiles = kMixWide;
      return p;
    }
  }
  if (nb >= 0) {
    p.tiles = kMixNarrow;
    p.nb = nb;
    p.ns = ns;
  } else {
    // a 192-row tile does 1.5x the work of a 128-row one in 1.41x the time
    p.tiles = tile_rounds(t192, slots, 1.41) < tile_rounds(t128, slots, 1.0) ? kPair192 : kPair128;
  }
  return p;
}

}  // namespace sphinx
