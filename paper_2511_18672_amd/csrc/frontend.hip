// Spatial refinement mask from the regression output (Sec. 5.3; Alg. 1
// laplacian_var, otsu(norm(.)), the opacity mask 1[O < tau_o] and their union,
// pooled to latent tokens by the block rule).
//
// Every step is integer-exact:
//   Y   = (77 R + 150 G + 29 B + 128) >> 8                 (luma, 0..255)
//   L   = Y(up) + Y(down) + Y(left) + Y(right) - 4 Y         (4-neighbour Laplacian)
//   V   = 81 sum9x9(L^2) - sum9x9(L)^2                       (81^2 x local variance)
//   Wm  = sum5x5(V)                                          (box smoothing)
//   inv = 255 - floor(255 (Wm - min) / (max - min))          (per-frame min-max, inverted)
//   t   = Otsu threshold of inv over the frame (exact 192-bit comparison)
//   pixel mask = (O < tau_o) | (inv > t); a token (16 x 16 pixels) is selected
//   iff any of its pixels is.
// Every stencil reads its input map with replicated borders.
//
// Kernels (one pass over each input, Wm stored as a double per pixel and inv
// as 1):
//   k_front_var     per tile of up to 240x16: the stencil chain in registers,
//                   Wm stored, tile min/max of Wm;
//   k_front_minmax  per frame of many tiles: min/max over them;
//   k_front_quant   per 4096 pixels: the frame's min/max from its tiles, inv
//                   as bytes from the stored Wm, LDS histogram merged into the frame's histogram with integer
//                   atomics;
//   k_front_otsu    per frame: Otsu threshold from the 256-bin histogram;
//   k_front_pool    per token: OR over its 16 x 16 pixels of both masks.
#include "kernels.hpp"

namespace sphinx {

namespace {
constexpr int kTPB = 256;
constexpr int kTY = 16;                      // output rows of a tile (image heights are multiples of 16)
constexpr int kTXMax = 240;                  // output columns of a tile, at most: 64 lanes x 4 less the halo
constexpr int kHaloX = 8;                    // 1 (Laplacian) + 4 (9-wide window) + 2 (5-wide box), to 4-column lanes
constexpr int kWinL = 9, kWinV = 5;          // rows of the variance window and of the box
constexpr int kQuantPix = 4096;              // pixels per k_front_quant workgroup
constexpr int kHistCopies = 16;
constexpr int kSplit4Tiles = 512;            // tiles up to which four waves share one,
constexpr int kSplit2Tiles = 1280;           // and up to which two do
constexpr int kFewTiles = 512;               // tiles per frame up to which k_front_quant takes their min/max itself

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return min(max(v, lo), hi); }

// Tiles across an image of W columns, and a tile's columns: the least number
// of tiles, their widths even to within 4 columns.
__host__ __device__ __forceinline__ int tiles_across(int W) { return (W + kTXMax - 1) / kTXMax; }
__host__ __device__ __forceinline__ int tile_cols(int W) {
  const int n = tiles_across(W);
  return 4 * ((W / 4 + n - 1) / n);
}

// Wave shifts by one lane (DPP; they run at the rate of a move and take no LDS).
// Lane 0 of from_left and lane 63 of from_right get 0; those are halo lanes.
__device__ __forceinline__ int from_left(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xf, 0xf, true); }
__device__ __forceinline__ int from_right(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x130, 0xf, 0xf, true); }
__device__ __forceinline__ double from_left(double v) {
  return __hiloint2double(from_left(__double2hiint(v)), from_left(__double2loint(v)));
}
__device__ __forceinline__ double from_right(double v) {
  return __hiloint2double(from_right(__double2hiint(v)), from_right(__double2loint(v)));
}
__device__ __forceinline__ double read_lane(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Luma of the four pixels of 12 interleaved RGB bytes.
struct Raw {
  uint32_t d[3];
};
__device__ __forceinline__ void luma4(const Raw& q, int (&y)[4]) {
  y[0] = (int)(__builtin_amdgcn_udot4(q.d[0], 0x001D964Du, 128u, false) >> 8);
  y[1] = (int)(__builtin_amdgcn_udot4(q.d[0], 0x4D000000u,
                                      __builtin_amdgcn_udot4(q.d[1], 0x00001D96u, 128u, false), false) >> 8);
  y[2] = (int)(__builtin_amdgcn_udot4(q.d[1], 0x964D0000u,
                                      __builtin_amdgcn_udot4(q.d[2], 0x0000001Du, 128u, false), false) >> 8);
  y[3] = (int)(__builtin_amdgcn_udot4(q.d[2], 0x1D964D00u, 128u, false) >> 8);
}

// The stencil chain, one wave per tile of up to 240 x 16 pixels: a lane owns
// four columns and streams down the rows.  Bound by VALU issue, so no stage
// goes through LDS with a neighbour and none is done twice down a column:
//  * vertical windows (9 rows of L and L^2, 5 of V) are running sums, whose
//    leaving rows come from a ring in LDS that only the lane itself reads;
//  * horizontal windows are a lane's own prefix and suffix sums plus those of
//    its two neighbours (DPP wave shifts);
//  * V and everything after it is whole numbers below 2^38 in doubles: exact,
//    at one instruction per addition where 64-bit integers take two;
//  * the next row's bytes are loaded a row ahead.
// 16 rows a tile, because 14 frames of 576 x 1024 then give 2.5 waves per SIMD;
// 14.5 KB of ring per wave lets 11 waves share a CU.
// Borders: columns past the image take the edge column's luma (clamped loads),
// vertical sums of L, L^2, and of V (one lane's value for all lanes outside);
// rows past it repeat the edge row's L and V (the stream does not advance).
// Stores Wm at the tile's pixels and the tile's min and max of Wm to
// part[2 tile .. 2 tile + 1]; the first tile of a frame clears its histogram.
// NW waves share a tile's rows: one wave walks 28 rows in series to give 16, so
// where the tiles would leave most of the 1024 SIMDs idle (up to 512 of them)
// four waves walk 16 rows for 4 each, for 1.7 times the work.  A whole call on
// small requests (a few hundred tokens on): 32 us with one wave, 24 with four (25 with
// the tiles in LDS described below).  Two waves walk 20 rows for 8 each (1.4 times
// the work) and their 29 KB of ring lets the 256 CUs hold 1280 such workgroups at
// once, so up to there they save a third of a lone wave's rows: 300 frames of
// 64 x 64 in 1200 tiles 43.8 us (45.1 with one wave, 43.0 with the tiles in LDS),
// 8 frames of 512 x 512 in 768 tiles 40.6 (42.5, 58.1).
// A 64 x 16 tile per workgroup with every stage in LDS took 100 us for
// 14 frames of 576 x 1024; this takes 35 us.
template <int NW>
__global__ __launch_bounds__(NW * kWave) void k_front_var(ReqTable T, FrontTiles F, const uint8_t* __restrict__ rgb,
                                                     double* __restrict__ part, double* __restrict__ wm,
                                                     uint32_t* __restrict__ hist) {
  typedef double f64x2 __attribute__((ext_vector_type(2)));
  constexpr int kRows = kTY / NW;
  __shared__ int2 rings_l[NW][kWinL][kWave];
  __shared__ f64x2 rings_v[NW][kWinV][2][kWave];
  __shared__ double red[2 * NW];
  const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
  auto& ring_l = rings_l[wave];
  auto& ring_v = rings_v[wave];
  const int tile = blockIdx.x;
  int r = 0;
  while (r + 1 < T.R && F.tile_off[r + 1] <= tile) ++r;
  const int H = 8 * T.h[r], W = 8 * T.w[r];
  const int ntx = tiles_across(W), nty = H / kTY, cols = tile_cols(W);
  const int loc = tile - F.tile_off[r];
  const int f = loc / (ntx * nty), rem = loc - f * ntx * nty;
  if (rem == 0 && wave == 0) reinterpret_cast<uint4*>(hist + 256 * (T.frame_off[r] + f))[lane] = make_uint4(0, 0, 0, 0);
  const int y0 = (rem / ntx) * kTY + wave * kRows, x0 = (rem % ntx) * cols, x1 = min(x0 + cols, W);
  const int64_t pix0 = 256 * (T.tok_off[r] + (int64_t)f * (T.h[r] >> 1) * (T.w[r] >> 1));  // the frame's first
  const int xs = x0 - kHaloX, x = xs + 4 * lane;
  const bool out_l = x < 0, out_r = x >= W;           // the lane's four columns lie left or right of the image
  const bool edge_l = xs < 0, edge_r = xs + 4 * kWave > W;  // the tile has such lanes
  const int last = (W - 4 - xs) >> 2;                 // the lane of the last image column (edge_r)
  const uint8_t* img = rgb + 3 * (pix0 + clampi(x, 0, W - 4));
  auto load = [&](int y) {
    const uint32_t* p = reinterpret_cast<const uint32_t*>(img + 3 * (int64_t)clampi(y, 0, H - 1) * W);
    return Raw{{p[0], p[1], p[2]}};
  };
  auto luma = [&](const Raw& q, int (&y)[4]) {
    luma4(q, y);
    if (edge_l || edge_r) {
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = out_l ? y[0] : y[e];
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = out_r ? y[3] : y[e];
    }
  };
#pragma unroll
  for (int i = 0; i < kWinL; ++i) ring_l[i][lane] = make_int2(0, 0);
#pragma unroll
  for (int i = 0; i < kWinV; ++i) ring_v[i][0][lane] = ring_v[i][1][lane] = f64x2{0.0, 0.0};

  // rows c - 1, c, c + 1 of luma around the Laplacian row c, and row c + 2's bytes
  const int v0 = clampi(y0 - 2, 0, H - 1);  // first row of V
  int rl = v0 - 4;                          // next row of L (may lie above the image)
  int c = clampi(rl, 0, H - 1);
  int up[4], cu[4], dn[4];
  luma(load(c - 1), up);
  luma(load(c), cu);
  luma(load(c + 1), dn);
  Raw ahead = load(c + 2);
  int s1[4] = {0, 0, 0, 0}, s2[4] = {0, 0, 0, 0};  // sums of L and L^2 over the last 9 rows of L, per column
  int slot_l = 0;
  auto push_l = [&]() {
    if (clampi(rl, 0, H - 1) != c) {
      ++c;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        up[e] = cu[e];
        cu[e] = dn[e];
      }
      luma(ahead, dn);
      ahead = load(c + 2);
    }
    ++rl;
    const int left = from_left(cu[3]), right = from_right(cu[0]);
    int l[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      l[e] = up[e] + dn[e] + (e == 0 ? left : cu[e - 1]) + (e == 3 ? right : cu[e + 1]) - 4 * cu[e];
    const int2 old = ring_l[slot_l][lane];  // |L| <= 1020: two to a word
    ring_l[slot_l][lane] = make_int2((l[0] & 0xffff) | (l[1] << 16), (l[2] & 0xffff) | (l[3] << 16));
    slot_l = slot_l + 1 == kWinL ? 0 : slot_l + 1;
    const int o[4] = {(int)(int16_t)old.x, old.x >> 16, (int)(int16_t)old.y, old.y >> 16};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s1[e] += l[e] - o[e];
      s2[e] += __mul24(l[e], l[e]) - __mul24(o[e], o[e]);
    }
  };
  for (int i = 0; i < kWinL - 1; ++i) push_l();

  double v[4] = {0.0, 0.0, 0.0, 0.0}, sv[4] = {0.0, 0.0, 0.0, 0.0};  // V, and its sum over the last 5 rows
  int slot_v = 0, cv = -1;
  double lo = __builtin_inf(), hi = -__builtin_inf();
  for (int k = 0; k < kRows + kWinV - 1; ++k) {
    const int cn = clampi(y0 - 2 + k, 0, H - 1);
    if (cn != cv) {
      cv = cn;
      push_l();
      int a[4], b[4];  // vertical sums, the edge column's in lanes outside the image
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        a[e] = s1[e];
        b[e] = s2[e];
      }
      if (edge_l) {
        const int a0 = __builtin_amdgcn_readlane(a[0], kHaloX / 4), b0 = __builtin_amdgcn_readlane(b[0], kHaloX / 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          a[e] = out_l ? a0 : a[e];
          b[e] = out_l ? b0 : b[e];
        }
      }
      if (edge_r) {
        const int a3 = __builtin_amdgcn_readlane(a[3], last), b3 = __builtin_amdgcn_readlane(b[3], last);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          a[e] = out_r ? a3 : a[e];
          b[e] = out_r ? b3 : b[e];
        }
      }
      // 9-wide window of column e: the left lane's last 4 - e columns, all four own, the right lane's first e + 1
      int wa[4], wb[4];
      auto window = [&](const int (&q)[4], int (&w)[4]) {
        const int p2 = q[0] + q[1], p3 = p2 + q[2], u2 = q[2] + q[3], u3 = q[1] + u2, all = p2 + u2;
        w[0] = from_left(all) + all + from_right(q[0]);
        w[1] = from_left(u3) + all + from_right(p2);
        w[2] = from_left(u2) + all + from_right(p3);
        w[3] = from_left(q[3]) + all + from_right(all);
      };
      window(a, wa);
      window(b, wb);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double da = (double)wa[e];
        v[e] = fma(-da, da, 81.0 * (double)wb[e]);
      }
    }
    const f64x2 o0 = ring_v[slot_v][0][lane], o1 = ring_v[slot_v][1][lane];
    ring_v[slot_v][0][lane] = f64x2{v[0], v[1]};
    ring_v[slot_v][1][lane] = f64x2{v[2], v[3]};
    slot_v = slot_v + 1 == kWinV ? 0 : slot_v + 1;
    sv[0] += v[0] - o0[0];
    sv[1] += v[1] - o0[1];
    sv[2] += v[2] - o1[0];
    sv[3] += v[3] - o1[1];
    if (k < kWinV - 1) continue;
    double q[4] = {sv[0], sv[1], sv[2], sv[3]};
    if (edge_l) {
      const double q0 = read_lane(q[0], kHaloX / 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) q[e] = out_l ? q0 : q[e];
    }
    if (edge_r) {
      const double q3 = read_lane(q[3], last);
#pragma unroll
      for (int e = 0; e < 4; ++e) q[e] = out_r ? q3 : q[e];
    }
    // 5-wide box of column e, in the same manner
    const double p2 = q[0] + q[1], u2 = q[2] + q[3], all = p2 + u2;
    const double w0 = from_left(u2) + (p2 + q[2]), w1 = from_left(q[3]) + all;
    const double w2 = all + from_right(q[0]), w3 = (q[1] + u2) + from_right(p2);
    if (x >= x0 && x < x1) {
      f64x2* o = reinterpret_cast<f64x2*>(wm + pix0 + (int64_t)(y0 + k - (kWinV - 1)) * W + x);
      o[0] = f64x2{w0, w1};
      o[1] = f64x2{w2, w3};
      lo = fmin(fmin(lo, fmin(w0, w1)), fmin(w2, w3));
      hi = fmax(fmax(hi, fmax(w0, w1)), fmax(w2, w3));
    }
  }
  for (int m = 32; m >= 1; m >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, m, kWave));
    hi = fmax(hi, __shfl_xor(hi, m, kWave));
  }
  if (NW > 1) {
    if (lane == 0) {
      red[2 * wave] = lo;
      red[2 * wave + 1] = hi;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      lo = fmin(lo, red[2 * i]);
      hi = fmax(hi, red[2 * i + 1]);
    }
  }
  if (threadIdx.x == 0) {
    part[2 * tile] = lo;
    part[2 * tile + 1] = hi;
  }
}

// Min and max of `n` (min, max) pairs, in every thread of a 256-thread workgroup.
__device__ __forceinline__ void block_minmax(const double* __restrict__ part, int n, double (&red)[2 * kTPB / kWave],
                                             double& lo, double& hi) {
  const int tid = threadIdx.x;
  lo = __builtin_inf();
  hi = -__builtin_inf();
  for (int i = tid; i < n; i += kTPB) {
    lo = fmin(lo, part[2 * i]);
    hi = fmax(hi, part[2 * i + 1]);
  }
  for (int m = 32; m >= 1; m >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, m, kWave));
    hi = fmax(hi, __shfl_xor(hi, m, kWave));
  }
  if (lane_id() == 0) {
    red[2 * (tid / kWave)] = lo;
    red[2 * (tid / kWave) + 1] = hi;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kTPB / kWave; ++w) {
    lo = fmin(lo, red[2 * w]);
    hi = fmax(hi, red[2 * w + 1]);
  }
}

// Tiles of one frame of request r.
__device__ __forceinline__ int frame_tiles(const ReqTable& T, int r) {
  return tiles_across(8 * T.w[r]) * (8 * T.h[r] / kTY);
}

// Per frame of more than kFewTiles tiles: min and max of Wm over them.
__global__ __launch_bounds__(kTPB) void k_front_minmax(ReqTable T, FrontTiles F, const double* __restrict__ part,
                                                       double* __restrict__ lohi) {
  __shared__ double red[2 * kTPB / kWave];
  const int g = blockIdx.x;
  int r = 0;
  while (r + 1 < T.R && T.frame_off[r + 1] <= g) ++r;
  const int per = frame_tiles(T, r);
  if (per <= kFewTiles) return;
  double lo, hi;
  block_minmax(part + 2 * (int64_t)(F.tile_off[r] + (g - T.frame_off[r]) * per), per, red, lo, hi);
  if (threadIdx.x == 0) {
    lohi[2 * g] = lo;
    lohi[2 * g + 1] = hi;
  }
}

// Quantisation of 4096 consecutive pixels of a frame's stored Wm with the
// frame's min/max, four at a time per thread: inv as bytes, and their
// histogram added to the frame's.  Bound by the reads of Wm; the LDS atomics
// would take longer than those where neighbouring pixels share a bin (a
// blurred region is one value), so a bin has 16 counters in 16 banks, one for
// every fourth lane of a wave.  One counter per bin and 64-bit integer
// products took 36 us for 14 frames of 576 x 1024; this takes 17 us (4.3 TB/s).
// The min/max of a frame of up to kFewTiles tiles is taken here, from their 16
// bytes each while the pixels' loads are in flight (at 512 tiles 8 KB from L2
// beside the 32 KB of Wm): 1 us, where a launch of its own took 4.4 us at the
// 180 tiles of those frames (whole call 73.1 -> 71.2 us).  Larger frames, where
// the repeated reads would grow past the pixels, keep the launch (lohi).
__global__ __launch_bounds__(kTPB) void k_front_quant(ReqTable T, FrontTiles F, FrontTiles Q,
                                                      const double* __restrict__ wm, const double* __restrict__ part,
                                                      const double* __restrict__ lohi, uint8_t* __restrict__ inv,
                                                      uint32_t* __restrict__ hist) {
  typedef double f64x2 __attribute__((ext_vector_type(2)));
  constexpr int U = kQuantPix / (4 * kTPB);
  __shared__ __attribute__((aligned(16))) uint32_t sh[256 * kHistCopies];
  __shared__ double red[2 * kTPB / kWave];
  const int tid = threadIdx.x;
  int r = 0;
  while (r + 1 < T.R && Q.tile_off[r + 1] <= (int)blockIdx.x) ++r;
  const int64_t pixels = (int64_t)64 * T.h[r] * T.w[r];  // of a frame
  const int per = (int)((pixels + kQuantPix - 1) / kQuantPix);
  const int loc = (int)blockIdx.x - Q.tile_off[r], f = loc / per, g = T.frame_off[r] + f;
  const int64_t in_frame = (int64_t)(loc - f * per) * kQuantPix + 4 * tid;
  const int64_t pix = 256 * T.tok_off[r] + f * pixels + in_frame;
  f64x2 w[U][2];
#pragma unroll
  for (int i = 0; i < U; ++i)
    if (in_frame + 4 * kTPB * i < pixels) {  // a frame is a multiple of 256 pixels: all four or none
      const f64x2* p = reinterpret_cast<const f64x2*>(wm + pix + 4 * kTPB * i);
      w[i][0] = p[0];
      w[i][1] = p[1];
    }
#pragma unroll
  for (int i = 0; i < kHistCopies; ++i) sh[tid + kTPB * i] = 0;
  const int tiles = frame_tiles(T, r);
  double flo, fhi;
  if (tiles <= kFewTiles) {
    block_minmax(part + 2 * (int64_t)(F.tile_off[r] + f * tiles), tiles, red, flo, fhi);
  } else {
    flo = lohi[2 * g];
    fhi = lohi[2 * g + 1];
  }
  const double span = fhi - flo;
  const double scale = span > 0.0 ? 1.0 / span : 0.0;
  __syncthreads();
  uint32_t* mine = sh + (tid & (kHistCopies - 1));
#pragma unroll
  for (int i = 0; i < U; ++i) {
    if (in_frame + 4 * kTPB * i >= pixels) continue;
    uint32_t packed = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      // floor(255 (w - lo) / span): a rounded product is at most one off, and the remainder, which the fma
      // gives exactly (all are whole numbers below 2^53), says which way
      const double num = 255.0 * (w[i][e >> 1][e & 1] - flo);
      const double q = floor(num * scale), rest = fma(-q, span, num);
      int iv = 255 - (int)q;
      if (span > 0.0) iv += rest < 0.0 ? 1 : (rest >= span ? -1 : 0);
      packed |= (uint32_t)iv << (8 * e);
      atomicAdd(mine + kHistCopies * iv, 1u);
    }
    *reinterpret_cast<uint32_t*>(inv + pix + 4 * kTPB * i) = packed;
  }
  __syncthreads();
  uint32_t sum = 0;
#pragma unroll
  for (int i = 0; i < kHistCopies / 4; ++i) {
    const uint4 v = reinterpret_cast<const uint4*>(sh)[kHistCopies / 4 * tid + i];
    sum += v.x + v.y + v.z + v.w;
  }
  if (sum != 0) atomicAdd(&hist[256 * g + tid], sum);
}

// 192-bit value of a (128-bit) * b (64-bit), as three 64-bit limbs.
struct U192 {
  uint64_t hi, mid, lo;
};
__device__ __forceinline__ U192 mul128x64(unsigned __int128 a, uint64_t b) {
  const unsigned __int128 p0 = (unsigned __int128)(uint64_t)a * b;
  const unsigned __int128 p1 = (unsigned __int128)(uint64_t)(a >> 64) * b + (uint64_t)(p0 >> 64);
  return U192{(uint64_t)(p1 >> 64), (uint64_t)p1, (uint64_t)p0};
}
__device__ __forceinline__ bool gt192(const U192& x, const U192& y) {
  if (x.hi != y.hi) return x.hi > y.hi;
  if (x.mid != y.mid) return x.mid > y.mid;
  return x.lo > y.lo;
}

struct OtsuCand {
  uint64_t nhi, nlo, d;  // score numerator (128 bits) and denominator
  int t;
};
// a scores above b, or scores equal and has the smaller threshold
__device__ __forceinline__ bool otsu_better(const OtsuCand& a, const OtsuCand& b) {
  const unsigned __int128 na = ((unsigned __int128)a.nhi << 64) | a.nlo;
  const unsigned __int128 nb = ((unsigned __int128)b.nhi << 64) | b.nlo;
  const U192 x = mul128x64(na, b.d), y = mul128x64(nb, a.d);
  if (gt192(x, y)) return true;
  if (gt192(y, x)) return false;
  return a.t < b.t;
}

// Otsu's threshold per frame, one thread per candidate t: the t in 0..254
// maximising (S w0 - W s0)^2 / (w0 w1) (an empty class scores 0), compared
// exactly as cross products; the smallest t among equal maxima.
__global__ __launch_bounds__(256) void k_front_otsu(const uint32_t* __restrict__ hist, int32_t* __restrict__ thr) {
  __shared__ int64_t sw[4], ss[4];
  __shared__ OtsuCand best[4];
  const int g = blockIdx.x, t = threadIdx.x, lane = lane_id(), wave = t >> 6;
  const int64_t h = hist[256 * g + t];
  // inclusive scans of the counts and of t * counts
  int64_t w0 = h, s0 = (int64_t)t * h;
  for (int d = 1; d < kWave; d <<= 1) {
    const int64_t a = __shfl_up(w0, d, kWave), b = __shfl_up(s0, d, kWave);
    if (lane >= d) {
      w0 += a;
      s0 += b;
    }
  }
  if (lane == kWave - 1) {
    sw[wave] = w0;
    ss[wave] = s0;
  }
  __syncthreads();
  int64_t Wt = 0, St = 0;
  for (int w = 0; w < 4; ++w) {
    if (w < wave) {
      w0 += sw[w];
      s0 += ss[w];
    }
    Wt += sw[w];
    St += ss[w];
  }
  OtsuCand c{0, 0, 1, t};
  const int64_t w1 = Wt - w0;
  if (t == 255) {
    c.d = 1;  // not a candidate: scores below every real one through the tie rule
  } else if (w0 != 0 && w1 != 0) {
    const __int128 a = (__int128)St * w0 - (__int128)Wt * s0;
    const unsigned __int128 m = (unsigned __int128)(a < 0 ? -a : a);
    const unsigned __int128 n = m * m;
    c.nhi = (uint64_t)(n >> 64);
    c.nlo = (uint64_t)n;
    c.d = (uint64_t)w0 * (uint64_t)w1;
  }
  for (int m = 1; m < kWave; m <<= 1) {
    OtsuCand o;
    o.nhi = __shfl_xor(c.nhi, m, kWave);
    o.nlo = __shfl_xor(c.nlo, m, kWave);
    o.d = __shfl_xor(c.d, m, kWave);
    o.t = __shfl_xor(c.t, m, kWave);
    if (otsu_better(o, c)) c = o;
  }
  if (lane == 0) best[wave] = c;
  __syncthreads();
  if (t == 0) {
    for (int w = 1; w < 4; ++w)
      if (otsu_better(best[w], c)) c = best[w];
    thr[g] = c.t;
  }
}

// Token pooling: lane = 4 * row + k handles pixel row `row` (0..15) of token
// base + k; the 16 rows of a token are OR-reduced across lanes.
__global__ __launch_bounds__(kTPB) void k_front_pool(ReqTable T, const float* __restrict__ opacity, float tau,
                                                     const uint8_t* __restrict__ inv,
                                                     const int32_t* __restrict__ thr, uint8_t* __restrict__ mask,
                                                     float* __restrict__ u) {
  const int64_t N = T.tok_off[T.R];
  const int lane = lane_id(), k = lane & 3, row = lane >> 2;
  const int64_t t = ((int64_t)blockIdx.x * kTPB + threadIdx.x) / kWave * 4 + k;
  bool any = false;
  if (t < N) {
    const TokPos p = decode_token(T, t);
    const int W = 8 * T.w[p.r];
    const int64_t tpf = (int64_t)(T.h[p.r] >> 1) * (T.w[p.r] >> 1);
    const int64_t pix = 256 * (T.tok_off[p.r] + (int64_t)p.f * tpf) + (int64_t)(16 * p.y + row) * W + 16 * p.x;
    const int th = thr[p.g];
    const f32x4* o = reinterpret_cast<const f32x4*>(opacity + pix);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 v = o[q];
      any |= (v[0] < tau) | (v[1] < tau) | (v[2] < tau) | (v[3] < tau);
    }
    const uint4 b = *reinterpret_cast<const uint4*>(inv + pix);
    const uint32_t wv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) any |= (int)((wv[q] >> (8 * e)) & 255u) > th;
  }
  int a = any ? 1 : 0;
  for (int m = 4; m < kWave; m <<= 1) a |= __shfl_xor(a, m, kWave);
  if (t < N && row == 0) {
    mask[t] = (uint8_t)a;
    if (u != nullptr) u[t] = a ? 1.0f : 0.0f;
  }
}
}  // namespace

int front_tiles(const ReqTable& T, FrontTiles* F) {
  int n = 0;
  for (int r = 0; r < T.R; ++r) {
    F->tile_off[r] = n;
    const int W = 8 * T.w[r], H = 8 * T.h[r];
    n += T.frames[r] * tiles_across(W) * (H / kTY);
  }
  F->tile_off[T.R] = n;
  return n;
}

// Workgroups of k_front_quant, likewise.
static int front_chunks(const ReqTable& T, FrontTiles* Q) {
  int n = 0;
  for (int r = 0; r < T.R; ++r) {
    Q->tile_off[r] = n;
    n += T.frames[r] * (int)(((int64_t)64 * T.h[r] * T.w[r] + kQuantPix - 1) / kQuantPix);
  }
  Q->tile_off[T.R] = n;
  return n;
}

size_t front_ws_bytes(const ReqTable& T, int G) {
  FrontTiles F;
  const int tiles = front_tiles(T, &F);
  const int64_t pixels = 256 * T.tok_off[T.R];
  auto a256 = [](size_t b) { return (b + 255) & ~(size_t)255; };
  return a256((size_t)tiles * 16) + a256((size_t)G * 16) + a256((size_t)G * 1024) + a256((size_t)G * 4) +
         a256((size_t)pixels) + a256((size_t)pixels * 8);
}

hipError_t launch_front(const ReqTable& T, int G, const uint8_t* rgb, const float* opacity, float tau,
                        uint8_t* mask, float* u, int32_t* thr_out, void* ws, hipStream_t s) {
  FrontTiles F, Q;
  const int tiles = front_tiles(T, &F), chunks = front_chunks(T, &Q);
  auto a256 = [](size_t b) { return (b + 255) & ~(size_t)255; };
  unsigned char* base = static_cast<unsigned char*>(ws);
  double* part = reinterpret_cast<double*>(base);
  base += a256((size_t)tiles * 16);
  double* lohi = reinterpret_cast<double*>(base);
  base += a256((size_t)G * 16);
  uint32_t* hist = reinterpret_cast<uint32_t*>(base);
  base += a256((size_t)G * 1024);
  int32_t* thr = thr_out != nullptr ? thr_out : reinterpret_cast<int32_t*>(base);
  base += a256((size_t)G * 4);
  const int64_t pixels = 256 * T.tok_off[T.R];
  uint8_t* inv = base;
  base += a256((size_t)pixels);
  double* wm = reinterpret_cast<double*>(base);
  if (tiles <= kSplit4Tiles)
    k_front_var<4><<<tiles, 4 * kWave, 0, s>>>(T, F, rgb, part, wm, hist);
  else if (tiles <= kSplit2Tiles)
    k_front_var<2><<<tiles, 2 * kWave, 0, s>>>(T, F, rgb, part, wm, hist);
  else
    k_front_var<1><<<tiles, kWave, 0, s>>>(T, F, rgb, part, wm, hist);
  bool large = false;
  for (int r = 0; r < T.R; ++r) large |= tiles_across(8 * T.w[r]) * (8 * T.h[r] / kTY) > kFewTiles;
  if (large) k_front_minmax<<<G, kTPB, 0, s>>>(T, F, part, lohi);
  k_front_quant<<<chunks, kTPB, 0, s>>>(T, F, Q, wm, part, lohi, inv, hist);
  k_front_otsu<<<G, 256, 0, s>>>(hist, thr);
  const int64_t N = T.tok_off[T.R];
  k_front_pool<<<(unsigned)((N + 15) / 16), kTPB, 0, s>>>(T, opacity, tau, inv, thr, mask, u);
  return hipGetLastError();
}

}  // namespace sphinx
