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

}  // namespace sphinx
