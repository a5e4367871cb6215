"""The library's own launch rules (csrc/launch_rules.hpp), compiled for the host."""
import ctypes
import functools
import os
import subprocess
import tempfile

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <string.h>
#include "launch_rules.hpp"
extern "C" void temporal(int R, const int32_t* frames, const int32_t* h, const int32_t* w, const int32_t* cu,
                         uint32_t* first, uint32_t* chunks) {
  const sphinx::TemporalWaves P = sphinx::temporal_waves(R, frames, h, w, cu);
  memcpy(first, P.first, 4 * (R + 1));
  memcpy(chunks, P.chunks, 4 * R);
}
extern "C" void gemm(int gated, int qcols, int M, int N, int K, int cus, int32_t* out) {
  const sphinx::GemmPlan p = sphinx::plan_gemm(gated != 0, qcols, M, N, K, cus);
  const int32_t v[8] = {p.tiles, p.bn, p.tall.t1, p.tall.n1, p.tall.t2, p.tall.n2, p.nb, p.ns};
  memcpy(out, v, sizeof(v));
}
"""


@functools.lru_cache(None)
def lib():
    with tempfile.TemporaryDirectory() as d:
        src, out = os.path.join(d, "rules.cpp"), os.path.join(d, "rules.so")
        with open(src, "w") as f:
            f.write(SOURCE)
        subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC",
                        "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2511_18672_amd", "csrc"),
                        src, "-o", out], check=True)
        return ctypes.CDLL(out)


def temporal_waves(shapes, selected):
    """(first wave of each request and their total, waves per column) for (frames, h, w) requests."""
    R = len(shapes)
    cols = [np.ascontiguousarray(c, np.int32) for c in zip(*shapes)]
    cu = np.concatenate([[0], np.cumsum(selected)]).astype(np.int32)
    first, chunks = np.empty(R + 1, np.uint32), np.empty(R, np.uint32)
    lib().temporal(R, *(c.ctypes.data_as(ctypes.c_void_p) for c in (*cols, cu, first, chunks)))
    return first.astype(np.int64), chunks.astype(np.int64)


TILES = ["deep64", "deep128", "deep192", "deep256", "tall", "mix_wide", "mix_narrow", "pair192", "pair128"]


def gemm_plan(which, M, D, mlp, cus=256):
    """(tiles, details) of a block GEMM of M rows: for tall tiles (columns, t1, n1, t2, n2), for mixes (nb, ns)."""
    N, K = {"qkv": (3 * D, D), "out": (D, D), "mlp1": (mlp, D), "mlp2": (D, mlp)}[which]
    v = np.empty(8, np.int32)
    lib().gemm(int(which in ("out", "mlp2")), D if which == "qkv" else 0, int(M), N, K, cus,
               v.ctypes.data_as(ctypes.c_void_p))
    v = v.tolist()
    name = TILES[v[0]]
    return name, tuple(v[1:6]) if name == "tall" else tuple(v[6:]) if name.startswith("mix") else ()
