"""The tall GEMM tiles (one eight-wave workgroup per CU) at the edges of their row
tiles: requests packed into one launch of just over the rows where tall tiles are
chosen give bit for bit what each request gives alone, on the deep-ring tiles of
small selections.  Every output starts at its bias and adds its products in
ascending k on both, so there is no tolerance.

Widths: 256-column tiles (hidden size 1024, MLP first layer), 192-column ones
(1152), the gated epilogue with one conditioning row per request (2048), and K of
eight stages (512).  Rows: one row in the last row tile, one short of a tile, whole
tiles only.  Two heights in one launch and long K are in the 12902-row packing of
test_few_tile_gemms_match_packed, the other heights in test_gemm_kernels_round_alike.
"""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
S = pytest.importorskip("paper_2511_18672_amd")

from test_gpu_gemm_tiles import kernels  # noqa: E402
from test_gpu_parity import _packed_vs_separate  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,hd,mlp,reqs,rows", [
    (1024, 64, 4096, [W.Request(6, 32, 32), W.Request(3, 10, 94)], 14 * 160 + 1),
    (1152, 72, 4608, [W.Request(6, 32, 32), W.Request(3, 26, 82)], 14 * 224 - 1),
    (2048, 64, 2048, [W.Request(5, 32, 32), W.Request(4, 32, 32), W.Request(9, 16, 32), W.Request(8, 16, 32)], 28 * 160),
    (512, 64, 512, [W.Request(9, 32, 32), W.Request(9, 32, 32), W.Request(7, 2, 398)], 6001),
])
def test_tall_tiles_match_small_ones(D, hd, mlp, reqs, rows):
    assert sum(r.tokens for r in reqs) == rows
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert any(k.startswith("tall") for k in kernels(rows, D, mlp, cus))
    assert all(k.startswith("deep") for r in reqs for k in kernels(r.tokens, D, mlp, cus))
    model = W.ModelCfg(D=D, heads=D // hd, head_dim=hd, mlp=mlp, L=1, dtype="bf16")
    wl = W.custom(f"tall_{D}", model, reqs, [1.0] * len(reqs), list(np.linspace(0.3, 0.7, len(reqs))),
                  [25] * len(reqs))
    print(f"[tall GEMM] D={D} rows={rows}", flush=True)
    assert _packed_vs_separate(wl) == 0.0
