"""Every bf16 GEMM kernel (tile family, epilogue and tile height) against the
deep-ring tiles: requests packed into one launch of the given rows give bit for
bit what each gives alone, cut small enough that all four of its GEMMs take the
deep-ring tiles.  Every output starts at its bias and adds its products in
ascending k on all of them, and the two MFMA forms they use round alike, so
there is no tolerance; weights whose exponents spread over 2^+-6 and sums with
cancellation would show another order.

Which kernels a packing takes is asked of the library's own launch rule, so a
change of the rule that moves a launch away from its kernel fails here.
"""
import numpy as np
import pytest

import workloads as W
from launch_rules import gemm_plan

torch = pytest.importorskip("torch")
S = pytest.importorskip("paper_2511_18672_amd")

from test_gpu_parity import _packed_vs_separate  # noqa: E402

pytestmark = pytest.mark.gpu

GEMMS = ["qkv", "out", "mlp1", "mlp2"]
EPILOGUE = {"qkv": "bias", "out": "gated", "mlp1": "gelu", "mlp2": "gated"}


def kernels(rows, D, mlp, cus):
    """Names of the kernels that the four GEMMs of a block take."""
    out = set()
    for g in GEMMS:
        tiles, p = gemm_plan(g, rows, D, mlp, cus)
        heights = {p[1], p[3]} if tiles == "tall" and p[4] else {p[1]} if tiles == "tall" else set()
        out |= {f"tall {p[0]} {EPILOGUE[g]} {32 * t}" for t in heights} or {f"{tiles} {EPILOGUE[g]}"}
    return out


def alone_rows(D, mlp, cus):
    """The most rows of which all four GEMMs take the deep-ring tiles."""
    m = 256
    while all(gemm_plan(g, m + 256, D, mlp, cus)[0].startswith("deep") for g in GEMMS):
        m += 256
    return m


def pieces(rows, most):
    """Requests of at most `most` tokens, one or more frames of one row each."""
    out = []
    while rows > 0:
        n = min(rows, most)
        f = -(-n // 1000)
        out.append(W.Request(f, 2, 2 * (n // f)))
        rows -= out[-1].tokens
    return out


@pytest.mark.parametrize("D,mlp,rows,expected", [
    (1152, 4096, 9418, "tall 192 bias 192, tall 192 bias 256, tall 192 gated 256, tall 256 gelu 160, "
                       "tall 256 gelu 224, pair192 gated"),
    (1792, 7168, 14503, "tall 256 bias 192, tall 256 bias 256, tall 256 gated 160, tall 256 gated 192, "
                        "tall 256 gated 224, tall 256 gated 256, tall 256 gelu 96, tall 256 gelu 256"),
    (1152, 1152, 10882, "tall 192 bias 128, tall 192 bias 224, tall 192 gelu 96, tall 192 gelu 192, pair128 gated"),
    (1152, 2304, 7222, "tall 192 bias 160, tall 192 gated 192, tall 192 gelu 128, tall 192 gelu 224"),
    (768, 1024, 10760, "tall 256 gated 128, mix_narrow gated, pair128 bias, pair192 gelu"),
    (1152, 1024, 8198, "tall 192 bias 96, tall 192 gated 224, mix_narrow gelu"),
    (1408, 4096, 4904, "tall 256 gelu 128, tall 256 gelu 192, pair192 bias"),
    (768, 3072, 4050, "tall 256 bias 160, tall 192 gelu 256"),
    (1024, 128, 6795, "tall 256 bias 128, tall 256 bias 224"),
    (256, 4096, 10760, "mix_narrow bias, mix_wide gelu"),
    (1408, 1408, 8869, "mix_wide bias, pair128 gelu"),
    (1280, 128, 30535, "tall 256 bias 96, tall 256 gated 96, mix_wide gated"),
    (1152, 1152, 13501, "tall 192 gelu 160"),
    (1920, 3840, 23020, "tall 192 gated 160"),
    (1152, 4096, 33040, "tall 192 gated 128"),
])
def test_gemm_kernels_round_alike(D, mlp, rows, expected):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    got = kernels(rows, D, mlp, cus)
    assert set(expected.split(", ")) <= got, got
    reqs = pieces(rows, alone_rows(D, mlp, cus))
    assert sum(r.tokens for r in reqs) == rows
    assert all(k.startswith("deep") for r in reqs for k in kernels(r.tokens, D, mlp, cus))
    model = W.ModelCfg(D=D, heads=D // 64, head_dim=64, mlp=mlp, L=1, dtype="bf16")
    wl = W.custom(f"tiles_{D}_{rows}", model, reqs, [1.0] * len(reqs), list(np.linspace(0.3, 0.6, len(reqs))),
                  [25] * len(reqs))
    rng = np.random.default_rng(rows)
    for name, w in wl.weights.items():
        if w.ndim == 2:  # powers of two keep the stored values exact
            w *= np.exp2(rng.integers(-6, 7, w.shape) - 4).astype(w.dtype)
    print(f"[GEMM tiles] D={D} mlp={mlp} rows={rows} in {len(reqs)} requests: {expected}", flush=True)
    assert _packed_vs_separate(wl) == 0.0
