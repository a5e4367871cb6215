"""GPU parity of the fp32 matrix-core kernels (attention and GEMM of fp32 models)
at the edges of their tiles, against the oracle in float64.

Attention: 32-query and 32-key tiles dealt to four waves, so segments of less
than one tile, of exactly one, and with one to four tiles and a remainder; head
dims of every rounding (16, 32, 64) with and without 16-byte rows.  Bound: scores
stay below about 24 in magnitude, so a score is off by at most 24 * 2^-24 * (a few
roundings) and a probability by that relatively; with |v| <= 5 and fp32 sums the
output is within 1e-5.

GEMM: 32-row and 64-column tiles, K steps of 64 in a ring of three: selections
around one row tile, and D and MLP widths of one, three, five and eight K steps.
"""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
S = pytest.importorskip("paper_2511_18672_amd")

from test_gpu_attention import check, rand  # noqa: E402
from test_gpu_parity import check_end_to_end  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd", [1, 10, 16, 20, 32, 33, 48, 64])
def test_fp32_attention_edges(hd):
    rng = np.random.default_rng(hd)
    heads = 3
    D = heads * hd
    lq, lk = [1, 31, 32, 33, 130, 5, 64], [1, 31, 32, 33, 130, 257, 7]
    cu_q, cu_k = (np.concatenate([[0], np.cumsum(v)]).astype(np.int32) for v in (lq, lk))
    ld = (D + 7) // 8 * 8
    q = rand(rng, int(cu_q[-1]), D, 0.5 if hd < 20 else 2.0 / np.sqrt(hd))
    k, v = rand(rng, int(cu_k[-1]), D), rand(rng, int(cu_k[-1]), D)
    check(q, k, v, heads, hd, cu_q, cu_k, dtype="f32", tag=f"fp32 hd{hd}", ldq=ld, ldkv=ld + 8)


@pytest.mark.parametrize("D,heads,mlp,n", [(64, 1, 64, 1), (64, 4, 192, 31), (192, 3, 320, 33), (512, 8, 2048, 70)])
def test_fp32_gemm_edges(D, heads, mlp, n):
    model = W.ModelCfg(D=D, heads=heads, head_dim=D // heads, mlp=mlp, L=1, dtype="f32")
    wl = W.custom(f"fp32_{D}_{n}", model, [W.Request(2, 16, 16)], [n / 128], [0.5], [2])
    R = check_end_to_end(wl)
    assert R.n_sel == n


@pytest.mark.parametrize("hd", [16, 64])
@pytest.mark.parametrize("tiles", [(0,), (1,), (1, 5, 9), (0, 4, 8, 1, 5, 9, 2, 6)])
def test_fp32_attention_keys_of_no_weight(hd, tiles):
    """Keys whose scores overflow to -inf (weight 0) fill whole 32-key tiles: the
    first tile of a wave, every tile of one wave, all tiles of three waves.  The
    other keys' softmax is what remains, so the bound is that of the edges above."""
    rng = np.random.default_rng(len(tiles))
    heads, n = 2, 300
    D = heads * hd
    q, k, v = rand(rng, n, D, 2.0 / np.sqrt(hd)), rand(rng, n, D), rand(rng, n, D)
    for t in tiles:
        k[32 * t:32 * t + 32, ::hd] = 3e38
    q[:, ::hd] = -2.0
    cu = np.array([0, n], np.int32)
    check(q, k, v, heads, hd, cu, cu, dtype="f32", tag=f"fp32 no weight hd{hd} tiles {tiles}")


def test_fp32_attention_beyond_one_launch():
    """131073 queries of 4096 heads of one dim: more workgroups than the 2^32
    threads of one launch hold.  Three keys, so that plain torch gives the
    reference; |score| < 40 and |v| < 6, hence the same 1e-5."""
    heads, n, kv = 4096, 131073, 3
    gen = torch.Generator(device="cuda").manual_seed(9)
    q = torch.randn(n, heads, generator=gen, device="cuda")
    k, v = (torch.randn(kv, heads, generator=gen, device="cuda") for _ in range(2))
    o = torch.full((n, heads), float("nan"), device="cuda")
    print(f"[attention] fp32 heads={heads} hd=1 n={n}", flush=True)
    S.sphinx_varlen_attention(S.F32, heads, 1, q, heads, k, v, heads, o, np.array([0, n], np.int32),
                              np.array([0, kv], np.int32))
    worst = 0.0
    for a in range(0, n, 16384):
        s = q[a:a + 16384].double()[:, None] * k.double()
        w = torch.exp2(s - s.amax(1, keepdim=True))
        ref = (w * v.double()).sum(1) / w.sum(1)
        worst = max(worst, float((o[a:a + 16384].double() - ref).abs().nan_to_num(nan=float("inf")).max()))
    print(f"[attention beyond one launch] max_abs = {worst:.3e}", flush=True)
    assert worst <= 1e-5
