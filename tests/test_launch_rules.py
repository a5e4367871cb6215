"""The rules that divide launches, on the CPU."""
import numpy as np
import pytest

from launch_rules import gemm_plan, temporal_waves


@pytest.mark.parametrize("seed", range(8))
def test_temporal_waves_follow_the_selection(seed):
    """Every column gets a wave and no more than its frames in fours; the waves
    of a launch stay near two per selected token whatever request is longest;
    requests are laid end to end."""
    rng = np.random.default_rng(seed)
    shapes, left = [], 64
    while left > 0 and len(shapes) < 6:
        f = int(min(left, np.exp(rng.uniform(0, np.log(64)))))
        shapes.append((max(1, f), 2 * int(rng.integers(1, 200)), 2 * int(rng.integers(1, 200))))
        left -= max(1, f)
    cols = np.array([h * w // 4 for _, h, w in shapes])
    frames = np.array([s[0] for s in shapes])
    sel = np.maximum(1, (np.exp(rng.uniform(np.log(0.01), 0, len(shapes))) * frames * cols).astype(int))
    first, chunks = temporal_waves(shapes, sel)
    assert np.array_equal(np.diff(first), chunks * cols) and first[0] == 0
    assert (chunks >= 1).all() and (chunks <= (frames + 3) // 4).all()
    assert (chunks * cols < 2 * sel + 2 * cols).all()
    assert ((chunks == (frames + 3) // 4) | (chunks * cols >= 2 * sel)).all()


def test_temporal_waves_of_mixed_requests():
    """One request of 60 frames leaves the single frames beside it at one wave per column."""
    first, chunks = temporal_waves([(60, 4, 4), (1, 1024, 1024), (1, 1024, 1024)], [120, 2621, 2621])
    assert chunks.tolist() == [15, 1, 1]
    assert first[-1] == 15 * 4 + 2 * 512 * 512


@pytest.mark.parametrize("which,M,D,mlp", [
    ("mlp2", 10816, 1536, 6144), ("mlp2", 31680, 768, 3072), ("mlp2", 27552, 768, 3072), ("mlp2", 31680, 1152, 4608),
    ("mlp2", 27552, 1152, 4608), ("mlp2", 12992, 1152, 4608), ("mlp2", 17952, 2048, 4096), ("out", 10816, 2048, 8192),
    ("out", 13920, 1536, 6144), ("out", 11232, 1920, 7680)])
def test_gated_launches_slower_on_tall_tiles(which, M, D, mlp):
    """Measured 3.6 to 14 % slower on tall tiles than on two tiles per CU."""
    assert gemm_plan(which, M, D, mlp)[0] != "tall"


@pytest.mark.parametrize("which,M,D,mlp", [
    ("mlp2", 31680, 1536, 6144), ("mlp2", 31680, 1024, 4096), ("mlp2", 15872, 1280, 5120), ("mlp2", 7744, 1152, 4608),
    ("mlp2", 31680, 1920, 7680), ("mlp2", 5776, 1536, 6144), ("qkv", 9600, 1280, 5120), ("mlp1", 8832, 1408, 5632)])
def test_launches_faster_on_tall_tiles(which, M, D, mlp):
    """Measured 10 to 20 % faster on tall tiles."""
    assert gemm_plan(which, M, D, mlp)[0] == "tall"


@pytest.mark.parametrize("seed", range(4))
def test_gemm_plans_cover_the_rows(seed):
    """Every plan covers all rows, with no row tile past them but one of a mix,
    which the kernel skips."""
    rng = np.random.default_rng(seed)
    for _ in range(2000):
        D, mlp = 128 * int(rng.integers(1, 17)), 128 * int(rng.integers(1, 65))
        M, which = int(np.exp(rng.uniform(0, np.log(70000)))), ["qkv", "out", "mlp1", "mlp2"][int(rng.integers(4))]
        tiles, p = gemm_plan(which, M, D, mlp)
        N = {"qkv": 3 * D, "mlp1": mlp}.get(which, D)
        if tiles == "tall":
            bn, t1, n1, t2, n2 = p
            assert bn in (192, 256) and N % bn == 0 and (which != "qkv" or D % bn == 0)
            assert 3 <= t1 <= 8 and 3 <= t2 <= 8 and n1 > 0 and n2 >= 0
            rows = 32 * t1 * n1 + 32 * t2 * n2
            assert rows >= M and rows - 32 * (t2 if n2 else t1) < M
        elif tiles == "mix_wide":
            assert min(p) > 0 and 192 * p[0] + 128 * p[1] >= M
        elif tiles == "mix_narrow":
            assert min(p) >= 0 and 192 * p[0] + 128 * p[1] >= (M + 7) // 8
