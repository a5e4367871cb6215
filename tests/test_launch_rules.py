"""The rules that divide launches, on the CPU."""
import numpy as np
import pytest

from launch_rules import temporal_waves


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
