"""Selection of rows too long for registers (binned, two reads) against the
oracle's comparison sort, bit for bit: row lengths at the ends of its range and
off every alignment, keep from 1 to T, and scores that defeat the sampled range."""
import numpy as np
import pytest

from test_gpu_parity import cb, orc, say, to_dev, to_host, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def rows(T, seed):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal(T).astype(np.float32)
    near = np.exp(x * np.float32(0.1)).astype(np.float32)
    wide = np.exp(x * 9).astype(np.float32)
    wide[rng.integers(0, T, 40)] *= np.float32(-1)
    few = rng.integers(0, 3, T).astype(np.float32)          # three values: ties at any threshold
    few[rng.integers(0, T, 5)] = np.float32("nan")
    const = np.full(T, 0.25, np.float32)
    const[T // 2] = np.float32("inf")
    zeros = np.where(rng.random(T) < 0.7, np.float32(0), near)   # most keys equal, ranks above them
    zeros[::7] *= np.float32(-1) * 0
    hidden = near.copy()                                    # the top lies outside any sample
    at = rng.choice(T, 900, replace=False)
    hidden[at] = (np.arange(900, dtype=np.float32) // 3) * np.float32(1e30)
    hidden[rng.choice(T, 900, replace=False)] = np.float32("-inf")
    return np.stack([near, wide, few, const, zeros, hidden])


@pytest.mark.parametrize("T", [32769, 40000, 65537, 100003, 131072, 262145, 524287, 524288, 524289])
def test_select_binned_rows(torch, cb, orc, T):   # noqa: F811
    imp = rows(T, T)
    dimp = to_dev(torch, imp)
    for ratio in (1e-9, 300 / T, 0.1, 0.31, 0.9995, 1.0):
        keep = cb.cb_keep_count(T, ratio)
        say(f"case T={T} keep={keep}")
        idx = torch.full((len(imp), keep), -7, dtype=torch.int32, device="cuda")
        assert cb.cb_select(dimp, len(imp), T, ratio, idx) == keep
        got, want = to_host(torch, idx), orc.select(imp, keep)
        for u in range(len(imp)):
            assert np.array_equal(got[u], want[u]), (T, keep, u)


def pair_rows(T, seed):
    """Rows for every place the threshold can take against the pair of sampled
    keys: ties at it, next to it and away from it, samples unlike the row."""
    rng = np.random.default_rng(seed)
    x = rng.standard_normal(T).astype(np.float32)
    near = np.exp(x * np.float32(0.1)).astype(np.float32)
    mid = np.where(rng.random(T) < 0.7, np.float32(1), near)      # one value holds most of the row
    tight = (1 + x * np.float32(1e-4)).astype(np.float32)         # far outliers on both sides
    far = rng.random(T)
    tight[far < 0.005], tight[far > 0.995] = np.float32(1e-20), np.float32(1e20)
    tied = tight.copy()
    tied[rng.random(T) < 0.5] = np.float32(1)
    up = np.sort(near)
    at = (np.arange(256) * T) // 256                               # where the sample is taken
    high, low = near.copy(), near.copy()
    high[at], low[at] = np.float32(1e9), np.float32(-1e9)
    alone = np.full(T, np.float32(-2))                             # all ties but the sample
    alone[at] = near[at]
    two = np.where(np.arange(T) % 2 == 0, np.float32(0), np.float32(-0.0))
    two[T // 3:T // 3 + 300] = np.float32("-inf")
    return np.stack([mid, tight, tied, up, up[::-1], high, low, alone, two])


@pytest.mark.parametrize("T", [32769, 65536, 100003, 524288])
def test_select_binned_pair(torch, cb, orc, T):   # noqa: F811
    imp = pair_rows(T, T + 1)
    dimp = to_dev(torch, imp)
    for ratio in (2 / T, 0.004, 0.05, 0.1, 0.3, 0.5, 0.85, 0.999, 1.0):
        keep = cb.cb_keep_count(T, ratio)
        say(f"case T={T} keep={keep}")
        idx = torch.full((len(imp), keep), -7, dtype=torch.int32, device="cuda")
        assert cb.cb_select(dimp, len(imp), T, ratio, idx) == keep
        got, want = to_host(torch, idx), orc.select(imp, keep)
        for u in range(len(imp)):
            assert np.array_equal(got[u], want[u]), (T, keep, u)
