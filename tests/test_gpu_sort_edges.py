"""Binning where its kernels' groups end: lists around the 256-key sub-lists, their merges and the
kernels' limits; tile counts around the rounds of the pair kernels; entries that meet every tile,
whose pairs run over many windows of 64. Bit for bit."""
import numpy as np
import pytest

from paper_2412_01217_amd import scenes
from tests.test_gpu_parity import _check_sort

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def projection(n, W, H, radius, seed):
    rng = np.random.default_rng(seed)
    hi = (rng.uniform(0, 1, (n, 2)) * [W, H]).astype(np.float32)
    lo = (rng.uniform(-1, 1, (n, 2)) * 1e-6).astype(np.float32)
    depth = rng.choice(np.linspace(0.5, 9.0, 1 + n // 3), n).astype(np.float32)   # ties: by index
    return hi, lo, radius(rng, n).astype(np.int32), depth


@pytest.mark.parametrize("sort_mode", [1, 2])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 256, 257, 511, 512, 513, 768, 1025, 1280, 1281, 2047, 2048, 2049,
                               4096, 4097, 5000, 8191, 8192, 8193])
def test_list_lengths(n, sort_mode):
    views = [scenes.identity_view(16, 16, levels=1)]
    assert _check_sort(views, n, *projection(n, 16, 16, lambda r, m: np.full(m, 3), n), sort_mode=sort_mode) == n


# 12288 tiles are the most that the bucket path takes
@pytest.mark.parametrize("tiles", [(1, 1), (5, 13), (32, 32), (33, 31), (64, 64), (17, 241), (128, 96)])
@pytest.mark.parametrize("n", [700, 1100])   # one block's entries, and more
def test_tile_counts(tiles, n):
    W, H = 16 * tiles[0], 16 * tiles[1]

    def radius(r, m):
        x = r.integers(0, 60, m)
        x[r.uniform(size=m) < 0.3] = 0
        x[[7, 200, 201, m - 1]] = W + H   # every tile
        return x
    views = [scenes.identity_view(W, H, levels=1)]
    D = _check_sort(views, n, *projection(n, W, H, radius, tiles[0]), sort_mode=2)
    assert D > 4 * tiles[0] * tiles[1]


def test_many_entries():
    """More entries than the pair kernels' waves take in one group each, over two items."""
    views = [scenes.identity_view(256, 192, levels=1), scenes.identity_view(96, 64, levels=1)]
    n = 300_000
    sizes = [(256, 192), (96, 64)]
    parts = [projection(n, W, H, lambda r, m: (r.uniform(size=m) < 0.05) * r.integers(1, 20, m), 40 + W)
             for W, H in sizes]
    hi, lo, rad, depth = (np.concatenate([p[i] for p in parts]) for i in range(4))
    assert _check_sort(views, n, hi, lo, rad, depth, sort_mode=2) > 50_000


# the automatic choice: by radix where a list can pass 8192 keys and the mean passes 2560 (2048 of
# several items)
@pytest.mark.parametrize("items", [1, 2])
@pytest.mark.parametrize("n,tiles", [(8192, (1, 1)), (8192, (2, 1)), (8193, (1, 1)), (8193, (2, 2)), (8193, (3, 1)),
                                     (8193, (5, 1)), (20000, (3, 3)), (20000, (4, 2)), (20000, (5, 2))])
def test_automatic_choice(n, tiles, items):
    W, H = 16 * tiles[0], 16 * tiles[1]
    views = [scenes.identity_view(W, H, levels=1)] * items
    parts = [projection(n, W, H, lambda r, m: np.full(m, 3), n + W + i) for i in range(items)]
    assert _check_sort(views, n, *(np.concatenate([p[i] for p in parts]) for i in range(4)), sort_mode=0) >= items * n
