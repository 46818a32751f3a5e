"""The clip search deals a row's values to lanes by the number of ratios: grids of 2, 3, 9, 11, 31 and 32 ratios (one to
eight subsets of lanes, with and without idle lanes) on rows whose groups of eight values divide unevenly among them."""
import numpy as np
import pytest

import workloads as wl
from test_gpu_next_rows import compare_search

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps", [2, 3, 9, 11, 31, 32])
@pytest.mark.parametrize("K,N", [(64, 16), (448, 16), (2048, 32), (8192, 16)])
def test_clip_search_grid_sizes(gpu, K, N, steps):
    print("case", K, N, steps, flush=True)
    rng = np.random.default_rng(K + steps)
    W = wl.to_f16_sat(rng.standard_normal((K, N)).astype(np.float32) * 0.02)
    W[:, 2] = 0
    W[:: max(K // 40, 1), 7] *= 25
    a = (np.abs(rng.standard_normal(K)) * (1 + 500 * (rng.random(K) < 0.004))).astype(np.float32)
    agree, idx = compare_search(gpu, W, a, 0.5, steps, 0.45, "K=%d N=%d steps=%d" % (K, N, steps))
    assert idx[2] == 0
