"""The searched fold takes its ratios from one pass over a row where they are multiples of a common fraction, and head-wise
folds from a sum per ratio.  One head that spans the whole row is the full transform: same ratios, codes and scales, bit for
bit, on grids with and without a common fraction, on normal rows and on rows made to tie or to sit on rounding boundaries."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


def columns(K, N, seed):
    rng = np.random.default_rng(seed)
    W = (rng.standard_normal((K, N)) * 0.02).astype(np.float32)
    W[:, 0] = 0
    for n in range(1, 9):                                   # one, two, .. eight weights: few distinct magnitudes, many ties
        W[:, n] = 0
        W[rng.choice(K, n, replace=False), n] = 0.5
    W[:, 9] = rng.integers(-7, 8, K) / 14.0
    W[:, 10] = np.float32(6e-8)                             # the smallest fp16
    W[:, 11] = 60000.0 * np.sign(W[:, 11])
    W[:, 12] = rng.standard_t(2, K) * 0.02                  # long tails: the smallest ratios win
    W[0, 13] = np.inf
    W[K // 2, 14] = np.nan
    return wl.to_f16_sat(W) if np.isfinite(W).all() else W.astype(np.float16)


@pytest.mark.parametrize("steps,lo", [(1, 0.9), (2, 0.5), (11, 0.5), (21, 0.5), (21, 0.8), (26, 0.5), (32, 0.69), (32, 0.25), (11, 0.37)])
@pytest.mark.parametrize("K,N", [(2048, 48), (4096, 1040), (8192, 32), (16384, 16)])
def test_one_pass_equals_a_sum_per_ratio(gpu, K, N, steps, lo):
    print("case", K, N, steps, lo, flush=True)
    W = torch.from_numpy(columns(K, N, K + steps)).cuda()
    full = gpu.sr_fold_smooth_rotate_quant_ex(W, None, 0.5, 0, False, steps, lo)
    head = gpu.sr_fold_smooth_rotate_quant_ex(W, None, 0.5, 1, False, steps, lo)
    torch.cuda.synchronize()
    for name, x, y in zip(("codes", "scales", "1/s", "ratios"), full, head):
        assert torch.equal(x.nan_to_num(7.0) if x.is_floating_point() else x, y.nan_to_num(7.0) if y.is_floating_point() else y), name
