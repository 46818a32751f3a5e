"""The one-pass clip search at every row length that has it, 28 2^p included: bit for bit the codes, scales and ratios of the sum
per ratio (forced by its knob) on normal rows and on rows made to tie, to sit on rounding boundaries, to hold one large value, to
be zero, infinite or NaN; on grids with a common fraction and without; and a minimiser of the oracle's errors."""
import numpy as np
import pytest
import torch

import workloads as wl
from test_gpu_fold_histogram import columns
from test_gpu_next_rows import compare_search

pytestmark = pytest.mark.gpu

ROWS = [(2048, 64), (4096, 64), (7168, 64), (8192, 32), (14336, 64), (16384, 32), (28672, 32)]


@pytest.mark.parametrize("steps,lo", [(2, 0.5), (11, 0.5), (21, 0.5), (21, 0.8), (32, 0.69), (11, 0.37)])
@pytest.mark.parametrize("K,N", ROWS)
def test_one_pass_equals_a_sum_per_ratio(gpu, tune, K, N, steps, lo):
    print("case search rows", K, N, steps, lo, flush=True)
    W = columns(K, N, K + steps)
    W[:, 15] = 0.02                                         # one sign: one large value among small ones, either way
    W[:, 16] = -0.02
    W[:, 17] = (np.random.default_rng(K).random(K) * 0.05).astype(np.float16)
    W[:, 18] = -W[:, 17]
    W = torch.from_numpy(W).cuda()
    a = torch.exp(torch.randn(K, generator=torch.Generator(device="cuda").manual_seed(K), device="cuda"))
    for absmax in (None, a):
        count = gpu.sr_fold_smooth_rotate_quant_ex(W, absmax, 0.5, 0, False, steps, lo)
        tune(gpu.SR_TUNE_CLIP_SEARCH, 1)
        sums = gpu.sr_fold_smooth_rotate_quant_ex(W, absmax, 0.5, 0, False, steps, lo)
        tune(gpu.SR_TUNE_CLIP_SEARCH, gpu.SR_TUNE_AUTO)
        for name, x, y in zip(("codes", "scales", "1/s", "ratios"), count, sums):
            assert torch.equal(x.nan_to_num(7.0) if x.is_floating_point() else x, y.nan_to_num(7.0) if y.is_floating_point() else y), name


@pytest.mark.parametrize("steps,lo", [(21, 0.5), (11, 0.37)])
@pytest.mark.parametrize("K,N", [(7168, 32), (14336, 32), (28672, 16)])
def test_choice_minimises_the_oracles_error(gpu, K, N, steps, lo):
    W = columns(K, N, K + steps)[:, :13]                    # the finite ones
    W = np.concatenate([W, wl.to_f16_sat(np.random.default_rng(K).standard_normal((K, 16 * ((N + 15) // 16) - 13)).astype(np.float32) * 0.02)], axis=1)
    a = (np.abs(np.random.default_rng(1).standard_normal(K)) + 0.1).astype(np.float32)
    compare_search(gpu, np.ascontiguousarray(W), a, 0.5, steps, lo, "search rows K=%d" % K)
