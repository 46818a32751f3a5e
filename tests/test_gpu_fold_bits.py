"""The searched fold has a kernel of its own for the full transform and the general one for head-wise transforms.  One head
that spans the whole row is the full transform: both kernels give the same codes, scales and ratios, bit for bit."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps", [2, 21])
@pytest.mark.parametrize("K,N", [(64, 1040), (512, 1040), (1024, 16), (2048, 528), (4096, 272), (8192, 80), (16384, 16), (32768, 16)])
def test_full_transform_equals_one_head(gpu, K, N, steps):
    print("case", K, N, steps, flush=True)
    rng = np.random.default_rng(K + N + steps)
    W = wl.to_f16_sat(rng.standard_normal((K, N)).astype(np.float32) * 0.02)
    W[:, 3] = 0
    W[:: max(K // 40, 1), 7] *= 25
    a = torch.from_numpy((np.abs(rng.standard_normal(K)) * (1 + 500 * (rng.random(K) < 0.004))).astype(np.float32)).cuda()
    W = torch.from_numpy(W).cuda()
    full = gpu.sr_fold_smooth_rotate_quant_ex(W, a, 0.5, 0, False, steps, 0.5)
    head = gpu.sr_fold_smooth_rotate_quant_ex(W, a, 0.5, 1, False, steps, 0.5)
    torch.cuda.synchronize()
    for name, x, y in zip(("codes", "scales", "1/s", "ratios"), full, head):
        assert torch.equal(x, y), (name, int((x != y).sum()))
