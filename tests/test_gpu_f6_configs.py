"""Every configuration of the FP6-pipe GEMM the launch rule can pick, forced where its indexing can go wrong: fewer K
chunks than waves, K remainders of the wave split and of the ring, one block of rows, ragged last tiles on both sides,
more tiles than workgroups.  INT32 accumulators are integers in fp32 and must equal the oracle's bit for bit."""
import numpy as np
import pytest
import torch

from oracle import smoothrot_oracle as o
import workloads as wl
from parity import check_output

pytestmark = pytest.mark.gpu

CONFIGS = [67, 68, 69, 72, 64064, 48064, 48032, 32064, 32032, 16032, 16016]
SHAPES = [(1, 16, 128), (9, 48, 1152), (17, 80, 2176), (65, 208, 384), (200, 1040, 3200), (40, 4112, 2304)]


@pytest.mark.parametrize("config", CONFIGS)
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_forced_configuration(gpu, tune, config, M, N, K):
    print("case", config, M, N, K, flush=True)
    tune(gpu.SR_TUNE_GEMM_TILE, config)
    cx, cw = wl.random_codes(M + K, M, K), wl.random_codes(N + 3 * K, N, K)
    X6, W6 = (gpu.sr_pack_f6_tiles(torch.from_numpy(o.pack_int4(c)).cuda()) for c in (cx, cw))
    want = o.gemm_i32_c(cx, cw)
    full = torch.full((M, N + 8), -7, dtype=torch.int32, device="cuda")
    gpu.sr_w4a4_gemm_f6(X6, None, W6, None, M, N, K, gpu.SR_I32, full[:, :N])
    # scales that are 4-byte aligned only, as the entry point allows
    rng = np.random.default_rng(K)
    xs, ws = rng.uniform(0.01, 2.0, M + 1).astype(np.float32), rng.uniform(1e-4, 1e-2, N + 1).astype(np.float32)
    xs_d, ws_d = torch.from_numpy(xs).cuda()[1:], torch.from_numpy(ws).cuda()[1:]
    Y = gpu.sr_w4a4_gemm_f6(X6, xs_d, W6, ws_d, M, N, K)
    torch.cuda.synchronize()
    assert bool((full[:, N:] == -7).all())
    assert np.array_equal(full[:, :N].cpu().numpy().astype(np.int64), want)
    check_output(Y.cpu().numpy(), o.dequant_out(want, xs[1:].astype(np.float64), ws[1:].astype(np.float64)))
