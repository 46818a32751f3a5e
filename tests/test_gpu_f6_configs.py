"""Every configuration of the FP6-pipe GEMM the launch rule can pick, forced where its indexing can go wrong: fewer K
chunks than waves, K remainders of the wave split and of the ring, one block of rows, ragged last tiles on both sides; and
the persistent ones with a grid of eight workgroups, so that each walks over several tiles, with fewer K stages than the ring
has slots and with K that leaves the ring at another slot than it began.  INT32 accumulators are integers in fp32 and must
equal the oracle's bit for bit."""
import numpy as np
import pytest
import torch

from oracle import smoothrot_oracle as o
import workloads as wl
from parity import check_output

pytestmark = pytest.mark.gpu

CONFIGS = [61, 65, 67, 68, 69, 72, 64064, 48064, 48032, 32064, 32032, 16032, 16016]
TILES = {61: (256, 256), 65: (256, 128), 67: (128, 128), 68: (128, 256), 69: (128, 64), 72: (192, 256)}      # persistent workgroups
SHAPES = [(1, 16, 128), (9, 48, 1152), (17, 80, 2176), (65, 208, 384), (200, 1040, 3200), (40, 4112, 2304)]


def compare(gpu, M, N, K):
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


@pytest.mark.parametrize("config", CONFIGS)
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_forced_configuration(gpu, tune, config, M, N, K):
    print("case", config, M, N, K, flush=True)
    tune(gpu.SR_TUNE_GEMM_TILE, config)
    compare(gpu, M, N, K)


@pytest.mark.parametrize("config", TILES)
@pytest.mark.parametrize("M,N,K", [(1100, 1040, 128), (1030, 784, 384), (777, 1168, 640), (1100, 1040, 1152)])
def test_several_tiles_per_workgroup(gpu, tune, config, M, N, K):
    print("case", config, M, N, K, flush=True)
    bm, bn = TILES[config]
    assert -(-M // bm) * -(-N // bn) > 2 * 8             # every workgroup has two tiles, some three or more
    tune(gpu.SR_TUNE_GEMM_TILE, config)
    tune(gpu.SR_TUNE_GEMM_GRID, 8)
    compare(gpu, M, N, K)


# 32 x 64 fetches its 8-byte tails for two fragments at a time up to 256 tiles in several rows, else each by itself
@pytest.mark.parametrize("M,N,K", [(130, 3312, 384), (130, 3216, 1152), (33, 8176, 2176), (32, 8176, 2176)])
def test_paired_tails_and_single_ones(gpu, tune, M, N, K):
    print("case", M, N, K, flush=True)
    tune(gpu.SR_TUNE_GEMM_TILE, 32064)
    compare(gpu, M, N, K)
