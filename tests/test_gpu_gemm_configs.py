"""Every configuration of the packed-nibble GEMM (M > 16) the launch rule can pick, forced where its indexing can go
wrong: fewer K chunks than waves, K remainders of the wave split, ragged last tiles on both sides, K that only the generic
kernel takes; and the persistent ones with a grid of eight workgroups, so that each walks over several tiles, with fewer K
stages than the ring has slots and with K that leaves the ring at another slot than it began.  INT32 accumulators must equal
the oracle's bit for bit."""
import numpy as np
import pytest
import torch

from oracle import smoothrot_oracle as o
import workloads as wl
from parity import check_output

pytestmark = pytest.mark.gpu

CONFIGS = [14, 15, 17, 18, 19, 20, 64064, 48064, 48032, 32064, 32032, 32016]
TILES = {14: (128, 128), 15: (256, 128), 17: (128, 64), 18: (192, 128), 19: (64, 128), 20: (128, 128)}      # persistent workgroups
SHAPES = [(17, 16, 256), (33, 80, 2304), (49, 208, 4352), (65, 48, 768), (200, 1040, 2560), (40, 4112, 4608), (70, 96, 192)]


def compare(gpu, M, N, K):
    cx, cw = wl.random_codes(M + K, M, K), wl.random_codes(N + 3 * K, N, K)
    Xq, Wq = (torch.from_numpy(o.pack_int4(c)).cuda() for c in (cx, cw))
    want = o.gemm_i32_c(cx, cw)
    full = torch.full((M, N + 8), -7, dtype=torch.int32, device="cuda")
    gpu.sr_w4a4_gemm(Xq, None, Wq, None, gpu.SR_I32, full[:, :N])
    rng = np.random.default_rng(K)
    xs, ws = rng.uniform(0.01, 2.0, M).astype(np.float32), rng.uniform(1e-4, 1e-2, N).astype(np.float32)
    Y = gpu.sr_w4a4_gemm(Xq, torch.from_numpy(xs).cuda(), Wq, torch.from_numpy(ws).cuda())
    torch.cuda.synchronize()
    assert bool((full[:, N:] == -7).all())
    assert np.array_equal(full[:, :N].cpu().numpy().astype(np.int64), want)
    check_output(Y.cpu().numpy(), o.dequant_out(want, xs.astype(np.float64), ws.astype(np.float64)))


@pytest.mark.parametrize("config", CONFIGS)
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_forced_configuration(gpu, tune, config, M, N, K):
    print("case", config, M, N, K, flush=True)
    tune(gpu.SR_TUNE_GEMM_TILE, config)
    compare(gpu, M, N, K)


@pytest.mark.parametrize("config", TILES)
@pytest.mark.parametrize("M,N,K", [(1100, 1040, 256), (1030, 784, 768), (777, 1168, 1280), (1100, 1040, 2304)])
def test_several_tiles_per_workgroup(gpu, tune, config, M, N, K):
    print("case", config, M, N, K, flush=True)
    bm, bn = TILES[config]
    assert -(-M // bm) * -(-N // bn) > 2 * 8             # every workgroup has two tiles, some three or more
    tune(gpu.SR_TUNE_GEMM_TILE, config)
    tune(gpu.SR_TUNE_GEMM_GRID, 8)
    compare(gpu, M, N, K)


# the kernel for tile grids that divide among the XCDs is another than the one for grids cut into runs (all but one of those above)
@pytest.mark.parametrize("config", TILES)
@pytest.mark.parametrize("tiles_m,tiles_n,K", [(4, 8, 256), (8, 3, 768), (2, 12, 1280), (4, 8, 2304)])
def test_several_tiles_per_workgroup_of_divided_grids(gpu, tune, config, tiles_m, tiles_n, K):
    bm, bn = TILES[config]
    assert (tiles_m % 2 == 0 and tiles_n % 4 == 0) or tiles_m % 8 == 0      # rectangles, and at least three tiles a workgroup
    M, N = tiles_m * bm - 5, tiles_n * bn - 16
    print("case divided", config, M, N, K, flush=True)
    tune(gpu.SR_TUNE_GEMM_TILE, config)
    tune(gpu.SR_TUNE_GEMM_GRID, 8)
    compare(gpu, M, N, K)
