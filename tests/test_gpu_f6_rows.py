"""Tiles of fewer rows than they could have (FP6 GEMM, row counts that would leave the last row of tiles short): every count of
fragments that the second row of waves can have, one and several rows of tiles, several tiles per workgroup; accumulators equal
to the oracle's bit for bit, nothing written past the last row."""
import pytest

from test_gpu_f6_configs import compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("config,M", [(61, 129), (61, 161), (61, 193), (61, 209), (61, 300), (61, 400), (61, 513), (61, 660), (61, 777), (72, 97), (72, 129),
                                      (72, 200), (72, 400), (72, 300), (72, 580), (68, 65), (68, 96), (68, 81), (68, 145)])
@pytest.mark.parametrize("N,K,grid", [(272, 640, 8), (2064, 256, None)])
def test_rows(gpu, tune, config, M, N, K, grid):
    print("case", config, M, N, K, flush=True)
    tune(gpu.SR_TUNE_GEMM_TILE, config)
    if grid:
        tune(gpu.SR_TUNE_GEMM_GRID, grid)
    compare(gpu, M, N, K)
