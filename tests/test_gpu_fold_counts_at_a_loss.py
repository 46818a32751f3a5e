"""Searched folds that count in vain, at a loss or not at all.  Weights whose rotated rows hold one large value and many small
ones (all weights of one sign, or equal): hardly any value decides between the ratios, so nearly every row needs a sum per ratio,
and counting its values first would be in vain.  Ratios that are multiples of a fine fraction only: many cells, some numbers of
them at odds with the LDS banks.  Row lengths that are to be counted.  Same ratios, codes and scales as from the sums alone, and
not much dearer than those."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


def weights(kind, K, N):
    rng = np.random.default_rng(K + N)
    if kind == "equal":
        W = np.full((K, N), 0.02)
    elif kind == "noise":
        W = 0.02 + 2e-4 * rng.standard_normal((K, N))
    else:
        W = 0.05 * rng.random((K, N))
    W[:, 1::2] *= -1
    return torch.from_numpy(wl.to_f16_sat(W.astype(np.float32))).cuda()


def fold_times(gpu, W, steps, *last):
    """Microseconds on the GPU of the fold with each of the last ratios: shortest of nine runs of four calls, taken in turn, each behind
    a wait long enough for the host to be ahead."""
    work = torch.empty(gpu.sr_fold_workspace_bytes(*W.shape), dtype=torch.uint8, device="cuda")
    times = [[] for _ in last]
    for _ in range(9):
        for lo, t in zip(last, times):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            torch.cuda._sleep(1000000)
            a.record()
            for _ in range(4):
                gpu.sr_fold_smooth_rotate_quant_ex(W, None, 0.5, 0, False, steps, lo, workspace=work)
            b.record()
            torch.cuda.synchronize()
            t.append(a.elapsed_time(b) * 250)
    return [min(t) for t in times]


# 21 ratios 0.025 apart share a fraction; with 0.499 as the last they do not, and every row takes a sum per ratio.  With the count
# in front of the sums these calls took 1.5 .. 1.7 times as long; without it 1.0 .. 1.2 (the other kernel's rotation and LDS).
@pytest.mark.parametrize("K,N", [(2048, 4096), (4096, 4096), (8192, 4096), (14336, 2048), (16384, 2048), (28672, 2048)])
def test_time(gpu, K, N):
    both, sums = fold_times(gpu, weights("noise", K, N), 21, 0.5, 0.499)
    print("case clustered", K, N, "%.1f %.1f us" % (both, sums), flush=True)
    assert both < 1.4 * sums


@pytest.mark.parametrize("kind", ["equal", "noise", "uniform"])
@pytest.mark.parametrize("K,N", [(2048, 32), (4096, 32), (8192, 32), (16384, 16)])
def test_bits(gpu, K, N, kind):
    print("case clustered bits", K, N, kind, flush=True)
    W = weights(kind, K, N)
    for steps, lo in ((21, 0.5), (32, 0.69), (2, 0.9), (5, 1.0)):
        full = gpu.sr_fold_smooth_rotate_quant_ex(W, None, 0.5, 0, False, steps, lo)
        head = gpu.sr_fold_smooth_rotate_quant_ex(W, None, 0.5, 1, False, steps, lo)
        for name, x, y in zip(("codes", "scales", "1/s", "ratios"), full, head):
            assert torch.equal(x, y), name


def test_time_of_a_fine_fraction(gpu):
    """6 ratios 1 / 70 apart: the runs of 16 cells that a thread had took twice as long as the sums."""
    W = (0.02 * torch.randn((2048, 4096), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")).half()
    both, sums = fold_times(gpu, W, 6, 65 / 70, 65 / 70 + 1.37e-4)
    print("case fine fraction %.1f %.1f us" % (both, sums), flush=True)
    assert both < 1.4 * sums


@pytest.mark.parametrize("steps,q", [(2, 100), (3, 71), (4, 100), (6, 56), (6, 64), (6, 70), (8, 98), (9, 75), (11, 100), (12, 100), (32, 62), (32, 99)])
@pytest.mark.parametrize("K,N", [(2048, 48), (4096, 32), (8192, 32), (16384, 16)])
def test_bits_of_fine_fractions(gpu, K, N, steps, q):
    print("case fine fractions bits", K, N, steps, q, flush=True)
    W = torch.from_numpy(wl.to_f16_sat(np.random.default_rng(K + q).standard_t(4, (K, N)).astype(np.float32) * 0.02)).cuda()
    full = gpu.sr_fold_smooth_rotate_quant_ex(W, None, 0.5, 0, False, steps, 1 - (steps - 1) / q)
    head = gpu.sr_fold_smooth_rotate_quant_ex(W, None, 0.5, 1, False, steps, 1 - (steps - 1) / q)
    for name, x, y in zip(("codes", "scales", "1/s", "ratios"), full, head):
        assert torch.equal(x, y), name


# normal weights, 21 ratios: with the count 0.6 .. 0.82 of the time of the sums
@pytest.mark.parametrize("K,N", [(4096, 4096), (7168, 4096), (8192, 4096), (14336, 2048), (16384, 2048), (28672, 2048)])
def test_count_is_ahead(gpu, K, N):
    W = (0.02 * torch.randn((K, N), generator=torch.Generator(device="cuda").manual_seed(K), device="cuda")).half()
    count, sums = fold_times(gpu, W, 21, 0.5, 0.499)
    print("case count ahead", K, N, "%.1f %.1f us" % (count, sums), flush=True)
    assert count < 0.9 * sums
