"""Head-wise rotation of rows of 4096: the codes bit for bit as fp32 additions in the stated order give them -- index bits
0 .. 11 in turn up to 1024 rows, bits 0, 1, 2, 9, 10, 11 and then 3 .. 8 beyond.  (A sum of 4096 values has many orders, all
correct to rounding; which one a row count takes is part of the result, or a code on a rounding boundary comes out one off.)"""
import numpy as np
import pytest
import torch

from oracle import smoothrot_oracle as o
import workloads as wl

RISING = tuple(range(12))
WAVE = (0, 1, 2, 9, 10, 11, 3, 4, 5, 6, 7, 8)


def rotate_f32(x, bits):
    """fp32 butterflies on the given index bits, one rounding per addition."""
    v = x.astype(np.float32)
    for b in bits:
        u = v.reshape(len(v), -1, 2, 1 << b)
        v = np.stack([u[:, :, 0] + u[:, :, 1], u[:, :, 0] - u[:, :, 1]], 2).reshape(len(v), -1)
    return v


def codes_f32(X, inv_s, bits, clip):
    x = X.astype(np.float32) if inv_s is None else X.astype(np.float32) * inv_s
    y = rotate_f32(x, bits)
    amax = np.abs(y).max(1)
    delta = np.where(amax == 0, np.float32(1), (np.float32(clip) * amax) / np.float32(7)).astype(np.float32)
    inv = np.float32(1) / delta
    return np.clip(np.rint(y.astype(np.float64) * inv[:, None].astype(np.float64)), -8, 7).astype(np.int8), delta


def case(M, nh, across, smooth):
    K = 4096
    X = wl.gauss_acts(3 * M + nh, M, K, 5, 300.0)
    inv_s = np.exp(np.random.default_rng(M + nh).standard_normal(K) * 0.5).astype(np.float32) if smooth else None
    d = K // nh
    return X, inv_s, (lambda order: [b for b in order if (1 << b >= d) == across])


def test_orders_differ_on_these_inputs():
    X, inv_s, bits = case(1025, 4, False, True)
    a, b = (codes_f32(X, inv_s, bits(order), 0.9)[0] for order in (RISING, WAVE))
    assert 0 < (a != b).sum() < 1e-4 * a.size
    ref = o.fwht_quant_act_heads(X[:8], 4, False, inv_s, 0.9)
    assert (a[:8] != ref["codes"]).mean() < 1e-4


@pytest.mark.gpu
@pytest.mark.parametrize("M,order", [(1024, RISING), (1025, WAVE), (1400, WAVE)])
@pytest.mark.parametrize("nh,across", [(32, True), (32, False), (4, False), (512, True)])
@pytest.mark.parametrize("smooth", [False, True])
def test_heads_codes_bit_for_bit(gpu, M, order, nh, across, smooth):
    print("case", M, nh, across, smooth, flush=True)
    X, inv_s, bits = case(M, nh, across, smooth)
    q, s = gpu.sr_fwht_quant_act_heads(torch.from_numpy(X).cuda(), nh, across, None if inv_s is None else torch.from_numpy(inv_s).cuda(), 0.9)
    torch.cuda.synchronize()
    codes, delta = codes_f32(X, inv_s, bits(order), 0.9)
    assert np.array_equal(s.cpu().numpy(), delta)
    assert np.array_equal(o.unpack_int4(q.cpu().numpy()), codes)
