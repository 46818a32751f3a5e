"""Rotation + quantiser in two passes (K = 2048, 4096, 8192, 14336): every K, with and without a gate row and factors, both
outputs, at the row counts where the launch changes (one row; a tile block and a row; K = 14336: as many rows as the chip
has CUs and one more), strided inputs, against the oracle under the boundary rule."""
import numpy as np
import pytest
import torch

from oracle import smoothrot_oracle as o
import workloads as wl
import f6_codec as fc
from parity import check_codes, check_scales

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gated", [False, True])
@pytest.mark.parametrize("smooth", [False, True])
@pytest.mark.parametrize("K,M", [(2048, 1), (2048, 73), (4096, 9), (8192, 1), (8192, 66), (14336, 1), (14336, 9), (14336, 256), (14336, 257)])
def test_two_pass(gpu, K, M, smooth, gated):
    print("case", K, M, smooth, gated, flush=True)
    G, U = wl.gate_up(K + M, M, K, 3, 400.0)
    U[M // 2] = 0                                        # an all-zero row: Delta = 1, codes 0
    inv_s = np.exp(np.random.default_rng(K + M).standard_normal(K) * 0.5).astype(np.float32) if smooth else None
    both = torch.from_numpy(np.concatenate([G, U], 1)).cuda()
    g, u = both[:, :K], both[:, K:]                      # rows 2 K apart
    inv = None if inv_s is None else torch.from_numpy(inv_s).cuda()
    if gated:
        (q4, s4), (q6, s6) = gpu.sr_swiglu_fwht_quant_act(g, u, inv, 0.9), gpu.sr_swiglu_fwht_quant_act_f6(g, u, inv, 0.9)
        ref = o.fwht_quant_swiglu(G, U, inv_s, 0.9)
    else:
        (q4, s4), (q6, s6) = gpu.sr_fwht_quant_act(u, inv, 0.9), gpu.sr_fwht_quant_act_f6(u, inv, 0.9)
        ref = o.fwht_quant_act(U, inv_s, 0.9)
    torch.cuda.synchronize()
    check_scales(s4.cpu().numpy(), ref["x_scale"])
    assert torch.equal(s4, s6) and s4[M // 2] == 1.0
    check_codes(o.unpack_int4(q4.cpu().numpy()), ref["codes"], ref["t"], "nibbles")
    check_codes(fc.f6_codes(fc.f6_tiles_unpack(q6.cpu().numpy(), M, K)), ref["codes"], ref["t"], "tiles")


@pytest.mark.parametrize("K,M,nh", [(2048, 3, 16), (2048, 70, 2), (4096, 5, 32), (4096, 1021, 8), (8192, 9, 64), (8192, 1, 4096)])
@pytest.mark.parametrize("across", [True, False])
@pytest.mark.parametrize("smooth", [False, True])
def test_two_pass_heads(gpu, K, M, nh, across, smooth):
    """Head-wise (4096: up to 1024 rows): lane bits that are left out flip no signs, whichever side of the split they are on."""
    print("case", K, M, nh, across, smooth, flush=True)
    X = wl.gauss_acts(K + M, M, K, 3, 200.0)
    inv_s = np.exp(np.random.default_rng(K + M).standard_normal(K) * 0.5).astype(np.float32) if smooth else None
    q, s = gpu.sr_fwht_quant_act_heads(torch.from_numpy(X).cuda(), nh, across, None if inv_s is None else torch.from_numpy(inv_s).cuda(), 0.9)
    torch.cuda.synchronize()
    ref = o.fwht_quant_act_heads(X, nh, across, inv_s, 0.9)
    check_scales(s.cpu().numpy(), ref["x_scale"])
    check_codes(o.unpack_int4(q.cpu().numpy()), ref["codes"], ref["t"])
