"""f6 tiles of rows whose rotation cancels exactly: a value that is zero gets the field 0, wherever it lies in the row."""
import numpy as np
import pytest
import torch

from oracle import smoothrot_oracle as o
import f6_codec as fc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,gated", [(1024, False), (1024, True), (2048, False), (2048, True), (4096, True), (8192, False),
                                     (8192, True), (14336, False), (14336, True)])
@pytest.mark.parametrize("M", [6, 263])
def test_exact_zeros(gpu, K, gated, M):
    print("case", K, gated, M, flush=True)
    rng = np.random.default_rng(K + M)
    U = np.zeros((M, K), np.float16)
    U[0] = 1.0                                           # cancels everywhere but in index 0 (14336: but in 28 places)
    U[1, [0, 1]] = 1.0
    U[2, [5, K // 2 + 5]] = 1.0
    for m in range(4, M):                                # row 3 stays zero; the others: two entries, values 0 and +-2
        U[m, rng.choice(K, 2, replace=False)] = rng.choice([-1.0, 1.0], 2)
    G = np.full((M, K), 20.0, np.float16)
    u = torch.from_numpy(U).cuda()
    X6, xs = gpu.sr_swiglu_fwht_quant_act_f6(torch.from_numpy(G).cuda(), u, None, 1.0) if gated else gpu.sr_fwht_quant_act_f6(u, None, 1.0)
    torch.cuda.synchronize()
    ref = o.fwht_quant_swiglu(G, U, None, 1.0) if gated else o.fwht_quant_act(U, None, 1.0)
    fields = fc.f6_tiles_unpack(X6.cpu().numpy(), M, K)
    zero = ref["t"] == 0
    assert zero.mean() > 0.2 and not fields[zero].any()
    assert np.array_equal(fc.f6_codes(fields), ref["codes"])
