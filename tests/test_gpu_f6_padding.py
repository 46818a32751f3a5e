"""The rows that pad the last block of 8 tile rows: every quantiser that writes f6 tiles leaves zero codes there, in a
buffer of its own as in one that held something else."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,M,gated", [(4096, 5, False), (4096, 1027, False), (4096, 3079, False), (2048, 9, False),
                                       (14336, 3, False), (14336, 201, True), (14336, 1101, False), (8192, 65, True)])
def test_padding_rows_are_zero(gpu, K, M, gated):
    print("case", K, M, gated, flush=True)
    g = torch.Generator(device="cuda").manual_seed(K + M)
    X, G = (torch.randn((M, K), generator=g, device="cuda").half() for _ in range(2))
    inv = torch.rand(K, generator=g, device="cuda") + 0.5
    X6 = torch.full((gpu.sr_f6_tiles_bytes(M, K),), 0xFF, dtype=torch.uint8, device="cuda")
    if gated:
        got = [gpu.sr_swiglu_fwht_quant_act_f6(G, X, inv, 0.9, b)[0] for b in (X6, None)]
    else:
        got = [gpu.sr_fwht_quant_act_f6(X, inv, 0.9, b)[0] for b in (X6, None)]
    torch.cuda.synchronize()
    for t in got:
        # piece (r, t, g) of block (R, C): 16 bytes at 256 t + 128 (g ^ (R & 1)) + 16 r, 8 at 512 + 128 (g ^ (R & 1)) + 16 r + 8 t
        last = t.view(K // 128, (M + 7) // 8, 768)[:, -1].cpu()
        for r in range(M % 8, 8):
            for step in range(2):
                for half in range(2):
                    a, b = 256 * step + 128 * half + 16 * r, 512 + 128 * half + 16 * r + 8 * step
                    assert not last[:, a:a + 16].any() and not last[:, b:b + 8].any(), (r, step, half)
        assert last.any()                                # (the rows before them are not)
