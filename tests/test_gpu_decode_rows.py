"""sr_w4a4_linear_decode of two to four tokens runs in one launch for K = 2048 and 4096 up to a number of channels, by two
launches beyond and for other token counts: bit for bit the codes, scales and outputs of sr_fwht_quant_act + sr_w4a4_gemm on
both sides of every edge (channel units that a workgroup lacks, the most units, the switch for two tokens)."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,N", [(2048, 16), (2048, 4112), (2048, 28672), (2048, 32768), (2048, 32784), (4096, 16), (4096, 2064),
                                 (4096, 6144), (4096, 20480), (4096, 20496), (4096, 28672), (4096, 28688)])
def test_one_launch_equals_the_two_calls(gpu, K, N):
    g = torch.Generator(device="cuda")
    g.manual_seed(K + N)
    Wq = torch.randint(0, 256, (N, K // 2), generator=g, dtype=torch.uint8, device="cuda")
    ws = 1e-3 + 1e-3 * torch.rand(N, generator=g, device="cuda")
    inv_s = torch.exp(0.5 * torch.randn(K, generator=g, device="cuda"))
    for M in (2, 3, 4, 5):
        print("case decode rows", M, K, N, flush=True)
        X = torch.full((M, K + 32), 9.0, dtype=torch.float16, device="cuda")
        X[:, :K] = torch.randn((M, K), generator=g, device="cuda").half()
        X[:, 5] = 300
        X[M - 1] = 0 if N % 32 else X[M - 1]
        for f in (inv_s, None):
            Xq, xs = gpu.sr_fwht_quant_act(X[:, :K], f, 0.9)
            want = gpu.sr_w4a4_gemm(Xq, xs, Wq, ws)
            Y = torch.full((M + 1, N + 8), -7.0, dtype=torch.float16, device="cuda")
            Xq1, xs1 = torch.zeros_like(Xq), torch.zeros_like(xs)
            gpu.sr_w4a4_linear_decode(X[:, :K], f, Wq, ws, 0.9, Y=Y[:M, :N], Xq_out=Xq1, x_scale_out=xs1)
            plain = gpu.sr_w4a4_linear_decode(X[:, :K], f, Wq, ws, 0.9)
            assert torch.equal(Xq, Xq1) and torch.equal(xs, xs1)
            assert torch.equal(Y[:M, :N], want) and torch.equal(plain, want)
            assert bool((Y[M:] == -7).all()) and bool((Y[:, N:] == -7).all())


def test_output_over_the_token_rows(gpu):
    """Y may lie over X, as with two launches one behind the other."""
    K = N = 4096
    X = torch.from_numpy(wl.cfg4_X(4, K)).cuda()
    Wq = torch.from_numpy(np.random.default_rng(1).integers(0, 256, (N, K // 2), dtype=np.uint8)).cuda()
    ws = torch.full((N,), 1e-3, device="cuda")
    want = gpu.sr_w4a4_linear_decode(X, None, Wq, ws, 0.9)
    for _ in range(20):
        Y = X.clone()
        gpu.sr_w4a4_linear_decode(Y, None, Wq, ws, 0.9, Y=Y)
        assert torch.equal(Y, want)


@pytest.mark.parametrize("M,K,N", [(3, 2048, 6144), (3, 2048, 28672), (2, 4096, 4096), (4, 4096, 4096), (2, 4096, 14336)])
def test_captured_calls(gpu, M, K, N):
    """Captured calls take two launches where the GPU is done sooner with them: the same outputs as eager ones, on every replay."""
    print("case captured decode rows", M, K, N, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    Wq = torch.randint(0, 256, (N, K // 2), generator=g, dtype=torch.uint8, device="cuda")
    ws = 1e-3 + 1e-3 * torch.rand(N, generator=g, device="cuda")
    X = torch.randn((M, K), generator=g, device="cuda").half()
    x, Y = X.clone(), torch.empty((M, N), dtype=torch.float16, device="cuda")
    work = torch.empty(gpu.sr_linear_decode_workspace_bytes(M, K), dtype=torch.uint8, device="cuda")
    gpu.sr_w4a4_linear_decode(x, None, Wq, ws, 0.9, Y=Y, workspace=work)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        gpu.sr_w4a4_linear_decode(x, None, Wq, ws, 0.9, Y=Y, workspace=work)
    for i in range(4):
        x.copy_(X * (1 + i))
        Y.zero_()
        graph.replay()
        assert torch.equal(Y, gpu.sr_w4a4_linear_decode(x, None, Wq, ws, 0.9)) and bool(Y.any())


@pytest.mark.parametrize("M,K,N", [(1, 4096, 4096), (2, 4096, 4096), (3, 4096, 4096), (4, 2048, 6144), (4, 4096, 28688), (7, 4096, 2048), (16, 8192, 2048)])
def test_one_launch_knob_leaves_the_gemm_alone(gpu, tune, M, K, N):
    """The knob value for one launch where there is one: inside that range, outside it and in the GEMM on its own, the same bits."""
    print("case decode knob 4", M, K, N, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N)
    Wq = torch.randint(0, 256, (N, K // 2), generator=g, dtype=torch.uint8, device="cuda")
    ws = 1e-3 + 1e-3 * torch.rand(N, generator=g, device="cuda")
    X = torch.randn((M, K), generator=g, device="cuda").half()
    Xq, xs = gpu.sr_fwht_quant_act(X, None, 0.9)
    work = torch.empty(max(gpu.sr_linear_decode_workspace_bytes(M, K), 16), dtype=torch.uint8, device="cuda")
    Y = torch.empty((M, N), dtype=torch.float16, device="cuda")
    want, gemm = gpu.sr_w4a4_linear_decode(X, None, Wq, ws, 0.9, workspace=work), gpu.sr_w4a4_gemm(Xq, xs, Wq, ws)
    tune(gpu.SR_TUNE_DECODE_KERNEL, 4)
    assert torch.equal(gpu.sr_w4a4_gemm(Xq, xs, Wq, ws), gemm)
    assert torch.equal(gpu.sr_w4a4_linear_decode(X, None, Wq, ws, 0.9, workspace=work), want)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        gpu.sr_w4a4_linear_decode(X, None, Wq, ws, 0.9, Y=Y, workspace=work)
    for _ in range(3):
        Y.zero_()
        graph.replay()
        assert torch.equal(Y, want)


@pytest.mark.parametrize("M,K", [(2, 2048), (3, 4096), (1, 8192), (4, 8192), (16, 4096)])
def test_output_over_the_token_rows_of_other_calls(gpu, M, K):
    """The same for the other calls that the header names: two tokens and more, any number of tokens of 8192."""
    print("case decode over rows", M, K, flush=True)
    X = torch.from_numpy(wl.cfg4_X(M, K)).cuda()
    Wq = torch.from_numpy(np.random.default_rng(K).integers(0, 256, (K, K // 2), dtype=np.uint8)).cuda()
    ws = torch.full((K,), 1e-3, device="cuda")
    want = gpu.sr_w4a4_linear_decode(X, None, Wq, ws, 0.9)
    for _ in range(10):
        Y = X.clone()
        gpu.sr_w4a4_linear_decode(Y, None, Wq, ws, 0.9, Y=Y)
        assert torch.equal(Y, want)
