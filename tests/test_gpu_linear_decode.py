"""The one-kernel form of the layer for one row against the separate kernels (a forced GEMM variant selects them;
the other tests hold them to the oracle), bit for bit."""
import numpy as np
import pytest
import torch

import paper_2402_17985_amd as fq
from tests.gpu_util import DEV, bytes_ws, dev_i32, scalar

pytestmark = pytest.mark.gpu
DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


def _compare(X, src, rep, W, bits, static, ydt, bias, pad=0):
    M, K = X.shape
    N = W.shape[0]
    Kpad = len(src)
    src_d = dev_i32(src)
    Wq = torch.empty((Kpad // 128, N, 96) if bits == 6 else (N, Kpad if bits == 8 else Kpad // 2), dtype=torch.uint8, device=DEV)
    s_w = torch.empty(1, dtype=torch.float32, device=DEV)
    fq.fq_flatten_weights(W, src_d, bits, Wq, s_w, bytes_ws(fq.fq_weights_workspace_bytes(K, Kpad)))
    rep_d = dev_i32(np.concatenate([[0], rep]))[1:]                        # 4-byte aligned only
    ws = bytes_ws(fq.fq_linear_workspace_bytes(M, K, Kpad, bits))
    out = []
    for variant in (-1, 2):
        Y = torch.full((M, N + pad), 7, dtype=ydt, device=DEV)
        fq.fq_gemm_select(variant)
        try:
            fq.fq_linear_bias(X, src_d, rep_d, Wq, s_w, bias, bits, Y[:, :N], ws, absmax_in=static)
        finally:
            fq.fq_gemm_select(-1)
        out.append(Y.view(torch.int16 if Y.element_size() == 2 else torch.int32))
    assert torch.equal(out[0], out[1])


def _x(rng, M, K, dtype):
    buf = torch.from_numpy(rng.standard_normal((M, (K + 15) // 16 * 16), dtype=np.float32) * np.float32(1.5)).to(DEV)
    buf[:, rng.choice(K, max(1, K // 100), replace=False)] *= 37.0
    return buf.to(DTYPES[dtype])[:, :K]


@pytest.mark.parametrize("bits", [8, 4, 6])
@pytest.mark.parametrize("scale", ["static", "dynamic", "zero"])
@pytest.mark.parametrize("dtype,M,K,N", [("bf16", 1, 16, 16), ("f32", 1, 257, 33), ("f16", 1, 1000, 200), ("bf16", 1, 4104, 8200),
                                         ("bf16", 1, 9000, 16500), ("f32", 1, 640, 47), ("bf16", 1, 30000, 70), ("bf16", 2, 640, 70)])
def test_planned_maps(dtype, M, K, N, scale, bits):
    rng = np.random.default_rng(K)
    X = _x(rng, M, K, dtype)
    W = torch.from_numpy(rng.standard_normal((N, (K + 15) // 16 * 16), dtype=np.float32)).to(DEV).to(torch.bfloat16)[:, :K]
    T = 4.0
    src, rep, _, _ = fq.fq_flatten_plan(X.float().abs().amax(dim=0).cpu().numpy(), T, 128 if bits == 6 else 32)
    if scale == "zero":
        X.zero_()
    static = scalar(T) if scale == "static" else None
    _compare(X, src, rep, W, bits, static, torch.bfloat16, None)
    _compare(X, src, rep, W, bits, static, torch.float32, torch.from_numpy(rng.standard_normal(N, dtype=np.float32)).to(DEV), pad=3)
    _compare(X, src, rep, W, bits, static, torch.int32, None)


@pytest.mark.parametrize("bits", [8, 4, 6])
@pytest.mark.parametrize("static", [False, True])
def test_maps_that_are_not_the_planners(static, bits):
    rng = np.random.default_rng(5)
    M, K, N, Kpad = 1, 500, 100, 1152
    X = _x(rng, M, K, "f32")
    W = torch.from_numpy(rng.standard_normal((N, 512), dtype=np.float32)).to(DEV)[:, :K]
    src = np.full(Kpad, -1, dtype=np.int32)
    rep = np.zeros(Kpad, dtype=np.int32)
    src[:K] = np.arange(K)
    rep[:K] = rng.integers(1, 4, K)
    src[16:32] = src[16:32][::-1]
    src[50], rep[70], rep[100], rep[101] = -1, 0, 256, 100000
    tail = np.arange(K + 3, Kpad - 20)
    src[tail] = rng.integers(0, K, tail.size)
    rep[tail] = rng.integers(1, 5, tail.size)
    src[tail[7]] = K + 5
    _compare(X, src, rep, W, bits, scalar(3.0) if static else None, torch.float16, None)


@pytest.mark.parametrize("M,N,bits", [(1, 300, 8), (1, 9000, 4), (16, 5000, 4), (70, 4000, 8), (500, 1000, 6)])
def test_replayed_from_a_graph(M, N, bits):
    """The kernels for few rows and few tiles inside a captured graph, replayed between eager work on other data."""
    rng = np.random.default_rng(M)
    K = 1024
    X = _x(rng, M, K, "bf16").contiguous()
    W = torch.from_numpy(rng.standard_normal((N, K), dtype=np.float32)).to(DEV).to(torch.bfloat16)
    layer = fq.FqLinear(W, X.float().abs().amax(dim=0).cpu().numpy(), 4.0, bits, device=DEV)
    Y = torch.zeros((M, N), dtype=torch.bfloat16, device=DEV)
    layer.forward(X, Y)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        layer.forward(X, Y)
    for _ in range(3):
        X.copy_(_x(rng, M, K, "bf16"))
        want = layer.forward(X).clone()
        Y.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("bits", [8, 4, 6])
@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("where", ["X", "second half of X", "map", "copy counts", "bound"])
def test_output_in_the_memory_of_an_input(where, static, bits):
    """Y may take the place of what only the quantizer reads (a row updated in place): the result is that of a Y apart."""
    rng = np.random.default_rng(bits)
    K = N = 5120
    X = _x(rng, 1, K, "bf16").contiguous()
    W = torch.from_numpy(rng.standard_normal((N, K), dtype=np.float32)).to(DEV).to(torch.bfloat16)
    layer = fq.FqLinear(W, X.float().abs().amax(dim=0).cpu().numpy(), 4.0, bits, device=DEV)
    bound = torch.full((N,), 4.0, dtype=torch.float32, device=DEV)
    absmax = bound[:1] if static or where == "bound" else None
    want = layer.forward(X, absmax_in=absmax)
    room = {"X": X.view(-1), "second half of X": torch.cat([X.view(-1), X.view(-1)]), "map": layer.src.view(torch.bfloat16),
            "copy counts": layer.rep.view(torch.bfloat16), "bound": bound.view(torch.bfloat16)}[where]
    if where == "second half of X":
        X, Y = room[:K].view(1, K), room[K // 2:K // 2 + N].view(1, N)
    else:
        Y = room[:N].view(1, N)
    layer.forward(X, Y, absmax_in=absmax)
    assert torch.equal(Y.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_what_is_not_finite(value, bits):
    """The accumulators of both forms for a row with an element that is not finite, static scale: padding slots add nothing,
    whatever the weights hold there."""
    rng = np.random.default_rng(3)
    K, N, Kpad = 500, 100, 1024
    X = _x(rng, 1, K, "f32")
    X[0, 0] = value
    src = np.full(Kpad, -1, dtype=np.int32)
    rep = np.zeros(Kpad, dtype=np.int32)
    src[:K], rep[:K] = np.arange(K), 1
    src[K:K + 300:7], rep[K:K + 300:7] = 3, 2                              # single copies among padding
    Wq = torch.randint(-128, 128, (N, Kpad if bits == 8 else Kpad // 2), dtype=torch.int8, device=DEV)
    ws = bytes_ws(fq.fq_linear_workspace_bytes(1, K, Kpad, bits))
    out = []
    for variant in (-1, 2):
        Y = torch.zeros((1, N), dtype=torch.int32, device=DEV)
        fq.fq_gemm_select(variant)
        try:
            fq.fq_linear(X, dev_i32(src), dev_i32(rep), Wq, scalar(1.0), bits, Y, ws, absmax_in=scalar(3.0))
        finally:
            fq.fq_gemm_select(-1)
        out.append(Y)
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("bits,K", [(8, 5000), (4, 70000), (8, 300000)])
def test_fewer_slots_than_channels(bits, K, static):
    """A map that drops most channels, the last one among those it reads."""
    rng = np.random.default_rng(K)
    Kpad, N = 256, 70
    X = _x(rng, 1, K, "bf16")
    W = torch.from_numpy(rng.standard_normal((N, (K + 15) // 16 * 16), dtype=np.float32)).to(DEV).to(torch.bfloat16)[:, :K]
    src = rng.integers(0, K, Kpad).astype(np.int32)
    src[:4], src[-3:] = [0, 1, K - 1, K - 1], -1
    rep = np.where(src >= 0, rng.integers(1, 4, Kpad), 0).astype(np.int32)
    _compare(X, src, rep, W, bits, scalar(2.0) if static else None, torch.float32, None)
