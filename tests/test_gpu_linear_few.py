"""The one-kernel form of the layer for a few rows against the separate kernels (a forced GEMM variant selects them; the
other tests hold them to the oracle), bit for bit."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2402_17985_amd as fq
from tests.gpu_util import DEV, scalar
from tests.test_gpu_linear_decode import _compare, _x
from tests.test_launch_rules import rules  # noqa: F401  (the launch rules, compiled for the host)

pytestmark = pytest.mark.gpu


def _w(rng, N, K):
    return torch.from_numpy(rng.standard_normal((N, (K + 15) // 16 * 16), dtype=np.float32)).to(DEV).to(torch.bfloat16)[:, :K]


# One group, a ragged one, one and several sets of quantizing waves, a thread's last row (and one more), the widest head; columns
# of one to four fragments with ragged ends, and several rounds of all workgroups.
@pytest.mark.parametrize("bits", [8, 4, 6])
@pytest.mark.parametrize("scale", ["static", "dynamic", "zero"])
@pytest.mark.parametrize("dtype,M,K,N", [("bf16", 2, 16, 16), ("f32", 16, 31, 33), ("f16", 16, 256, 70), ("bf16", 15, 1000, 4097), ("f32", 3, 1040, 5119),
                                         ("f16", 16, 1024, 8200), ("bf16", 1, 4096, 40), ("bf16", 1, 5120, 5121), ("f32", 4, 4100, 300),
                                         ("bf16", 8, 4368, 12290), ("f16", 9, 4368, 100), ("bf16", 2, 8207, 16387), ("bf16", 5, 2064, 33000)])
def test_planned_maps(dtype, M, K, N, scale, bits):
    rng = np.random.default_rng(K + M)
    X, W, T = _x(rng, M, K, dtype), _w(rng, N, K), 4.0
    src, rep, _, _ = fq.fq_flatten_plan(X.float().abs().amax(dim=0).cpu().numpy(), T, 128 if bits == 6 else 32)
    if scale == "zero":
        X.zero_()
    static = scalar(T) if scale == "static" else None
    _compare(X, src, rep, W, bits, static, torch.bfloat16, None)
    _compare(X, src, rep, W, bits, static, torch.float32, torch.from_numpy(rng.standard_normal(N, dtype=np.float32)).to(DEV), pad=3)
    _compare(X, src, rep, W, bits, static, torch.int32, None)


def _plan(rules, M, N, K, Kpad, bits, dtype, dynamic):
    """(sets of quantizing waves, rows that a thread holds, fragments of 16 columns) of the kernel that the call takes; None: another."""
    out = (ctypes.c_longlong * 7)()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    if not rules.few_scaled(M, N, K, Kpad, bits, 4 if dtype == "f32" else 2, int(dynamic), cus, out):
        return None
    return out[1], -(-M // out[1]), out[3]


# The shapes above that this kernel leaves to the separate ones (E3M2 beyond 16384 elements, one row by the rule for one row) are
# comparisons of those with themselves; here every one is taken, and by the kernel that is named: one set of quantizing waves and
# several, as many rows per thread as its registers hold, one to four fragments, each storage and type.
@pytest.mark.parametrize("scale", ["static", "dynamic"])
@pytest.mark.parametrize("bits,dtype,M,K,N,want", [
    (b, "bf16", 2, 4096, 12800, (2, 1, 4)) for b in (8, 4, 6)] + [
    (b, "bf16", 2, 8192, 4100, (1, 2, 2)) for b in (8, 4, 6)] + [
    (b, "f32", 4, 4096, 8300, (2, 2, 3)) for b in (8, 4, 6)] + [
    (b, "f16", 16, 1024, 12300, (8, 2, 4)) for b in (8, 4, 6)] + [
    (b, "bf16", 16, 4096, 11008, (2, 8, 3)) for b in (8, 4)] + [
    (b, "bf16", 16, 4096, 40, (2, 8, 1)) for b in (8, 4)] + [
    (b, "f16", 8, 8192, 8000, (1, 8, 2)) for b in (8, 4)] + [
    (b, "f32", 16, 2048, 12800, (4, 4, 4)) for b in (8, 4)] + [
    (b, "f32", 4, 8192, 8300, (1, 4, 3)) for b in (8, 4)] + [
    (6, "f32", 2, 8192, 12300, (1, 2, 4)), (6, "bf16", 8, 2048, 8300, (4, 2, 3)), (6, "bf16", 1, 8192, 1000, (1, 1, 1)), (6, "f32", 16, 1008, 5000, (8, 2, 2))])
def test_kernels_that_calls_take(rules, bits, dtype, M, K, N, want, scale):  # noqa: F811
    rng = np.random.default_rng(K + M)
    X, W, T = _x(rng, M, K, dtype), _w(rng, N, K), 4.0
    src, rep, _, _ = fq.fq_flatten_plan(X.float().abs().amax(dim=0).cpu().numpy(), T, 128 if bits == 6 else 32)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert _plan(rules, M, N, K, len(src), bits, dtype, scale == "dynamic") == want
    _compare(X, src, rep, W, bits, scalar(T) if scale == "static" else None, torch.bfloat16, None)


@pytest.mark.parametrize("bits", [8, 4, 6])
@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("copies", [254, 255, 256, 700])
def test_many_copies(copies, static, bits):
    """Channels of about as many copies as the table of multipliers and the byte counts hold."""
    rng = np.random.default_rng(copies)
    M, K, N = 7, 400, 100
    X, W = _x(rng, M, K, "bf16"), _w(rng, N, K)
    chmax = np.ones(K, dtype=np.float32)
    chmax[[3, 200, 399]] = [copies, copies, 2]
    X[:, 3] *= copies
    src, rep, _, _ = fq.fq_flatten_plan(chmax, 1.0, 128)
    assert rep[3] == copies
    _compare(X, src, rep, W, bits, scalar(3.0) if static else None, torch.float32, None)


@pytest.mark.parametrize("bits", [8, 4, 6])
@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("Kpad", [512, 1152, 8320])
def test_maps_that_are_not_the_planners(Kpad, static, bits):
    rng = np.random.default_rng(Kpad)
    M, K, N = 6, 500, 100
    X, W = _x(rng, M, K, "f32"), _w(rng, N, K)
    src = np.full(Kpad, -1, dtype=np.int32)
    rep = np.zeros(Kpad, dtype=np.int32)
    src[:K] = np.arange(K)
    rep[:K] = rng.integers(1, 4, K)
    src[16:32] = src[16:32][::-1]
    src[50], rep[70], rep[100], rep[101] = -1, 0, 256, 100000
    if Kpad > K + 30:
        tail = np.arange(K + 3, Kpad - 20)
        src[tail] = rng.integers(0, K, tail.size)
        rep[tail] = np.where(rng.random(tail.size) < 0.5, rep[src[tail]], rng.integers(-1, 5, tail.size))
        src[tail[7]], src[tail[400]] = K + 5, 100
        rep[tail[400]] = 256
    _compare(X, src, rep, W, bits, scalar(3.0) if static else None, torch.float16, None)


@pytest.mark.parametrize("static", [False, True])
def test_fewer_slots_than_channels(static):
    rng = np.random.default_rng(2)
    M, K, N, Kpad = 4, 1000, 70, 256
    X, W = _x(rng, M, K, "bf16"), _w(rng, N, K)
    src = rng.integers(0, K, Kpad).astype(np.int32)
    rep = rng.integers(1, 4, Kpad).astype(np.int32)
    _compare(X, src, rep, W, 8, scalar(2.0) if static else None, torch.float32, None)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("bits", [8, 4, 6])
@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_what_is_not_finite(value, static, bits, dtype):
    rng = np.random.default_rng(3)
    M, K, N = 5, 500, 100
    X, W = _x(rng, M, K, dtype), _w(rng, N, K)
    src, rep, _, _ = fq.fq_flatten_plan(X.float().abs().amax(dim=0).cpu().numpy(), 4.0, 128 if bits == 6 else 32)
    X[2, 7] = value
    _compare(X, src, rep, W, bits, scalar(3.0) if static else None, torch.int32, None)


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("where", ["X", "second row of X", "map"])
def test_output_in_the_memory_of_an_input(where, bits):
    """Y may take the place of what only the quantizer reads: the result is that of a Y apart."""
    rng = np.random.default_rng(bits)
    M, K = 4, 2048
    N = {"X": K, "second row of X": K, "map": 1024}[where]
    room = torch.cat([_x(rng, M, K, "bf16").contiguous().view(-1), torch.zeros(M * K, dtype=torch.bfloat16, device=DEV)])
    X = room[:M * K].view(M, K)
    layer = fq.FqLinear(_w(rng, N, K), X.float().abs().amax(dim=0).cpu().numpy(), 4.0, bits, device=DEV)
    want = layer.forward(X)
    Y = {"X": X, "second row of X": room[K:K + M * N].view(M, N) if N == K else None, "map": layer.src.view(torch.bfloat16)[:M * N].view(M, N) if N < K else None}[where]
    layer.forward(X, Y)
    assert torch.equal(Y.view(torch.int16), want.view(torch.int16))


# One row of 4-bit values beyond 64 columns per compute unit, whatever its length: short, ragged, with a partial last round of columns
@pytest.mark.parametrize("bits", [4, 6])
@pytest.mark.parametrize("scale", ["static", "dynamic"])
@pytest.mark.parametrize("dtype,K,N", [("bf16", 16, 16400), ("f32", 31, 17001), ("f16", 257, 24576), ("bf16", 1007, 33001), ("f32", 2005, 20480), ("bf16", 1024, 16385)])
def test_one_row_of_many_columns(dtype, K, N, scale, bits):
    rng = np.random.default_rng(K)
    X, W, T = _x(rng, 1, K, dtype), _w(rng, N, K), 4.0
    src, rep, _, _ = fq.fq_flatten_plan(X.float().abs().amax(dim=0).cpu().numpy(), T, 128 if bits == 6 else 32)
    static = scalar(T) if scale == "static" else None
    _compare(X, src, rep, W, bits, static, torch.bfloat16, None)
    _compare(X, src, rep, W, bits, static, torch.float32, torch.from_numpy(rng.standard_normal(N, dtype=np.float32)).to(DEV), pad=3)


# Weight rows of 4, 8 and 16 KiB, whose workgroups begin at different steps of the reduction, and of 12 KiB; several rounds of columns
@pytest.mark.parametrize("scale", ["static", "dynamic"])
@pytest.mark.parametrize("bits,dtype,M,K,Kpad,N", [
    (8, "bf16", 1, 8192, 8192, 8192), (8, "f16", 8, 8192, 8192, 4100), (8, "bf16", 2, 4096, 4096, 16500), (8, "f32", 3, 3001, 4096, 5000),
    (8, "bf16", 1, 8000, 12288, 24576), (4, "bf16", 1, 8192, 8192, 8192), (4, "f16", 16, 4000, 8192, 12300), (4, "bf16", 2, 8192, 16384, 20000),
    (8, "f32", 4, 8190, 8192, 33), (8, "bf16", 2, 8192, 16384, 8200)])
def test_rows_of_whole_4_kib(bits, dtype, M, K, Kpad, N, scale):
    rng = np.random.default_rng(Kpad + N)
    X, W = _x(rng, M, K, dtype), _w(rng, N, K)
    src, rep = np.full(Kpad, -1, np.int32), np.zeros(Kpad, np.int32)
    src[:K], rep[:K] = np.arange(K), 1
    more = (Kpad - K) // 2                                     # a second copy of the first channels, the rest padding
    src[K:K + more], rep[K:K + more], rep[:more] = np.arange(more), 2, 2
    _compare(X, src, rep, W, bits, scalar(4.0) if scale == "static" else None, torch.int32, None)
