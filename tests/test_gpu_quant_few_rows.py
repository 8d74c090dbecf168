"""The quantizer of few rows, whose workgroups with a dynamic scale may each take the maximum of all of X: every number of rows that is
left over by the rounds of rows, heads whose last group is ragged, and gathered groups, against the CPU oracle, byte for byte."""
import numpy as np
import pytest

import paper_2402_17985_amd as fq
from tests.test_gpu_quant_direct import _check

pytestmark = pytest.mark.gpu


def _layer(M, K, at, copies=3):
    """Rows whose largest element (over copies) lies at (row, channel) `at`, and a plan with a few copied channels."""
    rng = np.random.default_rng(M + K)
    X = rng.uniform(-1.0, 1.0, (M, K)).astype(np.float32)
    chmax = np.ones(K, dtype=np.float32)
    chmax[[K // 3, K // 2]] = [copies, 2]
    X[:, K // 3] *= copies
    X[at] = -3.25
    src, rep, _, _ = fq.fq_flatten_plan(chmax, 1.0, 128)
    return X, src, rep


# One set of threads for the head and several, one head group per thread and two
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("last", [False, True])
@pytest.mark.parametrize("dtype,M,K", [(d, M, K) for d in ("bf16", "f32") for M, K in
                                       ((1, 256), (2, 256), (5, 256), (9, 256), (13, 1024), (17, 256), (1, 4096), (3, 4096), (5, 4096), (1, 20480), (2, 16400), (3, 20480))])
def test_every_number_of_rows(dtype, M, K, last, bits):
    X, src, rep = _layer(M, K, (M - 1, K - 1) if last else (M // 2, 0))
    _check(X, dtype, src, rep, bits, None)


# The last group gathered from global memory: the maximum in it or before it, with further groups of that kind and without
@pytest.mark.parametrize("bits", [8, 4, 6])
@pytest.mark.parametrize("where", ["ragged", "head", "gathered"])
@pytest.mark.parametrize("dtype,M,K", [("bf16", 1, 20), ("f32", 7, 300), ("bf16", 64, 1000), ("f16", 8, 2500), ("f32", 20, 2500), ("bf16", 5, 16405), ("f32", 2, 20490)])
def test_ragged_heads(dtype, M, K, where, bits):
    X, src, rep = _layer(M, K, (M - 1, {"ragged": K - 1, "head": 0, "gathered": 14}[where]))
    if where == "gathered":
        src[[14, 15]] = src[[15, 14]]
    _check(X, dtype, src, rep, bits, None)


# Two head groups per thread, gathered groups of which either half, or both, differ from a plain one
@pytest.mark.parametrize("bits", [8, 4, 6])
@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("dtype,M,K", [("bf16", 3, 16400), ("f32", 3, 20480), ("f16", 70, 20490), ("f32", 300, 17000)])
def test_gathered_groups_of_wide_layers(dtype, M, K, static, bits):
    X, src, rep = _layer(M, K, (M - 1, 9))
    for base in (0, K // 2 // 16 * 16, K // 16 * 16 - 16):
        src[base + 1], src[base + 2] = base + 2, base + 1
    src[128 + 13], rep[256 + 3], rep[256 + 12] = -1, 0, 300
    _check(X, dtype, src, rep, bits, 3.0 if static else None)


# fp32: two rows left over, alone and after a round of four, by one set of threads for the head and by several
@pytest.mark.parametrize("bits", [8, 4, 6])
@pytest.mark.parametrize("at", [0, 1, -2, -1])
@pytest.mark.parametrize("M,K", [(2, 4096), (6, 4096), (10, 5001), (12, 2048), (24, 1024), (6, 8200)])
def test_two_rows_left_over(M, K, at, bits):
    X, src, rep = _layer(M, K, (at % M, K // 3 + 1))
    _check(X, "f32", src, rep, bits, None)


# Groups to be gathered in every row of a strip: the one with the channels of a ragged head, and copies of those.  Fewer waves than batches
# of appended groups, as many, and more; strips of one to four rows, several per workgroup
@pytest.mark.parametrize("bits", [8, 4, 6])
@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("copies", [{2: 30}, {2: 200, 5: 240, 8: 120, -1: 40}, {2: 250, 3: 100, 9: 250, -2: 70, 4: 254, 5: 250, 6: 250, 7: 250, -1: 9}])
@pytest.mark.parametrize("dtype,M,K", [("f16", 1500, 1003), ("bf16", 4683, 639), ("bf16", 700, 2005), ("f16", 20011, 555), ("f32", 1501, 1003), ("bf16", 1030, 31)])
def test_gathered_groups_of_every_row(dtype, M, K, copies, static, bits):
    rng = np.random.default_rng(M)
    X = rng.uniform(-1.0, 1.0, (M, K)).astype(np.float32)
    count = np.ones(K, dtype=np.int32)
    for c, n in copies.items():
        count[c if c < 0 else c * K // 11] = n
    X *= count
    X[M - 1, K - 1] = -1.25 * count[K - 1]
    slots = np.concatenate([np.arange(K), np.repeat(np.arange(K), count - 1)]).astype(np.int32)
    Kpad = (len(slots) + 127) // 128 * 128
    src, rep = np.full(Kpad, -1, np.int32), np.zeros(Kpad, np.int32)
    src[:len(slots)], rep[:len(slots)] = slots, count[slots]
    _check(X, dtype, src, rep, bits, 1.0 if static else None)
