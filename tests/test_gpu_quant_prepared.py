"""The flatten-quantize call whose absmax pass prepares the map for the quantizer, against the CPU oracle, byte for byte: heads
and tails around the 512 slots of a workgroup, copy counts around what a byte holds, and maps that are not the planner's."""
import numpy as np
import pytest

import paper_2402_17985_amd as fq
from tests.test_gpu_quant_direct import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [8, 4, 6])
@pytest.mark.parametrize("dtype,M,K,copies", [("bf16", 70, 16, 3), ("f32", 66, 31, 20), ("bf16", 65, 496, 2), ("f16", 100, 512, 254), ("bf16", 80, 530, 255),
                                              ("f32", 300, 1024, 256), ("bf16", 90, 700, 3000), ("bf16", 600, 16416, 40)])
def test_planned_maps(dtype, M, K, copies, bits):
    rng = np.random.default_rng(K)
    X = rng.standard_normal((M, K), dtype=np.float32)
    chmax = np.ones(K, dtype=np.float32)
    chmax[[K // 3, K - 1]] = [copies, 2]
    X[:, K // 3] *= copies
    src, rep, _, _ = fq.fq_flatten_plan(chmax, 1.0, 128)
    _check(X, dtype, src, rep, bits, None)


@pytest.mark.parametrize("bits", [8, 4, 6])
@pytest.mark.parametrize("M,K,Kpad", [(65, 1000, 1024), (70, 1000, 2560), (300, 516, 1536)])
def test_maps_that_are_not_the_planners(M, K, Kpad, bits):
    rng = np.random.default_rng(Kpad)
    X = rng.standard_normal((M, K), dtype=np.float32) * np.float32(3.0)
    src = np.full(Kpad, -1, dtype=np.int32)
    rep = np.zeros(Kpad, dtype=np.int32)
    src[:K] = np.arange(K)
    rep[:K] = rng.integers(1, 4, K)
    src[16:32] = src[16:32][::-1]
    src[50], rep[70], rep[100], rep[101] = -1, 0, 256, 100000
    n = Kpad - K
    src[K:] = np.where(rng.random(n) < 0.9, rng.integers(0, K, n), K + 5)
    own = rep[np.minimum(src[K:], K - 1)]
    rep[K:] = np.where(rng.random(n) < 0.8, own, rng.integers(-1, 5, n))
    src[K + 8:K + 24], rep[K + 8:K + 24] = 100, 256
    _check(X, "bf16", src, rep, bits, None)
