"""The quantizer's rounding and packing on every half-way point and clamp, through each kernel that quantizes: few rows, many
rows, one row ahead of the product, and layers whose row fills the LDS budget."""
import numpy as np
import pytest
import torch

import paper_2402_17985_amd as fq
from oracle import fq_oracle as O
from tests.gpu_util import DEV, bytes_ws, dev_i32, scalar

pytestmark = pytest.mark.gpu


def _packed(q, bits):
    return q.view(np.uint8) if bits == 8 else O.pack_i4(q) if bits == 4 else O.pack_e3m2_blocked(q)


def _halves(M, K, bits):
    """Multiples of 1/2 beyond both clamps, their fp32 neighbours and signed zeros; multiplier 1."""
    top = 140 if bits == 8 else 10
    v = np.arange(-2 * top, 2 * top + 1, dtype=np.float32) / np.float32(2)
    v = np.concatenate([v, np.nextafter(v, np.float32(np.inf)), np.nextafter(v, np.float32(-np.inf)), np.array([0.0, -0.0], np.float32)])
    return np.resize(np.concatenate([v, v[::-1]]), (M, K)).astype(np.float32)


@pytest.mark.parametrize("bits", [8, 4, 6])
@pytest.mark.parametrize("M,K", [(3, 1024), (300, 2048), (5, 32752), (3, 65536), (800, 16400)])
def test_ties_and_clamps(M, K, bits):
    qmax = 127 if bits == 8 else 7
    Kpad = (K + 255) // 256 * 256
    src, rep = np.full(Kpad, -1, np.int32), np.zeros(Kpad, np.int32)
    src[:K], rep[:K] = np.arange(K), 1
    X = _halves(M, K, bits)
    want = np.zeros((M, Kpad), np.int8)
    want[:, :K] = np.clip(np.rint(X), -qmax - 1, qmax)
    out = torch.full((Kpad // 128, M, 96) if bits == 6 else (M, Kpad if bits == 8 else Kpad // 2), 0x55, dtype=torch.uint8, device=DEV)
    s_x = torch.zeros(1, device=DEV)
    fq.fq_flatten_quant_act(torch.from_numpy(X).to(DEV), dev_i32(src), dev_i32(rep), bits, out, s_x,
                            bytes_ws(fq.fq_act_workspace_bytes(K, Kpad)), absmax_in=scalar(float(qmax)))
    np.testing.assert_array_equal(out.cpu().numpy().reshape(-1), _packed(want, bits).reshape(-1))


@pytest.mark.parametrize("bits", [8, 4, 6])
def test_ties_and_clamps_in_the_one_row_layer(bits):
    """Weights that select one slot each: the accumulators are the quantized row."""
    K = N = 256
    qmax = 127 if bits == 8 else 7
    src, rep = np.arange(K, dtype=np.int32), np.ones(K, np.int32)
    eye = np.eye(N, K, dtype=np.int8)
    Wq = torch.from_numpy(_packed(eye, bits)).to(DEV)
    for row in _halves(8, K, bits):
        Y = torch.empty((1, N), device=DEV)
        fq.fq_linear(torch.from_numpy(row).view(1, K).to(DEV), dev_i32(src), dev_i32(rep), Wq.view(torch.int8) if bits == 8 else Wq, scalar(1.0), bits,
                     Y, bytes_ws(fq.fq_linear_workspace_bytes(1, K, K, bits)), absmax_in=scalar(float(qmax)))
        np.testing.assert_array_equal(Y.cpu().numpy()[0], np.clip(np.rint(row), -qmax - 1, qmax) + np.float32(0))
