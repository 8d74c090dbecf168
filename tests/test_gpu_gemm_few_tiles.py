"""The GEMM kernels for few rows and few output tiles: every kernel and tile of the dispatch, at the edges of its rows,
columns, k-steps and waves.  Accumulators against the exact product; every output type bit for bit against the tiled
kernels, which the other tests hold to the oracle."""
import numpy as np
import pytest
import torch

import paper_2402_17985_amd as fq
from oracle import fq_oracle as O
from tests.gpu_util import DEV, scalar

pytestmark = pytest.mark.gpu


def _operand(rng, rows, K, bits):
    """(integer values, the same in storage) on the device."""
    lo, hi = (-128, 128) if bits == 8 else (-8, 8)
    q = rng.integers(lo, hi, (rows, K), dtype=np.int8)
    store = q if bits == 8 else O.pack_i4(q) if bits == 4 else O.pack_e3m2_blocked(q)
    return torch.from_numpy(q).to(DEV), torch.from_numpy(np.ascontiguousarray(store)).to(DEV)


def _gemm(bits, X, W, s_x, s_w, bias, Y):
    if bits == 8:
        fq.fq_gemm_i8_bias(X, W, s_x, s_w, bias, Y)
    elif bits == 4:
        fq.fq_gemm_i4_bias(X, W, s_x, s_w, bias, Y)
    else:
        fq.fq_gemm_i4_e3m2(X, W, s_x, s_w, bias, Y)


# (M, N): what 256 CUs make of it
SHAPES = [
    (1, 40), (3, 4100), (4, 9001), (16, 300), (16, 9000), (16, 16380),     # rows streamed into registers (16: 4-bit values)
    (5, 37), (33, 1000), (64, 4096),                                       # 32 x 32
    (32, 11008), (100, 2001),                                              # 32 x 64
    (130, 4000), (63, 16384), (8200, 20),                                  # 64 x 64
    (20, 20000),                                                           # 32 x 128
    (96, 16000), (90, 16001),                                              # 96 x 64
    (128, 16000), (125, 15999),                                            # 128 x 64
    (60, 30000),                                                           # 64 x 128
    (300, 10000), (257, 9999),                                             # 128 x 128
]


@pytest.mark.parametrize("bits,K", [(8, 32), (8, 128), (8, 1056), (8, 2080), (4, 32), (4, 256), (4, 2144), (6, 128), (6, 1152)])
@pytest.mark.parametrize("M,N", SHAPES)
def test_accumulators(M, N, bits, K):
    rng = np.random.default_rng(M + N + K)
    xq, X = _operand(rng, M, K, bits)
    wq, W = _operand(rng, N, K, bits)
    Y = torch.full((M, N), 0x55555555, dtype=torch.int32, device=DEV)
    _gemm(bits, X, W, None, None, None, Y)
    assert torch.equal(Y.double(), xq.double() @ wq.double().t().contiguous())


@pytest.mark.parametrize("bits", [8, 4, 6])
@pytest.mark.parametrize("ydt", [torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("M,N,pad", [(2, 130, 0), (2, 131, 2), (16, 9002, 6), (40, 333, 3), (70, 4096, 0), (128, 16000, 0), (300, 9999, 1)])
def test_output_types_and_strides(M, N, pad, ydt, bits):
    rng = np.random.default_rng(N)
    _, X = _operand(rng, M, 1152, bits)
    _, W = _operand(rng, N, 1152, bits)
    bias = torch.from_numpy(rng.standard_normal(N, dtype=np.float32)).to(DEV)
    for b in (None, bias):
        got = torch.full((M, N + pad), 7.0, dtype=ydt, device=DEV)
        want = got.clone()
        _gemm(bits, X, W, scalar(0.013), scalar(0.0021), b, got[:, :N])
        fq.fq_gemm_select(2)
        try:
            _gemm(bits, X, W, scalar(0.013), scalar(0.0021), b, want[:, :N])
        finally:
            fq.fq_gemm_select(-1)
        kind = torch.int32 if ydt == torch.float32 else torch.int16
        assert torch.equal(got.view(kind), want.view(kind))          # the padding columns stay untouched as well


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("batch,M,N,K", [(3, 40, 70, 1024), (160, 1, 128, 2048), (7, 4, 33, 1056), (12, 65, 130, 1024), (2, 1000, 1000, 1024)])
def test_batched(batch, M, N, K, bits):
    rng = np.random.default_rng(batch)
    xq, X = _operand(rng, batch * M, K, bits)
    wq, W = _operand(rng, batch * N, K, bits)
    Y = torch.full((batch, M, N), -1, dtype=torch.int32, device=DEV)
    (fq.fq_bmm_i8 if bits == 8 else fq.fq_bmm_i4)(X.view(batch, M, -1), W.view(batch, N, -1), None, None, Y)
    want = torch.bmm(xq.view(batch, M, K).double(), wq.view(batch, N, K).double().transpose(1, 2).contiguous())
    assert torch.equal(Y.double(), want)


# Outputs of the tiled kernels whose rows start at any element or that end inside a tile.  (variant, storage): 2 stores from
# the accumulator layout and is the reference; the others stage rows through LDS.
@pytest.mark.parametrize("ydt", [torch.int32, torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("variant,bits,K", [(6, 8, 256), (6, 4, 96), (7, 8, 160), (10, 4, 1024), (11, 8, 256), (12, 8, 384), (12, 4, 512), (6, 6, 256)])
@pytest.mark.parametrize("M,N,pad,shift", [(256, 256, 0, 0), (257, 255, 0, 0), (511, 513, 3, 0), (130, 1001, 0, 8), (300, 264, 8, 0), (128, 640, 64, 4)])
def test_ragged_outputs_of_the_tiled_kernels(M, N, pad, shift, variant, bits, K, ydt):
    rng = np.random.default_rng(M * N)
    _, X = _operand(rng, M, K, bits)
    _, W = _operand(rng, N, K, bits)
    kind = torch.int16 if ydt in (torch.float16, torch.bfloat16) else torch.int32
    for bias in (None,) if ydt == torch.int32 else (None, torch.from_numpy(rng.standard_normal(N, dtype=np.float32)).to(DEV)):
        out = []
        for v in (variant, 2 if bits != 6 else -1):
            buf = torch.full((M * (N + pad) + 2 * shift,), 7, dtype=ydt, device=DEV)     # shift: Y not on a cache line
            Y = buf[shift:shift + M * (N + pad)].view(M, N + pad)[:, :N]
            fq.fq_gemm_select(v)
            try:
                _gemm(bits, X, W, scalar(0.013), scalar(0.0021), bias, Y)
            finally:
                fq.fq_gemm_select(-1)
            out.append(buf)
        assert torch.equal(out[0].view(kind), out[1].view(kind))                         # nothing outside Y is touched


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("batch,M,N,K", [(5, 333, 150, 64), (3, 700, 701, 96), (150, 1, 300, 128), (9, 256, 129, 1024)])
def test_batched_tiles_and_their_order(batch, M, N, K, bits):
    rng = np.random.default_rng(M)
    xq, X = _operand(rng, batch * M, K, bits)
    wq, W = _operand(rng, batch * N, K, bits)
    Y = torch.full((batch, M, N), -1, dtype=torch.int32, device=DEV)
    (fq.fq_bmm_i8 if bits == 8 else fq.fq_bmm_i4)(X.view(batch, M, -1), W.view(batch, N, -1), None, None, Y)
    want = torch.bmm(xq.view(batch, M, K).double(), wq.view(batch, N, K).double().transpose(1, 2).contiguous())
    assert torch.equal(Y.double(), want)


def _device_operand(g, rows, K, bits):
    """(integer values as float64, the same in storage), made on the device: long reductions of many columns."""
    lo, hi = (-128, 128) if bits == 8 else (-8, 8)
    q = torch.randint(lo, hi, (rows, K), dtype=torch.int8, device=DEV, generator=g)
    if bits == 8:
        return q.double(), q
    if bits == 4:
        return q.double(), ((q[:, 0::2] & 15) | ((q[:, 1::2] & 15) << 4)).view(torch.uint8)
    # the quantizer with an identity map and the bound 7 multiplies by one: it stores these integers' codes
    codes, s = torch.empty((K // 128, rows, 96), dtype=torch.uint8, device=DEV), torch.empty(1, dtype=torch.float32, device=DEV)
    src, rep = torch.arange(K, dtype=torch.int32, device=DEV), torch.ones(K, dtype=torch.int32, device=DEV)
    ws = torch.empty(fq.fq_act_workspace_bytes(K, K), dtype=torch.uint8, device=DEV)
    fq.fq_flatten_quant_act(q.float(), src, rep, 6, codes, s, ws, absmax_in=scalar(7.0))
    return q.double(), codes


# Reductions long enough for every wave's main loop to reuse its registers or its stages: the weight-streaming kernel reloads
# a register slot from five k-steps per wave on (40 steps of 128 bytes, 96 in E3M2, with eight waves, 20 with four), the
# split-reduction kernels refill a buffer from 17 stages on at most, the ring from seven.  Lengths that give the waves four
# and five steps, six and seven, and more, the last step partial.
@pytest.mark.parametrize("bits,K", [(8, 4128), (8, 6304), (8, 12576), (4, 8256), (4, 12576), (4, 22048), (6, 4224), (6, 6400), (6, 9088)])
@pytest.mark.parametrize("M,N", [(1, 300), (4, 9001), (3, 20000), (16, 300), (16, 5000), (16, 16380),             # rows into registers
                                 (33, 1000), (32, 11008), (130, 4000), (20, 20000), (90, 16001),                  # split over waves
                                 (125, 15999), (60, 30000), (257, 9999)])                                         # the same, or the ring
def test_long_reductions(M, N, bits, K):
    g = torch.Generator(device=DEV).manual_seed(M + N + K)
    xq, X = _device_operand(g, M, K, bits)
    wq, W = _device_operand(g, N, K, bits)
    Y = torch.full((M, N), 0x55555555, dtype=torch.int32, device=DEV)
    _gemm(bits, X, W, None, None, None, Y)
    assert torch.equal(Y.double(), xq @ wq.t().contiguous())


# Batched: problems dealt to the XCDs in bands, with one tile each and with several, reductions that refill the buffers
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("batch,M,N,K", [(9, 60, 60, 4192), (7, 100, 200, 4192), (40, 250, 128, 2112), (12, 250, 500, 2112), (13, 65, 129, 1088),
                                         (3, 700, 701, 1088), (20, 40, 1500, 2624), (40, 768, 128, 1088)])
def test_batched_long_reductions(batch, M, N, K, bits):
    g = torch.Generator(device=DEV).manual_seed(M + N)
    xq, X = _device_operand(g, batch * M, K, bits)
    wq, W = _device_operand(g, batch * N, K, bits)
    Y = torch.full((batch, M, N), -1, dtype=torch.int32, device=DEV)
    (fq.fq_bmm_i8 if bits == 8 else fq.fq_bmm_i4)(X.view(batch, M, -1), W.view(batch, N, -1), None, None, Y)
    assert torch.equal(Y.double(), torch.bmm(xq.view(batch, M, K), wq.view(batch, N, K).transpose(1, 2).contiguous()))
