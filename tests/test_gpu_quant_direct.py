"""The flatten-quantize call on both sides of its dispatch rules, against the CPU oracle, byte for byte: the one-kernel
form for few rows (one or two head groups per thread; a' static, read by every workgroup, or from the candidates of the
absmax kernel) and the prepared form, with maps from the planner and maps that are not."""
import numpy as np
import pytest
import torch

import fq_workloads as WL
import paper_2402_17985_amd as fq
from oracle import fq_oracle as O
from tests.gpu_util import DEV, bytes_ws, dev_i32, scalar, to_dev

pytestmark = pytest.mark.gpu


def _packed(q, bits):
    return q.view(np.uint8) if bits == 8 else O.pack_i4(q) if bits == 4 else O.pack_e3m2_blocked(q)


def _padded(X, dtype):
    """Device tensor whose rows start on 16-byte boundaries, and the values it holds."""
    store, Xf = WL.round_to_dtype(X, dtype)
    M, K = X.shape
    buf = to_dev(np.pad(store, ((0, 0), (0, -K % 16))), dtype)
    return buf[:, :K], Xf


def _check(X, dtype, src, rep, bits, static, rep_offset=0):
    Xd, Xf = _padded(X, dtype)
    M, K = X.shape
    Kpad = len(src)
    valid = (src >= 0) & (src < K) & (rep > 0)                            # every other slot holds 0: padding to the oracle
    osrc, orep = np.where(valid, src, -1).astype(np.int32), np.where(valid, rep, 0).astype(np.int32)
    a = np.float32(static) if static else O.act_absmax_dynamic(Xf, osrc, orep)
    want, s_ref = O.flatten_quant_act(Xf, osrc, orep, bits if bits == 8 else 4, a)
    shape = (Kpad // 128, M, 96) if bits == 6 else (M, Kpad if bits == 8 else Kpad // 2)
    out = torch.full(shape, 0x55, dtype=torch.uint8, device=DEV)
    s_x = torch.zeros(1, dtype=torch.float32, device=DEV)
    rep_d = dev_i32(np.concatenate([np.zeros(rep_offset, np.int32), rep]))[rep_offset:]
    fq.fq_flatten_quant_act(Xd, dev_i32(src), rep_d, bits, out, s_x, bytes_ws(fq.fq_act_workspace_bytes(K, Kpad)),
                            absmax_in=scalar(static) if static else None)
    torch.cuda.synchronize()
    assert np.float32(s_x.item()) == s_ref
    np.testing.assert_array_equal(out.cpu().numpy().reshape(-1), _packed(want, bits).reshape(-1))


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("dtype,M,K,bits", [
    ("f32", 1, 16, 8), ("bf16", 3, 20, 4), ("f32", 5, 257, 6),            # narrow and ragged
    ("bf16", 64, 1000, 8), ("bf16", 65, 1000, 8),                         # a' read by every workgroup / candidates
    ("f16", 33, 4104, 4), ("bf16", 31, 4096, 6), ("f32", 16, 4096, 8),
    ("bf16", 1, 16384, 8), ("bf16", 5, 16400, 4), ("f32", 3, 22016, 6),   # one head group per thread, and two
    ("bf16", 768, 16384, 4), ("bf16", 769, 16384, 4),                     # last of the direct form, first of the other
    ("bf16", 700, 1024, 8), ("f32", 1500, 272, 4), ("bf16", 2, 33000, 8), # strips of several rows; too wide for it
])
def test_planned_maps(dtype, M, K, bits, static):
    rng = np.random.default_rng(K + M)
    X = rng.standard_normal((M, K), dtype=np.float32)
    out = rng.choice(K, max(1, K // 100), replace=False)
    X[:, out] *= np.float32(40.0)
    X[:, out[0]] *= np.float32(30.0)                                      # one channel with several hundred copies
    chmax = np.abs(WL.round_to_dtype(X, dtype)[1]).max(axis=0).astype(np.float32)
    T = float(np.float32(3.0 * np.median(chmax)))
    src, rep, _, _ = fq.fq_flatten_plan(chmax, T, 128 if bits == 6 else 32)
    _check(X, dtype, src, rep, bits, T if static else None)


# More elements than the one-kernel form takes, the last strip short: strips of four rows, and of two rows and one on both
# sides of the LDS size from which 512 threads walk them
@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("dtype,M,K,bits", [
    ("bf16", 1055, 12000, 8), ("bf16", 745, 17000, 4), ("bf16", 285, 45000, 8), ("bf16", 621, 20480, 4), ("bf16", 621, 20480, 8), ("f32", 603, 21000, 8), ("f16", 421, 30016, 4),
])
def test_wide_strips(dtype, M, K, bits, static):
    test_planned_maps(dtype, M, K, bits, static)


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("bits", [8, 4, 6])
@pytest.mark.parametrize("M,K", [(9, 200), (40, 4000), (200, 1200)])
def test_maps_that_are_not_the_planners(M, K, bits, static):
    rng = np.random.default_rng(M)
    X = (rng.standard_normal((M, K)) * rng.choice([1, 1, 10], K)).astype(np.float32)
    Kpad = (K + 512 + 127) // 128 * 128
    src = np.full(Kpad, -1, dtype=np.int32)
    rep = np.zeros(Kpad, dtype=np.int32)
    src[:K] = np.arange(K)
    rep[:K] = rng.integers(1, 4, K)
    src[16:32] = src[16:32][::-1]                                         # a head group that is a permutation
    src[50] = -1                                                          # a hole in the head
    rep[70] = 0                                                           # a head slot without copies
    rep[100] = 256                                                        # copy counts beyond a byte
    rep[101] = 100000
    tail = np.arange(K + 3, Kpad - 20)
    src[tail] = rng.integers(0, K, tail.size)
    rep[tail] = rep[src[tail]]
    rep[tail[::5]] += 1                                                   # not the channel's own copy count
    src[tail[7]] = K + 5                                                  # out of range
    _check(X, "f32", src, rep, bits, 3.0 if static else None, rep_offset=1)   # rep 4-byte aligned only
    _check(np.zeros_like(X), "f32", src, rep, bits, None)


@pytest.mark.parametrize("bits", [8, 4, 6])
@pytest.mark.parametrize("N,K", [(1, 16), (40, 1000), (300, 16400), (769, 16384)])
def test_weights(N, K, bits):
    """a' of the weights is their absmax over all channels, also those the map does not read."""
    rng = np.random.default_rng(N)
    W, Wf = _padded(rng.standard_normal((N, K), dtype=np.float32), "bf16")
    Kpad = (K + 200 + 127) // 128 * 128
    src = np.full(Kpad, -1, dtype=np.int32)
    src[:K] = np.arange(K)
    j = int(np.abs(Wf).max(axis=0).argmax())
    src[j] = -1                                                           # the largest channel is not read
    src[K:K + 150] = rng.integers(0, K, 150)
    want, s_ref = O.flatten_weights(Wf, src, bits if bits == 8 else 4)
    out = torch.full(((Kpad // 128, N, 96) if bits == 6 else (N, Kpad if bits == 8 else Kpad // 2)), 0x55, dtype=torch.uint8, device=DEV)
    s_w = torch.zeros(1, dtype=torch.float32, device=DEV)
    fq.fq_flatten_weights(W, dev_i32(src), bits, out, s_w, bytes_ws(fq.fq_weights_workspace_bytes(K, Kpad)))
    torch.cuda.synchronize()
    assert np.float32(s_w.item()) == s_ref
    np.testing.assert_array_equal(out.cpu().numpy().reshape(-1), _packed(want, bits).reshape(-1))


# A map that drops channels has fewer slots than X has columns: no kernel may look a channel's own slot up beyond its end.
# (Kpad, K): slots and columns, up to 4 MiB of map apart.
@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("dtype,M,K,Kpad,bits", [("f32", 5, 40, 32, 8), ("bf16", 33, 5000, 64, 4), ("f16", 700, 20000, 96, 8), ("bf16", 3, 200000, 256, 8),
                                                 ("f32", 2, 262144, 128, 4), ("bf16", 2, 524288, 256, 8)])
def test_fewer_slots_than_channels(dtype, M, K, Kpad, bits, static):
    rng = np.random.default_rng(K)
    X = rng.standard_normal((M, K), dtype=np.float32)
    src = rng.integers(0, K, Kpad).astype(np.int32)
    src[:5] = [0, 1, K - 1, K - 2, K - 1]
    src[-2:] = -1
    rep = np.where(src >= 0, rng.integers(1, 4, Kpad), 0).astype(np.int32)
    _check(X, dtype, src, rep, bits, 2.5 if static else None)


# Inputs with more than 1024 column blocks for the absmax pass (K > 262144 in fp32, > 524288 in two bytes), read through a map
# that drops most channels; the largest element lies in the last column block, in a channel that the map reads.
@pytest.mark.parametrize("dtype,M,K", [("f32", 2, 262400), ("f32", 70, 262148), ("bf16", 3, 524800)])
@pytest.mark.parametrize("bits", [8, 4])
def test_more_column_blocks_than_candidates(dtype, M, K, bits):
    rng = np.random.default_rng(K)
    X = rng.standard_normal((M, K), dtype=np.float32)
    X[M - 1, K - 2] = -77.0
    Kpad = 256
    src = np.full(Kpad, -1, dtype=np.int32)
    src[:200] = rng.choice(K, 200, replace=False)
    src[200:203] = K - 2
    rep = np.where(src >= 0, 1, 0).astype(np.int32)
    rep[200:203] = 3
    _check(X, dtype, src, rep, bits, None)
    _check(X, dtype, src, rep, bits, 2.0)
    Xd, Xf = _padded(X, dtype)
    for call, args in ((fq.fq_flatten_weights, ()), (fq.fq_flatten_quant_act_peel, (dev_i32(np.zeros(Kpad, np.int32)),))):
        out = torch.full((M, Kpad if bits == 8 else Kpad // 2), 0x55, dtype=torch.uint8, device=DEV)
        s = torch.zeros(1, dtype=torch.float32, device=DEV)
        ws = bytes_ws(fq.fq_act_workspace_bytes(K, Kpad))
        if args:
            call(Xd, dev_i32(src), *args, bits, 5.0, out, s, ws)
            want, s_ref = O.flatten_quant_act_peel(Xf, src, np.zeros(Kpad, np.int32), bits, 5.0, O.act_absmax_peel(Xf, 5.0))
        else:
            call(Xd, dev_i32(src), bits, out, s, ws)
            want, s_ref = O.flatten_weights(Xf, src, bits)
        assert np.float32(s.item()) == s_ref
        np.testing.assert_array_equal(out.cpu().numpy().reshape(-1), _packed(want, bits).reshape(-1))


# Padding slots hold 0 and finite elements keep their values whatever else X holds (static scale): infinities and NaN sit in
# column 0 and in a channel that is copied; padding stands in groups of copies, in the head and beside a slot that is gathered.
# (K, M): the one-kernel form with one and two groups per thread, the row-strip kernel, and a layer too wide for either.
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("dtype,M,K", [("f32", 3, 500), ("bf16", 70, 4096), ("bf16", 3, 16400), ("bf16", 800, 16384), ("f16", 5, 33000)])
def test_padding_beside_what_is_not_finite(dtype, M, K, bits):
    rng = np.random.default_rng(K)
    X = rng.standard_normal((M, K), dtype=np.float32)
    Kpad = (K + 300 + 31) // 32 * 32
    src = np.full(Kpad, -1, dtype=np.int32)
    rep = np.zeros(Kpad, dtype=np.int32)
    src[:K] = np.arange(K)
    rep[:K] = 1
    src[70] = -1                                                          # a hole in the head
    src[K:K + 40] = 5
    src[K + 50], src[K + 51], src[K + 90] = 7, K + 3, 9                    # single copies among padding
    rep[K:K + 120] = np.where((src[K:K + 120] >= 0) & (src[K:K + 120] < K), 2, 0)
    X[0, 0], X[M - 1, 0], X[1, 5], X[2, 9] = np.inf, -np.inf, np.nan, np.inf
    Xd, Xf = _padded(X, dtype)
    ok = np.isfinite(Xf)
    valid = (src >= 0) & (src < K)
    want, s_ref = O.flatten_quant_act(np.where(ok, Xf, 0).astype(np.float32), np.where(valid, src, -1).astype(np.int32), rep, bits, 3.0)
    out = torch.full((M, Kpad if bits == 8 else Kpad // 2), 0x55, dtype=torch.uint8, device=DEV)
    s_x = torch.zeros(1, dtype=torch.float32, device=DEV)
    fq.fq_flatten_quant_act(Xd, dev_i32(src), dev_i32(rep), bits, out, s_x, bytes_ws(fq.fq_act_workspace_bytes(K, Kpad)), absmax_in=scalar(3.0))
    got = out.cpu().numpy()
    got = got.view(np.int8) if bits == 8 else O.unpack_i4(got)
    defined = ~valid[None, :] | ok[:, np.where(valid, src, 0)]
    np.testing.assert_array_equal(got[defined], want[defined])
    assert np.float32(s_x.item()) == s_ref


# Copy counts on both sides of what a byte and the tables hold, one and two head groups per thread; a' from all of X in every
# workgroup (few rows), from the candidates, static; and the row-strip kernel.
@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("dtype,M,K,bits", [("bf16", 1, 640, 8), ("f32", 9, 640, 6), ("f16", 90, 640, 4), ("bf16", 5, 16500, 8), ("f32", 40, 16500, 4), ("bf16", 770, 16500, 8)])
def test_copy_counts_beyond_a_byte(dtype, M, K, bits, static):
    rng = np.random.default_rng(K + M)
    counts = np.array([253, 254, 255, 256, 300, 1023, 1024, 3000])
    at = np.concatenate([rng.choice(K - 20, counts.size - 1, replace=False), [K - 3]])      # the last one in the last group
    chmax = np.full(K, 0.5, dtype=np.float32)
    chmax[at] = counts - 0.5
    src, rep, _, _ = fq.fq_flatten_plan(chmax, 1.0, 128 if bits == 6 else 32)
    assert (rep[at] == counts).all()
    X = (rng.uniform(-1.0, 1.0, (M, K)) * chmax).astype(np.float32)
    X[M - 1, at[4]] = np.float32(299.25)                                                    # a' = 299.25 / 300
    _check(X, dtype, src, rep, bits, 1.0 if static else None)
    rep[src == at[4]] = rng.integers(250, 310, (src == at[4]).sum())                        # copies with other counts than the channel's
    _check(X, dtype, src, rep, bits, 1.0 if static else None)


# Tall and narrow (an attention operand): more strips than the matrix has columns, the largest element in the last row.
@pytest.mark.parametrize("dtype,M,K,bits", [("bf16", 70001, 64, 8), ("f32", 66000, 20, 4), ("bf16", 200000, 72, 8)])
def test_more_strips_than_columns(dtype, M, K, bits):
    rng = np.random.default_rng(K)
    X = rng.standard_normal((M, K), dtype=np.float32)
    X[M - 1, K - 1] = 9.5
    Kpad = (K + 31) // 32 * 32
    src = np.full(Kpad, -1, dtype=np.int32)
    src[:K] = np.arange(K)
    _check(X, dtype, src, np.where(src >= 0, 1, 0).astype(np.int32), bits, None)
