"""The launch rules that depend on sizes alone (csrc/fq_rules.h), compiled with the host compiler and walked on the CPU."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2402_17985_amd", "csrc")

DRIVER = """
#include "fq_rules.h"
extern "C" long long capacity(long long K) { return fq::candidate_capacity(K); }
extern "C" void absmax(long long M, long long K, long long ld, int vec, int* out)
{
    const fq::AbsmaxGrid a = fq::absmax_grid(M, K, ld, vec);
    out[0] = a.blocks; out[1] = a.strips; out[2] = a.rows_per_strip;
}
extern "C" int skinny(long long N) { return fq::skinny_holds(N); }
extern "C" void few_tiles(long long M, long long N, int rowbytes, int bits, long long count, long long cus, int* out)
{
    const fq::FewTilesChoice c = fq::few_tiles(M, N, rowbytes, bits, count, cus);
    out[0] = (int)c.kernel; out[1] = c.bm; out[2] = c.bn;
}
extern "C" int direct(int M, int R, int cus, int resident) { return fq::direct_workgroups(M, R, cus, resident); }
extern "C" int few_row(int N, int K, int bits, int x_bytes, int dynamic, int cus)
{
    return fq::few_takes_one_row(N, K, bits, x_bytes, dynamic, cus);
}
extern "C" int few_scaled(int M, int N, int K, int Kpad, int bits, int x_bytes, int dynamic, int cus, long long* out)
{
    fq::FewPlan p;
    if (!fq::few_plan(M, N, K, K, Kpad, bits, x_bytes, dynamic, cus, &p)) return 0;
    out[0] = p.sh.prep_waves; out[1] = p.sh.slots; out[2] = p.sh.cols; out[3] = p.fn; out[4] = p.threads; out[5] = p.grid; out[6] = p.lds;
    return 1;
}
extern "C" int few_turns(int M, int N, int K, int Kpad, int bits, int cus)
{
    fq::FewPlan p;
    return fq::few_plan(M, N, K, K, Kpad, bits, 2, true, cus, &p) ? p.sh.turns : -2;
}
extern "C" int few(int M, int N, int K, int Kpad, int bits, int x_bytes, int cus, long long* out)
{
    return few_scaled(M, N, K, Kpad, bits, x_bytes, 1, cus, out);
}
extern "C" int overlap(unsigned long long a, unsigned long long na, unsigned long long b, unsigned long long nb)
{
    return fq::overlap((const void*)a, na, (const void*)b, nb);
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("rules")
    src, so = str(d / "rules.cpp"), str(d / "rules.so")
    with open(src, "w") as f:
        f.write(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-static-libubsan",
                    "-shared", "-fPIC", "-I", CSRC, "-o", so, src], check=True)
    return ctypes.CDLL(so)


# (elements per 16 bytes, K): more column blocks than 1024 candidates from K = 262145 (fp32) and 524289 (2-byte types) on
@pytest.mark.parametrize("vec,K", [(4, 16), (4, 1024), (8, 64), (8, 4096), (8, 22016), (4, 262144), (4, 262145), (4, 262400),
                                   (8, 524288), (8, 524800), (4, 3000000), (8, 2**31 - 1)])
@pytest.mark.parametrize("M", [1, 2, 16, 64, 65, 500, 8192, 131072, 2**31 - 1])
def test_absmax_grid_covers_the_matrix_and_fits_the_candidates(rules, vec, K, M):
    out = (ctypes.c_int * 3)()
    rules.absmax(ctypes.c_longlong(M), ctypes.c_longlong(K), ctypes.c_longlong(-(-K // vec) * vec), vec, out)
    blocks, strips, rows = out
    rules.capacity.restype = ctypes.c_longlong
    capacity = rules.capacity(ctypes.c_longlong(K))
    assert rows > 0 and strips > 0 and (blocks - 1) * 64 * vec < K <= blocks * 64 * vec
    assert (strips - 1) * rows < M <= strips * rows
    assert blocks * strips <= capacity
    assert blocks * strips <= 1024 or strips == 1
    # a tall matrix gets the workgroups that its height allows, however narrow it is
    assert blocks * strips >= min(256, blocks * ((M + 63) // 64)) or blocks > 1024


def test_absmax_strips_follow_the_row_stride(rules):
    """Columns that fill a stride of whole 8 KiB up to its padding get the strips of that width; a part of a wider stride, and few
    rows, those of their own width."""
    def rows(M, K, ld, vec):
        out = (ctypes.c_int * 3)()
        rules.absmax(*(ctypes.c_longlong(v) for v in (M, K, ld)), vec, out)
        return out[2]
    for vec in (4, 8):
        for M in (2048, 4096, 8192, 16384):
            for K in (4000, 4088, 4090):
                assert rows(M, K, 4096, vec) == rows(M, 4096, 4096, vec)
            for K in (2500, 3000, 3600):
                assert rows(M, K, 4096, vec) == rows(M, K, 4100, vec)
            assert rows(M, 4096, 4112, vec) == rows(M, 4096, 8192, vec) == rows(M, 4096, 4096, vec)
        assert rows(2047, 8184, 8192, vec) == rows(2047, 8184, 8200, vec)
    assert rows(8192, 4088, 4096, 4) == 288 and rows(8192, 4088, 4112, 4) == 256


@pytest.mark.parametrize("a,na,b,nb,want", [(1000, 16, 1000, 16, 1), (1000, 16, 1015, 1, 1), (1000, 16, 1016, 1, 0), (1000, 16, 999, 1, 0),
                                            (1000, 16, 990, 11, 1), (1000, 16, 900, 500, 1), (1000, 500, 1100, 4, 1), (1000, 4, 2000, 4, 0)])
def test_overlap(rules, a, na, b, nb, want):
    u = ctypes.c_ulonglong
    assert rules.overlap(u(a), u(na), u(b), u(nb)) == want
    assert rules.overlap(u(b), u(nb), u(a), u(na)) == want


def test_weight_streaming_launches_stay_within_32_bits(rules):
    """Operands of less than 4 GiB admit N up to 2^27 - 1 (INT8, 32 slots) or 2^28 - 1 (nibbles, 32 slots)."""
    for N in (1, 16, 4097, 2**27 - 16, 2**27 - 15, 2**27 - 1, 2**27, 2**28 - 1):
        assert rules.skinny(ctypes.c_longlong(N)) == ((N + 15) // 16 * 512 < 2**32)
    assert not rules.skinny(ctypes.c_longlong(2**27 - 1))


TILED, SKINNY, STREAM, RING = range(4)


def _few_tiles(rules, bits, M, N, rowbytes, count=1, cus=256):
    out = (ctypes.c_int * 3)()
    q = ctypes.c_longlong
    rules.few_tiles(q(M), q(N), rowbytes, bits, q(count), q(cus), out)
    return tuple(out)


# Both sides of every line: (bits, M, N, batch, row bytes of a shorter reduction -> tiled kernels, of a longer one -> this)
@pytest.mark.parametrize("bits,M,N,count,short,long,want", [
    (8, 512, 2048, 1, 512, 640, (STREAM, 64, 64)), (4, 512, 2048, 1, 256, 384, (STREAM, 64, 64)), (8, 32, 256, 32, 480, 512, (STREAM, 32, 32)),
    (8, 384, 4096, 1, 896, 1024, (STREAM, 96, 64)), (4, 384, 4096, 1, 896, 1024, (STREAM, 96, 64)), (6, 384, 4096, 1, 288, 384, (STREAM, 96, 64)),
    (4, 512, 4096, 1, 1920, 2048, (STREAM, 128, 64)), (6, 512, 4096, 1, 1056, 1152, (STREAM, 128, 64)), (8, 2048, 1024, 1, 896, 1024, (RING, 128, 64)),
    (4, 64, 32768, 1, 1152, 1280, (STREAM, 64, 128)), (6, 64, 32768, 1, 672, 768, (STREAM, 64, 128)),
    (8, 256, 128, 40, 896, 1024, (STREAM, 96, 64)), (4, 256, 128, 40, 480, 512, (STREAM, 96, 64)), (4, 384, 128, 40, 896, 1024, (STREAM, 128, 64)),
    (4, 40, 1500, 20, 896, 1024, (STREAM, 64, 128)), (8, 768, 128, 40, 480, 512, (RING, 128, 128)), (4, 700, 700, 4, 480, 512, (RING, 128, 128)),
])
def test_reductions_too_short_to_split_stay_with_the_tiled_kernels(rules, bits, M, N, count, short, long, want):
    assert _few_tiles(rules, bits, M, N, short, count)[0] == TILED
    assert _few_tiles(rules, bits, M, N, long, count) == want


@pytest.mark.parametrize("bits,M,N,rowbytes,count,want", [
    (8, 4, 24576, 32, 1, (SKINNY, 0, 0)), (8, 5, 4096, 32, 1, (STREAM, 32, 32)), (4, 16, 16384, 16, 1, (SKINNY, 0, 0)), (4, 16, 16400, 128, 1, (STREAM, 32, 128)), (6, 16, 16384, 96, 1, (SKINNY, 0, 0)),
    (8, 1, 2**27 - 1, 32, 1, (TILED, 0, 0)), (8, 512, 4096, 128, 1, (RING, 128, 64)), (8, 512, 8192, 32, 1, (RING, 128, 128)), (6, 512, 8192, 3072, 1, (TILED, 0, 0)),
    (4, 768, 128, 2048, 40, (TILED, 0, 0)), (8, 8192, 4096, 4096, 1, (TILED, 0, 0)), (8, 1, 128, 480, 160, (TILED, 0, 0)), (8, 1, 128, 512, 160, (SKINNY, 0, 0)),
])
def test_products_of_few_tiles(rules, bits, M, N, rowbytes, count, want):
    assert _few_tiles(rules, bits, M, N, rowbytes, count) == want


@pytest.mark.parametrize("bits", [8, 4, 6])
def test_every_choice_has_a_kernel(rules, bits):
    stream = {(32, 32), (32, 64), (64, 64), (32, 128), (96, 64)} | ({(128, 64), (64, 128)} if bits != 8 else set())
    ring = {8: {(128, 64), (64, 128), (128, 128)}, 4: {(128, 128)}, 6: set()}[bits]
    seen = set()
    for cus in (32, 80, 256, 304):
        for M in (1, 4, 5, 16, 17, 40, 64, 96, 130, 300, 500, 1000, 2000, 9000):
            for N in (16, 100, 500, 1000, 2048, 4096, 9000, 16384, 16385, 30000):
                for rowbytes in (96, 384, 768, 1536, 6144):
                    for count in (1, 3, 40) if bits != 6 else (1,):
                        kernel, bm, bn = _few_tiles(rules, bits, M, N, rowbytes, count, cus)
                        assert kernel in (TILED, SKINNY) or (bm, bn) in (stream if kernel == STREAM else ring)
                        if kernel in (STREAM, RING):
                            assert -(-M // bm) * -(-N // bn) * count <= cus
                            seen.add((kernel, bm, bn))
    assert seen == {(STREAM, *t) for t in stream} | {(RING, *t) for t in ring}


def test_lines_follow_the_number_of_compute_units(rules):
    """64 columns per CU for 4-bit values of up to 16 rows; the quantizer's workgroups a row each up to the CUs, then strips."""
    for cus in (32, 64, 256):
        assert _few_tiles(rules, 4, 16, 64 * cus, 2048, cus=cus)[0] == SKINNY
        assert _few_tiles(rules, 4, 16, 64 * cus + 1, 2048, cus=cus)[0] != SKINNY
        assert [rules.direct(M, 4, cus, 2) for M in (1, cus, 2 * cus, 4 * cus, 6 * cus, 8 * cus, 100 * cus)] == \
            [1, cus, cus, cus, (6 * cus + 3) // 4, 2 * cus, 2 * cus]
    assert rules.direct(2**31 - 1, 1, 256, 16) == 4096


# The kernel of the whole layer for a few rows: threads cover the head and registers the rows, LDS holds them, and the columns of
# all rounds cover the output.
@pytest.mark.parametrize("bits", [8, 4, 6])
@pytest.mark.parametrize("x_bytes", [2, 4])
@pytest.mark.parametrize("cus", [1, 80, 256])
def test_few_rows_plan(rules, bits, x_bytes, cus):
    out = (ctypes.c_longlong * 7)()
    taken = 0
    for M in (1, 2, 3, 8, 9, 16, 17):
        for K in (1, 15, 16, 31, 1000, 1024, 1040, 4096, 4100, 5120, 8192, 8207, 8208, 30000):
            for Kpad in (K // 256 * 256, (K + 255) // 256 * 256, (K + 1000) // 128 * 128, 65408, 65536):
                for N in (1, 16, 17, 256, 4096, 4097, 5120, 11008, 16384, 16385, 100000, 2**31 - 1):
                    if Kpad <= 0 or not rules.few(M, N, K, Kpad, bits, x_bytes, cus, out):
                        continue
                    taken += 1
                    prep, slots, cols, fn, threads, grid, lds = out
                    assert M <= 16 and Kpad >= K // 16 * 16 and Kpad < 65536
                    assert 0 < prep <= 8 and prep < threads // 64 <= 16 and threads % 64 == 0
                    assert prep % slots == 0 and K // 16 <= prep // slots * 64
                    assert -(-M // slots) <= (8 if x_bytes == 2 else 4) and slots <= M
                    assert cols % 4 == 0 and 16 <= cols <= 64 and 16 * (fn - 1) < cols <= 16 * fn
                    assert 0 < grid <= cus and (grid == cus or (grid - 1) * cols < N <= grid * cols)
                    assert lds <= 160 * 1024
    assert taken > 0


# One row: both sides of the lines where the kernel of the whole layer begins and ends, each where it was measured
@pytest.mark.parametrize("bits,x_bytes,scales,K,N,want", [
    (8, 2, "sd", 2048, 4096, 0), (8, 2, "sd", 4096, 1024, 1), (8, 2, "sd", 2048, 4112, 1), (8, 2, "sd", 4096, 36000, 1), (8, 2, "sd", 4096, 40000, 0),
    (8, 2, "sd", 5120, 50000, 0), (8, 2, "sd", 3072, 65536, 1), (8, 2, "sd", 8192, 65536, 1), (4, 2, "sd", 1024, 4112, 0), (4, 2, "sd", 1024, 4300, 1),
    (4, 2, "sd", 2048, 4112, 1), (4, 2, "sd", 4096, 32000, 1), (4, 2, "sd", 4096, 50000, 0), (4, 2, "sd", 4096, 65536, 1), (4, 2, "sd", 4096, 100000, 0),
    (6, 2, "sd", 4096, 1024, 0), (6, 2, "sd", 8192, 1024, 1), (6, 2, "sd", 2048, 4112, 0), (6, 2, "sd", 2048, 12288, 1), (6, 2, "sd", 1024, 6000, 0),
    (6, 2, "sd", 1024, 16384, 0), (6, 2, "sd", 1024, 16385, 1), (6, 2, "sd", 1007, 24576, 1), (4, 4, "sd", 1024, 4300, 0), (4, 4, "sd", 1024, 12288, 1),
    (4, 4, "sd", 5120, 2000, 0), (4, 4, "sd", 8192, 2000, 1), (6, 4, "sd", 2048, 12288, 0), (6, 4, "sd", 3072, 4112, 0), (6, 4, "sd", 4096, 4300, 1),
    (8, 2, "d", 2507, 4100, 0), (8, 2, "d", 2507, 4300, 1), (8, 2, "d", 4090, 4100, 1), (8, 2, "d", 6503, 13000, 1), (8, 2, "d", 6503, 16384, 0),
    (8, 2, "d", 4090, 24576, 1), (8, 2, "d", 4090, 32000, 0), (8, 4, "d", 4090, 32000, 1), (8, 2, "s", 2005, 4100, 1), (8, 2, "s", 6503, 16384, 1),
    (8, 2, "sd", 1803, 8192, 0), (4, 2, "d", 2507, 4608, 0), (4, 2, "d", 2507, 10000, 1), (4, 2, "d", 3001, 4608, 1), (4, 2, "d", 6503, 4100, 0),
    (4, 2, "d", 8190, 4100, 1), (4, 2, "s", 2005, 5120, 1), (4, 4, "d", 3001, 11008, 0), (4, 4, "d", 4503, 4300, 1), (4, 4, "s", 2005, 8192, 0),
    (4, 4, "s", 2005, 11008, 1), (4, 4, "s", 2507, 4100, 0), (4, 2, "sd", 257, 16384, 0), (4, 2, "sd", 257, 16385, 1), (6, 2, "sd", 2005, 16384, 0),
])
def test_one_row_lines(rules, bits, x_bytes, scales, K, N, want):
    for scale in scales:
        assert rules.few_row(N, K, bits, x_bytes, int(scale == "d"), 256) == want


@pytest.mark.parametrize("bits", [8, 4, 6])
def test_few_rows_begin_at_a_step_of_the_reduction(rules, bits):
    for Kpad in range(128, 20000, 128):
        for M in (1, 2, 8):
            turns = rules.few_turns(M, 12288, min(Kpad, 8192), Kpad, bits, 256)
            if turns == -2:
                continue
            rowbytes = Kpad if bits == 8 else Kpad // 2
            assert turns == (rowbytes // 128 - 1 if bits != 6 and rowbytes in (4096, 8192, 16384) else -1)
