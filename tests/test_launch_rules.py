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
extern "C" void absmax(long long M, long long K, int vec, int* out)
{
    const fq::AbsmaxGrid a = fq::absmax_grid(M, K, vec);
    out[0] = a.blocks; out[1] = a.strips; out[2] = a.rows_per_strip;
}
extern "C" int skinny(long long N) { return fq::skinny_holds(N); }
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
    rules.absmax(ctypes.c_longlong(M), ctypes.c_longlong(K), vec, out)
    blocks, strips, rows = out
    rules.capacity.restype = ctypes.c_longlong
    capacity = rules.capacity(ctypes.c_longlong(K))
    assert rows > 0 and strips > 0 and (blocks - 1) * 64 * vec < K <= blocks * 64 * vec
    assert (strips - 1) * rows < M <= strips * rows
    assert blocks * strips <= capacity
    assert blocks * strips <= 1024 or strips == 1
    # a tall matrix gets the workgroups that its height allows, however narrow it is
    assert blocks * strips >= min(256, blocks * ((M + 63) // 64)) or blocks > 1024


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
