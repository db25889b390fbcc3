"""The linear's choice between its streaming and its tiled kernel: a host
function of the sizes, compiled here by itself. Both kernels give the same
values, so only its own values show which one a call takes."""

import ctypes
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2607_27744_amd", "csrc")
CUS = 256


@pytest.fixture(scope="module")
def pays(tmp_path_factory):
    cxx = os.environ.get("CXX", "g++")
    if shutil.which(cxx) is None:
        pytest.skip("no C++ compiler")
    tmp = tmp_path_factory.mktemp("rule")
    src, lib = tmp / "rule.cpp", tmp / "rule.so"
    src.write_text('#include "linear_rule.h"\n'
                   'extern "C" int pays(long long n, long long d, long long k, long long r, int c)'
                   ' { return rocs::stream_pays(n, d, k, r, c); }\n')
    subprocess.run([cxx, "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}", str(src), "-o", str(lib)],
                   check=True)
    fn = ctypes.CDLL(str(lib)).pays
    fn.argtypes = [ctypes.c_longlong] * 4 + [ctypes.c_int]
    return lambda *a: bool(fn(*a, CUS))


# N, D, K, R and whether streaming was measured as the faster one.
MEASURED = [
    # one round of 256 tiles
    (8192, 1024, 512, 0, False), (9011, 1024, 512, 0, True), (9011, 1024, 256, 0, True),
    (6553, 1024, 4096, 0, False), (8192, 1024, 4096, 0, True), (10000, 1024, 4096, 16, True),
    (8192, 512, 2048, 16, False), (32768, 512, 1024, 0, True),
    # several
    (64324, 512, 256, 64, False), (163840, 1024, 256, 16, True), (163840, 1024, 512, 16, True),
    (21299, 1024, 512, 0, False), (8192, 8192, 512, 16, True), (26214, 1024, 512, 0, True),
    (50000, 512, 512, 64, False), (100000, 1024, 512, 16, True),
    (18022, 1024, 1024, 0, False), (22937, 1024, 1024, 0, True),
    (21299, 1024, 2048, 0, True), (22937, 1024, 4096, 0, True), (32736, 1024, 2048, 1, True),
]


@pytest.mark.parametrize("n,d,k,r,want", MEASURED)
def test_the_faster_one_where_both_were_measured(pays, n, d, k, r, want):
    assert pays(n, d, k, r) == want


# The share of the rounds' area where each K's line lies, over two rounds.
@pytest.mark.parametrize("k,share", [(64, 3 / 4), (448, 3 / 4), (512, 2 / 3), (960, 2 / 3),
                                     (1024, 0.6), (1984, 0.6), (2048, 0.55), (8192, 0.55)])
def test_lines_over_two_rounds(pays, k, share):
    area = 2 * CUS * 256                        # rows of one feature tile in two rounds
    assert pays(int(area * share) + 64, 256, k, 0)
    assert not pays(int(area * share) - 64, 256, k, 0)


@pytest.mark.parametrize("k,at_half", [(64, None), (256, False), (1984, False), (2048, True)])
def test_line_of_one_round(pays, k, at_half):
    half = CUS * 256 // 2
    if at_half is None:                         # a short K keeps the line of more rounds
        assert not pays(half + 8192, 256, k, 0) and pays(CUS * 192, 256, k, 0)
        return
    assert pays(half, 256, k, 0) == at_half
    assert pays(half + 1, 256, k, 0) and not pays(half - 1, 256, k, 0)


def test_requests_count_at_most_their_partial_tiles(pays):
    # 32,736 rows of one request are 128 slots x 4 tiles: two rounds, not three.
    assert pays(32736, 1024, 512, 1) == pays(32736, 1024, 512, 0) is True
    # 200 requests may leave 199 partial tiles beside the 64 that hold the rows.
    assert pays(16384, 1024, 512, 1) and not pays(16384, 1024, 512, 200)
