"""Index arithmetic of the cascade's lists at the largest grids the library accepts (2^30
cells), compiled for the host and compared with Python's integers."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2110_08683_amd", "csrc")


@pytest.fixture(scope="module")
def index(tmp_path_factory):
    d = tmp_path_factory.mktemp("index")
    src, out = str(d / "index.cpp"), str(d / "index.so")
    with open(src, "w") as f:
        f.write('#include "gpmood_index.h"\n'
                'extern "C" unsigned groups(unsigned n, unsigned per) { return gpm::groups_of(n, per); }\n'
                'extern "C" int item(unsigned r, unsigned threads, unsigned t) { return (int)gpm::quad_item(r, threads, t); }\n'
                'extern "C" unsigned faces(int nx, int ny) { return gpm::faces_of(nx, ny); }\n')
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", CSRC, "-shared", "-fPIC", "-o", out, src])
    L = ctypes.CDLL(out)
    L.groups.restype = L.faces.restype = ctypes.c_uint
    L.item.restype = ctypes.c_int
    return L


# the claims after the first pass: 65536 threads a round in the single problem's kernel, 256
# a work block in a batch
@pytest.mark.parametrize("n", [1, 63, 64, 16384, 16385, (1 << 29) - 1, 1 << 29, (1 << 29) + 1, 600000001, 1 << 30])
@pytest.mark.parametrize("threads", [256, 65536])
def test_claims_cover_every_lowered_cell(index, n, threads):
    rounds = -(-n // (threads // 4))
    assert index.item(rounds - 1, threads, 0) < n <= index.item(rounds, threads, 0)
    for r in {0, 1, rounds // 2, rounds - 1}:
        for t in (0, 3, 4, threads - 1):
            assert index.item(r, threads, t) == r * (threads // 4) + t // 4, (r, t)


# wavefronts of eight faces and of sixteen cells
@pytest.mark.parametrize("n", [0, 1, 8, 9, 95, 96, 97, (1 << 28) - 1, 1 << 28, 1 << 29, 1 << 30])
def test_wavefronts_of_a_list(index, n):
    assert index.groups(n, 8) == -(-n // 8) and index.groups(n, 16) == -(-n // 16)


@pytest.mark.parametrize("nx,ny", [(1, 1), (62, 5), (32768, 1), (1, 32768), (32767, 32768), (32768, 32768)])
def test_face_count(index, nx, ny):
    assert index.faces(nx, ny) == (nx + 1) * ny + nx * (ny + 1)
