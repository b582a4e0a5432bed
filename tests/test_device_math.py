"""Arithmetic that the kernels share with the host, where only sizes that fit no card or millions of
values would show a mistake: compiled for the host alone and checked without a GPU."""
import ctypes as C
import os
import subprocess

import pytest

from paper_2507_08143_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def M(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("host_math") / "host_math.so")
    subprocess.run([build.HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-shared", "-fPIC",
                    "-I", build.INCLUDE, "-I", build.CSRC, os.path.join(HERE, "host_math.cpp"), "-o", lib], check=True)
    m = C.CDLL(lib)
    m.inplace_row.restype = C.c_longlong
    m.inplace_moves.argtypes = [C.c_int, C.c_longlong, C.c_int]
    return m


@pytest.mark.parametrize("run_rows", [256, 512, 1024])
def test_in_place_rows_up_to_the_largest_context(M, run_rows):
    """Every row below the count is covered, no row at or past it is taken for one of the list (indices
    are fetched three runs ahead of the last), and a row without an index never moves."""
    most = 2 ** 31 - 65
    for rows in (-(2 ** 31), -5, 0, 1, run_rows, run_rows + 1, 100003, most - 3 * run_rows, most - 1, most):
        runs = M.inplace_runs(rows, run_rows)
        assert runs == max(0, -(-rows // run_rows))
        for run in {0, runs - 1, runs, runs + 1, runs + 2} - {-1}:
            for jr in (0, 1, run_rows - 1):
                j = M.inplace_row(run, run_rows, jr)
                assert j == run * run_rows + jr
                assert not M.inplace_moves(-1, j, most)
                if 0 <= j < most:
                    assert not M.inplace_moves(j, j, most) and (j == 0 or not M.inplace_moves(j - 1, j, most))
                    assert bool(M.inplace_moves(j + 1, j, most)) == (j + 1 < most)
