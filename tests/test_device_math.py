"""Arithmetic that the kernels share with the host, where only sizes that fit no card or millions of
values would show a mistake: compiled for the host alone and checked without a GPU."""
import ctypes as C
import os
import subprocess

import numpy as np
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
                assert not M.inplace_moves(-1, j, most) and not M.inplace_moves(M.inplace_late_token(), j, most)
                if 0 <= j < most:
                    assert not M.inplace_moves(j, j, most) and (j == 0 or not M.inplace_moves(j - 1, j, most))
                    assert bool(M.inplace_moves(j + 1, j, most)) == (j + 1 < most)


@pytest.mark.parametrize("n", [1, 4, 5, 8192, 8193, 32771, 1000003, 2 ** 31 - 8191, 2 ** 31 - 1100, 2 ** 31 - 65])
def test_chunks_of_a_head_up_to_the_largest_context(M, n):
    """The chunks of the pooled selection cover a head's tokens once, and every load of four tokens that a thread
    issues for its rounds lies inside the head, also where the tokens themselves lie past its end."""
    blocks, chunk = C.c_int(), C.c_int()
    M.head_chunks(n, 8192, C.byref(blocks), C.byref(chunk))
    blocks, chunk = blocks.value, chunk.value
    assert 0 < chunk <= 8192 and chunk % 4 == 0
    for tile in {0, 1, blocks // 2, blocks - 2, blocks - 1} & set(range(blocks)):
        begin = tile * chunk
        tokens = M.chunk_tokens(begin, chunk, n)
        assert tokens == (chunk if tile + 1 < blocks else n - begin) and 0 < tokens <= chunk
        if n >= 4:
            for at in range(0, 8192, 4):
                first = M.quad_at(begin, at, tokens)
                assert 0 <= first <= n - 4
                if at + 4 <= tokens:
                    assert first == begin + at
                elif at < tokens:
                    assert first + 4 == begin + tokens


def _key(x):
    u = int(np.float32(x).view(np.uint32))
    return ~u & 0xffffffff if u >> 31 else u | 0x80000000


def test_selection_bins_partition_the_keys(M):
    """From the first key of one bin to the first of the next, through all 2^32: a bin's keys are those that
    bin_keys says, bins rise with the keys and fit the histogram, and none of scores that occur (magnitudes
    2^-42 to 2^28) is wider than the eighth of an octave that the top 12 key bits are."""
    lo, at, last = C.c_uint(), 0, -1
    while at < 2 ** 32:
        b = M.score_bin(at)
        assert last < b < 4096
        bits = M.bin_bits(b, 1, C.byref(lo))
        assert lo.value == at and 17 <= bits <= 23 and M.score_bin(at + (1 << bits) - 1) == b
        last, at = b, at + (1 << bits)
    assert M.score_bin(0) == 0 and M.score_bin(_key(-np.inf)) == 0 and M.score_bin(_key(np.inf)) == 4095
    for sign in (1.0, -1.0):
        for e in range(-42, 28):
            for f in (1.0, 1.3, 1.999):
                bits = M.bin_bits(M.score_bin(_key(sign * np.ldexp(f, e))), 1, C.byref(lo))
                assert bits == (17 if -18 <= e < 4 else 20)
    for b in (0, 1, 2047, 2048, 4095):
        assert M.bin_bits(b, 0, C.byref(lo)) == 20 and lo.value == b << 20


@pytest.mark.parametrize("n", [8224, 8300, 16385, 1000003, 2 ** 31 - 65])
def test_sampled_lines_lie_inside_the_pool(M, n):
    """Half lines of 16 scores, one in each of the equal stretches of the pool, from any alignment of its start."""
    groups = M.sample_lines()
    assert groups == 512
    for first in (0, 1, 15):
        lines = (n - first) // 16
        at = np.array([M.sample_line(g, lines) for g in range(groups)], dtype=np.int64)
        assert at[0] >= 0 and first + 16 * at[-1] + 16 <= n and np.all(np.diff(at) >= 0)
        stretch = lines / groups
        assert np.all(np.abs(at + 0.5 - (np.arange(groups) + 0.5) * stretch) <= 0.5 * stretch + 1)
