"""Bounds that the kernels take from csrc/cis_plan.h, checked on the host over their whole range (the
header is plain C++: it is compiled here with the host compiler)."""

import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_32444_amd", "csrc")

SOURCE = """
#include "cis_plan.h"
extern "C" {
uint32_t slab_bytes(uint32_t cols, uint32_t ld, int left) { return cis::slab_bytes(cols, ld, left); }
int64_t grad_rows(int64_t rows, int64_t V) { return cis::grad_rows(rows, V); }
int64_t seq_pieces(int64_t T, int64_t n_seq) { return cis::seq_pieces(T, n_seq, 128); }
int64_t seq_block() { return cis::kSeqBlock; }
int64_t grad_threads(int64_t V) { return cis::grad_tiles(V) * cis::kGradThreads; }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("clang++") or shutil.which("hipcc")
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(SOURCE)
    subprocess.run([cxx, "-std=c++20", "-shared", "-fPIC", "-I", CSRC, str(d / "plan.cpp"), "-o",
                    str(d / "plan.so")], check=True)
    lib = ctypes.CDLL(str(d / "plan.so"))
    lib.slab_bytes.argtypes = [ctypes.c_uint32, ctypes.c_uint32, ctypes.c_int]
    lib.slab_bytes.restype = ctypes.c_uint32
    lib.grad_rows.argtypes = [ctypes.c_int64, ctypes.c_int64]
    lib.grad_threads.argtypes = [ctypes.c_int64]
    lib.seq_pieces.argtypes = [ctypes.c_int64, ctypes.c_int64]
    lib.seq_pieces.restype = lib.seq_block.restype = ctypes.c_int64
    lib.grad_rows.restype = lib.grad_threads.restype = ctypes.c_int64
    return lib


# Offsets (bytes) of the 16-byte loads of one slab of a k-major operand: 64 rows, 256 columns.
ROWS, COLS = np.divmod(np.arange(64 * 32), 32)
COLS = COLS * 8


@pytest.mark.parametrize("ld", [*range(8, 257, 8), 320, 520, 4096, 1 << 16, 1 << 22])
def test_slab_loads_stay_in_the_matrix(plan, ld):
    """With `left` rows of the contraction and `cols` columns from the tile's first one on, the
    matrix ends at ((left - 1) ld + cols rounded up to 8) elements: no load that the resource lets
    through ends later, every chunk that holds an element of the slab is let through, and every
    row past the contraction is not."""
    off = (ROWS.astype(np.int64) * ld + COLS) * 2
    for cols in sorted({1, 7, 8, 9, ld // 2, ld - 7, ld - 1, ld} & set(range(1, ld + 1))):
        cols8 = (cols + 7) // 8 * 8
        for left in (*range(1, 131), 1000, 1 << 22):
            n = plan.slab_bytes(cols, ld, left)
            read = off + 16 <= n
            assert n % 16 == 0 and n <= 1 << 31
            assert np.all(off[read] + 16 <= ((left - 1) * ld + cols8) * 2), (cols, left)
            assert np.all(read[(ROWS < left) & (COLS < cols8)]), (cols, left)
            assert not np.any(read[ROWS >= left]), (cols, left)


def test_no_slab_beyond_the_contraction(plan):
    for left in (0, -1, -64, -1000):
        assert plan.slab_bytes(8, 8, left) == 0


@pytest.mark.parametrize("rows,V", [(1, 1), (4096, 151936), (8192, 1 << 18), (8192, 1 << 22),
                                    (1 << 16, 1 << 19), (1 << 16, 1 << 22)])
def test_grad_launch_within_the_runtime_limit(plan, rows, V):
    """HIP refuses a launch of 2^32 work items or more in a dimension; rows (up to a chunk of 2^16)
    and V (up to 2^22) at the ends of what the LM-head calls accept."""
    n = plan.grad_rows(rows, V)
    assert 1 <= n <= rows
    assert n * plan.grad_threads(V) < 1 << 32


@pytest.mark.parametrize("T", [1, 513, 1 << 20, 1 << 31, 1 << 33, 1 << 36])
def test_response_sums_within_the_runtime_limit(plan, T):
    """The launch that sums the responses' log K stays below 2^32 work items for any number of
    responses that a wave each allows (2^26 - 4), however long they are; several workgroups per
    response only where their sums fit."""
    most = (1 << 26) - 4
    for n in (1, 2, 7, 128, 129, min(T // 513 + 1, most), 1 << 20, (1 << 20) + 1, 1 << 22, most):
        p = plan.seq_pieces(T, n)
        assert (n * p * plan.seq_block() if p else (n + 3) // 4 * 256) < 1 << 32, n
        assert p <= 1 or n * p <= 128
