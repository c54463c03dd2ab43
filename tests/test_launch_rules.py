"""The launch code's choices (csrc/launch_rules.h), compiled for the host."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_SRC = r"""
#include "launch_rules.h"
extern "C" {
int32_t pop_chunk(int32_t a, int64_t c, int64_t p) { return bdfx::pop_chunk(a, c, p); }
int32_t persistent_grid(int32_t a, int r, int n, int64_t c, int64_t b) {
  return bdfx::persistent_grid(a, r, n, c, b);
}
int packed_min_cells_per_cu(int S, int R, int fp32, int waves) {
  return bdfx::packed_min_cells_per_cu(S, R, fp32 != 0, waves);
}
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, so = str(d / "rules.cpp"), str(d / "rules.so")
    with open(src, "w") as fh:
        fh.write(_SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2405_01713_amd", "csrc"), src, "-o", so], check=True)
    lib = ctypes.CDLL(so)
    lib.pop_chunk.argtypes = [ctypes.c_int32, ctypes.c_int64, ctypes.c_int64]
    lib.persistent_grid.argtypes = [ctypes.c_int32, ctypes.c_int, ctypes.c_int, ctypes.c_int64,
                                    ctypes.c_int64]
    return lib


@pytest.mark.parametrize("cells,poppers", [(1, 1), (64, 64), (8195, 16384), (131072, 16384),
                                           (2 ** 20, 8192), (2 ** 31 - 1, 16384),
                                           (2 ** 31 - 1, 1)])
@pytest.mark.parametrize("asked", [1, 4, 64, 2 ** 18, 2 ** 20, 2 ** 31 - 1])
def test_the_queue_counter_never_wraps(rules, asked, cells, poppers):
    """Every lane group pops once more than there are cells for it; the counter
    has to stay below 2^32 whatever chunk the options ask for."""
    chunk = rules.pop_chunk(asked, cells, poppers)
    assert 1 <= chunk <= asked
    assert (-(-cells // chunk) + poppers) * chunk < 2 ** 32
    # an ordinary request is taken as it is
    if (-(-cells // asked) + poppers + 1) * asked < 2 ** 32:
        assert chunk == asked


def test_persistent_grid(rules):
    g = rules.persistent_grid
    assert g(0, 4, 256, 10 ** 6, 16) == 1024  # as many blocks as reside
    assert g(0, 0, 256, 10 ** 6, 16) == 256  # at least one a CU
    assert g(2, 4, 256, 10 ** 6, 16) == 512  # as many as asked for
    assert g(0, 4, 256, 1001, 16) == 63  # no more than the cells fill
    assert g(2 ** 31 - 1, 4, 256, 2 ** 31 - 1, 1) == 2 ** 31 - 1
    assert g(0, 4, 256, 0, 16) == 0


def test_packing_looks_at_reactions_and_resident_waves(rules):
    """The measured pairs at which one cell per wave is faster are not packed,
    those at which packing is faster are (cells per CU 0: never)."""
    f = rules.packed_min_cells_per_cu
    at = lambda S, R, fp32, waves, cells: 0 < f(S, R, fp32, waves) <= cells
    for S, R, fp32, waves, cells in ((3, 3, 0, 16, 40), (9, 30, 0, 16, 32), (16, 64, 0, 10, 32),
                                     (9, 100, 0, 13, 48), (8, 150, 0, 10, 128),
                                     (16, 100, 1, 11, 128), (14, 100, 0, 9, 256), (21, 84, 1, 16, 96)):
        assert at(S, R, fp32, waves, cells), (S, R, fp32)
    for S, R, fp32, waves, cells in ((3, 3, 0, 16, 39), (9, 100, 0, 13, 32), (8, 150, 0, 10, 64),
                                     (16, 100, 0, 9, 128), (9, 200, 0, 8, 256), (9, 300, 1, 5, 256),
                                     (16, 400, 0, 4, 1024), (21, 84, 0, 13, 1024), (21, 325, 0, 7, 1024),
                                     (21, 84, 1, 16, 64), (21, 160, 1, 13, 192)):
        assert not at(S, R, fp32, waves, cells), (S, R, fp32)
