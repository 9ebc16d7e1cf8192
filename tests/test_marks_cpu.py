"""The running count behind the marks of a pool (32 bits, advanced by every
payload of every edit batch): no batch wraps it, and marks that stay are below
every mark of the next batch."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = """
#include "cvx_internal.h"
extern "C" int again(uint32_t epoch, uint64_t n_paint, int fresh) {
  return cvx::count_again(epoch, n_paint, fresh != 0);
}
extern "C" uint32_t runs() { return cvx::kLinkRuns; }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("marks")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(ROOT, "paper_1704_02724_amd", "csrc"), "-o",
                    str(d / "shim.so"), str(d / "shim.cpp")], check=True)
    lib = ctypes.CDLL(str(d / "shim.so"))
    lib.again.argtypes = [ctypes.c_uint32, ctypes.c_uint64, ctypes.c_int]
    lib.runs.restype = ctypes.c_uint32
    return lib


@pytest.mark.parametrize("seed", range(8))
def test_no_batch_wraps(lib, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    epoch, largest, runs, again = 0, 0, lib.runs(), 0
    for _ in range(2000):
        n = int(2 ** rng.uniform(0, 31))
        grow = rng.random() < 0.01
        if lib.again(epoch, n, grow):
            epoch = largest = 0
            again += not grow
        assert largest < epoch + 1           # the marks that stay are older
        largest = epoch + n + int(rng.integers(0, runs + 1))
        assert largest <= 0xFFFFFFFF         # the batch's own marks fit
        epoch = largest
    assert again > 0


def test_new_marks_start_from_zero(lib):
    """Marks that grow with the pool in the batch that would wrap."""
    assert lib.again(0xFFFFFFF0, 1000, 1)
    assert lib.again(0xFFFFFFF0, 1000, 0)
    assert lib.again(5, 0xFFFFFF00, 0) == 0
    assert not lib.again(5, 10, 0)
