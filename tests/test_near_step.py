"""The step rule of the search for a query's second rank next to its first one
(csrc/near.hpp), compiled for the host and run over sorted arrays: every rank
that lies in the first line looked at or the line next to it, the boundary
between the two included, is decided within those two lines, and what is
decided equals the bisection's rank."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_1208_3407_amd import build

HARNESS = r"""
#include "near.hpp"
// Looks taken until the rank of x from the line at w on is known (at most `most`; 0 = still open).
extern "C" uint32_t near_looks(const uint32_t* K, uint32_t n, uint32_t w, uint32_t x, uint32_t most, uint32_t* rank) {
    uint32_t r = bits::kNoLine;
    for (uint32_t k = 1; k <= most; ++k) {
        uint32_t cnt = 0;
        for (uint32_t i = w; i < w + 32u && i < n; ++i) cnt += K[i] < x ? 1u : 0u;
        if (bits::near_step(n, cnt, w, r)) {
            *rank = r;
            return k;
        }
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("near")
    src, out = os.path.join(d, "near.hip"), os.path.join(d, "near.so")
    with open(src, "w") as f:
        f.write(HARNESS)
    subprocess.run([build.hipcc(), "--cuda-host-only", "-O1", "-std=c++17", "-fPIC", "-shared", "-I", build.SRC, src, "-o", out],
                   check=True, capture_output=True, timeout=300)
    L = ctypes.CDLL(out)
    L.near_looks.restype = ctypes.c_uint32
    return L


@pytest.mark.parametrize("n", [1, 31, 32, 33, 64, 65, 96, 97, 1000, 1024])
@pytest.mark.parametrize("step", [1, 3, 40])   # 40: runs of equal keys longer than a line
def test_two_lines_decide(lib, n, step):
    K = (np.arange(n, dtype=np.uint32) // step) * 10 + 5
    kp = K.ctypes.data_as(ctypes.c_void_p)
    for x in range(0, int(K[-1]) + 11, 5):
        r = int(np.searchsorted(K, x, side="left"))
        for w in range(0, n, 32):
            got = ctypes.c_uint32(0)
            looks = lib.near_looks(kp, n, w, x, 40, ctypes.byref(got))
            assert looks and got.value == r, (n, x, w)
            # lines between the first one and the nearest that touches the rank, and the one that decides it
            away = max(0, w - r, r - w - 32)
            assert looks <= 2 + (away + 31) // 32, (n, x, w, r, looks)
            if w - 32 <= r <= w + 64 and away == 0:
                assert looks <= 2, (n, x, w, r, looks)
