"""The room for the O and W2 products' partial sums, from the library's own host
function: at least the K parts times rows of each launch that it is sized for.
Sized by the larger row count alone, 3310 prefill rows (one part) left no room
for the 3480 rows that rounds of 1740 in two parts write."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#include "split_k.h"
extern "C" int parts(int rows, int n, int k) { return hbsjd::split_for(rows, n, k); }
extern "C" long room(long a, long b, int d, int f, int f16) {
    return (long)hbsjd::partial_sum_rows(a, b, d, f, f16 != 0);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("split_k")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                           os.path.join(ROOT, "paper_2608_18183_amd", "csrc"),
                           str(d / "shim.cpp"), "-o", str(d / "shim.so")])
    so = ctypes.CDLL(str(d / "shim.so"))
    so.room.restype = ctypes.c_long
    so.room.argtypes = [ctypes.c_long, ctypes.c_long] + [ctypes.c_int] * 3
    return so


# d, f of the B, L and XL models and of a narrow one
@pytest.mark.parametrize("d,f", [(768, 2048), (1024, 2816), (1280, 3456), (128, 192)])
def test_room_holds_every_launch(lib, d, f):
    rng = np.random.default_rng(d)
    rows = [0, 1, 63, 64, 65, 1740, 3016, 3310, 8448]
    rows += np.exp(rng.uniform(0, np.log(20000), 60)).astype(int).tolist()
    need = {r: max(lib.parts(r, d, d), lib.parts(r, d, f)) * r if r else 0 for r in rows}
    for a in rows:
        for b in rows:
            assert lib.room(a, b, d, f, 1) == max(need[a], need[b])
            assert lib.room(a, b, d, f, 0) == max(a, b)


def test_fewer_rows_may_need_more_room(lib):
    assert lib.parts(3310, 768, 768) == lib.parts(3310, 768, 2048) == 1
    assert lib.parts(1740, 768, 2048) == 2
    assert lib.room(3310, 1740, 768, 2048, 1) == 3480
