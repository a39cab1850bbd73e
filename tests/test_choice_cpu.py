"""The size rules of csrc/choice.h, compiled for the host."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1912_02057_amd", "csrc")

SHIM = r"""
#include "choice.h"
extern "C" void pack_form(int planes, int64_t rows, int64_t Kpad, int *out)
{
    const rtn::PackRowsForm f = planes ? rtn::pack_rows_planes_form(rows, Kpad) : rtn::pack_rows_form(rows, Kpad);
    out[0] = f.waves, out[1] = f.steps, out[2] = f.step;
}
"""


@pytest.fixture(scope="module")
def L(tmp_path_factory):
    d = tmp_path_factory.mktemp("choice")
    (d / "shim.cpp").write_text(SHIM)
    so = str(d / "choice.so")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + CSRC, str(d / "shim.cpp"), "-o", so], check=True)
    lib = C.CDLL(so)
    lib.pack_form.argtypes = [C.c_int, C.c_int64, C.c_int64, C.c_void_p]
    return lib


@pytest.mark.parametrize("planes", [0, 1])
def test_row_pack_waves_have_work(L, planes):
    """Of the waves that share a row at most one has no elements of it, at any length."""
    out = (C.c_int * 3)()
    for rows in (1, 16, 500, 2047, 2048, 100000):
        for Kpad in list(range(64, 9000, 64)) + [1 << 20]:
            L.pack_form(planes, rows, Kpad, out)
            waves, turn = out[0], out[1] * out[2]
            assert waves in (1, 4) and turn > 0
            assert waves == 1 or (waves - 2) * turn < Kpad, (rows, Kpad, list(out))
