"""The rules that choose a kernel variant by size (csrc/fd_rules.h), compiled for the CPU: each
rule on both sides of its lines, at sizes where both variants were measured on an MI355X."""
import ctypes
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_12121_amd", "csrc")
CUS = 256

SHIM = r"""
#include "fd_rules.h"
extern "C" {
int score_one_pass(int regions, long long values, int cus) { return fd::score_one_pass(regions, values, cus); }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("needs a C++ compiler")
    d = tmp_path_factory.mktemp("rules")
    src, so = d / "rules.cpp", d / "rules.so"
    src.write_text(SHIM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", f"-I{CSRC}", str(src), "-o", str(so)],
                   check=True)
    lib = ctypes.CDLL(str(so))
    lib.score_one_pass.argtypes = [ctypes.c_int, ctypes.c_longlong, ctypes.c_int]
    return lib


@pytest.mark.parametrize("regions,values,one_pass", [
    (1, 8192, True), (64, 8192, True), (511, 8192, True),
    # few large regions are cut: one pass took up to 2.3 times as long
    (1, 65536, False), (4, 65536, False), (16, 16 * 1024, False), (16, 65536, False), (64, 16384, False), (64, 65536, False),
    (127, 16384, False), (140, 24576, False), (191, 65536, False),
    # enough of them are not
    (128, 16384, True), (140, 14976, True), (192, 65536, True), (511, 65536, True), (511, 65537, False), (512, 1 << 40, True),
])
def test_score_pass(rules, regions, values, one_pass):
    assert bool(rules.score_one_pass(regions, values, CUS)) == one_pass
