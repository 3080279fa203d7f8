"""The launch rules of csrc/launch_rules.h, compiled on their own for the host."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2312_09763_amd", "csrc")
SOURCE = """
#include "launch_rules.h"
extern "C" void tf_grid(int64_t max_m, int spb, int n_slot, int n_freq, int fg, int n_beam, int64_t *out) {
    const mv::TfGrid g = mv::tf_grid(max_m, spb, n_slot, n_freq, fg, n_beam);
    out[0] = g.x, out[1] = g.y, out[2] = g.z;
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, lib = str(d / "rules.cpp"), str(d / "rules.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, src, "-o", lib],
                   check=True)
    return ctypes.CDLL(lib)


@pytest.mark.parametrize("n_beam,ncomp,bytes_per,n_src,n_slot,n_freq", [
    (128, 4, 8, 3_145_728, 16, 1), (128, 4, 8, 3_145_728, 6, 3), (128, 4, 8, 3_145_728, 3, 5),
    (1, 4, 8, 1 << 22, 256, 1), (1, 4, 8, 1 << 22, 64, 5), (1, 1, 16, 1 << 18, 4096, 16), (8192, 4, 8, 1 << 14, 1, 1000)])
def test_beam_grid_within_launch_limits(rules, n_beam, ncomp, bytes_per, n_src, n_slot, n_freq):
    """Batches that fit the memory stay within HIP's limits per grid dimension, and the blocks cover them."""
    fg = 2 if n_freq <= 2 else 4
    spb = 256 // max(1, fg * ncomp * bytes_per // 16)
    out = (ctypes.c_int64 * 3)()
    rules.tf_grid(ctypes.c_int64(n_src), spb, n_slot, n_freq, fg, n_beam, out)
    x, y, z = out
    assert x * 256 < 1 << 32 and y <= 65535, (x, y)  # z is cut into launches
    assert x % 8 == 0 and x * spb >= n_src
    assert y == n_slot and z == -(-n_freq // fg) * -(-n_beam // 4)
