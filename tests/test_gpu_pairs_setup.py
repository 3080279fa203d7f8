"""Planning requested pairs: every pair of 128 polarised antennas."""
import ctypes
import statistics
import time

import numpy as np
import pytest

from helpers import say
from paper_2312_09763_amd import matvis as mv
from paper_2312_09763_amd import synth

pytestmark = pytest.mark.gpu


def _median_us(f):
    t = []
    for _ in range(15):
        t0 = time.perf_counter()
        f()
        t.append(time.perf_counter() - t0)
    return statistics.median(t) * 1e6


def test_tile_lists_cost_little_beside_the_plan():
    """matvis_set_pairs is the App. A plan (host), the tile lists and their upload; the lists took several times
    the plan's time when their tables were ordered maps."""
    n = 128
    pairs = np.array([(a, b) for a in range(n) for b in range(a, n)], dtype=np.int32)
    pa, pb = np.ascontiguousarray(pairs[:, 0]), np.ascontiguousarray(pairs[:, 1])
    L = mv.load_library()
    alpha, sizes, dens = np.empty(n, np.int32), np.empty(8, np.int32), np.empty(8)
    n_alpha, n_sub, size = ctypes.c_int32(), ctypes.c_int32(), ctypes.c_int64()
    plan = _median_us(lambda: L.matvis_submatrix_plan(pa.ctypes.data, pb.ctypes.data, len(pa), n, 3, alpha.ctypes.data,
                                                      sizes.ctypes.data, dens.ctypes.data, ctypes.byref(n_alpha),
                                                      ctypes.byref(n_sub)))
    wl = synth.workload(2, n_ant=n, n_src=300, n_time=1, n_freq=1)
    with mv.Context(mv.config_for(wl, "fp32")) as ctx:
        st = []
        whole = _median_us(lambda: st.append(L.matvis_set_pairs(ctx._h, pa.ctypes.data, pb.ctypes.data, len(pa), 3,
                                                                ctypes.byref(size))))
    say(f"set_pairs of {len(pa)} pairs: {whole:.0f} us, of which the plan {plan:.0f} us")
    assert st == [mv.OK] * 15
    assert whole <= 4 * plan
