"""The launch rules of csrc/launch_rules.h, compiled on their own for the host."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2312_09763_amd", "csrc")
SOURCE = """
#include "launch_rules.h"
extern "C" void tf_grid(int64_t max_m, int spb, int n_slot, int n_freq, int fg, int n_beam, int64_t *out) {
    const mv::TfGrid g = mv::tf_grid(max_m, spb, n_slot, n_freq, fg, n_beam);
    out[0] = g.x, out[1] = g.y, out[2] = g.z;
}
// k-splits of the product over sources: n and columns of each instance; out: launches, items and weights
extern "C" int sources_splits(int n_ant, int n_rows_pad, int64_t ksplit, int grid, int plain, int max_splits, int n_slot, int nfb,
                              const int64_t *K, int32_t *n, int64_t *kc, int32_t *items, int32_t *weight, int32_t *part) {
    mv::SplitRule r{};
    r.ksplit = ksplit, r.grid = grid, r.n_st = 1, r.n_bal = 1, r.max_splits = max_splits, r.plain_splits = plain;
    mv::sources_launches(n_ant, n_rows_pad, r);
    mv::OneThread g;
    const mv::SplitPlan p = mv::plan_splits(r, n_slot, nfb, [&](int s) { return K[s]; }, g);
    for (int i = 0; i < n_slot * nfb; i++) {
        const mv::Split s = mv::split_of(r, p, K[i / nfb], i);
        n[i] = s.n, kc[i] = s.kc;
    }
    for (int l = 0; l < 3; l++) items[l] = r.items[l], weight[l] = r.weight[l];
    *part = r.part_cost;
    return r.n_launch;
}
// the room that a context keeps for them: at most `most` splits of K columns or half of them
extern "C" int splits_room(int n_ant, int n_rows_pad, int64_t ksplit, int grid, int plain, int most, int n_slot, int nfb,
                           int64_t K) {
    mv::SplitRule r{};
    r.ksplit = ksplit, r.grid = grid, r.n_st = 1, r.n_bal = 1, r.max_splits = most, r.plain_splits = plain;
    mv::sources_launches(n_ant, n_rows_pad, r);
    const int n = r.n_launch > 1 ? mv::splits_wanted(r, n_slot, nfb, K) : most;
    return n > plain ? n : plain;
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


def _round(K, n):
    kc = -(-(-(-K // n)) // 64) * 64
    return -(-K // kc), kc


def _fill_grid(K, ksplit, grid, cap, n_bal):
    """Splits added until items (n_bal a split) fill whole waves of the grid, at most `cap` an instance."""
    n0 = [-(-k // ksplit) for k in K]
    t = sum(n0)
    n = 1 if t >= grid else n_bal
    extra = max(-(-t * n // grid) * grid // n - t, 0)
    out = []
    for i, k in enumerate(K):
        want = n0[i] + extra // len(K) + (i < extra % len(K))
        out.append(_round(k, max(n0[i], min(want, cap, -(-k // 64)))))
    return out


def _queue_time(splits, launches, part, K, grid=256):
    """Every launch's items taken by the workgroups in turn, each its columns and a fill; and the partials."""
    time = sum(n for n, _ in splits) * part
    length = np.array([min(kc, K[i] - s * kc) for i, (n, kc) in enumerate(splits) for s in range(n)])
    for items, weight in launches:
        item = np.repeat(weight * length + 24480, items)
        slot = np.zeros(-(-len(item) // grid) * grid)
        slot[:len(item)] = item
        time += slot.reshape(-1, grid).sum(0).max()
    return time


@pytest.mark.parametrize("up", [(0.5, 0.42, 0.47, 0.45, 0.49), (0.5, 0.42, 0.61, 0.47, 0.55)])
@pytest.mark.parametrize("n_src", [1000, 20_000, 40_000, 120_000])
@pytest.mark.parametrize("n_slot,nfb", [(1, 2), (2, 4), (3, 4), (4, 16), (3, 16), (7, 5), (15, 16), (5, 1)])
def test_splits_of_the_launches_over_sources(rules, up, n_src, n_slot, nfb):
    """Against the two simpler rules -- fill the grid with splits, of no more than the plain ones' capacity; and
    count the launches as one of an item per block -- the chosen splits' time is no longer, and rounding does
    not grow: no fewer splits than the first rule's unless they are short.  (12 % for the model's even splits; at
    1000 sources, where a whole split is a few stages and the last ones are shorter, 20 %.)"""
    grid, ksplit, slack = 256, 20_480, 1.2 if n_src == 1000 else 1.12
    vis = [int(n_src * f) for f in up]
    K = [2 * vis[s % 5] for s in range(n_slot) for _ in range(nfb)]
    plain = -(-2 * n_src // ksplit)
    slower = 0
    for n_ant in range(65, 361, 5):
        n_pad = -(-2 * n_ant // 256) * 256
        nb, B = n_pad // 256, n_slot * nfb
        most = max(plain, min(plain + -(-grid // B), -(-2 * n_src // 64), (1 << 30) // (B * n_pad * n_pad * 8)))
        most = rules.splits_room(n_ant, n_pad, ctypes.c_int64(ksplit), grid, plain, most, n_slot, nfb,
                                 ctypes.c_int64(2 * n_src))
        n, kc = (ctypes.c_int32 * B)(), (ctypes.c_int64 * B)()
        items, weight, part = (ctypes.c_int32 * 3)(), (ctypes.c_int32 * 3)(), ctypes.c_int32()
        slots = (ctypes.c_int64 * n_slot)(*K[::nfb])
        count = rules.sources_splits(n_ant, n_pad, ctypes.c_int64(ksplit), grid, plain, most, n_slot, nfb, slots, n, kc, items,
                                     weight, ctypes.byref(part))
        launches = list(zip(items[:count], weight[:count]))
        short = n_ant - (nb - 1) * 128 <= 96
        assert sum(i for i, _ in launches) == nb + (nb * (nb - 1) if nb > 1 else 0)
        assert count == (short and nb > 1) + 1 + (nb > 1)
        mine = list(zip(list(n), list(kc)))
        for i in range(B):
            assert 1 <= n[i] <= most and (n[i] - 1) * kc[i] < K[i] <= n[i] * kc[i] and kc[i] <= ksplit
        args = (launches, part.value, K)
        time = _queue_time(mine, *args)
        filled = _fill_grid(K, ksplit, grid, plain, 1)
        as_one = _fill_grid(K, ksplit, grid, most, nb)
        assert time <= slack * _queue_time(filled, *args), (n_ant, mine, filled)
        if sum(n for n, _ in as_one) >= sum(n for n, _ in filled) or max(kc for _, kc in as_one) <= 2048:
            assert time <= slack * _queue_time(as_one, *args), (n_ant, mine, as_one)
        if nb > 1:
            slower += _queue_time(as_one, *args) > 1.2 * time
            assert sum(n) >= sum(f for f, _ in filled) or max(kc) <= 2048
    if (n_src, n_slot, nfb, up[2]) == (40_000, 4, 16, 0.47):
        assert slower >= 38  # 130..220 and 260..350 antennas: what the count as one launch cost
