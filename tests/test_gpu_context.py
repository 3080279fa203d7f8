"""Contexts: what creating one costs, and that nothing depends on the memory it finds."""
import statistics
import time

import numpy as np
import pytest

from helpers import errors, grid_as_used, oracle_vis, say

pytestmark = pytest.mark.gpu


def test_small_context_costs_no_more_than_an_unfused_one():
    """A small context that multiplies tiles uploads their list; an unfused one holds the Z of a batch instead.
    A transfer of its own in the middle of the allocations made the former take twice the latter's time."""
    import torch
    from paper_2312_09763_amd import matvis as mv
    from paper_2312_09763_amd import synth
    wl = synth.workload(1, n_ant=37, n_src=2000, n_time=4, n_freq=2)
    times = []
    for unfused in (True, False, True, False):  # (one kind after another: the allocator keeps the last one's pieces)
        cfg = mv.config_for(wl, "fp64", unfused=unfused)
        t = []
        for _ in range(50):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            with mv.Context(cfg):
                t.append(time.perf_counter() - t0)
        times.append(statistics.median(t))
    unfused, fused = min(times[0::2]), min(times[1::2])
    say(f"context creation: {fused * 1e6:.0f} us, unfused {unfused * 1e6:.0f} us")
    assert fused <= 1.15 * unfused


@pytest.mark.parametrize("precision,unfused", [("fp64", False), ("fp64", True), ("fp32", False), ("fp32", True),
                                               ("bf16x3", False), ("bf16x3", True)])
def test_results_do_not_depend_on_the_memory_found(precision, unfused):
    """Contexts whose buffers lie in memory full of NaNs, for the whole call and for the product step alone."""
    import torch
    from paper_2312_09763_amd import matvis as mv
    from paper_2312_09763_amd import synth
    tol = {"fp64": 1e-10, "fp32": 1e-5, "bf16x3": 3e-5}[precision]
    for workload, n_ant in ((1, 37), (2, 20), (2, 70)):
        say(f"context in NaNs: {precision}, unfused {unfused}, workload {workload}, {n_ant} antennas")
        wl = synth.workload(workload, n_ant=n_ant, n_src=300, n_time=2, n_freq=2)
        cfg = mv.config_for(wl, precision, unfused=unfused)
        d = mv.device_inputs(wl, precision)
        junk = [torch.full((1 << 20,), float("nan"), dtype=torch.float64, device="cuda") for _ in range(64)]
        torch.cuda.synchronize()
        del junk
        torch.cuda.empty_cache()
        with mv.Context(cfg) as ctx:
            V = ctx.simulate(**d).cpu().numpy().astype(np.complex128)
            ctx.finish()
            n_row = n_ant * wl.beam.shape[2] - 3
            g = torch.Generator(device="cuda").manual_seed(1)
            dt = torch.complex128 if precision == "fp64" else torch.complex64
            Z = torch.randn((n_row, 130), generator=g, device="cuda", dtype=dt)
            P = ctx.step_herk(Z).cpu().numpy().astype(np.complex128)
        ef, ec = errors(V.reshape((-1,) + V.shape[2:]), oracle_vis(wl, grid=grid_as_used(wl, precision)))
        Zh = Z.cpu().numpy().astype(np.complex128)
        scale = np.sqrt(np.outer((abs(Zh) ** 2).sum(1), (abs(Zh) ** 2).sum(1)))
        ep = (abs(P - Zh @ Zh.conj().T) / scale).max()
        say(f"  err_F={ef:.3e} err_CS={ec:.3e}, product step {ep:.3e}")
        assert ef <= tol and ec <= tol and ep <= tol
