"""The beam step's layout at its edges: values per grid point around the tile widths of the channel
interleaving (odd counts, one more than a tile), beams around the group of 4 that one block
evaluates, one to five channels, few and odd source counts."""
import numpy as np
import pytest

import oracle
from helpers import TOL, errors, gpu_simulate, grid_as_used, say
from paper_2312_09763_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("workload,n_beam,n_freq,n_src", [(1, 1, 1, 7), (1, 3, 3, 130), (1, 4, 8, 65), (1, 5, 9, 300),
                                                          (1, 2, 17, 90), (1, 1, 33, 64), (2, 1, 1, 33), (2, 5, 2, 257),
                                                          (2, 8, 3, 120), (2, 9, 5, 40), (2, 2, 17, 70)])
def test_beam_step_edges(precision, workload, n_beam, n_freq, n_src):
    import torch
    wl = synth.workload(workload, n_ant=12, n_src=n_src, n_time=3, n_freq=n_freq)
    say(f"beam groups {precision}: workload {workload}, {n_beam} beams, {n_freq} channels, {n_src} sources")
    wl.beam = np.concatenate([wl.beam * (1 - 0.05 * b) * np.exp(0.3j * b) for b in range(n_beam)])
    bidx = (np.arange(12) * 7 % n_beam).astype(np.int32)
    V = gpu_simulate(wl, precision, beam_idx=torch.from_numpy(bidx).cuda())
    ref = oracle.simulate(wl.antpos, wl.freqs, wl.lsts, wl.ra, wl.dec, wl.flux, grid_as_used(wl, precision), wl.latitude,
                          wl.dza, wl.daz, wl.interp, beam_idx=bidx)
    # instances whose few sources all lie where the beam is below the smallest complex64 value have no
    # FP32 answer but zero
    big = np.abs(ref).max(axis=(1, 2, 3, 4)) > (np.finfo(np.float32).tiny if precision == "fp32" else 0.0)
    assert (np.abs(V[~big]) <= np.finfo(np.float32).tiny).all()
    V, ref = V[big], ref[big]
    if not len(V):
        return
    ef, ec = errors(V, ref)
    say(f"  err_F={ef:.3e} err_CS={ec:.3e}")
    assert ef <= TOL[precision] and ec <= TOL[precision]
