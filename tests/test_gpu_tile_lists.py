"""The full product over 16 x 16 tiles (kernels_tiles.hip) at its edges: one antenna, rows around a block
of 16, the row and tile counts where a workgroup goes from 4 to 8 to 16 waves and a product to two
bundles and to rectangles, one and several beams, one and two feeds, few columns and several chunks.
Operands are exact to FP32 rounding on FP32 (three bf16 terms) and to 2^-16 on BF16X3 (two roundings to
8 bits)."""
import numpy as np
import pytest

import oracle
from helpers import errors, gpu_simulate, grid_as_used, say
from paper_2312_09763_amd import synth

pytestmark = pytest.mark.gpu

# FP32: sine and cosine on the hardware to 2^-21 each: 1e-6, twice that; BF16X3: both operands, 2 x 2^-16
# of the Cauchy-Schwarz scale, which a single source can reach
TOL = {"fp32": 2e-6, "bf16x3": 2.0**-15}


@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
@pytest.mark.parametrize("workload,n_ant,n_beam,n_src", [
    (1, 1, 1, 40), (1, 16, 1, 15), (1, 17, 1, 16), (1, 80, 1, 65), (1, 81, 1, 100), (1, 128, 2, 90), (2, 1, 1, 64),
    (2, 16, 1, 300), (2, 17, 1, 33), (2, 32, 1, 100), (2, 49, 1, 50), (2, 64, 1, 200), (2, 8, 3, 100), (2, 41, 5, 40),
    (2, 193, 2, 60)])
def test_full_product_tiles(precision, workload, n_ant, n_beam, n_src):
    import torch
    wl = synth.workload(workload, n_ant=n_ant, n_src=n_src, n_time=2, n_freq=2)
    say(f"tile lists {precision}: workload {workload}, {n_ant} antennas, {n_beam} beams, {n_src} sources")
    wl.beam = np.concatenate([wl.beam * (1 - 0.05 * b) * np.exp(0.3j * b) for b in range(n_beam)])
    bidx = (np.arange(n_ant) * 7 % n_beam).astype(np.int32)
    ref = oracle.simulate(wl.antpos, wl.freqs, wl.lsts, wl.ra, wl.dec, wl.flux, grid_as_used(wl, precision), wl.latitude,
                          wl.dza, wl.daz, wl.interp, beam_idx=bidx)
    for kw in ({}, {"src_chunk": 64}):
        V = gpu_simulate(wl, precision, beam_idx=torch.from_numpy(bidx).cuda(), **kw)
        # instances whose few sources all lie where the beam's square is below the smallest complex64 value
        # have no FP32 answer but zero
        big = np.abs(ref).max(axis=(1, 2, 3, 4)) > np.finfo(np.float32).tiny
        assert (np.abs(V[~big]) <= np.finfo(np.float32).tiny).all()
        if not big.any():
            continue
        ef, ec = errors(V[big], ref[big])
        say(f"  {kw}: err_F={ef:.3e} err_CS={ec:.3e}")
        assert ef <= TOL[precision] and ec <= TOL[precision]


@pytest.mark.parametrize("n_ant,n_beam", [(129, 1), (208, 1), (209, 1), (256, 1), (300, 2)])
def test_scalar_fp32_bundles(n_ant, n_beam):
    import torch
    wl = synth.workload(1, n_ant=n_ant, n_src=150, n_time=1, n_freq=2)
    wl.beam = np.concatenate([wl.beam * (1 - 0.05 * b) for b in range(n_beam)])
    bidx = (np.arange(n_ant) % n_beam).astype(np.int32)
    ref = oracle.simulate(wl.antpos, wl.freqs, wl.lsts, wl.ra, wl.dec, wl.flux, grid_as_used(wl, "fp32"), wl.latitude,
                          wl.dza, wl.daz, wl.interp, beam_idx=bidx)
    V = gpu_simulate(wl, "fp32", beam_idx=torch.from_numpy(bidx).cuda())
    ef, ec = errors(V, ref)
    say(f"scalar fp32, {n_ant} antennas: err_F={ef:.3e} err_CS={ec:.3e}")
    assert ef <= 2e-6 and ec <= 2e-6
    assert np.array_equal(V, np.conj(np.transpose(V, (0, 2, 1, 4, 3))))


@pytest.mark.parametrize("workload,n_ant,n_beam,n_src", [
    (1, 1, 1, 40), (1, 16, 1, 31), (1, 17, 1, 33), (1, 112, 1, 90), (1, 113, 1, 64), (1, 160, 2, 100), (1, 161, 1, 70),
    (1, 256, 1, 120), (1, 300, 1, 90), (2, 8, 3, 100), (2, 41, 5, 40), (2, 100, 2, 60)])
def test_fp64_tiles(workload, n_ant, n_beam, n_src):
    import torch
    wl = synth.workload(workload, n_ant=n_ant, n_src=n_src, n_time=2, n_freq=2)
    say(f"tile lists fp64: workload {workload}, {n_ant} antennas, {n_beam} beams, {n_src} sources")
    wl.beam = np.concatenate([wl.beam * (1 - 0.05 * b) * np.exp(0.3j * b) for b in range(n_beam)])
    bidx = (np.arange(n_ant) * 7 % n_beam).astype(np.int32)
    ref = oracle.simulate(wl.antpos, wl.freqs, wl.lsts, wl.ra, wl.dec, wl.flux, wl.beam, wl.latitude, wl.dza, wl.daz,
                          wl.interp, beam_idx=bidx)
    for kw in ({}, {"src_chunk": 64}):
        V = gpu_simulate(wl, "fp64", beam_idx=torch.from_numpy(bidx).cuda(), **kw)
        ef, ec = errors(V, ref)
        say(f"  {kw}: err_F={ef:.3e} err_CS={ec:.3e}")
        assert ef <= 1e-10 and ec <= 1e-10
