"""Z in device memory (MATVIS_FLAG_UNFUSED) in every precision against the oracle: antennas around the
product's super-tiles (64 rows in FP64, 128 otherwise) and the antenna groups of the Z step, several
beams, a polarised sky, k-splits added to fill the grid (calls below their context's capacities, fewer
columns than a split keeps and columns for several splits), sources in chunks, and requested pairs."""
import numpy as np
import pytest

import oracle
from helpers import errors, grid_as_used, say
from paper_2312_09763_amd import matvis as mv
from paper_2312_09763_amd import synth

pytestmark = pytest.mark.gpu

# BF16X3: both operands to 2^-16 and lo lo^H (2^-16) left out, of the Cauchy-Schwarz scale, which a single
# source can reach; the other two are the bars of every parity test
TOL = {"fp64": 1e-10, "fp32": 1e-5, "bf16x3": 3 * 2.0**-16}
PRECISIONS = ["fp64", "fp32", "bf16x3"]


def _workload(workload, n_ant, n_beam, n_src, n_time=2, n_freq=2):
    wl = synth.workload(workload, n_ant=n_ant, n_src=n_src, n_time=n_time, n_freq=n_freq)
    wl.beam = np.concatenate([wl.beam * (1 - 0.05 * b) * np.exp(0.3j * b) for b in range(n_beam)])
    return wl, (np.arange(n_ant) * 7 % n_beam).astype(np.int32)


def _check(V, ref, precision):
    assert np.array_equal(V, np.conj(np.transpose(V, (0, 2, 1, 4, 3))))
    # instances below the smallest value of the output's type have no answer but zero
    low = np.finfo(np.float32).tiny if precision != "fp64" else 0.0
    big = np.abs(ref).reshape(len(ref), -1).max(1) > low
    assert (np.abs(V[~big]) <= low).all()
    if big.any():
        ef, ec = errors(V[big], ref[big])
        say(f"  err_F={ef:.3e} err_CS={ec:.3e}")
        assert ef <= TOL[precision] and ec <= TOL[precision]


def _simulate(wl, bidx, precision, stokes=None, **kw):
    import torch
    cfg = mv.config_for(wl, precision, unfused=True, polarised_sky=stokes is not None, **kw)
    with mv.Context(cfg) as ctx:
        assert ctx.product_path == "z_in_hbm"
        V = ctx.simulate(**mv.device_inputs(wl, precision, stokes=stokes), beam_idx=torch.from_numpy(bidx).cuda())
        ctx.finish()
        V = V.cpu().numpy().astype(np.complex128)
    return V.reshape((-1,) + V.shape[2:])


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("workload,n_ant,n_beam,n_src", [
    (1, 1, 1, 40), (1, 37, 1, 3), (1, 63, 1, 129), (1, 64, 2, 90), (1, 65, 1, 1500), (1, 128, 1, 127), (1, 130, 3, 200),
    (1, 200, 1, 300), (2, 17, 1, 65), (2, 32, 2, 100), (2, 33, 1, 64), (2, 65, 1, 700), (2, 70, 5, 90)])
def test_full_product(precision, workload, n_ant, n_beam, n_src):
    wl, bidx = _workload(workload, n_ant, n_beam, n_src)
    ref = oracle.simulate(wl.antpos, wl.freqs, wl.lsts, wl.ra, wl.dec, wl.flux, grid_as_used(wl, precision), wl.latitude,
                          wl.dza, wl.daz, wl.interp, beam_idx=bidx)
    # its own sizes; capacities above them; chunks; plain k-splits of 64 columns
    for kw in ({}, {"max_time": 5, "max_freq": 3, "max_src": n_src + 700}, {"src_chunk": 64}, {"ksplit": 64}):
        say(f"unfused {precision}: workload {workload}, {n_ant} antennas, {n_beam} beams, {n_src} sources, {kw}")
        _check(_simulate(wl, bidx, precision, **kw), ref, precision)


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("n_ant,n_beam,chunk", [(20, 1, 0), (40, 3, 0), (70, 1, 300)])
def test_polarised_sky(precision, n_ant, n_beam, chunk):
    wl, bidx = _workload(2, n_ant, n_beam, 900)
    st = synth.polarised_stokes(wl.flux, wl.freqs, seed=4)
    say(f"unfused {precision}, polarised sky: {n_ant} antennas, {n_beam} beams, chunk {chunk}")
    ref = oracle.simulate(wl.antpos, wl.freqs, wl.lsts, wl.ra, wl.dec, st, grid_as_used(wl, precision), wl.latitude,
                          wl.dza, wl.daz, wl.interp, beam_idx=bidx)
    _check(_simulate(wl, bidx, precision, stokes=st, src_chunk=chunk), ref, precision)


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("workload,n_ant,n_beam,n_src,n_sub,kw", [
    (1, 37, 1, 1500, 3, {}), (1, 90, 4, 130, 2, {}), (2, 19, 1, 900, 2, {"src_chunk": 256}), (2, 40, 3, 200, 1, {}),
    (1, 64, 1, 300, 2, {"ksplit": 64})])
def test_requested_pairs(precision, workload, n_ant, n_beam, n_src, n_sub, kw):
    import torch
    wl, bidx = _workload(workload, n_ant, n_beam, n_src)
    rng = np.random.default_rng(5)
    pairs = sorted({(int(a), int(b)) for a, b in rng.integers(0, n_ant, (200, 2))} | {(a, a) for a in range(n_ant)})
    say(f"unfused {precision}: {len(pairs)} pairs, workload {workload}, {n_ant} antennas, {n_beam} beams, {kw}")
    with mv.Context(mv.config_for(wl, precision, unfused=True, **kw)) as ctx:
        ctx.set_pairs(pairs, n_sub)
        V = ctx.simulate_pairs(**mv.device_inputs(wl, precision), beam_idx=torch.from_numpy(bidx).cuda())
        ctx.finish()
        V = V.cpu().numpy().astype(np.complex128)
    V = V.reshape((-1,) + V.shape[2:])
    ref = oracle.simulate_pairs(wl.antpos, wl.freqs, wl.lsts, wl.ra, wl.dec, wl.flux, grid_as_used(wl, precision),
                                wl.latitude, wl.dza, wl.daz, wl.interp, beam_idx=bidx,
                                instances=[(t, f) for t in range(2) for f in range(2)], pairs=pairs)
    auto = [u for u, (a, b) in enumerate(pairs) if a == b]
    scale = np.abs(np.einsum("iupp->iup", ref[:, auto])).max(axis=(1, 2))
    e = float((np.abs(V - ref).max(axis=(1, 2, 3)) / scale).max())
    say(f"  error {e:.2e}")
    assert e <= TOL[precision]
