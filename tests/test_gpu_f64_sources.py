"""FP64 product over sources (k_herk_coh64) against the FP64 oracle at 1e-10: one block of 64 antennas
(both halves of the workgroup share its sources), an odd and an even number of blocks, short last
blocks of every tile count, sources around the stage (16) and its halves, a polarised sky, and the
sub-matrix product of the same context."""
import numpy as np
import pytest

from helpers import errors, say
from paper_2312_09763_amd import matvis as mv
from paper_2312_09763_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_ant,n_src", [(1, 30), (16, 200), (33, 1), (33, 40), (48, 33), (64, 31), (64, 1000), (65, 300),
                                         (100, 70), (128, 500), (129, 90), (180, 64), (192, 130), (250, 41)])
def test_against_oracle(n_ant, n_src):
    import oracle
    wl = synth.workload(2, n_ant=n_ant, n_src=n_src, n_time=2, n_freq=2)
    say(f"fp64 over sources: {n_ant} antennas, {n_src} sources")
    d = mv.device_inputs(wl, "fp64")
    with mv.Context(mv.config_for(wl, "fp64")) as ctx:
        V = ctx.simulate(**d).cpu().numpy()
        ctx.finish()
    V = V.reshape((-1,) + V.shape[2:])
    assert np.array_equal(V, np.conj(np.transpose(V, (0, 2, 1, 4, 3))))
    ref = oracle.simulate(wl.antpos, wl.freqs, wl.lsts, wl.ra, wl.dec, wl.flux, wl.beam, wl.latitude, wl.dza, wl.daz,
                          wl.interp)
    seen = np.abs(ref).reshape(len(ref), -1).max(1) > 0
    assert np.all(V[~seen] == 0)
    if seen.any():
        ef, ec = errors(V[seen], ref[seen])
        say(f"  err_F={ef:.3e} err_CS={ec:.3e}")
        assert ef <= 1e-10 and ec <= 1e-10


@pytest.mark.parametrize("n_ant", [40, 100])
def test_against_z_in_memory(n_ant):
    """The same inputs with Z in device memory (unfused), for a polarised sky, several source
    chunks, and the sub-matrix product, which takes Z on both."""
    wl = synth.workload(2, n_ant=n_ant, n_src=900, n_time=2, n_freq=3)
    st = synth.polarised_stokes(wl.flux, wl.freqs, seed=4)
    d = mv.device_inputs(wl, "fp64", stokes=st)
    pairs = [(0, 0), (n_ant - 1, 3), (5, n_ant - 1), (7, 7)]
    out = []
    for kw in (dict(), dict(src_chunk=250), dict(unfused=True)):
        with mv.Context(mv.config_for(wl, "fp64", polarised_sky=True, **kw)) as ctx:
            V = ctx.simulate(**d).cpu().numpy()
            ctx.set_pairs(pairs, 2)
            S = ctx.simulate_pairs(**d).cpu().numpy()
            ctx.finish()
        out.append((V, S))
    for V, S in out:
        assert errors(V.reshape((-1,) + V.shape[2:]), out[-1][0].reshape((-1,) + V.shape[2:]))[1] <= 1e-12
        scale = np.abs(out[-1][1]).max()
        assert np.abs(S - out[-1][1]).max() <= 1e-12 * scale
        want = V[:, :, [a for a, _ in pairs], [b for _, b in pairs]]
        assert np.abs(S - want).max() <= 1e-12 * scale
