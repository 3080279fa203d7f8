"""The requested pairs' tiles in FP64 (k_tiles64) at their edges: a bundle holds 64 tiles and 16 blocks of
16 rows, in 8 waves, or in 4 up to 32 tiles and 7 blocks; one pair, rows around a block, either order of
a pair, autocorrelations, one and two feeds, a beam per antenna, columns around a stage of 16."""
import numpy as np
import pytest

import oracle
from helpers import say
from paper_2312_09763_amd import matvis as mv
from paper_2312_09763_amd import synth

pytestmark = pytest.mark.gpu


def _pairs(kind, n_ant):
    if kind == "one":
        return [(n_ant - 1, 0)]
    if kind == "all":
        return [(a, b) for a in range(n_ant) for b in range(a, n_ant)]
    if kind == "both":  # either order, and the autocorrelations
        return [(a, b) for a in range(n_ant) for b in range(n_ant) if (a + b) % 3 == 0]
    rng = np.random.default_rng(5)
    return sorted({(int(a), int(b)) for a, b in rng.integers(0, n_ant, (300, 2))})


@pytest.mark.parametrize("workload,n_ant,kind,n_beam,n_src", [
    (1, 2, "one", 1, 40), (1, 16, "all", 1, 33), (1, 17, "all", 3, 31), (1, 112, "all", 1, 47), (1, 113, "all", 1, 48),
    (1, 130, "both", 1, 64), (1, 160, "all", 1, 70), (1, 230, "all", 1, 300), (1, 360, "random", 1, 120),
    (2, 8, "both", 1, 200), (2, 9, "all", 9, 65), (2, 64, "all", 64, 50), (2, 200, "random", 2, 120)])
def test_pair_tiles_fp64(workload, n_ant, kind, n_beam, n_src):
    import torch
    wl = synth.workload(workload, n_ant=n_ant, n_src=n_src, n_time=2, n_freq=2)
    wl.beam = np.concatenate([wl.beam * (1 - 0.005 * b) * np.exp(0.3j * b) for b in range(n_beam)])
    bidx = (np.arange(n_ant) * 7 % n_beam).astype(np.int32)
    pairs = _pairs(kind, n_ant)
    say(f"pair tiles fp64: workload {workload}, {n_ant} antennas, {len(pairs)} pairs ({kind}), {n_beam} beams")
    d = mv.device_inputs(wl, "fp64")
    with mv.Context(mv.config_for(wl, "fp64")) as ctx:
        ctx.set_pairs(pairs, 2)
        V = ctx.simulate_pairs(**d, beam_idx=torch.from_numpy(bidx).cuda()).cpu().numpy()
        ctx.finish()
    V = V.reshape((-1,) + V.shape[2:])
    auto = [(a, a) for a in sorted({p[0] for p in pairs} | {p[1] for p in pairs})]
    ref = oracle.simulate_pairs(wl.antpos, wl.freqs, wl.lsts, wl.ra, wl.dec, wl.flux, wl.beam, wl.latitude, wl.dza,
                                wl.daz, wl.interp, beam_idx=bidx, instances=[(t, f) for t in range(2) for f in range(2)],
                                pairs=pairs + auto)
    scale = np.abs(np.einsum("iupp->iup", ref[:, len(pairs):])).max(axis=(1, 2))
    e = float((np.abs(V - ref[:, :len(pairs)]).max(axis=(1, 2, 3)) / scale).max())
    say(f"  error {e:.2e}")
    assert e <= 1e-10
