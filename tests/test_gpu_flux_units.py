"""FP32 results do not depend on the unit of the fluxes: 1 Jy is 1e-26 W / (m^2 Hz), and faint pixels in such
units come near the end of FP32's range, which the low terms of a split operand must not reach first."""
import numpy as np
import pytest

import oracle
from helpers import errors, grid_as_used, gpu_simulate, say
from paper_2312_09763_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("workload,n_ant", [(1, 37), (1, 150), (1, 300), (2, 20), (2, 70), (2, 90), (2, 200), (2, 300)])
def test_fp32_over_the_range_of_fluxes(workload, n_ant):
    wl = synth.workload(workload, n_ant=n_ant, n_src=300, n_time=1, n_freq=2)
    ref = oracle.simulate(wl.antpos, wl.freqs, wl.lsts, wl.ra, wl.dec, wl.flux, grid_as_used(wl, "fp32"), wl.latitude,
                          wl.dza, wl.daz, wl.interp)
    flux = wl.flux
    for unit in (1e30, 1.0, 1e-26, 1e-33, 1e-35, 1e-36):
        wl.flux = flux * unit
        ef, ec = errors(gpu_simulate(wl, "fp32") / unit, ref)
        say(f"flux unit {unit:.0e}: workload {workload}, {n_ant} antennas: err_F={ef:.2e} err_CS={ec:.2e}")
        assert ef <= 1e-5 and ec <= 1e-5
