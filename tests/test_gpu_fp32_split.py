"""FP32 products as six bf16 products (kernels_herk_x6.hip) at the edges of antenna blocks and tile
rows: product over sources (diagonal blocks, short last blocks, block pairs) and the three-block
scalar product.  The products are exact to FP32 rounding, so what is left is the hardware sine and
cosine (2^-21 of a unit, both operands: 1e-6); the bar is twice that, a fifth of FP32's own."""
import numpy as np
import pytest

from helpers import errors, grid_as_used, say
from paper_2312_09763_amd import matvis as mv
from paper_2312_09763_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("workload,n_ant,n_src", [(2, 65, 300), (2, 80, 33), (2, 96, 500), (2, 97, 200), (2, 128, 300),
                                                  (2, 129, 200), (2, 145, 100), (2, 200, 150), (2, 225, 90),
                                                  (2, 300, 120), (1, 257, 300), (1, 272, 64), (1, 273, 65),
                                                  (1, 320, 200), (1, 352, 100), (1, 384, 333)])
def test_fp32_products(workload, n_ant, n_src):
    import oracle
    wl = synth.workload(workload, n_ant=n_ant, n_src=n_src, n_time=1, n_freq=2)
    say(f"fp32 split products: workload {workload}, {n_ant} antennas, {n_src} sources")
    d = mv.device_inputs(wl, "fp32")
    ref = oracle.simulate(wl.antpos, wl.freqs, wl.lsts, wl.ra, wl.dec, wl.flux, grid_as_used(wl, "fp32"), wl.latitude,
                          wl.dza, wl.daz, wl.interp)
    for tile in (0, 2):
        with mv.Context(mv.config_for(wl, "fp32", tile=tile)) as ctx:
            assert ctx.product_path == ("sources" if workload == 2 else "fused_blocks")
            V = ctx.simulate(**d).cpu().numpy().astype(np.complex128)
            ctx.finish()
        V = V.reshape((-1,) + V.shape[2:])
        ef, ec = errors(V, ref)
        say(f"  tile {tile}: err_F={ef:.3e} err_CS={ec:.3e}")
        assert ef <= 2e-6 and ec <= 2e-6
