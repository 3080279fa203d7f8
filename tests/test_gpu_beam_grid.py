"""A batch whose beam step has more than 2^32 threads in all (one launch dimension cannot hold them)."""
import numpy as np
import pytest

from helpers import say

pytestmark = pytest.mark.gpu


def test_beam_step_of_a_very_large_batch():
    """64 times of 5 channels and 2^22 sources in one batch against the same call in batches of one time.  Sums
    of 2.1 million terms of one sign (flux 1 a source, a beam of 1) in 256 splits or more: a split adds at most
    8192 / 16 stages of 16 in FP32, about 2^-24 sqrt(512) = 1.3e-6, and the splits are added in FP64; the bar
    is 1e-5, the FP32 bar of the other tests."""
    import torch
    from paper_2312_09763_amd import matvis as mv
    free = torch.cuda.mem_get_info()[0]
    if free < 100 << 30:
        pytest.skip("needs 100 GB of free device memory")
    n_src, n_time, n_freq = 1 << 22, 64, 5
    g = torch.Generator(device="cuda").manual_seed(3)
    u = torch.rand((2, n_src), generator=g, device="cuda", dtype=torch.float64)
    radec = torch.stack([2 * np.pi * u[0], torch.asin(2 * u[1] - 1)]).contiguous()
    freqs = torch.linspace(100e6, 200e6, n_freq, device="cuda", dtype=torch.float64)
    lsts = torch.arange(n_time, device="cuda", dtype=torch.float64) * (2 * np.pi / n_time)
    antpos = torch.tensor([[0.0, 0, 0], [14.6, 0, 0]], device="cuda", dtype=torch.float64)
    flux = torch.ones((n_freq, n_src), device="cuda", dtype=torch.float64)
    beam = torch.zeros((1, n_freq, 2, 2, 19, 72), device="cuda", dtype=torch.complex64)
    beam[:, :, 0, 0] = beam[:, :, 1, 1] = 1.0
    out = []
    for batch in (n_time, 1):
        say(f"beam grid: {n_time} x {n_freq} instances of {n_src} sources, {batch} times a batch")
        cfg = mv.Config(n_ant=2, n_feed=2, n_ax=2, n_beam=1, max_src=n_src, max_time=n_time, max_freq=n_freq,
                        latitude_rad=-0.5, precision="fp32", beam_mode="bilinear", n_za=19, n_az=72,
                        dza_rad=np.radians(5.0), daz_rad=np.radians(5.0), batch_time=batch, src_chunk=n_src,
                        ksplit=32768)
        with mv.Context(cfg) as ctx:
            vis = ctx.simulate(antpos, freqs, lsts, radec, flux, beam)
            ctx.finish()
            out.append(vis.cpu().numpy())
        torch.cuda.empty_cache()
    up = out[1][:, :, 0, 0, 0, 0].real
    assert (np.abs(up - n_src / 2) < 0.01 * n_src).all()  # half of a uniform sky is up
    err = np.abs(out[0] - out[1]).max() / up.min()
    say(f"  largest difference {err:.2e} of the autocorrelation")
    assert err <= 1e-5
