"""Network evaluation around the sizes where its tasks change from 16 to 32 points: every point's outputs are
those of the same point in a small call, bit for bit."""
import numpy as np
import pytest

from paper_2312_09763_amd import matvis as mv
from paper_2312_09763_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [7 * 16384, 7 * 16384 + 1, 120_000, 131_072, 131_073, 9 * 16384 + 5, 200_001, 262_143])
def test_forward_around_the_steps(n):
    import torch
    P = torch.from_numpy(synth.surrogate_init(1, sigma_v=1.0, az_max=4)).cuda()
    g = torch.Generator().manual_seed(7)
    x = torch.rand((n, 3), generator=g).cuda()
    whole = mv.mlp_forward(P, x)
    parts = torch.cat([mv.mlp_forward(P, x[a:a + 60_000].contiguous()) for a in range(0, n, 60_000)])
    assert np.array_equal(whole.cpu().numpy(), parts.cpu().numpy())
