"""Network evaluation at the edges of its tasks (16 points, 32 past 2^18) and with more calls in flight
than there are weight images: each call's outputs are those of the same points in other company."""
import threading

import numpy as np
import pytest

from paper_2312_09763_amd import matvis as mv
from paper_2312_09763_amd import synth

pytestmark = pytest.mark.gpu


def _inputs(n, seed=3):
    import torch
    g = torch.Generator().manual_seed(seed)
    return torch.rand((n, 3), generator=g).cuda()


@pytest.mark.parametrize("n", [1, 15, 16, 17, 4095, 65537, (1 << 18) - 1, 1 << 18, (1 << 18) + 1, (1 << 18) + 33])
def test_forward_does_not_depend_on_the_call(n):
    import torch
    P = torch.from_numpy(synth.surrogate_init(0, sigma_v=1.0, az_max=4)).cuda()
    x = _inputs((1 << 18) + 40)
    whole = mv.mlp_forward(P, x[:n].contiguous()).cpu().numpy()
    part = np.concatenate([mv.mlp_forward(P, x[a:min(a + 999, n)].contiguous()).cpu().numpy()
                           for a in (0, max(0, n - 999))])
    ref = np.concatenate([whole[:min(999, n)], whole[max(0, n - 999):]])
    assert np.array_equal(part, ref)  # the same products in the same order for every point


def test_forward_from_several_threads():
    import torch
    Ps = [torch.from_numpy(synth.surrogate_init(i, sigma_v=1.0, az_max=4)).cuda() for i in range(7)]
    x = _inputs(20_000)
    want = [mv.mlp_forward(P, x).cpu().numpy() for P in Ps]
    bad = []

    def work(i):
        stream = torch.cuda.Stream()
        for _ in range(20):
            with torch.cuda.stream(stream):
                got = mv.mlp_forward(Ps[i], x, stream=stream)
            if not np.array_equal(got.cpu().numpy(), want[i]):
                bad.append(i)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(7)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert not bad
