"""The learned beam's loss and gradient on bf16 products (kernels_mlp_train.hip) at the edges of its
row tiles (16), bias chunks (256), weight chunks (128 from 512 rows on) and of several chunks per
workgroup, against the float64 gradient: bf16 operands are 2^-9 off each, through four layers and
back, so 2e-2 of each block's norm is five times what they add up to.  Parameters may be aligned to
one float only."""
import numpy as np
import pytest

from helpers import say
from oracle import mlp as om
from paper_2312_09763_amd import matvis as mv
from paper_2312_09763_amd import synth

pytestmark = pytest.mark.gpu


def _case(n):
    import torch
    rng = np.random.Generator(np.random.PCG64(n))
    x = rng.uniform(0.0, 1.0, (n, 3)).astype(np.float32)
    y = rng.normal(0.0, 0.3, (n, 8)).astype(np.float32)
    return synth.surrogate_init(3), x, y, torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()


@pytest.mark.parametrize("n", [1, 15, 16, 17, 255, 257, 511, 512, 513, 4097, 9001])
def test_gradient_at_chunk_edges(n):
    import torch
    p, x, y, xd, yd = _case(n)
    say(f"training gradient: n={n}")
    g, loss = mv.mlp_loss_grad(torch.from_numpy(p).cuda(), xd, yd)
    ref, ref_loss = om.loss_grad(p, x.astype(np.float64), y.astype(np.float64))
    assert float(loss.item()) == pytest.approx(ref_loss, rel=2e-2)
    G, R = om.unpack(g.cpu().numpy().astype(np.float64)), om.unpack(np.asarray(ref, dtype=np.float64))
    assert np.all(G["B"] == 0)
    for k in R:
        if k != "B":
            e = np.linalg.norm(G[k] - R[k]) / np.linalg.norm(R[k])
            assert e <= 2e-2, (k, e)


def test_parameters_aligned_to_one_float():
    import torch
    p, _, _, xd, yd = _case(300)
    room = torch.empty(p.size + 1, dtype=torch.float32, device="cuda")
    room[1:] = torch.from_numpy(p).cuda()
    a, la = mv.mlp_loss_grad(room[1:], xd, yd)
    b, lb = mv.mlp_loss_grad(torch.from_numpy(p).cuda(), xd, yd)
    assert torch.equal(a, b) and torch.equal(la, lb)
