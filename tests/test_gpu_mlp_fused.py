"""The fused cost-model kernels at the edges of their range, against the
binary64 oracle (oracle.mlp).

Tolerances, relative 2-norm per parameter block: every value is a chain of
binary32 dot products of at most 64 terms and depth + 1 layers, and the
batch sums add at most 20000 rows in partial sums of at most 20000 / 256 tiles:
outputs 1e-5, gradients 1e-4 (as for the layer-wise kernels)."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import note
from oracle import mlp as omlp

pytestmark = pytest.mark.gpu

tg = pytest.importorskip("paper_2606_15991_amd")
DEV = "cuda:0"


def _rel(a, b):
    return float(np.linalg.norm(np.asarray(a, np.float64) - b) /
                 max(np.linalg.norm(b), 1e-300))


# one row; a tile less one and plus one row; the workspace's smallest number
# of partial gradients; several tiles per workgroup; the widest and the
# narrowest layers; the deepest fused network and the first one past it; one
# input more than the fused kernels take
@pytest.mark.parametrize("n_in,hidden,depth,batch", [
    (24, 64, 3, 1), (24, 64, 3, 31), (24, 64, 3, 33), (24, 64, 3, 70),
    (24, 64, 3, 20000), (64, 64, 4, 100), (1, 1, 2, 65), (17, 49, 1, 300),
    (24, 64, 5, 100), (65, 64, 2, 100)])
def test_mlp_edges_match_oracle(n_in, hidden, depth, batch):
    note("mlp fused", n_in, hidden, depth, batch)
    p = synth.mlp_init(n_in, hidden, depth, 31)
    p = p + synth.normal(p.shape, 32, std=0.05)
    X, y = synth.normal((batch, n_in), 33), synth.normal((batch,), 34)
    pd, Xd, yd = p.to(DEV), X.to(DEV), y.to(DEV)
    out = tg.tile_mlp_forward(pd, Xd, n_in, hidden, depth)
    loss, g = tg.tile_mlp_loss_grad(pd, Xd, yd, n_in, hidden, depth)
    _, g2 = tg.tile_mlp_loss_grad(pd, Xd, yd, n_in, hidden, depth)
    torch.cuda.synchronize()
    p64, X64, y64 = (t.double().numpy() for t in (p, X, y))
    assert _rel(out.cpu(), omlp.forward(p64, X64, n_in, hidden, depth)[0]) \
        <= 1e-5
    want = omlp.loss(p64, X64, y64, n_in, hidden, depth)
    assert abs(loss.item() - want) <= 1e-5 * want
    gr = omlp.grad(p64, X64, y64, n_in, hidden, depth)
    off = 0
    for o, i in omlp.shapes(n_in, hidden, depth):
        for n in (o * i, o):
            assert _rel(g.cpu()[off:off + n], gr[off:off + n]) <= 1e-4, off
            off += n
    assert torch.equal(g, g2)
