"""Infinite inputs of the cost model in networks whose width the fused kernels
pad: a unit that ReLU sets to zero stays zero, whatever the padding columns
multiply.  Against the binary64 oracle, non-finite values where it has them.

Tolerances as for finite inputs: outputs 1e-5, gradients 1e-4 (relative
2-norm per parameter block, over its finite entries)."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import note
from oracle import mlp as omlp

pytestmark = pytest.mark.gpu

tg = pytest.importorskip("paper_2606_15991_amd")
DEV = "cuda:0"


def close(got, want, tol):
    got, want = np.asarray(got, np.float64), np.asarray(want)
    fin = np.isfinite(want)
    assert np.array_equal(fin, np.isfinite(got))
    return np.linalg.norm(got[fin] - want[fin]) <= \
        tol * max(np.linalg.norm(want[fin]), 1e-300)


@pytest.mark.parametrize("n_in,hidden,depth", [
    (24, 40, 3), (5, 1, 2), (17, 63, 4), (24, 64, 3)])
def test_infinite_inputs(n_in, hidden, depth):
    note("mlp infinite", n_in, hidden, depth)
    batch = 70
    p = synth.mlp_init(n_in, hidden, depth, 41).clone()
    p += synth.normal(p.shape, 42, std=0.05)
    W0 = p[:hidden * n_in].view(hidden, n_in)
    W0[:, 0] = -W0[:, 0].abs() - 0.01
    X, y = synth.normal((batch, n_in), 43), synth.normal((batch,), 44)
    X[3::7, 0] = float("inf")        # every first-layer unit becomes zero
    pd, Xd, yd = p.to(DEV), X.to(DEV), y.to(DEV)
    out = tg.tile_mlp_forward(pd, Xd, n_in, hidden, depth)
    loss, g = tg.tile_mlp_loss_grad(pd, Xd, yd, n_in, hidden, depth)
    torch.cuda.synchronize()
    p64, X64, y64 = (t.double().numpy() for t in (p, X, y))
    with np.errstate(invalid="ignore"):
        want = omlp.forward(p64, X64, n_in, hidden, depth)[0]
        lw = omlp.loss(p64, X64, y64, n_in, hidden, depth)
        gr = omlp.grad(p64, X64, y64, n_in, hidden, depth)
    assert np.isfinite(want).all()
    assert close(out.cpu(), want, 1e-5)
    assert abs(loss.item() - lw) <= 1e-5 * lw
    off, g = 0, g.cpu().numpy()
    for o, i in omlp.shapes(n_in, hidden, depth):
        for n in (o * i, o):
            assert close(g[off:off + n], gr[off:off + n], 1e-4), off
            off += n
