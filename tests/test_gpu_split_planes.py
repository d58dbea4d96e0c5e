"""Split-precision products whose planes are stored once (whole K tiles in
each plane, 256 x 256 sub-tensors) and once per product (everything else),
with operands whose rows take 16-byte chunks and ones that do not, against
binary64: bf16x6 within 2e-6 and bf16x3 within 6e-6 of the result's norm."""
import pytest
import torch

import synth
from gpu_util import note, reference, rel_err

pytestmark = pytest.mark.gpu

tg = pytest.importorskip("paper_2606_15991_amd")
DEV = "cuda:0"


@pytest.mark.parametrize("prec,bar", [("bf16x6", 2e-6), ("bf16x3", 6e-6)])
@pytest.mark.parametrize("nk", [True, False])
@pytest.mark.parametrize("M,N,K,pad,tile", [
    (300, 264, 64, 0, 256),     # one K tile a plane
    (513, 256, 192, 1, 256),    # odd row stride: one element a lane
    (256, 520, 128, 4, 256),
    (260, 264, 72, 0, 256),     # K tiles that straddle two planes
    (260, 264, 128, 0, 64)])    # another kernel
def test_split_planes(prec, bar, nk, M, N, K, pad, tile):
    note("split planes", prec, nk, M, N, K, pad, tile)
    A = synth.normal((M, K), 71)
    B = synth.normal((N, K) if nk else (K, N), 72)

    def put(x):
        big = torch.full((x.shape[0], x.shape[1] + pad), float("nan"),
                         device=DEV)
        v = big[:, :x.shape[1]]
        v.copy_(x)
        return v
    C = torch.full((M, N), float("nan"), device=DEV)
    wc = torch.zeros((M, N), dtype=torch.int32, device=DEV)
    tg.tile_gemm(put(A), put(B), C, tile, tile, b_trans=nk, precision=prec,
                 write_count=wc)
    torch.cuda.synchronize()
    assert torch.all(wc == 1)
    assert rel_err(C.cpu(), reference(A, B, nk)) <= bar
