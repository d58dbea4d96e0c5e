"""The kernel for unaligned and mixed-type operands, at the edges of its
programs' blocks (64 x 64 and 128 x 128 outputs), K tiles (64 bf16, 32
binary32) and chunks, for every dtype pair and layout.

Small-integer operands: every partial sum is an integer below 2^24, so the
result is exact.  N(0,1) operands: 1e-5 relative Frobenius error (binary32
accumulation of exactly represented products)."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import exact64, note, reference, rel_err

pytestmark = pytest.mark.gpu

tg = pytest.importorskip("paper_2606_15991_amd")
DEV = "cuda:0"
BF, F8, F32 = torch.bfloat16, torch.float8_e4m3fn, torch.float32


def offset_view(t, pad, shift):
    """The values of t on the GPU, rows `cols + pad` elements apart, the
    first one `shift` elements into the buffer."""
    rows, cols = t.shape
    raw = t.view(torch.uint8) if t.dtype == F8 else t
    ld = cols + pad
    buf = torch.zeros(rows * ld + shift, dtype=raw.dtype, device=DEV)
    v = buf[shift:shift + rows * ld].view(rows, ld)[:, :cols]
    v.copy_(raw.to(DEV))
    return v.view(F8) if t.dtype == F8 else v


# one element; a block less one, whole and plus one in each direction; K of
# one chunk less one, of a tile less one and plus one, of several tiles; more
# programs than compute units with 64 x 64 and with 128 x 128 blocks
@pytest.mark.parametrize("M,N,K", [
    (17, 1, 1), (63, 65, 7), (64, 64, 63), (65, 129, 65), (128, 127, 33),
    (200, 140, 191), (1000, 2100, 37), (2100, 2200, 71)])
@pytest.mark.parametrize("adt,bdt", [(BF, BF), (BF, F8), (F8, F8),
                                     (F32, F32)])
@pytest.mark.parametrize("b_trans", [True, False])
def test_blocks_and_tails(M, N, K, adt, bdt, b_trans):
    bshape = (N, K) if b_trans else (K, N)
    note("simple blocks", M, N, K, adt, bdt, b_trans)
    cfg = {"kind": "simple"}
    for gen, exact in ((synth.small_int, True), (synth.normal, False)):
        A, B = gen((M, K), 81).to(adt), gen(bshape, 82).to(bdt)
        Ad, Bd = offset_view(A, 1, 1), offset_view(B, 3, 1)
        R = reference(A, B, b_trans)
        for out in (F32, BF):
            C = torch.full((M, N), float("nan"), dtype=out, device=DEV)
            wc = torch.zeros((M, N), dtype=torch.int32, device=DEV)
            tg.tile_gemm(Ad, Bd, C, b_trans=b_trans, config=cfg,
                         write_count=wc)
            torch.cuda.synchronize()
            assert torch.all(wc == 1)
            if exact:
                want = R if out == F32 else exact64(
                    torch.from_numpy(R).to(BF))
                assert np.array_equal(exact64(C.cpu()), want), out
            else:
                assert rel_err(C.cpu(), R) <= (1e-5 if out == F32 else 4e-3)


@pytest.mark.parametrize("bm,bn", [(64, 64), (48, 64), (33, 7)])
def test_partition_scales_and_ownership(bm, bn):
    """Explicit partitions, scales, and the program map the launch walks."""
    M, N, K = 300, 200, 99
    note("simple partition", bm, bn)
    A, B = synth.normal((M, K), 83).to(BF), synth.normal((N, K), 84).to(F8)
    sa, sb = synth.uniform_pm1((M,), 85) + 2, synth.uniform_pm1((N,), 86) + 2
    Ad, Bd = A.to(DEV), B.to(DEV)
    C = torch.full((M, N), float("nan"), device=DEV)
    wc = torch.zeros((M, N), dtype=torch.int32, device=DEV)
    tg.tile_gemm(Ad, Bd, C, bm, bn, b_trans=True, scale_a=sa.to(DEV),
                 scale_b=sb.to(DEV), write_count=wc)
    torch.cuda.synchronize()
    assert torch.all(wc == 1)
    assert rel_err(C.cpu(), reference(A, B, True, sa, sb)) <= 1e-5
    cfg, n_prog, offs, ids = tg.tile_gemm_plan(Ad, Bd, C, bm, bn,
                                               b_trans=True)
    assert (cfg["bm"], cfg["bn"]) == (bm, bn)
    assert sorted(ids) == list(range(len(ids))) and len(offs) == n_prog + 1
