"""The kernel for unaligned and mixed-type operands under explicit partitions
whose width is no multiple of a 16-byte chunk, B stored K x N with N a multiple
of it and K a whole number of K tiles: chunks of the last block straddle N in
the operand's last row.  Small integers: exact; NaN behind the operand."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import exact64, note, reference

pytestmark = pytest.mark.gpu

tg = pytest.importorskip("paper_2606_15991_amd")
DEV = "cuda:0"
BF, F8, F32 = torch.bfloat16, torch.float8_e4m3fn, torch.float32


def fenced(t):
    """t on the GPU, NaN in front of it and behind it."""
    raw = t.view(torch.uint8) if t.dtype == F8 else t
    nan = 0x7f if t.dtype == F8 else float("nan")
    big = torch.full((t.numel() + 64,), nan, dtype=raw.dtype, device=DEV)
    v = big[32:-32].view(t.shape)
    v.copy_(raw.to(DEV))
    return v.view(F8) if t.dtype == F8 else v


@pytest.mark.parametrize("bm,bn", [(64, 7), (64, 12), (33, 33), (5, 60)])
@pytest.mark.parametrize("adt,bdt", [(BF, BF), (BF, F8), (F8, F8),
                                     (F32, F32)])
def test_straddling_blocks(bm, bn, adt, bdt):
    M, N, K = 70, 136, 128
    note("simple partitions", bm, bn, adt, bdt)
    A = synth.small_int((M, K), 91).to(adt)
    B = synth.small_int((K, N), 92).to(bdt)
    C = torch.full((M, N), float("nan"), device=DEV)
    wc = torch.zeros((M, N), dtype=torch.int32, device=DEV)
    tg.tile_gemm(fenced(A), fenced(B), C, bm, bn,
                 config={"kind": "simple"}, write_count=wc)
    torch.cuda.synchronize()
    assert torch.all(wc == 1)
    assert np.array_equal(exact64(C.cpu()), reference(A, B))


# operands of whole dwords (no shifting of chunks), default partition: one
# 64 x 64 block a program, and 2 x 2 of them (more than 128 programs of those)
@pytest.mark.parametrize("M,N,K", [(33, 136, 132), (1400, 1500, 132)])
@pytest.mark.parametrize("adt,bdt", [(BF, BF), (BF, F8), (F8, F8),
                                     (F32, F32)])
@pytest.mark.parametrize("b_trans", [True, False])
def test_whole_dwords(M, N, K, adt, bdt, b_trans):
    note("simple whole dwords", M, N, K, adt, bdt, b_trans)
    A = synth.small_int((M, K), 93).to(adt)
    B = synth.small_int((N, K) if b_trans else (K, N), 94).to(bdt)
    C = torch.full((M, N), float("nan"), device=DEV)
    tg.tile_gemm(fenced(A), fenced(B), C, b_trans=b_trans,
                 config={"kind": "simple"})
    torch.cuda.synchronize()
    assert np.array_equal(exact64(C.cpu()), reference(A, B, b_trans))
