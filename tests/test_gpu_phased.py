"""The phased schedule (the two-stage cross-tile configurations of 256 x 256
sub-tensors) at the edges of its K loop and of its stores.

Small-integer operands: every partial sum is an integer below 2^24, so the
product is exact (bf16 output: exact but for the one rounding).  Scaled e4m3
products of N(0,1) values: 1e-4, the bar of the 8-bit instructions."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import exact64, note, reference, rel_err

pytestmark = pytest.mark.gpu

tg = pytest.importorskip("paper_2606_15991_amd")
DEV = "cuda:0"
BF, F8, F32 = torch.bfloat16, torch.float8_e4m3fn, torch.float32


def padded(t, pad, shift=0):
    """t on the GPU with rows cols + pad elements apart, `shift` elements
    into its buffer."""
    raw = t.view(torch.uint8) if t.dtype == F8 else t
    rows, cols = raw.shape
    ld = cols + pad
    buf = torch.zeros(rows * ld + shift, dtype=raw.dtype, device=DEV)
    v = buf[shift:shift + rows * ld].view(rows, ld)[:, :cols]
    v.copy_(raw.to(DEV))
    return v.view(F8) if t.dtype == F8 else v


def run(M, N, K, dt, b_trans, out, ldc_pad, shift, sched=3):
    A = synth.small_int((M, K), 91).to(dt)
    B = synth.small_int((N, K) if b_trans else (K, N), 92).to(dt)
    mult = 16 // A.element_size()
    pa = -K % mult
    Ad = padded(A, pa)
    Bd = padded(B, pa if b_trans else -N % mult)
    buf = torch.full((M * (N + ldc_pad) + shift,), float("nan"), dtype=out,
                     device=DEV)
    C = buf[shift:].view(M, N + ldc_pad)[:, :N]
    wc = torch.zeros((M, N), dtype=torch.int32, device=DEV)
    cfg = {"kind": "tiled", "bm": 256, "bn": 256, "sched": sched,
           "stages": 2}
    tg.tile_gemm(Ad, Bd, C, 256, 256, b_trans=b_trans, config=cfg,
                 write_count=wc)
    torch.cuda.synchronize()
    assert torch.all(wc == 1)
    R = reference(A, B, b_trans)
    want = R if out == F32 else exact64(torch.from_numpy(R).to(BF))
    assert np.array_equal(exact64(C.cpu()), want)
    # nothing between the rows, or in front of the first, is written
    rest = torch.cat([buf[:shift], buf[shift:].view(M, N + ldc_pad)[:, N:]
                      .reshape(-1)])
    assert bool(torch.isnan(rest).all())


# one to seven K tiles, whole, with a partial one and with a chunk that
# straddles K (e4m3 tiles are twice as deep)
@pytest.mark.parametrize("K", [1, 9, 64, 120, 128, 192, 200, 257, 320, 384,
                               449, 896])
@pytest.mark.parametrize("dt,b_trans", [(BF, True), (BF, False), (F8, True)])
def test_k_loop_edges(K, dt, b_trans):
    note("phased K", K, dt, b_trans)
    run(272, 264, K, dt, b_trans, F32, 0, 0)
    run(272, 264, K, dt, b_trans, BF, 0, 0)


# last column blocks with a partial 16-byte piece, none and one element;
# output rows that start inside a dword or a 16-byte piece
@pytest.mark.parametrize("M,N", [(257, 265), (255, 513), (1, 300), (300, 258),
                                 (512, 256), (250, 31)])
@pytest.mark.parametrize("out", [F32, BF])
@pytest.mark.parametrize("ldc_pad,shift", [(0, 0), (1, 1), (3, 0), (2, 2)])
def test_store_edges(M, N, out, ldc_pad, shift):
    note("phased store", M, N, out, ldc_pad, shift)
    run(M, N, 136, BF, True, out, ldc_pad, shift)


def test_several_sub_tensors_per_program_and_long_k_name():
    note("phased 4352^2 x 328, both names")
    run(4352, 4352, 328, BF, True, BF, 0, 0)
    run(520, 600, 328, BF, True, F32, 0, 0, sched=6)


@pytest.mark.parametrize("sa,sb", [(True, True), (True, False),
                                   (False, True)])
@pytest.mark.parametrize("out", [F32, BF])
def test_scales(sa, sb, out):
    M, N, K = 4400, 4360, 272
    note("phased scales", sa, sb, out)
    qa, va = synth.quant_e4m3_rows(synth.normal((M, K), 93))
    qb, vb = synth.quant_e4m3_rows(synth.normal((N, K), 94))
    C = torch.full((M, N), float("nan"), dtype=out, device=DEV)
    tg.tile_gemm(qa.to(DEV), qb.to(DEV), C, 256, 256, b_trans=True,
                 scale_a=va.to(DEV) if sa else None,
                 scale_b=vb.to(DEV) if sb else None)
    torch.cuda.synchronize()
    rows = np.arange(0, M, 61)
    R = reference(qa[rows], qb, True, va[rows] if sa else None,
                  vb if sb else None)
    got = C.cpu()[torch.from_numpy(rows)]
    assert rel_err(got, R) <= (1e-4 if out == F32 else 4e-3)
