"""The phased schedule of 128 x 128 sub-tensors at the edges of its K loop and
of its stores: small-integer operands, exact (bf16 output: but for the one
rounding); scaled e4m3 products of N(0,1) values within 1e-4, the bar of the
8-bit instructions."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import exact64, note, reference, rel_err
from test_gpu_phased import BF, DEV, F8, F32, padded

pytestmark = pytest.mark.gpu

tg = pytest.importorskip("paper_2606_15991_amd")
CFG = {"kind": "tiled", "bm": 128, "bn": 128, "wm": 4, "wn": 2, "stages": 4}


def run(M, N, K, dt, out, ldc_pad=0, shift=0):
    A = synth.small_int((M, K), 91).to(dt)
    B = synth.small_int((N, K), 92).to(dt)
    pad = -K % (16 // A.element_size())
    Ad, Bd = padded(A, pad), padded(B, pad)
    buf = torch.full((M * (N + ldc_pad) + shift,), float("nan"), dtype=out,
                     device=DEV)
    C = buf[shift:].view(M, N + ldc_pad)[:, :N]
    wc = torch.zeros((M, N), dtype=torch.int32, device=DEV)
    tg.tile_gemm(Ad, Bd, C, b_trans=True, config=CFG, write_count=wc)
    torch.cuda.synchronize()
    assert torch.all(wc == 1)
    rows = np.unique(np.linspace(0, M - 1, 300).astype(int))
    R = reference(A[rows], B, True)
    want = R if out == F32 else exact64(torch.from_numpy(R).to(BF))
    assert np.array_equal(exact64(C.cpu()[torch.from_numpy(rows)]), want)
    rest = torch.cat([buf[:shift], buf[shift:].view(M, N + ldc_pad)[:, N:]
                      .reshape(-1)])
    assert bool(torch.isnan(rest).all())


@pytest.mark.parametrize("K", [1, 9, 64, 120, 128, 192, 200, 257, 320, 449,
                               896])
@pytest.mark.parametrize("dt", [BF, F8])
def test_k_loop_edges(K, dt):
    note("phased128 K", K, dt)
    run(136, 136, K, dt, F32)
    run(144, 264, K, dt, BF)


@pytest.mark.parametrize("M,N", [(129, 137), (127, 257), (1, 300), (300, 130),
                                 (128, 128), (122, 31)])
@pytest.mark.parametrize("out", [F32, BF])
@pytest.mark.parametrize("ldc_pad,shift", [(0, 0), (1, 1), (2, 2)])
def test_store_edges(M, N, out, ldc_pad, shift):
    note("phased128 store", M, N, out, ldc_pad, shift)
    run(M, N, 136, BF, out, ldc_pad, shift)


def test_several_sub_tensors_per_program():
    note("phased128 several")
    run(2700, 2312, 328, BF, BF)


@pytest.mark.parametrize("out", [F32, BF])
def test_scales(out):
    M, N, K = 2700, 2312, 272
    note("phased128 scales", out)
    qa, va = synth.quant_e4m3_rows(synth.normal((M, K), 93))
    qb, vb = synth.quant_e4m3_rows(synth.normal((N, K), 94))
    C = torch.full((M, N), float("nan"), dtype=out, device=DEV)
    tg.tile_gemm(qa.to(DEV), qb.to(DEV), C, b_trans=True, config=CFG,
                 scale_a=va.to(DEV), scale_b=vb.to(DEV))
    torch.cuda.synchronize()
    rows = np.arange(0, M, 61)
    R = reference(qa[rows], qb, True, va[rows], vb)
    got = C.cpu()[torch.from_numpy(rows)]
    assert rel_err(got, R) <= (1e-4 if out == F32 else 4e-3)


# bf16 rows by e4m3 weights: at least 128 programs of 128 x 128
@pytest.mark.parametrize("M,N,K", [(300, 5500, 16), (300, 5505, 48),
                                   (257, 5633, 64), (300, 5500, 80),
                                   (511, 4097, 208), (384, 5504, 512)])
@pytest.mark.parametrize("out", [F32, BF])
def test_mixed(M, N, K, out):
    note("phased128 mixed", M, N, K, out)
    A = synth.small_int((M, K), 91).to(BF)
    B = synth.small_int((N, K), 92).to(F8)
    scale = torch.from_numpy(
        2.0 ** np.random.default_rng(54).integers(-2, 3, N)).float()
    Ad = torch.full((M, K + 8), float("nan"), dtype=BF, device=DEV)[:, :K]
    Ad.copy_(A)
    Bd = torch.full((N, K + 16), 0x7f, dtype=torch.uint8, device=DEV)[:, :K]
    Bd.copy_(B.view(torch.uint8))
    C = torch.full((M, N), float("nan"), dtype=out, device=DEV)
    wc = torch.zeros((M, N), dtype=torch.int32, device=DEV)
    tg.tile_gemm(Ad, Bd.view(F8), C, b_trans=True, scale_b=scale.to(DEV),
                 write_count=wc)
    torch.cuda.synchronize()
    assert torch.all(wc == 1)
    want = reference(A, B, True) * scale.double().numpy()
    if out == BF:
        want = exact64(torch.from_numpy(want).float().to(BF))
    assert np.array_equal(exact64(C.cpu()), want)
