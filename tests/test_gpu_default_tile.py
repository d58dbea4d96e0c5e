"""Default sub-tensor sizes of the tiled products on either side of the
rule's lines (256 compute units): the size and LDS stages chosen, the product
of small integers exact and every element stored once."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import exact64, note, reference

pytestmark = pytest.mark.gpu

tg = pytest.importorskip("paper_2606_15991_amd")
DEV = "cuda:0"
BF, F8, F32 = torch.bfloat16, torch.float8_e4m3fn, torch.float32


@pytest.mark.parametrize("tile", [128, 64, 32])
@pytest.mark.parametrize("nk", [True, False])
@pytest.mark.parametrize("M,N,K", [(131, 260, 4), (129, 132, 100),
                                   (40, 516, 32), (257, 384, 68)])
def test_f32_tiles(tile, nk, M, N, K):
    """Rows, columns and K tiles cut off by the operands' ends, which lie in
    larger buffers of NaN; small integers, exact."""
    note("f32 tile", tile, nk, M, N, K)
    A = synth.small_int((M, K), 97).float()
    B = synth.small_int((N, K) if nk else (K, N), 98).float()

    def inside(x):
        big = torch.full((x.shape[0] + 2, x.shape[1] + 12), float("nan"),
                         device=DEV)
        v = big[1:-1, 4:4 + x.shape[1]]
        v.copy_(x)
        return v
    C = torch.full((M, N), float("nan"), device=DEV)
    wc = torch.zeros((M, N), dtype=torch.int32, device=DEV)
    tg.tile_gemm(inside(A), inside(B), C, b_trans=nk, config=dict(
        kind="tiled", bm=tile, bn=tile), write_count=wc)
    torch.cuda.synchronize()
    assert torch.all(wc == 1)
    assert np.array_equal(exact64(C.cpu()), reference(A, B, nk))


@pytest.mark.parametrize("dt,M,N,K,size,stages", [
    (BF, 2816, 3072, 72, 256, 2),     # t(256) = 132 of 256
    (BF, 2304, 2304, 72, 128, 2),     # t(256) = 81, t(128) = 324
    (BF, 2048, 2048, 72, 128, 4),     # t(128) = 256
    (BF, 129, 65536, 72, 256, 2), (BF, 128, 65536, 72, 128, 2),
    (BF, 64, 65536, 72, 64, 2),       # at most 64 rows
    (BF, 1024, 1024, 72, 128, 4),     # t(128) = 64
    (BF, 1024, 896, 72, 64, 2),       # t(128) = 56, t(64) = 224
    (BF, 1024, 1024, 512, 64, 8),     # eight K tiles, t(64) = 256: shared K
    (BF, 1025, 1024, 512, 128, 4),    # t(64) = 272
    (BF, 512, 512, 256, 32, 16),       # four, t(32) = 256: shared K
    (F8, 1025, 512, 1024, 64, 8), (F8, 1024, 576, 896, 32, 2),
    (F8, 1408, 1664, 144, 128, 4),    # e4m3: t(128) = 143 >= 140.8
    (F8, 1408, 1536, 144, 64, 2),     # t(128) = 132, t(64) = 528
    (BF, 64, 20000, 2304, 64, 4), (BF, 64, 20000, 2296, 64, 2),
    (F8, 64, 20000, 4608, 64, 4), (F8, 64, 20000, 4592, 64, 2),
    (F32, 32, 24576, 128, 32, 16),     # three rounds, four K tiles
    (F32, 32, 24580, 128, 32, 2), (F32, 33, 20000, 36, 64, 2),
    (F32, 2048, 1536, 36, 64, 2),     # three rounds of 64, one of 128
    (F32, 2048, 1540, 4, 128, 2)])    # four, one

def test_default_tile_lines(dt, M, N, K, size, stages):
    note("default tile", dt, M, N, K)
    old = tg.tile_picker_mode(0)
    try:
        A = synth.small_int((M, K), 95).to(dt)
        B = synth.small_int((N, K), 96).to(dt)
        Ad, Bd = A.to(DEV), B.to(DEV)
        C = torch.full((M, N), float("nan"), device=DEV)
        wc = torch.zeros((M, N), dtype=torch.int32, device=DEV)
        cfg = tg.tile_gemm_plan(Ad, Bd, C, b_trans=True, want_map=False)[0]
        assert (cfg["bm"], cfg["stages"]) == (size, stages), cfg
        tg.tile_gemm(Ad, Bd, C, b_trans=True, write_count=wc)
        torch.cuda.synchronize()
    finally:
        tg.tile_picker_mode(old)
    assert torch.all(wc == 1)
    rows = np.unique(np.linspace(0, M - 1, 97).astype(int))
    assert np.array_equal(exact64(C.cpu()[torch.from_numpy(rows)]),
                          reference(A[rows], B, True))


@pytest.mark.parametrize("dt,nk", [(BF, True), (BF, False), (F8, True),
                                   (F32, True), (F32, False)])
@pytest.mark.parametrize("tile,waves", [(32, 8), (64, 4)])
@pytest.mark.parametrize("M,N,K", [(40, 72, 16), (33, 100, 64), (70, 136, 68),
                                   (64, 64, 512), (129, 200, 1100),
                                   (65, 40, 4112), (2100, 1100, 528)])
def test_shared_k(dt, nk, tile, waves, M, N, K):
    """Wavefronts that share K: fewer K tiles than wavefronts, tails, several
    sub-tensors per program; operands inside larger buffers of NaN."""
    if dt == F32 and tile == 64:
        pytest.skip("binary32 has the 32 x 32 form only")
    mult = 16 // torch.empty((), dtype=dt).element_size()
    if not nk:
        N -= N % mult
    if dt == F32:
        K -= K % mult
    note("shared K", dt, nk, tile, M, N, K)
    A = synth.small_int((M, K), 97).to(dt)
    B = synth.small_int((N, K) if nk else (K, N), 98).to(dt)

    def inside(x):
        raw = x.view(torch.uint8) if dt == F8 else x
        cols = -(-x.shape[1] // mult) * mult + mult
        big = torch.full((x.shape[0] + 2, cols),
                         0x7f if dt == F8 else float("nan"), dtype=raw.dtype,
                         device=DEV)
        v = big[1:-1, :x.shape[1]]
        v.copy_(raw)
        return v.view(F8) if dt == F8 else v
    for out in (F32, BF):
        C = torch.full((M, N), float("nan"), dtype=out, device=DEV)
        wc = torch.zeros((M, N), dtype=torch.int32, device=DEV)
        tg.tile_gemm(inside(A), inside(B), C, b_trans=nk, config=dict(
            kind="tiled", bm=tile, bn=tile, wm=waves, wn=1), write_count=wc)
        torch.cuda.synchronize()
        assert torch.all(wc == 1)
        R = reference(A, B, nk)
        want = R if out == F32 else exact64(torch.from_numpy(R).to(BF))
        assert np.array_equal(exact64(C.cpu()), want)
