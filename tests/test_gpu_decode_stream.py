"""Decode products whose programs are dealt to one workgroup per compute unit
(unsplit K, at least 85 in 100 of the workgroups' worth of programs, more than
eleven 128-byte blocks of K): runs of columns that end inside a row tile, a
last workgroup with fewer programs, K that ends inside a block, operands that
stand in larger buffers of NaN.  Small integers: exact (bf16 output: but for
its one rounding)."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import exact64, note, reference

pytestmark = pytest.mark.gpu

tg = pytest.importorskip("paper_2606_15991_amd")
DEV = "cuda:0"
BF, F8, F32 = torch.bfloat16, torch.float8_e4m3fn, torch.float32


def inside(x, pad):
    """x on the GPU, in rows pad elements longer, NaN around it."""
    raw = x.view(torch.uint8) if x.dtype == F8 else x
    nan = 0x7f if x.dtype == F8 else float("nan")
    big = torch.full((x.shape[0] + 2, x.shape[1] + pad), nan,
                     dtype=raw.dtype, device=DEV)
    v = big[1:-1, :x.shape[1]]
    v.copy_(raw)
    return v.view(F8) if x.dtype == F8 else v


@pytest.mark.parametrize("wdt,M,N,K,bn,out", [
    (BF, 1, 2048, 712, 0, F32),        # 11.125 blocks of K, 8 columns each
    (F8, 1, 2048, 1424, 0, BF),
    (F8, 8, 4000, 1552, 0, F32),       # 250 workgroups
    (BF, 5, 2600, 784, 0, BF),         # 11 columns; the last has 4
    (BF, 16, 7936, 1024, 0, F32),      # 31 columns: a tile and 15
    (F8, 16, 8192, 2000, 0, BF),
    (BF, 3, 12800, 800, 25, F32),      # 50 columns: three tiles and two
    (F8, 2, 25500, 1600, 16, F32),     # seven programs each, N inside one
    (F8, 7, 51200, 2048, 0, BF),
    (BF, 8, 12288, 5120, 0, F32)])     # 160 KiB of LDS
def test_decode_stream(wdt, M, N, K, bn, out):
    note("decode stream", wdt, M, N, K, bn, out)
    x = synth.to_bf16(synth.small_int((M, K), 51))
    W = synth.small_int((N, K), 52).to(wdt)
    res = synth.small_int((M, N), 53).float()
    scale = torch.from_numpy(
        2.0 ** np.random.default_rng(54).integers(-2, 3, N)).float()
    xd, Wd = inside(x, 8), inside(W, 16)
    C = torch.full((M, N), float("nan"), dtype=out, device=DEV)
    wc = torch.zeros((M, N), dtype=torch.int32, device=DEV)
    cfg = {"kind": "skinny", "bn": bn, "ksplit": 4, "splitk": 1} if bn \
        else {"kind": "skinny", "splitk": 1}
    tg.tile_gemm(xd, Wd, C, b_trans=True, config=cfg, write_count=wc,
                 scale_b=scale.to(DEV), residual=res.to(DEV))
    torch.cuda.synchronize()
    want = reference(x, W, True) * scale.double().numpy() + \
        res.double().numpy()
    if out == BF:
        want = exact64(torch.from_numpy(want).float().to(BF))
    assert torch.all(wc == 1)
    assert np.array_equal(exact64(C.cpu()), want)
