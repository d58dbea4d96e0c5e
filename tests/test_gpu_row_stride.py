"""One-row operands whose descriptor names no stride (ld = 0), through the C
entry points: accepted, so the product is the one with ld = cols, whichever
kernel runs it.  Small integers: exact."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import exact64, note, reference

pytestmark = pytest.mark.gpu

tg = pytest.importorskip("paper_2606_15991_amd")
DEV = "cuda:0"
BF, F8, F32 = torch.bfloat16, torch.float8_e4m3fn, torch.float32


@pytest.mark.parametrize("adt,bdt,N,K,b_trans,kind", [
    (BF, BF, 4096, 1536, True, None),          # decode, streaming
    (BF, F8, 4096, 2048, True, None),
    (BF, BF, 300, 256, True, None),            # decode, plain
    (BF, F8, 16384, 128, True, "simple"),      # 128 x 128 blocks, direct loads
    (BF, BF, 200, 256, True, "tiled"),
    (BF, BF, 200, 256, False, "tiled"),
    (BF, BF, 200, 1, False, "tiled"),          # B is a single row as well
    (F32, F32, 200, 128, True, None),
    (F32, F32, 200, 128, False, "simple"),
    (F8, F8, 200, 256, True, None)])
def test_one_row_without_stride(adt, bdt, N, K, b_trans, kind):
    note("row stride", adt, bdt, N, K, b_trans, kind)
    A = synth.small_int((1, K), 95).to(adt)
    B = synth.small_int((N, K) if b_trans else (K, N), 96).to(bdt)
    Ad, Bd = A.to(DEV), B.to(DEV)
    C = torch.full((1, N), float("nan"), device=DEV)
    a, b, c = tg.make_in(Ad), tg.make_in(Bd, b_trans), tg.make_out(C)
    a.ld = c.ld = 0
    if b.rows == 1:
        b.ld = 0
    o = tg.make_opts(config={"kind": kind} if kind else None)
    assert tg.lib.tile_gemm(a, b, c, o, tg._stream(None)) == tg.TG_OK
    torch.cuda.synchronize()
    assert np.array_equal(exact64(C.cpu()), reference(A, B, b_trans))


def test_grouped_row_without_stride():
    note("row stride, grouped")
    A, B = synth.to_bf16(synth.small_int((1, 256), 97)), \
        synth.to_bf16(synth.small_int((256, 200), 98))
    Ad, Bd = A.to(DEV), B.to(DEV)
    C = torch.full((1, 200), float("nan"), device=DEV)
    a, b, c = tg.make_in(Ad), tg.make_in(Bd), tg.make_out(C)
    a.ld = 0
    ws = torch.empty(tg.tile_gemm_grouped_workspace_size(1),
                     dtype=torch.uint8, device=DEV)
    plan = tg.tg_grouped_plan()
    st = tg._stream(None)
    assert tg.lib.tile_gemm_grouped_prepare(
        1, a, b, c, None, ws.data_ptr(), ws.numel(), plan, st) == tg.TG_OK
    assert tg.lib.tile_gemm_grouped(plan, st) == tg.TG_OK
    torch.cuda.synchronize()
    assert np.array_equal(exact64(C.cpu()), reference(A, B))
