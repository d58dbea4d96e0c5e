"""The fused normalisation and product does not depend on what LDS held."""
import pytest
import torch

import oracle
import synth
from gpu_util import exact64, note, rel_err

pytestmark = pytest.mark.gpu

tg = pytest.importorskip("paper_2606_15991_amd")
DEV = "cuda:0"


@pytest.mark.parametrize("d,wdt", [(2672, "bf16"), (1040, "bf16"),
                                   (1104, "fp8"), (2480, "fp8")])
def test_fused_norm_ignores_what_lds_held(d, wdt):
    """K whose last super-step is partial: the steps past K read
    normalisation weights from LDS that no load filled.  A product of NaN
    operands leaves NaNs in the LDS of every compute unit first."""
    note("fused norm after NaNs", d, wdt)
    nan = torch.full((2048, 2048), float("nan"), dtype=torch.bfloat16,
                     device=DEV)
    sink = torch.empty((2048, 2048), device=DEV)
    x = synth.to_bf16(synth.normal((1, d), 17))
    nw = (1.0 + synth.normal((d,), 18, std=0.1)).to(torch.bfloat16)
    w = synth.normal((d, d), 19, std=0.02)
    if wdt == "bf16":
        W, sw = synth.to_bf16(w), None
    else:
        W, sw = synth.quant_e4m3_rows(w)
    xd, nd, Wd = x.to(DEV), nw.to(DEV), W.to(DEV)
    swd = None if sw is None else sw.to(DEV)
    want = oracle.rms_norm_matvec(
        exact64(x), exact64(nw), exact64(W), 1e-6,
        sw=None if sw is None else exact64(sw))
    for _ in range(3):
        tg.tile_gemm(nan, nan, sink, 256, 256, b_trans=True)
        y = torch.empty((1, d), device=DEV)
        tg.tile_rms_norm_matvec(xd, nd, Wd, y, 1e-6, scale_w=swd)
        torch.cuda.synchronize()
        assert rel_err(y.cpu(), want) <= 1e-5
