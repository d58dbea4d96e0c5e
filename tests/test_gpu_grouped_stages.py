"""Grouped launches of 128 x 128 sub-tensors past one round of the compute
units: even K (programs of two stages) and uneven K, both layouts of B.
Small integers: exact, every element stored once."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import exact64, note, reference

pytestmark = pytest.mark.gpu

tg = pytest.importorskip("paper_2606_15991_amd")
DEV = "cuda:0"


@pytest.mark.parametrize("b_trans", [True, False])
@pytest.mark.parametrize("ks", [(200,), (72, 136, 1032)])
def test_grouped_128_past_one_round(b_trans, ks):
    note("grouped 128", b_trans, ks)
    shapes = [(500, 520, ks[i % len(ks)]) for i in range(15)]   # 300
    As = [synth.to_bf16(synth.small_int((m, k), 60 + i))
          for i, (m, n, k) in enumerate(shapes)]
    Bs = [synth.to_bf16(synth.small_int((n, k) if b_trans else (k, n),
                                        80 + i))
          for i, (m, n, k) in enumerate(shapes)]
    Ad, Bd = [a.to(DEV) for a in As], [b.to(DEV) for b in Bs]
    Cs = [torch.full((m, n), float("nan"), device=DEV) for m, n, _ in shapes]
    wc = torch.zeros(sum(m * n for m, n, _ in shapes), dtype=torch.int32,
                     device=DEV)
    launch = tg.tile_gemm_grouped_prepare(
        Ad, Bd, Cs, b_trans=b_trans, write_count=wc,
        config={"kind": "tiled", "bm": 128, "bn": 128})
    tg.tile_gemm_grouped(launch)
    torch.cuda.synchronize()
    assert torch.all(wc == 1)
    for a, b, c in zip(As, Bs, Cs):
        assert np.array_equal(exact64(c.cpu()), reference(a, b, b_trans))
