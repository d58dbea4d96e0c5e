"""Grouped launches of a whole number of rows of programs and of some more
or less (256 x 256 sub-tensors, one program per compute unit): every element
of every product exact and stored once."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import exact64, note, reference

pytestmark = pytest.mark.gpu

tg = pytest.importorskip("paper_2606_15991_amd")
DEV = "cuda:0"


@pytest.mark.parametrize("rows,more", [(0, 3), (1, 0), (1, 1), (2, -1),
                                       (2, 0), (2, 5), (3, 255)])
def test_grouped_rows(rows, more):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    total = rows * cus + more
    note("grouped rows", rows, more, total)
    # `total` sub-tensors of 256 x 256 over problems of rising K, one row of
    # sub-tensors each
    counts = [total // 3, total - 2 * (total // 3), total // 3]
    shapes = [(190, 256 * c - 120, 64 * (i + 1))
              for i, c in enumerate(counts) if c]
    As = [synth.small_int((m, k), 60 + i).to(torch.bfloat16)
          for i, (m, n, k) in enumerate(shapes)]
    Bs = [synth.small_int((k, n), 70 + i).to(torch.bfloat16)
          for i, (m, n, k) in enumerate(shapes)]
    Ad, Bd = [a.to(DEV) for a in As], [b.to(DEV) for b in Bs]
    Cs = [torch.full((m, n), float("nan"), device=DEV) for m, n, k in shapes]
    wc = torch.zeros(sum(m * n for m, n, k in shapes), dtype=torch.int32,
                     device=DEV)
    launch = tg.tile_gemm_grouped_prepare(
        Ad, Bd, Cs, config={"bm": 256, "bn": 256}, write_count=wc)
    tg.tile_gemm_grouped(launch)
    torch.cuda.synchronize()
    assert torch.all(wc == 1)
    for A, B, C in zip(As, Bs, Cs):
        pick = torch.arange(0, A.shape[0], 13)
        assert torch.isfinite(C).all()
        assert np.array_equal(exact64(C.cpu()[pick]), reference(A[pick], B))
