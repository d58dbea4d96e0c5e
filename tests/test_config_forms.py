"""Configurations that name wavefronts, stages, bk or a schedule but no size
take the largest square sub-tensor that gives every compute unit close to one,
whatever the defaults are, so that they find their kernel (planned for 256
compute units, without a GPU)."""
import ctypes
import os
import subprocess

import pytest
import torch

from conftest import ROOT
import paper_2606_15991_amd as tg

BF, F8, F32 = torch.bfloat16, torch.float8_e4m3fn, torch.float32


@pytest.mark.parametrize("dt,M,N,K,b_trans,cfg,want", [
    # narrow outputs whose own default is 64 or 128
    (BF, 64, 65536, 512, True, dict(sched=3, stages=2), (256, 2, 4, 64, 2)),
    (BF, 100, 49152, 256, True, dict(bk=32), (256, 2, 4, 32, 4)),
    (BF, 65536, 64, 512, False, dict(stages=5), (256, 2, 4, 32, 5)),
    (F8, 17, 51200, 512, True, dict(sched=2), (256, 2, 4, 64, 4)),
    # an output whose own default is 256
    (BF, 3072, 3072, 1024, False, dict(wm=2, wn=2, sched=1),
     (128, 2, 2, 32, 4)),
    # small ones, whose wavefronts share K by default
    (BF, 512, 512, 512, True, dict(wm=1, wn=1), (32, 1, 1, 64, 2)),
    (BF, 1024, 1024, 1024, True, dict(wm=2, wn=2, stages=2),
     (64, 2, 2, 64, 2)),
    (F32, 512, 512, 512, True, dict(stages=2), (32, 1, 1, 32, 2)),
    (F32, 4096, 4096, 512, False, dict(wm=2, wn=2), (128, 2, 2, 32, 2))])
def test_named_configurations_find_their_kernel(dt, M, N, K, b_trans, cfg,
                                                want):
    A = torch.empty((M, K), dtype=dt)
    B = torch.empty((N, K) if b_trans else (K, N), dtype=dt)
    C = torch.empty((M, N))
    got = tg.tile_gemm_plan(A, B, C, b_trans=b_trans, want_map=False,
                            config={"kind": "tiled", **cfg})[0]
    assert got["bm"] == got["bn"]
    assert (got["bm"], got["wm"], got["wn"], got["bk"], got["stages"]) == \
        want, got


@pytest.mark.parametrize("dt,M,N,K,b_trans,size,stages", [
    (BF, 4096, 2048, 2048, False, 128, 2),     # 512 of 128 x 128: resident
    (F8, 4096, 2048, 2048, True, 128, 2),
    (BF, 2300, 3500, 4096, True, 128, 2),      # 504, and 126 of 256 x 256
    (F8, 4096, 2176, 2048, True, 256, 2),      # 544
    (BF, 3072, 3072, 512, False, 256, 2)])     # 576
def test_256_from_more_than_two_programs_of_128(dt, M, N, K, b_trans, size,
                                                stages):
    A = torch.empty((M, K), dtype=dt)
    B = torch.empty((N, K + (-K) % 16 + 16) if b_trans else (K, N), dtype=dt)
    if b_trans:
        B = B[:, :K]
    C = torch.empty((M, N))
    old = tg.tile_picker_mode(0)
    try:
        got = tg.tile_gemm_plan(A, B, C, b_trans=b_trans, want_map=False)[0]
    finally:
        tg.tile_picker_mode(old)
    assert (got["bm"], got["stages"]) == (size, stages), got


@pytest.mark.parametrize("dt,M,N,K,b_trans,stages", [
    (BF, 2048, 2048, 512, True, 4), (BF, 2048, 2049, 512, True, 2),
    (BF, 2048, 2048, 512, False, 4), (BF, 2304, 2304, 512, False, 2),
    (F8, 2048, 2048, 512, True, 4), (F8, 4096, 4096, 512, True, 2),
    (F32, 4096, 4096, 512, True, 2)])
def test_partition_of_128_past_one_round(dt, M, N, K, b_trans, stages):
    """An explicit 128 x 128 partition takes the programs that the default
    takes of that size: past one round two of two stages per compute unit."""
    A = torch.empty((M, K), dtype=dt)
    B = torch.empty((N, K) if b_trans else (K, N), dtype=dt)
    C = torch.empty((M, N))
    got = tg.tile_gemm_plan(A, B, C, 128, 128, b_trans=b_trans,
                            want_map=False)[0]
    assert got["stages"] == stages, got


GROUPED = """
#include "tg_internal.hpp"
extern "C" int stages(int64_t tiles, int64_t longest, int64_t sum, int b_nk) {
    return tg::grouped_stages_128(tiles, longest, sum, b_nk, 256);
}
"""


def test_grouped_partition_of_128(tmp_path):
    """The rule of a grouped launch, by (problems, sub-tensors of each, K from,
    K to): two stages where they were measured ahead of, or level with, one
    program per compute unit."""
    src, lib = tmp_path / "g.cpp", tmp_path / "g.so"
    src.write_text(GROUPED)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC",
                    "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
                    os.path.join(ROOT, "paper_2606_15991_amd", "csrc"),
                    str(src), "-o", str(lib)], check=True)
    f = ctypes.CDLL(str(lib)).stages
    f.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int]

    def rule(n, tiles, lo, hi, nk):
        ks = [lo + (hi - lo) * i // (n - 1) for i in range(n)]
        return f(n * tiles, max(ks), tiles * sum(ks), nk)
    for n, tiles, lo, hi, by_nk, by_kn in (
            (200, 16, 512, 512, 2, 2), (12, 256, 512, 512, 2, 2),
            (100, 4, 1024, 1024, 2, 2), (12, 256, 2048, 2048, 0, 2),
            (40, 16, 2048, 2048, 0, 2), (20, 16, 2048, 3450, 0, 2),
            (20, 16, 2048, 4300, 0, 0), (40, 16, 2048, 6200, 0, 2),
            (20, 16, 512, 790, 2, 2), (16, 16, 512, 512, 0, 0)):
        assert rule(n, tiles, lo, hi, 1) == by_nk, (n, tiles, lo, hi)
        assert rule(n, tiles, lo, hi, 0) == by_kn, (n, tiles, lo, hi)


@pytest.mark.parametrize("M,N,K,size,wm", [
    (512, 512, 128, 32, 8), (512, 512, 124, 64, 2),      # one round of 32
    (640, 640, 256, 32, 8), (640, 640, 252, 64, 2),      # two
    (800, 800, 512, 32, 8), (800, 800, 508, 64, 2),      # three
    (103, 6000, 144, 64, 2)])
def test_binary32_shares_k_where_it_is_long(M, N, K, size, wm):
    old = tg.tile_picker_mode(0)
    try:
        got = tg.tile_gemm_plan(torch.empty((M, K)), torch.empty((N, K)),
                                torch.empty((M, N)), b_trans=True,
                                want_map=False)[0]
    finally:
        tg.tile_picker_mode(old)
    assert (got["bm"], got["wm"]) == (size, wm), got
