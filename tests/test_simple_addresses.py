"""Addresses that the kernel for unaligned operands (gemm_simple.hip) reads of
a B stored K x N without checks, at every block of explicit partitions: all of
them inside the operand.  The rules are compiled from the kernel's own header;
the loader's addresses are formed here as it forms them."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from conftest import ROOT

CSRC = os.path.join(ROOT, "paper_2606_15991_amd", "csrc")

SOURCE = """
#include "tg_internal.hpp"
extern "C" int whole_tiles(int K, int bk, int b_nk, int N, int n0, int bn,
                           int epc) {
    return tg::simple_whole_tiles(K, bk, b_nk, N, n0, bn, epc);
}
extern "C" int shift(uintptr_t base, int64_t ld, int64_t es, int64_t step) {
    return tg::simple_shift(base, ld, es, step);
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, lib = d / "rules.cpp", d / "rules.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC",
                    "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", CSRC, str(src), "-o", str(lib)], check=True)
    return ctypes.CDLL(str(lib))


def ends(K, N, ld, n0, BN, epc, tiles, bk):
    """Last element (plus one) of every chunk that the unchecked tiles read;
    chunks past N read column 0."""
    col = n0 + np.arange(0, BN, epc)
    col = np.where(col < N, col, 0)
    k = np.arange(tiles * bk)
    return (k[:, None] * ld + col[None, :]) + epc


@pytest.mark.parametrize("es,epc,bk", [(4, 4, 32), (2, 8, 64), (1, 8, 64)])
@pytest.mark.parametrize("N", [1, 5, 8, 63, 64, 65, 72, 130, 136, 200])
def test_unchecked_loads_stay_inside(rules, es, epc, bk, N):
    for K in (1, bk - 1, bk, 2 * bk, 3 * bk + 5):
        for bn in list(range(1, 65)) + [128]:
            BN = 128 if bn == 128 else 64
            for n0 in range(0, N, bn):
                t = rules.whole_tiles(K, bk, 0, N, n0, BN, epc)
                assert 0 <= t <= K // bk
                for ld in (N, N + 1, N + 8):
                    if t:
                        last = ends(K, N, ld, n0, BN, epc, t, bk).max()
                        assert last <= (K - 1) * ld + N, (K, bn, n0, ld)
                # rows of whole tiles are left out only where they must be
                if N - n0 >= BN or (N - n0) % epc == 0:
                    assert t == K // bk
                assert rules.whole_tiles(K, bk, 1, N, n0, BN, epc) == K // bk


@pytest.mark.parametrize("es,epc", [(4, 4), (2, 8), (1, 8)])
def test_unshifted_chunks_are_whole_dwords(rules, es, epc):
    i64 = ctypes.c_int64
    rules.shift.argtypes = [ctypes.c_size_t, i64, i64, i64]
    for base in range(0, 8, es):
        for ld in range(128, 136):
            for step in range(0, 65):
                n0 = step * np.arange(4)
                k = np.arange(8)
                at = base + (k[:, None, None] * ld + n0[:, None] +
                             np.arange(0, 64, epc)) * es
                assert bool(rules.shift(base, ld, es, step)) == \
                    bool((at % 4).any()), (base, ld, step)
