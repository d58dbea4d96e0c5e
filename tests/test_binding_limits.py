"""Arguments that the binding's call frame cannot take as they are: they come
to what the descriptor objects make of them, and to the same errors."""
import ctypes

import pytest
import torch

import paper_2606_15991_amd as tg

BF = torch.bfloat16


def status(f):
    with pytest.raises(tg.TileGemmError) as e:
        f()
    return e.value.status


def test_integers_past_their_field():
    A = torch.empty((8, 64), dtype=BF)
    B = torch.empty((64, 32), dtype=BF)
    C = torch.empty((8, 32))
    x = torch.empty(64, dtype=BF)
    for bm in (2 ** 31, 2 ** 32 - 1, -1):
        assert tg.make_out(C, bm, 4).bm < 0
        assert status(lambda: tg.tile_gemm(A, B, C, bm, 4)) == tg.TG_E_ARG
        assert status(lambda: tg.tile_add(A, A, A.clone(), bm, 4)) == \
            tg.TG_E_ARG
        assert status(lambda: tg.tile_rms_norm(A, x, A.clone(), bm=bm)) == \
            tg.TG_E_ARG
    assert status(lambda: tg.tile_gemm(A, B, C, precision=2 ** 40 + 7)) == \
        tg.TG_E_ARG


def test_wrapped_fields_equal_the_descriptors():
    A = torch.empty((8, 64), dtype=BF)
    f = tg._Frame()
    for v in (2 ** 31, 2 ** 32 + 64, -2 ** 31 - 1):
        tg._fill(f, tg._in(A, 1) + tg._in(A) + tg._NO_IN + tg._in(A) +
                 (v, 16) + tg._opts(v, True, None, None, None, None, None, 0))
        want = tg.make_out(A, v, 16)
        assert (f.c.bm, f.c.bn, f.c.ld) == (want.bm, want.bn, want.ld)
        assert f.o.precision == ctypes.c_int32(v).value
        assert f.a.data == A.data_ptr() and f.a.trans == 1


@pytest.mark.parametrize("b_trans,error", [
    (2, tg.TileGemmError), (-1, tg.TileGemmError),
    (torch.tensor(2), tg.TileGemmError), (None, TypeError),
    ("x", ValueError)])
def test_b_trans_is_zero_or_one(b_trans, error):
    A = torch.empty((8, 64), dtype=BF)
    B = torch.empty((64, 32), dtype=BF)
    C = torch.empty((8, 32))
    for f in (tg.tile_gemm, tg.tile_gemm_noalloc, tg.tile_gemm_plan):
        with pytest.raises(error):
            f(A, B, C, b_trans=b_trans)


@pytest.mark.parametrize("call,entry", [
    (lambda t: tg.tile_gemm(t[0], t[1], t[2], residual=t[2]), "tile_gemm"),
    (lambda t: tg.tile_add(t[0], t[0], t[3]), "tile_add"),
    (lambda t: tg.tile_rms_norm(t[0], t[4], t[3]), "tile_rms_norm"),
    (lambda t: tg.tile_rms_norm_matvec(t[0], t[4], t[5], t[6]),
     "tile_rms_norm_matvec")])
def test_a_call_inside_another_leaves_it_alone(monkeypatch, call, entry):
    """What a signal handler or a finalizer between filling the frame and the
    library's reading it does: another call of the same thread."""
    t = [torch.empty(s, dtype=d) for s, d in (
        ((8, 64), BF), ((64, 32), BF), ((8, 32), torch.float32),
        ((8, 64), BF), ((64,), BF), ((48, 64), BF), ((8, 48), BF))]
    other = torch.empty((3, 16), dtype=BF)
    seen = []

    def library(*args):
        descs = [a._obj for a in args if hasattr(a, "_obj")]
        before = [bytes(d) for d in descs]
        if not seen:
            seen.append(1)
            tg.tile_add(other, other, other)
        assert [bytes(d) for d in descs] == before
        return 0
    for e in {entry, "tile_add"}:
        monkeypatch.setattr(tg.lib, e, library)
    call(t)
    assert seen
    assert not tg._call.held.busy
