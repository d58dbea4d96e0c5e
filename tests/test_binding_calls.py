"""The binding's call frame: the fields it packs are those of the descriptor
objects, the errors it raises theirs, and threads do not share a frame."""
import ctypes
import threading

import pytest
import torch

import paper_2606_15991_amd as tg

BF = torch.bfloat16


def fields(d):
    return tuple(getattr(d, f) or 0 for f, _ in d._fields_)


@pytest.mark.parametrize("make", [
    lambda: torch.empty((3, 5), dtype=BF),
    lambda: torch.empty((1, 5)),
    lambda: torch.empty((4, 16), dtype=BF)[:, :5],
    lambda: torch.empty((7, 3))[:1],
    lambda: torch.empty((2, 9, 8), dtype=torch.float8_e4m3fn)[:, 0],
    lambda: torch.empty((1, 8)).t()[:1],          # one element, stride 1
    lambda: torch.empty((0, 4)), lambda: torch.empty((4, 0)),
    lambda: torch.empty((1, 0)), lambda: torch.empty(6)[2:4].view(1, 2),
    lambda: torch.empty((8, 1)), lambda: torch.empty((5, 4)).t()[:, :1]])
def test_packed_fields_equal_the_descriptors(make):
    t = make()
    for trans in (0, 1):
        assert tg._in(t, trans) == fields(tg.make_in(t, trans))


@pytest.mark.parametrize("t,status", [
    (torch.empty((2, 2), dtype=torch.int32), tg.TG_E_DTYPE),
    (torch.empty((2, 2, 2)), tg.TG_E_SHAPE),
    (torch.empty((4, 4)).t(), tg.TG_E_SHAPE)])
def test_same_errors(t, status):
    for f in (tg._in, tg.make_in):
        with pytest.raises(tg.TileGemmError) as e:
            f(t)
        assert e.value.status == status


def test_options_and_frame_layout():
    scale, ws = torch.ones(4), torch.empty(64, dtype=torch.uint8)
    cfg = tg.make_config({"kind": "tiled", "bm": 64, "bn": 64})
    o = tg.make_opts("bf16x3", scale, scale, cfg, ws, None, False)
    vals = tg._opts(tg.TG_PREC_BF16X3, False, scale, scale, cfg, ws, None, 0)
    f = tg._Frame()
    ins = [torch.empty((i + 2, 5), dtype=BF) for i in range(4)]
    tg._pack.pack_into(f, 0, *tg._in(ins[0]), *tg._in(ins[1], 1),
                       *tg._in(ins[2]), *tg._in(ins[3]), 7, 9, *vals)
    for got, want in ((f.a, tg.make_in(ins[0])),
                      (f.b, tg.make_in(ins[1], True)),
                      (f.x, tg.make_in(ins[2])),
                      (f.c, tg.make_out(ins[3], 7, 9))):
        assert fields(got) == fields(want)
    for name, _ in tg.tg_opts._fields_:
        a, b = getattr(f.o, name), getattr(o, name)
        if name == "config":
            a, b = ctypes.addressof(a.contents), ctypes.addressof(b.contents)
        if name != "residual":
            assert a == b, name


def test_one_frame_per_thread():
    seen = []

    def work():
        seen.append(ctypes.addressof(tg._call.f))

    ts = [threading.Thread(target=work) for _ in range(2)]
    for t in ts:
        t.start()
        t.join()
    work()
    assert len({seen[2]} | {ctypes.addressof(tg._call.f)}) == 1
    assert seen[2] not in seen[:2]
