"""The plan names the form of the decode and of the simple kernel that a launch
runs, on both sides of each line that chooses between them, and at every shape
by which the GPU tests mean to run one of them (planned for 256 compute
units)."""
import pytest
import torch

import paper_2606_15991_amd as tg
import test_gpu_decode_stream
import test_gpu_phased128

BF, F8, F32 = torch.bfloat16, torch.float8_e4m3fn, torch.float32


def plan(M, N, K, wdt, cfg, pad=(0, 0), adt=BF, want_map=False, b_trans=True):
    A = torch.empty((M, K + pad[0]), dtype=adt, device="meta")[:, :K]
    B = torch.empty((N, K + pad[1]) if b_trans else (K, N), dtype=wdt,
                    device="meta")
    if b_trans:
        B = B[:, :K]
    C = torch.empty((M, N), device="meta")
    da, db, dc = tg.make_in(A), tg.make_in(B, b_trans), tg.make_out(C)
    da.data, db.data, dc.data = 1 << 40, 2 << 40, 3 << 40
    c = tg.tg_config()
    st = tg.lib.tile_gemm_plan(da, db, dc, tg.make_opts(config=cfg), c, None,
                               None, None)
    assert st == tg.TG_OK
    return c.as_dict()


def cases(test):
    mark = next(m for m in test.pytestmark if m.name == "parametrize" and
                m.args[0].count(",") > 1)
    return mark.args[1]


def decode(bn=0):
    return {"kind": "skinny", "bn": bn, "ksplit": 4 if bn else 0,
            "splitk": 1}


@pytest.mark.parametrize("wdt,M,N,K,bn,stream", [
    # 85 in 100 workgroups' worth of programs: 218 of 256, 435 of 512
    (BF, 8, 217 * 16, 1024, 16, 0), (BF, 8, 218 * 16, 1024, 16, 4),
    (F8, 2, 435 * 16, 4096, 16, 0), (F8, 2, 436 * 16, 4096, 16, 4),
    # several programs a workgroup, few rows: 25 blocks of K, 17 with three
    # or four rows, e4m3 17 with one or two in up to five programs
    # (rows are K + 8 long); 33, 36 and 37 blocks round eight wavefronts
    (BF, 2, 16384, 1528, 16, 0), (BF, 2, 16384, 1976, 16, 4),
    (BF, 2, 16384, 2104, 16, 0), (BF, 2, 16384, 2296, 16, 0),
    (BF, 2, 16384, 2360, 16, 4), (BF, 3, 16384, 2104, 16, 4),
    # rows of no whole 128 bytes: 65 blocks
    (BF, 2, 16384, 1984, 16, 0), (BF, 2, 16384, 4096, 16, 0),
    (BF, 2, 16384, 4160, 16, 4),
    (BF, 3, 16384, 1024, 16, 0), (BF, 4, 16384, 1032, 16, 4),
    (BF, 2, 16384, 1024, 25, 4), (BF, 5, 16384, 1024, 16, 4),
    (F8, 2, 20480, 2048, 16, 0), (F8, 2, 20480, 2064, 16, 4),
    (F8, 2, 23040, 2048, 16, 4), (F8, 3, 20480, 2048, 16, 4),
    # two programs a workgroup, 256 KiB apart (rows padded by eight elements)
    (BF, 1, 8192, 4088, 16, 0), (BF, 4, 8192, 8184, 16, 0),
    (BF, 1, 8192, 5112, 16, 4), (BF, 5, 8192, 4088, 32, 4),
    (BF, 1, 16384, 4088, 16, 4),
    # up to 20 columns a workgroup: 320 blocks
    (BF, 1, 5120, 20480, 20, 4), (BF, 1, 5120, 20488, 20, 0),
    (BF, 1, 5376, 20488, 21, 4), (F8, 1, 5120, 40960, 20, 4),
    # a second row tile of one or two columns
    (BF, 4, 4608, 4096, 18, 0), (BF, 4, 4864, 4096, 19, 4),
    (BF, 5, 4608, 4096, 18, 4), (BF, 4, 4096, 4096, 16, 4),
    # more than eleven blocks of 128 bytes of K
    (BF, 1, 4096, 704, 16, 0), (BF, 1, 4096, 712, 16, 4),
    (F8, 1, 4096, 1408, 16, 0), (F8, 1, 4096, 1424, 16, 4),
    # activations beside the ring within 160 KiB of LDS
    (BF, 8, 12288, 5120, 16, 4), (BF, 16, 12288, 5120, 16, 0),
    # K of whole 16-byte chunks of the weights
    (F8, 1, 4096, 2040, 16, 0), (F8, 1, 4096, 2048, 16, 4)])
def test_decode_lines(wdt, M, N, K, bn, stream):
    got = plan(M, N, K, wdt, decode(bn), (8, 8 if wdt == BF else
                                          16 - K % 16))
    assert (got["kind"], got["stages"]) == (tg.TG_KIND_SKINNY, stream), got


def test_decode_split_runs_the_plain_form():
    cfg = {"kind": "skinny", "bn": 16, "ksplit": 4, "splitk": 2}
    o = plan(8, 4096, 2048, BF, cfg)
    assert (o["splitk"], o["stages"]) == (2, 0)


@pytest.mark.parametrize("case",
                         cases(test_gpu_decode_stream.test_decode_stream))
def test_stream_tests_run_the_streaming_form(case):
    wdt, M, N, K, bn, _ = case
    assert plan(M, N, K, wdt, decode(bn), (8, 16))["stages"] == 4


# simple kernel: (wavefronts down, across, K tile, LDS stages)
@pytest.mark.parametrize("adt,bdt,M,N,K,b_trans,want", [
    (BF, F8, 300, 5500, 64, True, (4, 2, 64, 4)),      # 129 blocks of 128
    (BF, F8, 300, 5200, 64, True, (2, 2, 64, 2)),      # 123
    (BF, F8, 300, 5500, 72, True, (2, 4, 64, 2)),      # half a chunk of K
    (BF, F8, 300, 5504, 64, False, (2, 4, 64, 2)),     # B stored K x N
    (BF, BF, 1111, 1531, 1003, False, (2, 2, 64, 2)),
    (F32, F32, 2100, 2200, 71, True, (2, 4, 32, 2))])
def test_simple_forms(adt, bdt, M, N, K, b_trans, want):
    got = plan(M, N, K, bdt, {"kind": "simple"}, (0, 16 - K % 16), adt,
               b_trans=b_trans)
    assert (got["wm"], got["wn"], got["bk"], got["stages"]) == want, got


@pytest.mark.parametrize("case", cases(test_gpu_phased128.test_mixed))
def test_mixed_tests_run_the_mixed_form(case):
    M, N, K = case
    got = plan(M, N, K, F8, None, (8, 16))
    assert (got["kind"], got["wm"], got["stages"]) == \
        (tg.TG_KIND_SIMPLE, 4, 4), got


def launch_of(cfg):
    """What tells two launches apart: the streaming form has no use for
    ksplit, the two-stage cross-tile schedules are one kernel."""
    c = dict(cfg)
    if c["kind"] == tg.TG_KIND_SKINNY and c["stages"]:
        c["ksplit"] = 0
    if c["sched"] == tg.TG_SCHED_CROSS_WARM:
        c["sched"] = tg.TG_SCHED_CROSS
    return tuple(sorted(c.items()))


@pytest.mark.parametrize("dt,wdt,M,N,K,bns", [
    (BF, F8, 8, 51200, 5120, {16, 32, 25}), (BF, BF, 1, 5120, 5120, {20}),
    (BF, F8, 1, 5120, 5120, {20}), (BF, BF, 8192, 8192, 8192, None),
    (BF, BF, 4096, 4096, 32768, None), (F8, F8, 2048, 2048, 2048, None)])
def test_candidates_name_each_launch_once(dt, wdt, M, N, K, bns):
    A = torch.empty((M, K), dtype=dt)
    B = torch.empty((N, K), dtype=wdt)
    C = torch.empty((M, N))
    old = tg.tile_picker_mode(0)
    try:
        dflt = tg.tile_gemm_plan(A, B, C, b_trans=True, want_map=False,
                                 workspace_bytes=1 << 40)[0]
    finally:
        tg.tile_picker_mode(old)
    cands = tg.tile_gemm_candidates(A, B, C, b_trans=True)
    assert len({launch_of(c) for c in cands}) == len(cands)
    if bns is None:
        assert dflt in cands
    else:
        assert {c["bn"] for c in cands if c["kind"] == tg.TG_KIND_SKINNY and
                c["stages"]} >= bns
