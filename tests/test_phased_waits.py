"""The phased schedule's LDS reads (gemm_phased.hip) are complete when the other
group loads over what they read, in the assembly that the compiler makes of it.

A half is loaded over four slots after the first group read it.  The second
group reads one slot later, so its read must be covered by a counter wait
before the third barrier after it: a read that only its use waits for, two
slots further on, leaves the order to the latencies."""
import os
import re
import subprocess

import pytest

from conftest import ROOT
from paper_2606_15991_amd import build as lib_build


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm") / "phased.s"
    subprocess.run([lib_build.HIPCC, *lib_build.COMMON,
                    *lib_build.DEVICE_FLAGS, "-S", "--offload-device-only",
                    os.path.join(lib_build.CSRC, "gemm_phased.hip"),
                    "-o", str(out)], check=True, capture_output=True)
    return out.read_text()


def kernels(text):
    name, body = None, []
    for line in text.split("\n"):
        m = re.match(r"^(_Z\w*gemm_\w*kernel\w*):", line)
        if m:
            name, body = m.group(1), []
        elif name and line.startswith(".Lfunc_end"):
            yield name, body
            name = None
        elif name:
            body.append(line.split(";")[0].strip())


def k_loop(body):
    """The smallest loop that holds two K tiles' matrix instructions (eight
    phases of 16, e4m3 of 8) and fragment reads (24 a tile, 32 where B's are
    transposing ones)."""
    reads = 64 if any(l.startswith("ds_read_b64_tr") for l in body) else 48
    need = 64 if any("_f8f6f4" in l for l in body) else 128
    label = {l[:-1]: i for i, l in enumerate(body) if l.endswith(":")}
    loops = []
    for i, l in enumerate(body):
        m = re.match(r"s_c?branch\w*\s+(\S+)", l)
        if m and label.get(m.group(1), i) < i:
            part = body[label[m.group(1)]:i]
            if sum(x.startswith("v_mfma") for x in part) >= need and \
                    sum(x.startswith("ds_read") for x in part) >= reads:
                loops.append(part)
    return min(loops, key=len)


def barriers_to_wait(loop):
    """Most barriers between an LDS read and the wait that covers it, in two
    rounds of the loop.  A wavefront's LDS accesses complete in order."""
    flight, barriers, worst = [], 0, 0
    for l in loop + loop:
        if l.startswith("ds_"):
            flight.append(barriers)
        elif l.startswith("s_barrier"):
            barriers += 1
        m = re.match(r"s_waitcnt.*lgkmcnt\((\d+)\)", l)
        if m and len(flight) > int(m.group(1)):
            done = len(flight) - int(m.group(1))
            worst = max([worst] + [barriers - b for b in flight[:done]])
            flight = flight[done:]
    return worst


def test_reads_are_waited_for_before_their_half_is_loaded_over(assembly):
    seen = 0
    for name, body in kernels(assembly):
        if "Li256ELi256E" in name:
            assert barriers_to_wait(k_loop(body)) <= 2, name
            seen += 1
    assert seen == 14


def test_accumulators_stay_in_their_registers(assembly):
    """The matrix instructions are inline assembly, so the compiler puts no
    wait states between them and a spill or copy of an accumulator: there is
    none.  Of the accumulation registers only the stores' own reads appear,
    after the drain."""
    spills = re.findall(r"\.(vgpr_spill_count|private_segment_fixed_size):"
                        r"\s+(\d+)", assembly)
    assert len(spills) >= 2 * 22
    assert all(n == "0" for _, n in spills), spills
    for name, body in kernels(assembly):
        acc = [l for l in body if "accvgpr" in l]
        assert acc and all(l.startswith("v_accvgpr_read_b32")
                           for l in acc), name
        first = next(i for i, l in enumerate(body) if "accvgpr" in l)
        assert "s_nop 15" in body[:first], name


REMARKS = """x.hip:9:1: remark: Function Name: _Z1av [-Rpass-analysis]
x.hip:9:1: remark:     ScratchSize [bytes/lane]: %d [-Rpass-analysis]
x.hip:9:1: remark:     SGPRs Spill: 3 [-Rpass-analysis]
x.hip:9:1: remark:     VGPRs Spill: %d [-Rpass-analysis]
"""


def test_the_build_refuses_spills():
    assert "gemm_phased.hip" in lib_build.NO_SPILL
    lib_build.check_no_spill("x.hip", REMARKS % (0, 0) + REMARKS % (0, 0))
    for bad in (REMARKS % (0, 0) + REMARKS % (8, 0), REMARKS % (0, 1), ""):
        with pytest.raises(RuntimeError):
            lib_build.check_no_spill("x.hip", bad)


def test_inline_assembly_names_what_it_overwrites():
    """M0 and SCC: the compiler may keep a value of its own in either."""
    seen = 0
    for f in sorted(os.listdir(lib_build.CSRC)):
        text = open(os.path.join(lib_build.CSRC, f)).read()
        for block in re.findall(r"asm volatile\((.*?)\);", text, re.S):
            code = " ".join(re.findall(r'"([^"]*)"', block))
            code = re.sub(r"\\[nt]", " ", code)
            clobbers = block.rsplit(":", 1)[-1]
            if re.search(r"\bs_\w+ m0,", code):
                seen += 1
                assert '"m0"' in clobbers, (f, block)
            if re.search(r"\bs_(add|sub|and|or|lshl|cmp)_", code):
                assert '"scc"' in clobbers, (f, block)
    assert seen == 7
