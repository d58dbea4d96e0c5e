"""The sources whose hash ties a traffic profile to the headline kernel hold
that kernel and what it includes."""
import os
import re
import sys

from conftest import ROOT

sys.path.insert(0, ROOT)


def test_hashed_sources_hold_the_headline_kernel():
    import bench
    named = {os.path.basename(f) for f in bench.KERNEL_SOURCES}
    csrc = os.path.join(ROOT, "paper_2606_15991_amd", "csrc")
    holders = [f for f in os.listdir(csrc)
               if "gemm_phased_kernel(" in open(os.path.join(csrc, f)).read()]
    assert holders == ["gemm_phased.hip"]
    todo, seen = list(holders), set()
    while todo:
        f = todo.pop()
        if f in seen:
            continue
        seen.add(f)
        todo += re.findall(r'#include "(tg_\w+\.hpp)"',
                           open(os.path.join(csrc, f)).read())
    assert seen <= named, seen - named
