"""Pinned host memory that kernels of several devices' contexts write has to be
mapped on all of them.  One GPU cannot show the difference, so the allocations
are read in the source."""
import os
import re

CTX = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_1503_08366_amd", "csrc", "ctx.hpp")


def test_blocks_that_kernels_write_are_portable():
    text = open(CTX).read()
    for name in ("PinnedSlab", "PinnedOut"):
        body = text[text.index(f"class {name} {{"):]
        body = body[:body.index("\n};")]
        calls = re.findall(r"hipHostMalloc\(([^;{]*?)\) != hipSuccess", body)
        assert calls and all("hipHostMallocPortable" in c for c in calls), name
