"""The tables of a batched rebuild and of a batch's replicas are compared byte by byte to see whether a replica's storage
moved, so their structures hold no padding, whose bytes nothing sets."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TABLES = {"grid.hip": ["GridJob", "WrapArgs", "SortArgs"], "pairlist.hip": ["ListJob", "SearchArgsT", "FinishArgs"],
          "forces.hip": ["RepDesc"]}


@pytest.mark.parametrize("source", sorted(TABLES))
def test_no_padding(source):
    from paper_1306_1737_amd import build
    hipcc = build._hipcc()
    if shutil.which(hipcc) is None:
        pytest.skip("no hipcc")
    r = subprocess.run([hipcc, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-fsyntax-only",
                        "-Wpadded", os.path.join(build.CSRC, source)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    text = open(os.path.join(build.CSRC, source)).read()
    for name in TABLES[source]:
        assert re.search(r"struct %s\b" % name, text), name
        hits = [line for line in r.stderr.splitlines() if "padding" in line and re.search(r"\b%s\b" % name, line)]
        assert not hits, hits
