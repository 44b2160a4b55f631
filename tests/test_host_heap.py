"""The host path of a transform on a plan that exists takes nothing from the heap: an allocation
can fail, and the exception would leave a C entry point.  Read from the assembly of the host side
(functions not inlined, so that each one's calls stand in it)."""
import os
import re
import subprocess

import pytest

from paper_1308_5706_amd import build as B

INCLUDE = os.path.join(B.HERE, "..", "include")


def test_transforms_take_nothing_from_the_heap(tmp_path):
    if not os.path.exists(B.HIPCC):
        pytest.skip("needs hipcc")
    out = tmp_path / "api.s"
    subprocess.run([B.HIPCC, "-x", "hip", "-S", "--cuda-host-only", os.path.join(B.CSRC, "api.cpp"), "-o", str(out),
                    "-O1", "-fno-inline", "-std=c++17", f"--offload-arch={B.ARCH}", "-I", INCLUDE, "-I", B.CSRC],
                   check=True, capture_output=True)
    text = out.read_text()
    for name in ("run_inverse", "run_forward"):
        m = re.search(rf"^(_ZN4s2dw\S*{name}\S*):.*?^\.Lfunc_end", text, re.S | re.M)
        assert m, name
        calls = set(re.findall(r"\bcallq?\s+(\S+)", m.group(0)))
        assert any("launch_wig" in c for c in calls)
        grows = ("_Znw", "malloc", "push_back", "emplace", "_M_realloc", "_M_insert", "resize")
        assert not [c for c in calls if any(g in c for g in grows)], name
