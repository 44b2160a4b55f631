"""The host path of a transform on a plan that exists takes nothing from the heap: an allocation
can fail, and the exception would leave a C entry point.  Read from the assembly of the host side
(functions not inlined, so that each one's calls stand in it)."""
import os
import re
import subprocess

import pytest

from paper_1308_5706_amd import build as B

INCLUDE = os.path.join(B.HERE, "..", "include")
# event records while stages are timed; look-ups of keys that the plan holds
ASIDE = ("5Stage", "prof_", "St3map", "St8_Rb_tree")
GROWS = ("_Znw", "malloc", "push_back", "emplace", "_M_realloc", "_M_insert", "resize")


def test_transforms_take_nothing_from_the_heap(tmp_path):
    if not os.path.exists(B.HIPCC):
        pytest.skip("needs hipcc")
    out = tmp_path / "api.s"
    subprocess.run([B.HIPCC, "-x", "hip", "-S", "--cuda-host-only", os.path.join(B.CSRC, "api.cpp"), "-o", str(out),
                    "-O1", "-fno-inline", "-std=c++17", f"--offload-arch={B.ARCH}", "-I", INCLUDE, "-I", B.CSRC],
                   check=True, capture_output=True)
    calls = {m.group(1): {c.split("@")[0] for c in re.findall(r"\b(?:callq?|jmp)\s+(_Z\S+)", m.group(2))}
             for m in re.finditer(r"^(_Z\S+):(.*?)^\.Lfunc_end", out.read_text(), re.S | re.M)}
    for name in ("run_inverse", "run_forward"):
        todo = [f for f in calls if name in f]
        assert todo, name
        seen = set()
        while todo:
            f = todo.pop()
            if f in seen or any(a in f for a in ASIDE):
                continue
            seen.add(f)
            assert not any(g in f for g in GROWS), (name, f)
            todo += calls.get(f, ())
        assert any("launch_wig" in f for f in seen)
