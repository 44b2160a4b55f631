"""What the inline assembly of the Wigner kernels promises the compiler, read from the assembly
that it writes for small kernels around the statement (compiled here, nothing runs)."""
import os
import re
import subprocess

import pytest

from paper_1308_5706_amd import build as B

INCLUDE = os.path.join(B.HERE, "..", "include")

# the five loads of a block, operands that the compiler cannot prove uniform
LOADS = """load_lds16_5<32, 8>(
        lds_load(desc_of(src), off[threadIdx.x], lds_off(buf + 512)), threadIdx.x * 16u, off[threadIdx.x + 64],
        lds_off(buf + 640), lds_load(desc_of(src), off[threadIdx.x + 128], lds_off(buf + 768)), threadIdx.x * 8u,
        lds_load(desc_of(src), off[threadIdx.x + 192], lds_off(buf + 896)), threadIdx.x * 16u,
        lds_load(desc_of(src), off[threadIdx.x + 256], lds_off(buf + 960)), threadIdx.x * 8u)"""


def assembly(tmp_path, body):
    if not os.path.exists(B.HIPCC):
        pytest.skip("needs hipcc")
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text('#include "wigner_k.h"\nnamespace s2dw {\n' + body + "\n}\n")
    subprocess.run([B.HIPCC, "-x", "hip", "-S", "--cuda-device-only", str(src), "-o", str(out), "-O3", "-std=c++17",
                    f"--offload-arch={B.ARCH}", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", INCLUDE, "-I", B.CSRC], check=True, capture_output=True)
    text = out.read_text()
    body = text[text.index("\n_ZN4s2dw5probe"):]
    body = body[:body.index("s_endpgm")]
    lines = [line.split(";")[0].strip() for line in body.splitlines()]
    return [x for x in lines if x and not x.endswith(":") and not x.startswith(".")]


def loads_to_lds(lines):
    return [i for i, x in enumerate(lines) if x.startswith("buffer_load") and x.endswith("lds")]


def test_loads_to_lds_say_that_they_write_m0(tmp_path):
    """Two loads of the compiler's own to one LDS address, with the statement's to others between
    them: m0 has to be set again for the second."""
    lines = assembly(tmp_path, """
__global__ void probe(const void *src, const unsigned *off, double *out) {
    __shared__ double buf[1024];
    const __amdgpu_buffer_rsrc_t b = buf_of(src);
    auto *l = (__attribute__((address_space(3))) void *)buf;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(b, l, 4, threadIdx.x * 4u, 0, 0, 0);
    %s;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(b, l, 4, threadIdx.x * 4u, 512, 0, 0);
    wait_lds<0>();
    out[threadIdx.x] = buf[threadIdx.x];
}""" % LOADS)
    at = loads_to_lds(lines)
    assert len(at) == 7
    m0 = [i for i, x in enumerate(lines) if re.match(r"s_mov(k_i32|_b32) m0,", x)]
    assert any(at[5] < i < at[6] for i in m0)


def test_loads_to_lds_wait_for_scalars_that_a_vector_instruction_wrote(tmp_path):
    """Five wait states between a readfirstlane and the load that takes its result as the offset; m0
    one before its load; the lane mask as it was afterwards."""
    lines = assembly(tmp_path, """
__global__ void probe(const void *src, const unsigned *off, double *out) {
    __shared__ double buf[1024];
    %s;
    wait_lds<0>();
    out[threadIdx.x] = buf[threadIdx.x];
}""" % LOADS)
    at = loads_to_lds(lines)
    assert len(at) == 5
    for load in at:
        soffset = lines[load].split(",")[2].split()[0]
        write = max(i for i, x in enumerate(lines[:load]) if re.match(rf"\S+ {soffset},", x))
        assert lines[write].startswith("v_readfirstlane_b32")
        states = sum(int(x.split()[1]) + 1 if x.startswith("s_nop") else 1 for x in lines[write + 1:load])
        assert states >= 5
        assert lines[load - 2].startswith("s_mov_b32 m0,") and lines[load - 1].startswith("s_nop")
    masks = [x for x in lines[at[2]:] if "exec" in x and x.startswith("s_")]
    assert masks[0].startswith("s_mov_b64") and masks[0].endswith("exec")
    saved = masks[0].split()[1].rstrip(",")
    assert masks[1:3] == ["s_lshr_b64 exec, -1, 32", "s_lshr_b64 exec, -1, 56"]
    assert masks[3] == f"s_mov_b64 exec, {saved}"
