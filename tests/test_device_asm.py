"""What the inline assembly of the Wigner kernels promises the compiler, read from the assembly
that it writes for small kernels around the statements (compiled here, nothing runs)."""
import os
import re
import subprocess

import pytest

from paper_1308_5706_amd import build as B

INCLUDE = os.path.join(B.HERE, "..", "include")


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
    return [x for x in (line.split(";")[0].strip() for line in body.splitlines()) if x and not x.endswith(":")]


def test_loads_to_lds_say_that_they_write_m0(tmp_path):
    """Two loads of the compiler's own to one LDS address, with one of load_lds16 to another between
    them: m0 has to be set again for the second."""
    lines = assembly(tmp_path, """
__global__ void probe(const void *src, double *out) {
    __shared__ double buf[512];
    const __amdgpu_buffer_rsrc_t b = buf_of(src);
    auto *l = (__attribute__((address_space(3))) void *)buf;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(b, l, 4, threadIdx.x * 4u, 0, 0, 0);
    load_lds16(desc_of(src), threadIdx.x * 16u, 0, lds_off(buf + 256));
    __builtin_amdgcn_raw_ptr_buffer_load_lds(b, l, 4, threadIdx.x * 4u, 512, 0, 0);
    wait_lds<0>();
    out[threadIdx.x] = buf[threadIdx.x];
}""")
    loads = [i for i, x in enumerate(lines) if x.startswith("buffer_load") and x.endswith("lds")]
    assert len(loads) == 3
    m0 = [i for i, x in enumerate(lines) if re.match(r"s_mov(k_i32|_b32) m0,", x)]
    assert any(loads[1] < i < loads[2] for i in m0)


@pytest.mark.parametrize("call,loads", [
    ("load_lds16(desc_of(src), threadIdx.x * 16u, off[threadIdx.x], lds_off(buf))", 1),
    ("load_lds16_3(desc_of(src), threadIdx.x * 16u, off[threadIdx.x], off[threadIdx.x + 64], lds_off(buf), "
     "lds_off(buf + 128), desc_of(src), threadIdx.x * 16u, off[threadIdx.x + 128], lds_off(buf + 256))", 3)])
def test_loads_to_lds_wait_for_scalars_that_a_vector_instruction_wrote(tmp_path, call, loads):
    """Five wait states between a readfirstlane and the load that takes its result as the offset."""
    lines = assembly(tmp_path, """
__global__ void probe(const void *src, const unsigned *off, double *out) {
    __shared__ double buf[512];
    %s;
    wait_lds<0>();
    out[threadIdx.x] = buf[threadIdx.x];
}""" % call)
    at = [i for i, x in enumerate(lines) if x.startswith("buffer_load") and x.endswith("lds")]
    assert len(at) == loads
    for load in at:
        soffset = lines[load].split(",")[2].split()[0]
        write = max(i for i, x in enumerate(lines[:load]) if re.match(rf"\S+ {soffset},", x))
        assert lines[write].startswith("v_readfirstlane_b32")
        states = 0
        for x in lines[write + 1:load]:
            states += int(x.split()[1]) + 1 if x.startswith("s_nop") else 1
        assert states >= 5
