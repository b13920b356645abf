"""The staged kernel's requests to LDS are inline assembly, which the compiler does not look into: what they need of the code around
them, read off the assembly of small kernels compiled here (no GPU)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2512_17970_amd import build

SOURCE = r"""
#include "gemm_staged_impl.h"
using namespace cg;
typedef __attribute__((address_space(3))) void lds_void;

extern "C" __global__ void fresh_descriptor(const unsigned char* const* p, unsigned* out)
{
    extern __shared__ unsigned char smem[];
    const u32x4_t words = buffer_words(p[threadIdx.x], 4096);
    load_to_lds<false>(0, threadIdx.x * 16, words, 0);
    wait_requests<0>();
    out[threadIdx.x] = smem[threadIdx.x];
}

extern "C" __global__ void among_others(unsigned char* p, unsigned* out)
{
    extern __shared__ unsigned char smem[];
    const u32x4_t words = buffer_words(p, 4096);
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(p, 0, 4096, 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void*)smem, 4, threadIdx.x * 4, 0, 0, 0);
    load_to_lds<STREAM>(1024, threadIdx.x * 16, words, 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void*)smem, 4, threadIdx.x * 4, 512, 0, 0);
    wait_requests<0>();
    out[threadIdx.x] = smem[threadIdx.x];
}
"""

pytestmark = pytest.mark.skipif(shutil.which(build.HIPCC) is None, reason="no hipcc")


def instructions(tmp_path, kernel, stream="false"):
    src, asm = tmp_path / "requests.hip", tmp_path / "requests.s"
    src.write_text(SOURCE.replace("STREAM", stream))
    subprocess.run([build.HIPCC, *build.FLAGS, "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, "--cuda-device-only", "-S", str(src), "-o", str(asm)],
                   check=True, capture_output=True)
    body = asm.read_text().split(f"\n{kernel}:", 1)[1].split("s_endpgm", 1)[0]
    lines = (line.split(";")[0].strip() for line in body.splitlines())
    return [line for line in lines if line and not line.startswith(".") and not line.endswith(":")]


def test_a_request_waits_for_its_descriptor(tmp_path):
    """Five wait states between a vector instruction that writes a scalar register and the buffer instruction that reads it."""
    code = instructions(tmp_path, "fresh_descriptor")
    use = next(i for i, line in enumerate(code) if line.startswith("buffer_load"))
    last = max(i for i, line in enumerate(code[:use]) if re.match(r"v_read(first)?lane", line))
    states = sum(int(line.split()[1]) + 1 if line.startswith("s_nop") else 1 for line in code[last + 1:use])
    assert states >= 5, code[last:use + 1]


@pytest.mark.parametrize("stream", ["false", "true"])
def test_requests_share_m0_with_the_compiler(tmp_path, stream):
    """A request of the compiler's own behind one of these sets its LDS address again."""
    code = instructions(tmp_path, "among_others", stream)
    loads = [i for i, line in enumerate(code) if line.startswith("buffer_load") and line.endswith("lds")]
    assert [line.split()[0] for line in (code[i] for i in loads)] == ["buffer_load_dword", "buffer_load_dwordx4", "buffer_load_dword"]
    for before, at in zip([0] + loads, loads):
        assert any(re.match(r"s_\w+ m0,", line) for line in code[before:at]), code[before:at + 1]
