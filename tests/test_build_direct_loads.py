"""CPU: the loads that go to LDS without passing through registers, as the compiler takes them."""
import os
import re
import subprocess

from paper_2505_02351_amd import build

SOURCE = """
#include "prefill_kernels.hpp"
using namespace optgqa;
__global__ void copy(const unsigned char* p, uint32_t* out, int n)
{
    extern __shared__ uint32_t tile[];
    const uint32_t lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint32_t*)tile;
    for (int i = 0; i < n; ++i) {
        load_direct(lds + 1024 * __builtin_amdgcn_readfirstlane(i & 3), p + 1024 * i, threadIdx.x * 16);
        load_direct(lds + 4096, p + 1024 * i + 16 * threadIdx.x);
    }
    wait_direct();
    out[threadIdx.x] = tile[threadIdx.x];
}
"""


def test_direct_loads_compile_without_a_warning(tmp_path):
    """m0, which holds the loads' LDS address, is the compiler's to set: a statement that writes it by itself may find it gone."""
    src, asm = tmp_path / "copy.hip", tmp_path / "copy.s"
    src.write_text(SOURCE)
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    res = subprocess.run(["hipcc", *flags, "--cuda-device-only", "-S", "-I" + os.path.join(build.ROOT, "include"),
                          "-I" + os.path.join(build.PKG, "csrc"), str(src), "-o", str(asm)], capture_output=True, text=True)
    assert res.returncode == 0 and "m0" not in res.stderr, res.stderr[-2000:]
    code = [line.split(";")[0].split() for line in asm.read_text().splitlines()]
    code = [line for line in code if line and re.match(r"[sv]_|global_", line[0])]
    loads = [i for i, line in enumerate(code) if line[0] == "global_load_lds_dwordx4"]
    assert len(loads) >= 2
    for i in loads:                             # set right before, and a wait state in between
        assert code[i - 1][0] == "s_nop" and any("m0," in line[1:2] for line in code[i - 12:i - 1]), code[i - 12:i + 1]
