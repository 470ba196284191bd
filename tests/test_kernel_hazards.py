"""Wait states that the compiler leaves to whoever writes inline assembly, looked for in the assembly of the helpers that the
kernels share (built from source here, no GPU needed)."""
import os
import re
import subprocess

import pytest

from paper_2511_05811_amd import build

COPIES = """
#include "moss_gemm.h"
using namespace moss;
__global__ void copies(const uint8_t *p, uint32_t lds, uint32_t k)
{
    dma16(p, threadIdx.x * 16, lds);
    dma16(p, threadIdx.x * 16 + 64, lds + k);
#pragma unroll
    for (int x = 0; x < 3; x++) dma16_at(p, threadIdx.x * 16 + k, lds, x * 1024);
    wait_vmcnt<0>();
}
"""


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    src = tmp_path_factory.mktemp("hazards") / "copies.hip"
    src.write_text(COPIES)
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    res = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags + ["-I", build.INCLUDE, "-I", build.CSRC, "-S", "--offload-device-only",
                          "-o", "-", str(src)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return [l.split(";")[0].split() for l in res.stdout.splitlines() if l.startswith("\t") and not l.strip().startswith((".", ";"))]


def test_a_copy_into_lds_waits_one_state_behind_the_write_of_m0(assembly):
    copies = [i for i, l in enumerate(assembly) if l and l[0].startswith("global_load_lds")]
    assert len(copies) == 5
    for i in copies:
        assert not (len(assembly[i - 1]) > 1 and assembly[i - 1][1].startswith("m0")), (assembly[i - 1], assembly[i])


def test_the_kernels_copy_into_lds_through_these_helpers_only():
    for name in os.listdir(build.CSRC):
        text = open(os.path.join(build.CSRC, name)).read()
        assert len(re.findall(r"load_lds|lds_dword|buffer_load\w* .*lds", text)) == (2 if name == "moss_gemm.h" else 0), name
