"""The asm copies global -> LDS set the register m0 and have to say so: between two of the compiler's own copies to one LDS
address, which both need m0, it must not take the value it set for the first one to be still there.  Compiled to gfx950
assembly on the CPU; nothing runs."""
import re
import subprocess

import pytest

from paper_2605_16732_amd import build as BLD

KERNEL = r"""
#include "dirotq_internal.h"
typedef const __attribute__((address_space(1))) void* gp;
typedef __attribute__((address_space(3))) void* lp;
extern "C" __global__ void probe(const char* p, const char* q, float* out) {
  __shared__ __align__(16) float s[1024];
  __builtin_amdgcn_global_load_lds((gp)(p + 4 * threadIdx.x), (lp)s, 4, 0, 0);
  dirotq::%s(dirotq::lds_address(s) + 2048, 16 * threadIdx.x, q);
  __builtin_amdgcn_global_load_lds((gp)(q + 4 * threadIdx.x), (lp)s, 4, 0, 0);
  __syncthreads();
  out[threadIdx.x] = s[threadIdx.x];
}
"""


@pytest.mark.parametrize("copy", ["copy_to_lds", "copy4_to_lds"])
def test_m0_is_set_again_after_an_asm_copy(copy, tmp_path):
    src, asm = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(KERNEL % copy)
    subprocess.run([BLD.hipcc(), *BLD.HIPCC_FLAGS, "-I", BLD.ROOT + "/include", "-I", BLD.CSRC, "--offload-device-only", "-S", str(src),
                    "-o", str(asm)], check=True, capture_output=True)
    text = [ln.split(";")[0].strip() for ln in asm.read_text().splitlines()]
    seen = [ln for ln in text if re.search(r"\bm0\b", ln) or ln.startswith("global_load_lds")]
    loads = [i for i, ln in enumerate(seen) if ln.startswith("global_load_lds")]
    assert len(loads) == 3, seen
    for i in loads:                                        # each load has its own write of m0 in front of it
        assert i > 0 and "m0" in seen[i - 1] and not seen[i - 1].startswith("global_load_lds"), seen
