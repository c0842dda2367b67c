"""The load straight into shared memory, in the code compiled for the card: where a vector instruction has just written the scalar
pair of its address the five wait states stand before it (or a scalar instruction has copied it since), m0 is the compiler's to write, and it has
nothing to say about the statement."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2512_15550_amd import build

SOURCE = r"""
#include "arith.hpp"
using namespace ctkvr;
__global__ void from_uniform_pointer(const char *const *from, float *out)
{
    extern __shared__ float s[];
    const uint64_t p = (uint64_t)from[threadIdx.x];
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)p), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32));
    load_to_lds(0u, (const char *)(((uint64_t)hi << 32) | lo), threadIdx.x * 16u);
    __builtin_amdgcn_s_waitcnt(0x0f70);
    out[threadIdx.x] = s[threadIdx.x];
}
"""


@pytest.mark.skipif(not shutil.which(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")), reason="needs hipcc")
def test_wait_states_and_m0(tmp_path):
    src = tmp_path / "load.hip"
    src.write_text(SOURCE)
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *build.HIPCC_FLAGS, "-I", build.CSRC, "--cuda-device-only", "-S", "-o", str(tmp_path / "load.s"), str(src)]
    run = subprocess.run(cmd, capture_output=True, text=True)
    assert run.returncode == 0 and "inline-asm" not in run.stderr, run.stderr
    code = [x.split(";")[0].strip() for x in (tmp_path / "load.s").read_text().splitlines()]
    code = [x for x in code if re.match(r"[sv]_|global_|ds_", x)]
    at = next(i for i, x in enumerate(code) if x.startswith("global_load_lds"))
    pair = re.search(r"s\[(\d+):(\d+)\]", code[at])
    regs = {f"s{r}" for r in range(int(pair.group(1)), int(pair.group(2)) + 1)}
    by_vector = [i for i, x in enumerate(code[:at]) if x.startswith("v_readfirstlane") and x.split()[1].rstrip(",") in regs]
    by_scalar = [i for i, x in enumerate(code[:at]) if re.match(r"s_mov_b64 s\[%s:%s\]," % pair.groups(), x)]
    if max(by_vector, default=-1) > max(by_scalar, default=-1):
        states = sum(int(x.split()[1]) + 1 if x.startswith("s_nop") else 1 for x in code[max(by_vector) + 1:at])
        assert states >= 5, code[max(by_vector):at + 1]
    # m0: the compiler's own doing, so that it knows what is in it; one wait state to the load
    m0 = [i for i, x in enumerate(code) if re.match(r"s_\w+ m0,", x)]
    assert len(m0) == 1 and m0[0] < at - 1, code[:at + 1]
