"""The staged kernels' global->LDS copy takes its LDS base from M0: the
compiler knows that (compiled here for gfx950, nothing is run), so a value it
keeps in M0 across a copy is there again afterwards."""
import os
import re
import subprocess

import pytest

from paper_1202_4748_amd import build

SRC = """
#include <hip/hip_runtime.h>
#include "lbfss_fused.hpp"
using namespace lbfss;
extern "C" __global__ void probe(const float *src, float *out, int v) {
    __shared__ float s[64 * 4];
    int keep;
    asm volatile("s_mov_b32 %%0, %%1 ; set" : "={m0}"(keep) : "s"(v));
    copy_to_lds<%d>(src + 4 * threadIdx.x, (lptr_t)&s[0]);
    asm volatile("; use %%0" ::"{m0}"(keep));
    __builtin_amdgcn_s_waitcnt(vmcnt_wait(0));
    __syncthreads();
    out[threadIdx.x] = s[threadIdx.x];
}
"""


@pytest.mark.parametrize("width", [16, 4])
def test_m0_kept_across_a_copy(tmp_path, width):
    (tmp_path / "p.hip").write_text(SRC % width)
    out = tmp_path / "p.s"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-Wall")]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--cuda-device-only", "-S", "-I",
                    os.path.join(build.HERE, "csrc"), "-o", str(out), str(tmp_path / "p.hip")], check=True,
                   capture_output=True)
    lines = build.asm_functions(out.read_text())["probe"]
    i = next(k for k, t in enumerate(lines) if "; set" in t)
    copy = next(k for k, t in enumerate(lines) if "global_load_lds" in t)
    j = next(k for k, t in enumerate(lines) if "; use" in t)
    assert i < copy < j
    saved = [m.group(1) for t in lines[i:copy] if (m := re.match(r"\s*s_mov_b32 (s\d+), m0", t))]
    restored = [m.group(1) for t in lines[copy:j] if (m := re.match(r"\s*s_mov_b32 m0, (s\d+)", t))]
    assert restored and restored[-1] in saved
