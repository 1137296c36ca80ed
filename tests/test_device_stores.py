"""Stores written in inline assembly (csrc/device_util.h): the wait states behind them, seen in the assembly that hipcc writes."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_05699_amd import build as build_module

# The data of a store of more than 8 bytes must not be overwritten by a vector instruction within two wait states (gfx940 and
# later).  The compiler sees to that behind stores that it knows; here the first register of the data is overwritten at once.
KERNEL = """
#include "device_util.h"
__global__ void overwritten_at_once(float* p, floatx4 v) {
    v[0] += threadIdx.x, v[1] += threadIdx.x, v[2] += threadIdx.x, v[3] += threadIdx.x;
    float* at = p + 7 * threadIdx.x;
    for (int i = 0; i < 3; ++i) {
        stream_store_at(at, v);
        asm volatile("v_add_f32 %0, 1.0, %0" : "+v"(v[0]));
        at += 4096;
    }
}
"""


def test_the_data_of_an_assembly_store_stays_for_two_wait_states(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    (tmp_path / "k.hip").write_text(KERNEL)
    subprocess.run([hipcc, *build_module.FLAGS, "-I", build_module.CSRC, "--cuda-device-only", "-S", str(tmp_path / "k.hip"), "-o", str(tmp_path / "k.s")],
                   check=True, capture_output=True)
    lines = [s for s in (re.sub(r";.*", "", x).strip() for x in (tmp_path / "k.s").read_text().splitlines()) if s and not s.startswith((".", "#"))]
    stores = [i for i, s in enumerate(lines) if s.startswith("global_store_dwordx4")]
    assert len(stores) == 3
    for i in stores:
        first, last = map(int, re.search(r"v\[\d+:\d+\], v\[(\d+):(\d+)\], off", lines[i]).groups())
        waited = 0
        for s in lines[i + 1:]:
            nop = re.match(r"s_nop (\d+)", s)
            written = re.match(r"v_\w+ v\[?(\d+)(?::(\d+))?", s)
            if written and int(written[1]) <= last and int(written[2] or written[1]) >= first:
                assert waited >= 2, lines[i:i + 4]
                break
            waited += int(nop[1]) + 1 if nop else 1
