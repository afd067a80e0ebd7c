"""The inline assembly of adjoint_linear.hip's pull-back, compiled for gfx950 with
equal operands: no accumulator shares a register with an input that a later
instruction of the block still reads."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2603_20525_amd import build

PROBE = '''
#include "adjoint_linear.hip"
namespace plan {
__global__ void probe(const float *p, const Column *c, float *o) {
    const float v = p[threadIdx.x];
    o[threadIdx.x] = pull_back(v, v, c[threadIdx.x].q2.z, c[threadIdx.x]);
}
}
'''


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="no hipcc")
def test_accumulators_share_no_register_with_inputs(tmp_path):
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(PROBE)
    flags = [f for f in build.HIPCC_FLAGS if f != "-fPIC"]
    subprocess.run(["hipcc", *flags, "-I", build.CSRC, "--offload-device-only", "-S", "-o",
                    str(out), str(src)], check=True, capture_output=True)
    body = re.search(r"^_Z\w*probe\w*:(.*?)s_endpgm", out.read_text(), re.S | re.M).group(1)
    lines = re.findall(r"v_(?:mul|fmac)_f32_dpp (v\d+), (v\d+), (v\d+) row_newbcast", body)
    assert len(lines) == 13
    written = {d for d, _, _ in lines}
    read = {r for _, a, b in lines for r in (a, b)}
    assert len(written) == 3 and not written & read
