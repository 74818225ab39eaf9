"""The marching kernels read each direction with a scalar plane offset.

The planes of a march are the same in every lane, but a buffer load takes that
part of its address from a scalar register: where the compiler holds it in a
vector register instead, it wraps the load into a loop over the lanes' values
with a wait of its own, and 48 such loops cost the two-node march half its time
again.  Compiles the periodic kernels for gfx950 and looks for such loops.
"""
import os
import re
import subprocess

import pytest

from paper_1805_08643_amd import build

KERNELS = """
#include <hip/hip_runtime.h>
#include "%s"
using namespace lbm;
#define STEP(s) template __global__ void lbm::k_step<s, OP_NONORTH, false>( \\
    const Storage<s>::T *, Storage<s>::T *, const Storage<s>::R *, GridDesc, PhysD);
#define STEP2(s) template __global__ void lbm::k_step2<s, OP_NONORTH, false>( \\
    const Storage<s>::T *, Storage<s>::T *, const Storage<s>::R *, GridDesc, PhysD); \\
    template __global__ void lbm::k_batch_step<s, OP_NONORTH, true>(unsigned char *, const RunDesc *, int, int, int);
#define SPLIT(s) template __global__ void lbm::k_step_split<s, OP_NONORTH, false, false, false>( \\
    const Storage<s>::T *, Storage<s>::T *, const float *, GridDesc, PhysD);
STEP(ST_F64) STEP(ST_F32) STEP(ST_F16S) STEP2(ST_F32) STEP2(ST_F16S) SPLIT(ST_F32) SPLIT(ST_F16S) SPLIT(ST_F16N)
template __global__ void lbm::k_step4<OP_NONORTH, false>(const uint16_t *, uint16_t *, const float *, GridDesc, PhysD);
"""
LANE_LOOP = re.compile(r"\n\s+buffer_load[^\n]*\n(?:\s+(?:s_nop|;)[^\n]*\n)*\s+s_xor_b64 exec, exec, \S+\n\s+s_cbranch_execnz")


def test_no_loops_over_lanes(tmp_path):
    try:
        compiler = build.hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    src, asm = tmp_path / "march.hip", tmp_path / "march.s"
    src.write_text(KERNELS % os.path.join(build.HERE, "csrc", "lbm_kernels.hpp"))
    flags = [f for f in build.flags() if f not in ("-fPIC", "-shared")]
    subprocess.run([compiler, *flags, "--offload-device-only", "-S", str(src), "-o", str(asm)], check=True,
                   capture_output=True)
    text = asm.read_text()
    loops, seen = {}, 0
    for m in re.finditer(r"\n(_ZN3lbm\w*(?:k_step|k_batch_step)\w*):", text):
        body = text[m.end():text.index(".Lfunc_end", m.end())]
        assert "buffer_load" in body
        seen += 1
        loops[m.group(1)] = len(LANE_LOOP.findall(body))
    assert seen == 11
    assert not any(loops.values()), loops
