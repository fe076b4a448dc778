"""Wait states that gfx950 leaves to whoever writes the instructions, in the assembly of the counts of positive outputs."""
import os
import re
import subprocess

import pytest

from paper_2301_08527_amd import build

KERNEL = """
#include "rocket_device.hpp"
template <int R>
__device__ void pool(const float *x, float bound, uint32_t *out)
{
    float z[R];
    for (int i = 0; i < R; ++i) z[i] = x[threadIdx.x + 64 * i];
    PoolState st = {-INFINITY, 0.f, 0};
    rk_pool<R>(z, MASK, bound, 0.f, 0.f, st);
    out[threadIdx.x] = static_cast<uint32_t>(st.cnt) + __float_as_uint(st.vmax);
}
__global__ void count(const float *x, float bound, uint32_t *out) { pool<ROWS>(x, bound, out); }
"""
NEEDED = 2       # between a vector instruction that writes a scalar register and a vector instruction that reads it


def scalars(operand):
    """Scalar registers of an operand."""
    found = {"vcc"} if "vcc" in operand else set()
    for first, last in re.findall(r"\bs\[(\d+):(\d+)\]", operand):
        found |= {"s%d" % i for i in range(int(first), int(last) + 1)}
    return found | {"s" + n for n in re.findall(r"\bs(\d+)\b", operand)}


def too_early(asm):
    """Vector instructions of a straight piece of assembly that read a scalar register which one wrote fewer than
    NEEDED wait states before."""
    age, bad = {}, []
    for line in asm.splitlines():
        line = line.split(";")[0].strip()
        if not line or line.startswith(".") or line.endswith(":"):
            continue
        name, _, rest = line.partition(" ")
        operands = [o.strip() for o in rest.split(",")]
        writes = set()
        if name.startswith("v_"):
            carries = "_co_" in name or name.startswith(("v_div_scale", "v_mad_u64", "v_mad_i64"))     # the second operand is written
            reads = set().union(*[scalars(o) for o in operands[2 if carries else 1:]]) if len(operands) > 1 else set()
            bad += [line for r in reads if age.get(r, NEEDED) < NEEDED]
            if carries:
                writes = scalars(operands[1])
            elif name.startswith(("v_cmp", "v_readlane", "v_readfirstlane")):
                writes = scalars(operands[0])
        steps = 1 + int(operands[0]) if name == "s_nop" else 1
        age = {r: a + steps for r, a in age.items()}
        age.update({w: 0 for w in writes})
    return bad


def test_scanner():
    assert too_early("v_cmp_lt_f32 vcc, s4, v1\nv_addc_co_u32 v0, vcc, 0, v0, vcc")
    assert too_early("v_cmp_lt_f32 vcc, s4, v1\ns_nop 0\nv_addc_co_u32 v0, vcc, 0, v0, vcc")
    assert too_early("v_cmp_lt_f32 s[6:7], s4, v1\nv_mov_b32 v2, v3\nv_cndmask_b32 v0, 0, v1, s[6:7]")
    assert not too_early("v_mad_u64_u32 v[0:1], s[6:7], v2, s4, 0\nv_mad_u64_u32 v[0:1], s[6:7], v3, s4, 0")
    assert not too_early("v_cmp_lt_f32 vcc, s4, v1\ns_nop 1\nv_addc_co_u32 v0, vcc, 0, v0, vcc\nv_addc_co_u32 v5, vcc, v1, v2, s[6:7]")


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="hipcc not found")
@pytest.mark.parametrize("mask", [2, 3])
@pytest.mark.parametrize("rows", [1, 2, 3, 8, 16, 32])      # the strips' heights: one, two and no outputs beyond threes
def test_counts_wait_for_their_comparisons(tmp_path, rows, mask):
    source, asm = tmp_path / "count.hip", tmp_path / "count.s"
    source.write_text(KERNEL.replace("ROWS", str(rows)).replace("MASK", str(mask)))
    subprocess.run([build.HIPCC, "-S", "--cuda-device-only"] + build.DEVICE + build.COMMON + [str(source), "-o", str(asm)],
                   check=True, stderr=subprocess.DEVNULL)
    text = asm.read_text()
    assert text.count("v_addc_co_u32") >= rows       # the counts are in it
    assert too_early(text) == []
