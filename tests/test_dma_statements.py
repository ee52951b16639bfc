"""The direct-to-LDS load statements of a2sf_dev.h on the CPU: compiled with a base address that a
vector instruction forms right before them, the distances that gfx950 does not interlock are kept --
five states between that instruction and a load that reads its scalar result, one between the M0 write
and the load."""
import os
import re
import subprocess

import pytest

from paper_2407_20485_amd import build

KERNEL = """
#include "a2sf_dev.h"
using namespace a2sf;
extern "C" __global__ void probe(const unsigned long long* table, float* out, int n) {
  __shared__ __attribute__((aligned(1024))) char smem[8192];
  const int lane = threadIdx.x & 63;
  float x = out[lane];
  for (int i = 0; i < n; ++i) {
    const unsigned long long a = table[64 * i + lane];
    const char* base = (const char*)((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(a >> 32)) << 32 |
                                     (uint32_t)__builtin_amdgcn_readfirstlane((int)a));
    STATEMENT
    wait_vm<0>();
    x += ((volatile float*)smem)[lane];
  }
  out[lane] = x;
}
"""


def scalar_registers(text):
    out = set()
    for lo, hi, one in re.findall(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b", text):
        out.update(range(int(lo), int(hi) + 1) if lo else [int(one)])
    return out


def too_close(lines):
    """(instruction, states since the write) of every load that follows a write too soon, and the number
    of loads seen."""
    clock, vector_wrote, m0, found, loads = 0, {}, -10, [], 0
    for ln in lines:
        op, _, rest = ln.partition(" ")
        if op.startswith("global_load_lds"):
            loads += 1
            found += [(ln, clock - vector_wrote[r]) for r in scalar_registers(rest) if clock - vector_wrote.get(r, -10) < 6]
            if clock - m0 < 2:
                found.append((ln, "m0"))
        dst = rest.split(",")[0]
        if op.startswith("v_") and (op.startswith("v_read") or op.startswith("v_cmp") or "s[" in dst):
            vector_wrote.update((r, clock) for r in scalar_registers(dst))
        elif op.startswith("s_"):
            for r in scalar_registers(dst):
                vector_wrote.pop(r, None)
            if dst.strip() == "m0":
                m0 = clock
        clock += int(rest) + 1 if op == "s_nop" else 1
    return found, loads


@pytest.mark.parametrize("statement", ["dma16(base, lane * 16, (uint32_t)(size_t)smem);", "dma4(base, lane * 4, (uint32_t)(size_t)smem);",
                                       "dma16_at(base + lane * 16, (uint32_t)(size_t)smem);"])
def test_distances(tmp_path, statement):
    src, asm = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(KERNEL.replace("STATEMENT", statement))
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *build.COMMON, "-I", build.CSRC, "--cuda-device-only", "-S",
                    str(src), "-o", str(asm)], check=True, capture_output=True)
    text = asm.read_text()
    body = text[text.index("probe:"):text.index("s_endpgm")]
    lines = [ln.split(";")[0].strip() for ln in body.splitlines()[1:]]
    found, loads = too_close([ln.replace("\t", " ") for ln in lines if ln and not ln.startswith(".") and not ln.endswith(":")])
    assert loads >= 1 and not found


def test_catches_a_base_read_too_soon():
    """Planted mistake: the load reads the vector instruction's result itself."""
    lines = ["v_readfirstlane_b32 s4, v1", "s_mov_b32 m0, s6", "s_nop 0", "global_load_lds_dwordx4 v2, s[4:5]"]
    assert too_close(lines)[0] and not too_close(lines[:1] + ["s_nop 3"] + lines[1:])[0]
