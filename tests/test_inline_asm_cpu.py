"""Inline assembly keeps the distance that the hardware asks for between a scalar register's write by a vector instruction and
its next read by one: two instructions.  The compiler keeps it between its own instructions and does not look into an inline
block, so the blocks are compiled here with operands that a vector instruction has just written (a lane read, a comparison),
as a spilled register would be, and the distances are counted in the assembly."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "slimdp_device.h"
using namespace slimdp;
extern "C" __global__ void borrow(const uint32_t* in, uint32_t* out)
{
    const uint32_t i = threadIdx.x;
    const uint32_t r[4] = {in[i], in[i + 64], in[i + 128], in[i + 192]};
    uint32_t d[4], acc = in[i + 256];
    sub4_borrow(r, (uint32_t)__builtin_amdgcn_readlane((int)acc, 7), d, acc);
    out[i] = acc ^ d[0] ^ d[1] ^ d[2] ^ d[3];
}
extern "C" __global__ void masked(const float4* in, const uint32_t* bits, float* out)
{
    const float4 x = in[threadIdx.x];
    const uint32_t b = bits[threadIdx.x];
    out[threadIdx.x] = first_masked(x, Masks4{__ballot(b & 1u), __ballot(b & 2u), __ballot(b & 4u), 0ull});
}
"""
SCALARS = re.compile(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b")


def scalars(text):
    out = set()
    for m in SCALARS.finditer(text):
        out |= {int(m.group(3))} if m.group(3) else set(range(int(m.group(1)), int(m.group(2)) + 1))
    return out


def shortest_distances(assembly):
    """Per kernel: the fewest instructions between a vector instruction's write of a scalar register and a vector read of it."""
    found, kernel, written, at = {}, None, {}, 0
    for line in assembly.splitlines():
        label = re.match(r"^(\w+):", line)
        if label and not label.group(1).startswith("L"):
            kernel, written, at = label.group(1), {}, 0
        text = line.split(";")[0].strip()
        if not re.match(r"^[sv]_|^(global|buffer|ds|flat)_", text):
            continue
        op, _, operands = text.partition(" ")
        if op == "s_nop":
            at += int(operands, 0) + 1
            continue
        at += 1
        if op.startswith("v_"):
            parts = [p.strip() for p in operands.split(",")]
            results = 2 if "_co_" in op or "mad_u64" in op else 1
            for reg in scalars(",".join(parts[results:])):
                if reg in written:
                    found[kernel] = min(found.get(kernel, 1 << 30), at - written[reg] - 1)
            for reg in scalars(",".join(parts[:results])):
                written[reg] = at
        elif op.startswith("s_"):
            for reg in scalars(operands.split(",")[0]):
                written.pop(reg, None)
    return found


def test_vector_reads_of_scalars_keep_their_distance(tmp_path):
    src, out = tmp_path / "blocks.hip", tmp_path / "blocks.s"
    src.write_text(SOURCE)
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "-O3", "-std=c++17", "-ffp-contract=off",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1709_09393_amd", "csrc"), "--cuda-device-only", "-S", "-o", str(out), str(src)],
                   check=True, capture_output=True)
    found = shortest_distances(out.read_text())
    assert set(found) == {"borrow", "masked"}, found           # both read scalars that a vector instruction wrote
    assert min(found.values()) >= 2, found
