"""The split of the tiles into groups, compiled for the host and walked over sizes and devices of every kind: no group is
empty or holds more tiles than a block has counters for, the groups fit their table, and both directions of the rule agree.
Nothing the interface serves (2^31 parameters, 65,536 segments) is out of reach on a device with few compute units."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = r"""
#include <cstdio>
#include "slimdp_split.h"
using namespace slimdp;
int main()
{
    const uint32_t most = (1u << 31) / 4096u + 65536u, cus[] = {1, 4, 32, 38, 64, 128, 255, 256, 304};
    unsigned long long seen = 0;
    for (uint32_t c : cus)
        for (uint64_t T = 1; T <= most; T = T < 5000 ? T + 1 : (T < most ? (T * 9 / 8 < most ? T * 9 / 8 : most) : most + 1ull)) {
            const uint32_t t = (uint32_t)T, groups = core_groups(t, c);
            if (groups == 0 || groups > CORE_GROUPS || groups > t) { std::printf("T=%u cus=%u: %u groups\n", t, c, groups); return 1; }
            for (uint32_t g = 0; g < groups; ++g) {
                const uint32_t a = group_first(g, t, groups), b = group_first(g + 1, t, groups);
                if (b <= a || b - a > GROUP_MAX || group_of(a, t, groups) != g || group_of(b - 1, t, groups) != g) {
                    std::printf("T=%u cus=%u group %u of %u: tiles %u..%u\n", t, c, g, groups, a, b);
                    return 1;
                }
            }
            if (group_first(0, t, groups) != 0 || group_first(groups, t, groups) != t) { std::printf("T=%u: ends\n", t); return 1; }
            ++seen;
        }
    std::printf("ok %llu\n", seen);
    return 0;
}
"""


def test_every_number_of_tiles_splits_into_groups_that_a_block_can_count(tmp_path):
    src, exe = tmp_path / "split.cpp", tmp_path / "split"
    src.write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_1709_09393_amd", "csrc"),
                    "-o", str(exe), str(src)], check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0 and run.stdout.startswith("ok"), run.stdout
