"""The rule for how much device memory one wave of exclusive evaluations takes
(host): all of it at once up to 4 GiB, then at most half of what is free, or
what the trace's buffer holds anyway."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r'''
#include <cstdio>
#include <cstdlib>
#include "kv_internal.h"
int main(int argc, char** argv) {
  for (int i = 1; i + 2 < argc; i += 3)
    std::printf("%llu\n", (unsigned long long)kv::excl_budget(strtoull(argv[i], 0, 10), strtoull(argv[i + 1], 0, 10),
                                                              strtoull(argv[i + 2], 0, 10)));
}
'''


def test_budget(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
                    os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2603_08739_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    gib = 1 << 30
    cases = [((1, 0, 0), 1), ((4 * gib, gib, 0), 4 * gib), ((5 * gib, 200 * gib, 0), 5 * gib), ((237 * gib, 280 * gib, 0), 140 * gib),
             ((237 * gib, 2 * gib, 0), gib), ((237 * gib, 2 * gib, 130 * gib), 130 * gib), ((6 * gib, 2 * gib, 130 * gib), 6 * gib)]
    out = subprocess.run([str(exe)] + [str(x) for c, _ in cases for x in c], capture_output=True, text=True, check=True).stdout
    assert [int(x) for x in out.split()] == [want for _, want in cases]
