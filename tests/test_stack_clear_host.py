"""Sizes of the joint histograms and the rule that picks who clears them, on
the host: a word count past 32 bits must reach a fill that counts in 64 bits,
and the clearing loop of the stack pass's first kernel, whose index is 32 bits
and moves on by rows * 1,024, must stay below 2^32."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r'''
#include <cstdio>
#include <cstdlib>
#include "kv_internal.h"
int main(int argc, char** argv) {
  for (int i = 1; i + 1 < argc; i += 2) {
    const uint64_t words = kv::joint_words(strtoull(argv[i], 0, 10), 16 * 1023, 16);
    std::printf("%llu %d\n", (unsigned long long)words,
                (int)kv::rows_clear(words, strtoull(argv[i + 1], 0, 10)));
  }
}
'''


def test_joint_clear_sizes(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
                    os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2603_08739_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    extra = 16 * 1023 + 16
    # a batch accepts up to 2^31 - 1 joint bins; 16 groups of 65,536 x 1,024 bins are 2^30
    cases = [(b, rows) for b in (1, 1000, 1 << 26, (1 << 30) - 4096, (1 << 30) - 4095, 1 << 30, (1 << 31) - 1)
             for rows in (1, 233, 4096, 65_536, 524_288)]
    out = subprocess.run([str(exe)] + [str(x) for c in cases for x in c], capture_output=True, text=True, check=True).stdout
    for (bins, rows), line in zip(cases, out.splitlines()):
        words, by_rows = (int(x) for x in line.split())
        assert words == 4 * bins + extra
        if by_rows:  # the index of the last thread's last step, and one step on
            assert words - 1 + rows * 1024 < 1 << 32
        assert not (by_rows and words > rows * 16_384)
    assert out.splitlines()[1].endswith(" 1")  # 233 rows do clear a small table
