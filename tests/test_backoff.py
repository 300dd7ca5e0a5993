"""When resident kernels are attempted on a shared GPU (Backoff in mdot_internal.h), on the CPU: a program
built from the header plays chunks whose attempts succeed or fail."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "mdot_internal.h"
#include <cstdio>
using namespace mdot;
int main()
{
    Backoff b;
    int tries = 0;
    for (int k = 0; k < 1000; ++k) {  // alone: every chunk is resident
        tries += b.resident();
        b.met();
    }
    std::printf("%d\n", tries);
    tries = 0;
    int last = 0, gap = 0;
    for (int k = 0; k < 10000; ++k)  // a GPU that stays busy: fewer and fewer attempts, never none
        if (b.resident()) {
            gap = k - last;
            last = k;
            ++tries;
            b.missed();
        }
    std::printf("%d %d\n", tries, gap);
    int after = 0;
    while (!b.resident()) ++after;  // and free again: at most kMost chunks later
    b.met();
    std::printf("%d\n", after);
    tries = 0;
    for (int k = 0; k < 100; ++k) {
        tries += b.resident();
        b.met();
    }
    b.missed();  // one failure: two chunks
    int skipped = 0;
    while (!b.resident()) ++skipped;
    std::printf("%d %d\n", tries, skipped);
}
"""


def test_attempts_are_seldom_made_where_they_fail(tmp_path):
    src, exe = tmp_path / "b.cpp", tmp_path / "b"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2307_08507_amd", "csrc"),
                           "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)])
    out = [tuple(map(int, x.split())) for x in subprocess.check_output([str(exe)], text=True).splitlines()]
    assert out[0] == (1000,)
    tries, gap = out[1]
    assert 10000 // 17 <= tries <= 10000 // 17 + 8 and gap == 17
    assert out[2][0] <= 16
    assert out[3] == (100, 2)


def test_a_resident_launch_ends_within_milliseconds():
    src = open(os.path.join(ROOT, "paper_2307_08507_amd", "csrc", "mdot_api.cpp")).read()
    steps = int(re.search(r"kResidentMax = (\d+);", src).group(1))
    assert steps * 33e-6 < 10e-3  # at the slowest step, n = 4096 in FP64
