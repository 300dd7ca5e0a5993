"""The limit of a wait inside the resident kernels (WaitClock in mdot_internal.h), on the CPU: a program
built from the header runs it over sequences of looks. Four seconds of looks a millisecond apart run out;
a queue that is preempted for any time between two looks is not taken to have waited."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "mdot_internal.h"
#include <cstdio>
using namespace mdot;
// looks until the wait runs out (at most 100000), `gap` ticks apart, the first at `start`; every
// `each`-th gap is `stall` ticks instead
static int looks(uint64_t start, uint64_t gap, int each, uint64_t stall)
{
    WaitClock c;
    uint64_t t = start;
    for (int k = 1; k <= 100000; ++k) {
        if (c.ran_out((uint32_t)t)) return k;
        t += each && k % each == 0 ? stall : gap;
    }
    return -1;
}
int main()
{
    const uint64_t ms = 100000, s = 1000 * ms;
    std::printf("%d\n", looks(12345, ms, 0, 0));               // a look per ms
    std::printf("%d\n", looks((1ull << 32) - 2 * s, ms, 0, 0)); // across the wrap of the low word
    std::printf("%d\n", looks(7, ms, 10, 60 * s));             // preempted for a minute every 10 looks
    std::printf("%d\n", looks(7, 3600 * s, 0, 0));             // an hour between any two looks
    WaitClock c;
    bool out = false;                                          // ten stalls of ten seconds in all
    for (int k = 0; k < 10; ++k) out |= c.ran_out((uint32_t)((k + 1) * 10 * s));
    std::printf("%d\n", (int)out);
}
"""


def test_waits_run_out_by_looks_and_not_by_stalls(tmp_path):
    src, exe = tmp_path / "wait.cpp", tmp_path / "wait"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2307_08507_amd", "csrc"),
                           "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)])
    steady, wrapped, stalled, slow, few = map(int, subprocess.check_output([str(exe)], text=True).split())
    assert 3990 <= steady <= 4010 and 3990 <= wrapped <= 4010
    # 9 looks of 1 ms and a stall of at most 10 ms each time: 19 ms of waiting, not a minute
    assert 2080 <= stalled <= 2130
    assert 400 <= slow <= 402
    assert few == 0
