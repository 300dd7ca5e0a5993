"""The limit of a wait inside the resident kernels, on the CPU: a count of looks, which a preempted queue
does not advance. From the header: whole numbers of flag reads, seconds at the time a look takes, and far
from wrapping."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_waits_are_limited_by_looks():
    src = open(os.path.join(ROOT, "paper_2307_08507_amd", "csrc", "mdot_internal.h")).read()
    flag = int(re.search(r"kWaitFlag = (\d+);", src).group(1))
    looks = 1 << int(re.search(r"kWaitLooks = 1u << (\d+);", src).group(1))
    assert looks % flag == 0 and looks < 1 << 31
    # a look is a load from memory: 0.1 us at the least, about 1 us with the other workgroups polling
    assert 0.5 < looks * 0.1e-6 and looks * 1e-6 < 20
    assert flag * 1e-6 < 0.01  # and the others' giving up is seen within some milliseconds
    kern = open(os.path.join(ROOT, "paper_2307_08507_amd", "csrc", "mdot_kernels.hip")).read()
    wait = kern[kern.index("struct Wait {"):]
    assert "wall_clock64" not in wait[:wait.index("\n};")]
