"""Which launches add up their own partial results: the rule, compiled from its header and run on the CPU.  Workgroups that wait hold
their places, so those of all launches that can be under way must leave a compute unit of every XCD to the others."""
import ctypes
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2102_08124_amd", "csrc")
QUEUES, UNITS_OF_XCD = 4, 32         # hardware queues that HIP makes for a process; compute units of an XCD

SOURCE = """
#include "tmask_sum_choice.hpp"
using namespace tmask;
extern "C" int itself(const uint32_t *workgroups, const int *wanted, int n, uint32_t threads, int score)
{
    LaunchSums sums;
    for (int k = 0; k < n; k++)
        sums.add(workgroups[k], wanted[k] != 0);
    return adds_up_itself(sums, threads, score != 0);
}
"""


@pytest.fixture(scope="module")
def itself(tmp_path_factory):
    """(workgroups of each matrix, whether its sum is asked for, threads, score) -> the launch adds up its own partial results"""
    folder = tmp_path_factory.mktemp("sums")
    src, lib = folder / "sums.cpp", folder / "sums.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(lib), str(src)], check=True)
    dll = ctypes.CDLL(str(lib))

    def ask(workgroups, wanted=None, threads=256, score=False):
        n = len(workgroups)
        wanted = [1] * n if wanted is None else wanted
        return bool(dll.itself((ctypes.c_uint32 * n)(*workgroups), (ctypes.c_int * n)(*wanted), n, threads, int(score)))
    return ask


@pytest.mark.parametrize("threads,score", [(256, False), (64, False), (256, True), (64, True)])
def test_waiting_workgroups_leave_a_compute_unit_of_every_xcd(itself, threads, score):
    """Each queue has one launch of which workgroups have yet to start; its waiting workgroups may all be on one XCD, which is so
    where every matrix has a multiple of eight workgroups."""
    rng = random.Random(5)
    seen = set()
    for n in [1, 2, 3, 4, 5, 6, 7, 8, 9, 16, 31, 32, 33, 52, 64, 96, 128, 224, 256]:
        for _ in range(50):
            workgroups = [rng.choice([1, 2, 8, 16, 24, 64, 256]) for _ in range(n)]
            wanted = [rng.choice([0, 1, 1, 1]) for _ in range(n)]
            waiting = sum(w > 1 and asked for w, asked in zip(workgroups, wanted))
            took = itself(workgroups, wanted, threads, score)
            if took:
                assert waiting * QUEUES < UNITS_OF_XCD, (workgroups, wanted)
            seen.add((took, waiting * QUEUES < UNITS_OF_XCD))
    assert (True, True) in seen and (False, False) in seen


def test_the_limits(itself):
    assert itself([256] * 7) and not itself([256] * 8)
    assert itself([1] * 200) and itself([1] * 200 + [256] * 7) and not itself([1] * 200 + [256] * 8)
    assert itself([256] * 8, [1] * 7 + [0])                                    # nobody asked for the eighth
    assert itself([2048]) and not itself([2049]) and itself([512], threads=64) and not itself([513], threads=64)
    assert itself([2048] * 7) and itself([2048] * 7 + [1] * 200)               # whatever they have in all
    assert itself([256], score=True) and not itself([257], score=True) and not itself([128, 129], score=True)
