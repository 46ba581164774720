"""How the last workgroup of a matrix takes the records of the others (take_words): the function, read from the header and run on the
CPU with a thread for each lane of a small wavefront.  Nothing that comes or stays away keeps a wavefront longer than its reads."""
import os
import re
import subprocess

import pytest

HEADER = os.path.join(os.path.dirname(__file__), "..", "paper_2102_08124_amd", "csrc", "tmask_device.hpp")
MOST = 1000                                # reads in vain that a wavefront has here

PROGRAM = r"""
#include <atomic>
#include <cstdint>
#include <cstdio>
#include <pthread.h>
#include <thread>
#include <vector>
#define __device__
#define __forceinline__ inline
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __builtin_amdgcn_s_sleep(n) ((void)0)
struct Tags { uint32_t a, b; };
constexpr int LANES = 4, RECORDS = 8, W = 2;
static unsigned long long memory[LANES * RECORDS * W];
static long comes[LANES * RECORDS];        // after how many reads of the wavefront a record is there (-1: never)
static long rounds = 0;                    // reads of the wavefront
static pthread_barrier_t barrier;
static std::atomic<int> missing{0};
static unsigned long long sim_load(const unsigned long long *at)
{
    const long record = (at - memory) / W, k = (at - memory) % W;
    if (comes[record] >= 0 && rounds >= comes[record])
        return ((unsigned long long)(k ? 22 : 11) << 32) | (unsigned long long)(100 * record + k);
    return *at;
}
static void sim_store(unsigned long long *at, unsigned long long v) { *at = v; comes[(at - memory) / W] = -2; }
static bool any_lane(bool x)
{
    if (x)
        missing++;
    pthread_barrier_wait(&barrier);
    const bool any = missing.load() != 0;
    if (pthread_barrier_wait(&barrier) == PTHREAD_BARRIER_SERIAL_THREAD) {
        missing = 0;
        rounds++;
    }
    pthread_barrier_wait(&barrier);
    return any;
}
#define __any(x) any_lane(x)
#define __hip_atomic_load(at, order, scope) sim_load(at)
#define __hip_atomic_store(at, v, order, scope) sim_store(at, v)
@TEXT@
int main(int argc, char **argv)
{
    for (int r = 0; r < LANES * RECORDS; r++) {
        if (scanf("%ld", &comes[r]) != 1)
            return 1;
        memory[W * r] = 11ull << 32;       // the first word of another call's record with this call's tag, the second one stale
        memory[W * r + 1] = (33ull << 32) | 5;
    }
    pthread_barrier_init(&barrier, nullptr, LANES);
    std::vector<std::thread> lanes;
    static int came[LANES * RECORDS];
    static uint32_t got[LANES * RECORDS][W], rest[LANES];
    for (int l = 0; l < LANES; l++)
        lanes.emplace_back([l] {
            uint32_t left = kMostReads;
            for (int r = 0; r < RECORDS; r++) {
                const int record = r * LANES + l;
                uint32_t v[W];
                came[record] = take_words<W>(memory + W * record, Tags{11, 22}, v, left);
                got[record][0] = v[0]; got[record][1] = v[1];
            }
            rest[l] = left;
        });
    for (auto &t : lanes)
        t.join();
    printf("%ld", rounds);
    for (int l = 0; l < LANES; l++)
        printf(" %u", rest[l]);
    printf("\n");
    for (int r = 0; r < LANES * RECORDS; r++)
        printf("%d %u %u %llu %llu\n", came[r], got[r][0], got[r][1], memory[W * r], memory[W * r + 1]);
}
"""


@pytest.fixture(scope="module")
def take(tmp_path_factory):
    text = open(HEADER).read()
    m = re.search(r"constexpr uint32_t kMostReads = [^;]+;.*?(?=__device__ __forceinline__ double words_as_double)", text, re.S)
    assert m and "take_words" in m.group(0)
    code = re.sub(r"(kMostReads = )[^;]+;", r"\g<1>%d;" % MOST, m.group(0), count=1)
    folder = tmp_path_factory.mktemp("take")
    src, exe = folder / "take.cpp", folder / "take"
    src.write_text(PROGRAM.replace("@TEXT@", code))
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread", "-o", str(exe), str(src)], check=True)

    def run(comes):
        out = subprocess.run([str(exe)], input=" ".join(map(str, comes)), capture_output=True, text=True, check=True, timeout=60).stdout.split("\n")
        head = list(map(int, out[0].split()))
        return head[0], head[1:], [list(map(int, line.split())) for line in out[1:] if line]
    return run


LANES, RECORDS = 4, 8
STALE = [11 << 32, (33 << 32) | 5]


def test_records_that_come_are_taken_and_cleared(take):
    rounds, rest, records = take([(7 * r) % 40 for r in range(LANES * RECORDS)])
    assert rounds <= 40 + RECORDS + 1 and len(set(rest)) == 1
    for r, (came, v0, v1, w0, w1) in enumerate(records):
        assert (came, v0, v1) == (1, 100 * r, 100 * r + 1) and (w0, w1) == (0, 0)


@pytest.mark.parametrize("never", [[0], [31], [0, 5, 10, 15], [0, 4, 8, 12, 16, 20, 24, 28], list(range(32))])
def test_a_wavefront_has_one_number_of_reads_for_all_records(take, never):
    """Each lane's, and each record's, own number would add up: four missing records in four lanes, eight in one."""
    rounds, rest, records = take([-1 if r in never else 0 for r in range(LANES * RECORDS)])
    assert rounds == MOST + RECORDS and rest == [0] * LANES
    for r, (came, v0, v1, w0, w1) in enumerate(records):
        assert came == (r not in never)
        assert [w0, w1] == (STALE if r in never else [0, 0])           # another call's record stays what it is


def test_late_records_use_up_the_same_reads(take):
    rounds, rest, records = take([300 * (r // LANES) if r % LANES == r // LANES % LANES else 0 for r in range(LANES * RECORDS)])
    assert rounds <= MOST + RECORDS and rest == [0] * LANES
    assert [rec[0] for rec in records[:LANES * 4]] == [1] * LANES * 4 and 0 in [rec[0] for rec in records]
