// Whether a launch adds up its own partial results.  Host arithmetic in plain C++: the CPU tests compile this header by itself.
#pragma once
#include <cstdint>

namespace tmask {

// What of a launch decides: its workgroups, those of its largest matrix, and how many matrices have one that would wait.
struct LaunchSums {
    uint32_t total = 0, most = 0, waiting = 0;

    void add(uint32_t workgroups, bool wanted)              // a matrix; wanted: its sum is asked for
    {
        total += workgroups;
        most = most > workgroups ? most : workgroups;
        waiting += wanted && workgroups > 1u;
    }
};

// The last workgroup of a matrix waits for the others in its place on a compute unit (hand_over, hand_over_score), and one that it
// waits for may not have started yet.  Were every place of an XCD held by waiting workgroups, a launch on another queue whose next
// workgroup belongs there would stop, and with it what waits for that workgroup elsewhere: two launches could stop each other.  A
// queue starts the workgroups of one launch after the other, and a launch whose workgroups have all started ends by itself, so
// of each queue the waiting workgroups of one launch count.  Seven each on the four queues that HIP makes hold 28 of the
// 32 compute units of an XCD at the worst (all on the same one, each on a compute unit of its own): a unit that none of them holds is
// left, and any workgroup fits there once the others on it are done.  With streams of all three priorities, four queues each, it is 84
// waiting workgroups, of 96 places that an XCD has for the largest of these kernels (three to a compute unit).  A launch alone ends
// on however few compute units: workgroups start in the order of their numbers on each XCD, and only lower ones are waited for.
// Beyond that (streams confined to the same few compute units, queues of many processes) the wait is bounded.  Larger
// batches leave their sums to a second launch, which they hardly notice: 52 matrices of 5724 workgroups 22.8 us in one launch, 23.5
// in two.
constexpr uint32_t kQueues = 4, kUnitsOfXcd = 32;
constexpr uint32_t kMostWaiting = (kUnitsOfXcd - 1) / kQueues;

// Workgroups of `threads`.  Objectives: whatever seven matrices of at most eight results per thread of the adding workgroup have in
// all (up to there the second launch has 256 threads, and the order of additions is the same).  Two launches / one, us, fp32 2:4: one
// matrix of 512 workgroups 4.8 / 4.5, of 2048 11.3 / 10.4, two 17.3 / 16.5, four 30.6 / 29.5, seven (14336) 50.6 / 48.9; bf16 4:8
// 7.7 / 7.5 ... 119.6 / 117.4; optimal 4:8 17.4 / 17.2 ... 226 / 224.  (With many more that wait the readers slow down what they wait
// for: 144 matrices, 36864 workgroups, 147 / 153.)
// Scores: 256 workgroups, whose records are seven words each.  512^2 and 1024^2 mask, compression and score (256 workgroups)
// 17.1 / 16.7, 1024 x 2048 (512) 18.6 / 19.3, six matrices (3072) 60 / 67; the score alone 384 7.6 / 6.6, 512 7.8 / 7.3, 1024 8.6 / 12.1.
inline bool adds_up_itself(const LaunchSums &launch, uint32_t threads, bool score)
{
    if (launch.waiting > kMostWaiting)
        return false;
    return score ? launch.total <= 256u : launch.most <= 8u * threads;
}

}  // namespace tmask
