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
// left, and any workgroup fits there once the others on it are done.  (Queues of other processes come on top; launches would
// have to fill five or more of them, each with seven waiting workgroups on one XCD.)  Larger batches leave their sums to a second
// launch, which they hardly notice: 52 matrices of 5724 workgroups 22.8 us in one launch, 23.5 in two.
constexpr uint32_t kQueues = 4, kUnitsOfXcd = 32;
constexpr uint32_t kMostWaiting = (kUnitsOfXcd - 1) / kQueues;

// Workgroups of `threads`.  Back to back, two launches / one, us: 512^2 .. 1536^2 masks at 2:4 and 4:8 9.3-10.2 / 6.9-7.3, 4096^2
// bf16 14.6 / 13.0, six matrices fp32 2:4 (3072 workgroups) 15.2 / 13.7.  Eight results per thread of the adding workgroup at most:
// up to there the second launch has 256 threads, and the order of additions is the same.  A score's record is seven words:
// 512^2 and 1024^2 mask, compression and score (256 workgroups) 17.1 / 16.7, 1024 x 2048 (512) 18.6 / 19.3, six matrices (3072)
// 60 / 67.
inline bool adds_up_itself(const LaunchSums &launch, uint32_t threads, bool score)
{
    if (launch.waiting > kMostWaiting)
        return false;
    return score ? launch.total <= 256u : launch.total <= 8192u && launch.most <= 8u * threads;
}

}  // namespace tmask
