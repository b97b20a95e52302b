// The rounds of a perturbation phase in one workgroup, its trials decided by
// wave 0.  Plain C++, so that the order of its reads, writes and barriers can be
// run on the host as well.
#pragma once

namespace smx {

// decide() (wave 0 alone) takes every decision it can and returns the trials
// the workgroup has to sum before it can go on, 0 once the phase is over;
// sum(n) (every thread) sums them and records the outcome.  Every wave goes by
// `todo` (a word of LDS), never by the phase's state, which wave 0 may be
// writing while another wave is still at the head of the loop: todo is written
// before one barrier and read between it and the next, so all waves take the
// same rounds, and what they read of the state after the last one is ordered.
// Ends when decide() returns 0.
template <typename Word, typename Decide, typename Sum, typename Barrier>
__device__ inline void phase_rounds(bool wave0, Word &todo, Decide &&decide, Sum &&sum, Barrier &&barrier)
{
    for (;;) {
        if (wave0) todo = decide(); // the same value from every lane
        barrier();
        const int n = todo;
        if (n == 0) return;
        sum(n);
        barrier();
    }
}

} // namespace smx
