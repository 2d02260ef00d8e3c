// schedule.hpp -- how a call of n steps is cut into launches (host code without HIP).
#pragma once
#include <cstdint>

namespace lbfv {

// Launches of at most `per` steps for the n steps left of a call.  exact: an even or odd number of
// them as n is, so that the state ends in the buffer that n one-step launches would leave it in.
inline int tail_launches(int n, int per, bool exact) {
    int launches = (n + per - 1) / per;
    if (exact) launches += (launches ^ n) & 1;
    return launches;
}
// Steps of the next of those launches: the same for all to within one step, none shorter than need
// be; or as many as a launch takes, and the rest in the last one.
inline int launch_steps(int left, int launches, int per, bool exact) {
    return exact ? (left + launches - 1) / launches : (left < per ? left : per);
}

// Steps of an autotuner's trial of launches of `per` steps that end where one-step launches do:
// whole launches, an even number of them (they have then all `per` steps), at least as many steps
// as asked for.  20 steps would run as 4 launches of 5 for every `per` from 5 to 8, and the widest
// would never be timed at the length that it is made for.
inline int trial_length(int per, int trial_steps) {
    const int64_t pair = 2 * (int64_t)per, n = (trial_steps + pair - 1) / pair * pair;
    return n <= INT32_MAX ? (int)n : trial_steps;
}

}  // namespace lbfv
