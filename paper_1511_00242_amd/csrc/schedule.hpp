// schedule.hpp -- how a call of n steps is cut into launches (host code without HIP).
#pragma once
#include <cstdint>

namespace lbfv {

// The n steps left of a call in launches of at most `per`.  exact: an even or odd number of launches
// as n is, so that the state ends in the buffer that n one-step launches would leave it in; the
// launches then have the same steps to within one, and are no more than need be.  Otherwise as many
// steps as a launch takes, and the rest in the last one.
// no_twos (exact): three steps and one instead of two and two, for meshes on which one step is
// marched and a launch of two gains nothing on two marches.
class Cut {
public:
    Cut(int n, int per, bool exact, bool no_twos = false)
        : left_(n), per_(per), exact_(exact), no_twos_(exact && no_twos && per >= 3), launches_((n + per - 1) / per) {
        if (exact_) launches_ += (launches_ ^ n) & 1;
    }
    // steps of the next launch, 0 after the last
    int next() {
        if (launches_ <= 0) return 0;
        int k = exact_ ? (left_ + launches_ - 1) / launches_ : (left_ < per_ ? left_ : per_);
        --launches_;
        if (no_twos_ && k == 2 && left_ >= 4) {
            k = 3;
            const int least = (left_ - k + per_ - 1) / per_;
            launches_ = least + ((least ^ launches_) & 1);
        }
        left_ -= k;
        return k;
    }

private:
    int left_, per_;
    bool exact_, no_twos_;
    int launches_;
};

// Steps of an autotuner's trial of launches of `per` steps that end where one-step launches do:
// whole launches, an even number of them (they have then all `per` steps), at least as many steps
// as asked for.  20 steps would run as 4 launches of 5 for every `per` from 5 to 8, and the widest
// would never be timed at the length that it is made for.
inline int trial_length(int per, int trial_steps) {
    const int64_t pair = 2 * (int64_t)per, n = (trial_steps + pair - 1) / pair * pair;
    return n <= INT32_MAX ? (int)n : trial_steps;
}

}  // namespace lbfv
