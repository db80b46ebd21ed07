// The layout tuner's result, shared by the clones of a deferred handle: one of them times the
// layouts, whichever is set up first, and all take its choice and report its times. Set-ups of
// one LP may run on several threads at once: a second one waits for the trial instead of
// disturbing it with one of its own. Host code without HIP types.
#pragma once

#include <mutex>

namespace lpgpu {

struct LayoutTrial {
    int layout = -1;              // the faster layout (0 panels, 1 row tiles; -1 before the trial)
    double us[2] = {0.0, 0.0};    // mean time of one A x + A^T y pair in each
};

class SharedLayoutTrial {
public:
    // *out: the result of the trial, made by run(LayoutTrial*) (0 on success) unless there is one.
    // A trial that failed leaves none, and its code is returned.
    template <class Run>
    int get(LayoutTrial* out, Run&& run) {
        std::lock_guard<std::mutex> lk(mu_);
        if (trial_.layout < 0) {
            LayoutTrial t;
            if (int rc = run(&t)) return rc;
            trial_ = t;
        }
        *out = trial_;
        return 0;
    }

private:
    std::mutex mu_;
    LayoutTrial trial_;
};

}  // namespace lpgpu
