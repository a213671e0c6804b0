// What the host keeps of an iterative solve on the device (internal header).
#pragma once

namespace etpic {

// Pinned memory the solve's kernels write.  word: (k + 1) << 1 | done of the
// last product launch that ran, or of the whole solve where it is one launch;
// r2, b2 are read once the stream has drained.  gave_up: a block of a
// one-launch solve left a wait that ran out.
struct SolveWatch {
    unsigned long long word;
    double r2, b2;
    unsigned long long gave_up;
};

// Whether a one-launch solve whose stream has drained left its result.  Block
// 0's report alone does not say so: another block may have left the last
// exchange without its rows.
inline bool one_launch_took(const SolveWatch &w) {
    return __atomic_load_n(&w.word, __ATOMIC_RELAXED) != 0 && __atomic_load_n(&w.gave_up, __ATOMIC_RELAXED) == 0;
}

}   // namespace etpic
