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

// Whether a solver's next solve tries one launch.  One that fails costs the
// wait for its blocks (0.5 ms) before the same iterations go by launches; while
// other work holds the compute units they would need, that is every solve.  So
// after a failure the next solves go by launches at once: 4, then twice as many
// after each further one up to 64; a success forgets it.  59,900 edges beside a
// kernel that holds 128 of 256 compute units: 1753 us a solve when each tried,
// 1292 now, 1402 by the launches of before; two contexts solving at once meet
// nearly always (750 us each, 1215 by launches) and lose nothing.
struct OneLaunchTrials {
    unsigned left_out = 0, after_next = 4;

    bool tries() {
        if (left_out == 0) return true;
        --left_out;
        return false;
    }
    void ended(bool took) {
        left_out = took ? 0 : after_next;
        after_next = took ? 4 : after_next < 64 ? 2 * after_next : 64;
    }
};

}   // namespace etpic
