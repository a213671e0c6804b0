// Checks of what the host keeps of an iterative solve (solve_host.hpp).
#include <cstdio>
#include <cstdlib>

#include "solve_host.hpp"

#define CHECK(x)                                                     \
    do {                                                             \
        if (!(x)) {                                                  \
            std::printf("failed at line %d: %s\n", __LINE__, #x);    \
            std::exit(1);                                            \
        }                                                            \
    } while (0)

static void a_block_that_left_a_wait_is_not_a_result() {
    using etpic::SolveWatch;
    CHECK(!etpic::one_launch_took(SolveWatch{0, 0.0, 0.0, 0}));          // the blocks did not meet
    CHECK(etpic::one_launch_took(SolveWatch{2 * 5 + 1, 1.0, 1.0, 0}));   // converged
    CHECK(etpic::one_launch_took(SolveWatch{2 * 5, 1.0, 1.0, 0}));       // the last allowed iteration
    CHECK(!etpic::one_launch_took(SolveWatch{2 * 5 + 1, 1.0, 1.0, 1}));  // block 0 got through, another did not
    CHECK(!etpic::one_launch_took(SolveWatch{0, 0.0, 0.0, 1}));
}

// solves of a context whose blocks never meet: how many try one launch
static void few_solves_wait_while_other_work_holds_the_chip() {
    etpic::OneLaunchTrials t;
    int tried = 0;
    for (int i = 0; i < 1000; ++i)
        if (t.tries()) {
            ++tried;
            t.ended(false);
        }
    CHECK(tried <= 20 && tried >= 10);   // and it does not stop trying
    // the work is gone: the next trial succeeds, and from then on every solve tries
    int later = 0;
    while (!t.tries()) ++later;
    CHECK(later <= 64);
    t.ended(true);
    for (int i = 0; i < 10; ++i) {
        CHECK(t.tries());
        t.ended(true);
    }
    // one failure among successes costs four solves by launches
    CHECK(t.tries());
    t.ended(false);
    for (int i = 0; i < 4; ++i) CHECK(!t.tries());
    CHECK(t.tries());
}

int main() {
    few_solves_wait_while_other_work_holds_the_chip();
    a_block_that_left_a_wait_is_not_a_result();
    std::printf("all checks passed\n");
    return 0;
}
