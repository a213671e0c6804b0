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

int main() {
    a_block_that_left_a_wait_is_not_a_result();
    std::printf("all checks passed\n");
    return 0;
}
