// Prints what csrc/step_plan.h says of steps, a line each: 1 one launch, 0 two.
// Usage: step_plan CHUNKS ROW_CHUNKS TILES LOGITS_BYTES FP32 GREEDY LARGE HEAD [...]
#include <cstdio>
#include <cstdlib>

#include "step_plan.h"

int main(int argc, char** argv) {
    for (int i = 1; i + 7 < argc; i += 8) {
        auto n = [&](int k) { return atoll(argv[i + k]); };
        const s4c::StepScan s = {n(0), n(1), n(2), n(3), n(4) != 0, n(5) != 0, n(6) != 0, (int)n(7)};
        printf("%d\n", (int)s4c::one_launch_pays(s));
    }
    return 0;
}
