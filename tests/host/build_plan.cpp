// Prints the lists that a row of the candidate tree's scan leaves, for every "rows chunks" pair on the command line.
#include <cstdio>
#include <cstdlib>

#include "build_plan.h"

int main(int argc, char** argv) {
    for (int i = 1; i + 1 < argc; i += 2) {
        const int chunks = atoi(argv[i + 1]), seg = s4c::build_segment(atoll(argv[i]), chunks);
        printf("%d %d\n", seg, 4 * ((chunks + seg - 1) / seg));
    }
    return 0;
}
