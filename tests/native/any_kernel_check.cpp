// The choice of the any-N kernel on the host.  Exit status 0 when all hold.
#include <cstdio>

#include "kernels.hpp"

int main() {
    using namespace phub;
    // a piece of the stream walk takes at least two blocks: never below
    for (int n = 1; n <= kMaxWorkers; ++n)
        if ((any_kernel(n) == kAnyBatches) != (n <= kManyBlock)) {
            std::fprintf(stderr, "%d workers\n", n);
            return 1;
        }
    return 0;
}
