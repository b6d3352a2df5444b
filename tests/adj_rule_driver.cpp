// The rule for the many-steps reverse kernel, host code: reads tiles in x and y, waves a
// tile, bytes a value and compute units, prints 1 where it is taken, else 0.
#include <cstdio>

#include "lbm_internal.h"

int main() {
    int ntx, nty, waves, bytes, cus;
    while (std::scanf("%d %d %d %d %d", &ntx, &nty, &waves, &bytes, &cus) == 5) {
        lbm::ChanMultiPlan p;
        p.ntx = ntx;
        p.nty = nty;
        p.cus = cus;
        std::printf("%d\n", int(lbm::adj_multi_pays(p, waves, size_t(bytes))));
    }
    return 0;
}
