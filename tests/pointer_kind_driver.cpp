// Which memory the macro kernels may write to straight away, host code: reads the
// memory type and GPU of a pointer and the context's GPU, prints 1 or 0.
#include <cstdio>

#include "lbm_internal.h"

int main() {
    const hipMemoryType types[4] = {hipMemoryTypeDevice, hipMemoryTypeHost, hipMemoryTypeManaged,
                                    hipMemoryTypeUnregistered};
    int type, owner, device;
    while (std::scanf("%d %d %d", &type, &owner, &device) == 3) {
        hipPointerAttribute_t a{};
        a.type = types[type];
        a.device = owner;
        std::printf("%d\n", int(lbm::kernel_may_write(a, device)));
    }
    return 0;
}
