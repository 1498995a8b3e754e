// A launch that the runtime refuses is reported once, by the launch itself: what it leaves in the thread's last error
// would be taken for the next caller's.  (A workgroup of 2,048 threads is refused on every device, and without one
// every launch is.)
#include <cstdio>

#include "../../paper_2510_20878_amd/csrc/ha_rag_attend_dev.h"

struct Args {
    int *out;
};
__global__ void one_argument(const Args a)
{
    if (a.out) *a.out = 1;
}

int main()
{
    Args a = {nullptr};
    const hipError_t e = ha_rag::launch_args(one_argument, dim3(1), dim3(2048), 0, nullptr, a);
    if (e == hipSuccess) {
        std::fprintf(stderr, "launch_host: the launch was not refused\n");
        return 1;
    }
    const hipError_t left = hipGetLastError();
    if (left != hipSuccess) {
        std::fprintf(stderr, "launch_host: %s is left behind\n", hipGetErrorName(left));
        return 1;
    }
    std::printf("launch_host ok: %s\n", hipGetErrorName(e));
    return 0;
}
