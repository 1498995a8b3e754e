// A launch that the runtime refuses is reported once, by the launch itself: what it leaves in the thread's last error
// would be taken for the next caller's.  The runtime's two calls are this program's own, which refuses every launch (without
// a device the real one sets the error anew in whatever call comes next).
#include <cstdio>

#include "../../paper_2510_20878_amd/csrc/ha_rag_attend_dev.h"

static hipError_t last = hipSuccess;

extern "C" hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t)
{
    return last = hipErrorOutOfMemory;
}
extern "C" hipError_t hipGetLastError()
{
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}

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
    const hipError_t e = ha_rag::launch_args(one_argument, dim3(1), dim3(64), 0, nullptr, a);
    if (e != hipErrorOutOfMemory || last != hipSuccess) {
        std::fprintf(stderr, "launch_host: reported %d, left behind %d\n", (int)e, (int)last);
        return 1;
    }
    std::printf("launch_host ok\n");
    return 0;
}
