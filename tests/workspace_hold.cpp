// Two host threads ask for the workspace of one stream: the second gets it when the first one's call is over.  No GPU: the
// few runtime calls on the way are answered here.
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <thread>

#include "../paper_1801_00829_amd/csrc/runtime.h"

extern "C" {
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
}

int main()
{
    using namespace fuse;
    std::string err;
    std::atomic<int> got{0};
    std::thread other[2];
    {
        Workspace ws;
        if (Runtime::get().workspace(nullptr, 10, ws, err) || !ws.partials || !ws.ticket)
            return std::printf("workspace: %s\n", err.c_str()), 2;
        for (int t = 0; t < 2; ++t)                   // the same stream, and another one
            other[t] = std::thread([t, &got] {
                std::string e;
                Workspace w;
                if (!Runtime::get().workspace(reinterpret_cast<hipStream_t>((size_t)t * 64), 100000, w, e))
                    got += t ? 10 : 1;
            });
        other[1].join();
        std::this_thread::sleep_for(std::chrono::milliseconds(300));
        if (got != 10) {
            std::printf("while it is held: %d\n", (int)got);
            std::fflush(stdout);
            std::_Exit(1);
        }
    }
    other[0].join();
    return std::printf("after: %d\n", (int)got), got == 11 ? 0 : 1;
}
