// Driver of the device pool's host code without a GPU: a thread that ends while
// another one waits for the device may have left work behind that the wait does not
// cover.  Its blocks are not handed out before the next wait.
#include "../paper_2103_07537_amd/csrc/memory.hip"

#include <cstdlib>
#include <thread>

extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return ""; }
hipError_t hipMalloc(void** p, size_t n) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
}

using mbamg::DevBuf;

static void* block_of_a_thread_that_ends(size_t n) {
    void* p = nullptr;
    std::thread([&] { DevBuf<float> a(n); p = a.p; }).join();
    return p;
}

int main() {
    const size_t n = 1 << 16;
    void* before = block_of_a_thread_that_ends(n);
    uint64_t mark = mbamg::pool_mark();
    void* during = block_of_a_thread_that_ends(n);   // the device is being waited for
    mbamg::pool_device_idle(mark);
    DevBuf<float> a(n), b(n);
    if (a.p != before) return 1;                      // handed over before the wait: idle
    if (b.p == during) return 2;                      // a kernel may still use it
    mark = mbamg::pool_mark();
    mbamg::pool_device_idle(mark);
    DevBuf<float> c(n);
    return c.p == during ? 0 : 3;                     // idle after the next wait
}
