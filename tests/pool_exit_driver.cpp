// Driver of the device pool's host code without a GPU: stand-ins for the HIP calls
// it makes, a thread whose buffer grows and outlives the thread's list of freed
// blocks, and the blocks' reuse afterwards.
#include "../paper_2103_07537_amd/csrc/memory.hip"

#include <cstdlib>
#include <set>
#include <thread>

static std::set<void*> live;
extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return ""; }
hipError_t hipMalloc(void** p, size_t n) { live.insert(*p = std::malloc(n)); return hipSuccess; }
hipError_t hipFree(void* p) { live.erase(p); std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
}

using mbamg::DevBuf;

static void use(size_t n) {
    static thread_local DevBuf<float> scratch;   // kept for the thread's life, as the gradient's is
    if (scratch.n < n) scratch.alloc(n);
}

int main() {
    for (int round = 0; round < 3; ++round) {
        std::thread t([] { for (size_t n = 1; n <= 64; n *= 2) use(n * 4096); });
        t.join();
        mbamg::pool_device_idle();
    }
    const size_t before = live.size();
    if (before == 0 || before > 7) return 1;     // every round's blocks served the next one
    {
        DevBuf<float> a(4096), b(64 * 4096);
        if (live.size() != before) return 2;     // and serve this thread
    }
    for (size_t n = 1; n <= 64; n *= 2) use(n * 4096);   // the main thread's own, released at its end
    return 0;
}
