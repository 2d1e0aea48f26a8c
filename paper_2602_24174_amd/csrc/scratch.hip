// Scratch memory of the synchronous calls (table builds, tokenizer enrichment).
//
// A build of 32 M tokens needs 1.2 GB for 5 ms.  Memory that goes back to the driver is cleared before it is handed out again, at
// about 80 GB/s: allocated on each call, that build takes 5.6 ms until the cleared memory of the card is used up and 15 ms from
// then on.  So one block per device, of TASC_CFG_KEEP_SCRATCH_KIB at most, stays with the library between calls, as long as the process
// holds a model or a table; it goes with the last of them, when the option is set to less, and when the device has no memory left
// for something else of the library's.
#include "tasc_internal.h"
#include <mutex>

namespace {
size_t g_most = (size_t)2 << 30;
constexpr int kDevices = 16;
struct Kept { char* p; size_t bytes; };
Kept g_kept[kDevices];
int64_t g_handles = 0;
std::mutex g_mu;

int device() {
    int dev = 0;
    (void)hipGetDevice(&dev);
    return dev >= 0 && dev < kDevices ? dev : -1;
}
void drop(int dev) {          // under g_mu
    if (g_kept[dev].p) (void)hipFree(g_kept[dev].p);
    g_kept[dev] = Kept{nullptr, 0};
}
}  // namespace

void tasc_handles_add(int n) {
    std::lock_guard<std::mutex> lock(g_mu);
    g_handles += n;
    if (g_handles == 0)
        for (int d = 0; d < kDevices; ++d) drop(d);
}

void tasc_scratch_limit(size_t bytes) {
    std::lock_guard<std::mutex> lock(g_mu);
    g_most = bytes;
    for (int d = 0; d < kDevices; ++d)
        if (g_kept[d].bytes > bytes) drop(d);
}

tasc_status tasc_device_malloc(void** p, size_t bytes) {
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        {
            std::lock_guard<std::mutex> lock(g_mu);
            const int dev = device();
            if (dev >= 0) drop(dev);
        }
        e = hipMalloc(p, bytes);
    }
    TASC_HIP(e);
    return TASC_OK;
}

tasc_status TascScratch::get(size_t need) {
    {
        std::lock_guard<std::mutex> lock(g_mu);
        const int dev = device();
        if (dev >= 0 && g_kept[dev].p && g_kept[dev].bytes >= need) {
            p = g_kept[dev].p;
            bytes = g_kept[dev].bytes;
            g_kept[dev] = Kept{nullptr, 0};
            return TASC_OK;
        }
    }
    const tasc_status rc = tasc_device_malloc((void**)&p, need);
    bytes = rc == TASC_OK ? need : 0;
    return rc;
}

bool tasc_scratch_kept(size_t bytes) {
    std::lock_guard<std::mutex> lock(g_mu);
    return g_handles != 0 && bytes <= g_most;
}

void TascScratch::keep() {
    std::lock_guard<std::mutex> lock(g_mu);
    const int dev = device();
    if (dev < 0 || g_handles == 0 || bytes > g_most || bytes <= g_kept[dev].bytes) return;      // (the destructor frees it)
    drop(dev);
    g_kept[dev] = Kept{p, bytes};
    p = nullptr;
}

TascScratch::~TascScratch() {
    if (p) (void)hipFree(p);
}
