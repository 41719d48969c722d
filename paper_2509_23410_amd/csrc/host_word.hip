// The words of host_word.h
#include "host_word.h"

#include <hip/hip_runtime_api.h>

#include <mutex>
#include <new>

namespace {
constexpr int kWords = 64, kWordStride = 16;   // a cache line each, one page of memory
}  // namespace

struct HostWordPage {
    uint32_t *host = nullptr, *device = nullptr;
    uint64_t held = 0;                         // bit = word
    HostWordPage* next = nullptr;
};

namespace {
std::mutex g_mutex;                            // of the list and its `held`
HostWordPage* g_pages = nullptr;

HostWordPage* new_page() {
    HostWordPage* p = new (std::nothrow) HostWordPage;
    if (!p) return nullptr;
    void *host = nullptr, *device = nullptr;
    if (hipHostMalloc(&host, kWords * kWordStride * sizeof(uint32_t), hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess ||
        hipHostGetDevicePointer(&device, host, 0) != hipSuccess) {
        (void)hipGetLastError();
        if (host) (void)hipHostFree(host);
        delete p;
        return nullptr;
    }
    p->host = static_cast<uint32_t*>(host);
    p->device = static_cast<uint32_t*>(device);
    return p;
}
}  // namespace

HostWord::HostWord() {
    std::unique_lock<std::mutex> lock(g_mutex);
    for (page_ = g_pages; page_ && page_->held == ~0ull;) page_ = page_->next;
    if (!page_) {
        lock.unlock();                         // (nobody waits for this allocation, not even a call that gives its word back)
        page_ = new_page();
        if (!page_) return;
        lock.lock();
        page_->next = g_pages;
        g_pages = page_;
    }
    slot_ = __builtin_ctzll(~page_->held);
    page_->held |= 1ull << slot_;
    __atomic_store_n(page_->host + slot_ * kWordStride, 0u, __ATOMIC_RELEASE);
}

HostWord::~HostWord() {
    if (!page_) return;
    std::lock_guard<std::mutex> lock(g_mutex);
    page_->held &= ~(1ull << slot_);
}

uint32_t* HostWord::device() const { return page_->device + slot_ * kWordStride; }
uint32_t HostWord::value() const { return __atomic_load_n(page_->host + slot_ * kWordStride, __ATOMIC_ACQUIRE); }
