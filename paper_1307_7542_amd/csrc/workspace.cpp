// Device memory for the duration of one call.
//
// Blocks above kOwn come from the allocator that the caller has set
// (hub_set_allocator; the Python binding sets PyTorch's caching allocator) and go
// back to it when the call ends, so that the program that owns the device sees
// them, reuses them and can have them back.  They are not taken from the driver
// call by call, because memory that the driver takes back is wiped before it can
// be allocated again, about 25 ms per GB once fresh memory has run out (14-site
// ring FP64, energy with gradient, 18 GB of Lanczos vectors: 180 to 440 ms per call
// from the driver, 30 ms from the allocator).
//
// Smaller blocks, and without an allocator all of them, come from the driver and
// go back to a per-device list of idle blocks, at most kIdle bytes of them, the
// longest unused given up first; the list is emptied (and the allocator asked for
// its idle memory) before an allocation of the library is reported as failed, and
// by hub_workspace_trim.  A block is handed to one caller at a time under a lock
// and comes back only after the caller's stream has been waited for, so it may be
// used on any other stream next.
#include <map>
#include <mutex>
#include <new>
#include <unordered_map>

#include "internal.h"

namespace hub {
namespace {

constexpr size_t kIdle = (size_t)256 << 20;
constexpr size_t kOwn = (size_t)32 << 20;

struct Allocator {
    hub_alloc_fn alloc = nullptr;
    hub_release_fn release = nullptr;
    hub_idle_fn idle = nullptr;
    hub_trim_fn trim = nullptr;
};

struct Block {
    size_t bytes = 0;
    hub_release_fn release = nullptr;  // of the allocator that it came from, or NULL: from the driver
};

struct IdleBlock {
    void *p = nullptr;
    uint64_t since = 0;
};

struct DeviceList {
    std::multimap<size_t, IdleBlock> idle;  // by size
    size_t idle_bytes = 0;
};

struct Lists {
    std::mutex mu;
    std::map<int, DeviceList> dev;
    std::unordered_map<void *, Block> blocks;  // every block handed out or idle
    uint64_t clock = 0;
    Allocator caller;
};

// never destroyed: the HIP runtime may end before static destructors run
Lists &lists()
{
    static Lists *l = new Lists();
    return *l;
}

// Takes idle blocks off the list, longest unused first, until at most `keep` bytes are left.
void trim(Lists &l, DeviceList &d, size_t keep, std::vector<void *> &out)
{
    while (d.idle_bytes > keep && !d.idle.empty()) {
        auto old = d.idle.begin();
        for (auto it = d.idle.begin(); it != d.idle.end(); ++it)
            if (it->second.since < old->second.since) old = it;
        out.push_back(old->second.p);
        d.idle_bytes -= old->first;
        l.blocks.erase(old->second.p);
        d.idle.erase(old);
    }
}

void free_all(const std::vector<void *> &p)
{
    for (void *q : p) (void)hipFree(q);
}

size_t trim_all()
{
    Lists &l = lists();
    std::vector<void *> out;
    size_t bytes = 0;
    {
        std::lock_guard<std::mutex> lk(l.mu);
        for (auto &d : l.dev) {
            bytes += d.second.idle_bytes;
            trim(l, d.second, 0, out);
        }
    }
    free_all(out);
    return bytes;
}

Allocator caller_allocator()
{
    Lists &l = lists();
    std::lock_guard<std::mutex> lk(l.mu);
    return l.caller;
}

hub_status no_memory(size_t bytes, const char *why)
{
    set_error("workspace allocation of " + std::to_string(bytes) + " bytes: " + why);
    return HUB_ERR_OOM;
}

}  // namespace

void ws_reclaim()
{
    (void)trim_all();
    const Allocator a = caller_allocator();
    if (a.trim) a.trim();
}

hipError_t device_alloc(void **p, size_t bytes)
{
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipSuccess) return e;
    (void)hipGetLastError();
    ws_reclaim();
    return hipMalloc(p, bytes);
}

// owner: the stream on which the block is taken from the caller's allocator;
// external: it was (work of another stream then waits for that one).  What the
// allocator refuses (a limit of its own, say) comes from the driver if the call needs
// it, and not at all if it is spare.
hub_status ws_alloc(void **p, size_t bytes, hipStream_t owner, bool spare, bool &external)
try {
    *p = nullptr;
    external = false;
    const size_t unit = bytes < ((size_t)1 << 20) ? 256 : (size_t)1 << 20;
    bytes = (std::max<size_t>(bytes, 1) + unit - 1) / unit * unit;
    int device = 0;
    HUB_HIP(hipGetDevice(&device));
    Lists &l = lists();
    const Allocator a = caller_allocator();
    Block b{bytes, nullptr};
    if (a.alloc && bytes > kOwn) {
        *p = a.alloc(bytes, device, owner);
        if (!*p && spare) return no_memory(bytes, "refused by the caller's allocator");
    }
    if (*p) {
        b.release = a.release;
        external = true;
    } else {
        {
            std::lock_guard<std::mutex> lk(l.mu);
            DeviceList &d = l.dev[device];
            auto it = d.idle.lower_bound(bytes);
            if (it != d.idle.end() && it->first <= bytes + bytes / 4) {
                *p = it->second.p;
                d.idle_bytes -= it->first;
                d.idle.erase(it);
                return HUB_OK;
            }
        }
        const hipError_t e = device_alloc(p, bytes);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            *p = nullptr;
            (void)no_memory(bytes, hipGetErrorString(e));
            return (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation) ? HUB_ERR_OOM : HUB_ERR_DEVICE;
        }
    }
    try {
        std::lock_guard<std::mutex> lk(l.mu);
        l.blocks[*p] = b;
    } catch (...) {
        if (b.release) b.release(*p);
        else (void)hipFree(*p);
        *p = nullptr;
        throw;
    }
    return HUB_OK;
} catch (const std::bad_alloc &) {
    return no_memory(bytes, "host allocation failed");
}

void ws_free(int device, void *p, bool reusable)
{
    if (!p) return;
    Lists &l = lists();
    hub_release_fn release = nullptr;
    std::vector<void *> out;
    try {
        std::lock_guard<std::mutex> lk(l.mu);
        auto it = l.blocks.find(p);
        const Block b = it != l.blocks.end() ? it->second : Block{};
        release = b.release;
        if (!release && reusable && b.bytes > 0 && b.bytes <= kIdle) {
            DeviceList &d = l.dev[device];
            trim(l, d, kIdle - b.bytes, out);
            d.idle.emplace(b.bytes, IdleBlock{p, ++l.clock});
            d.idle_bytes += b.bytes;
            p = nullptr;
        } else if (it != l.blocks.end()) {
            l.blocks.erase(it);
        }
    } catch (const std::bad_alloc &) {  // no room to note it as idle: back to the driver
    }
    free_all(out);
    if (!p) return;
    if (release) release(p);
    else (void)hipFree(p);
}

size_t ws_idle_bytes(int device)
{
    Lists &l = lists();
    std::lock_guard<std::mutex> lk(l.mu);
    auto it = l.dev.find(device);
    return it != l.dev.end() ? it->second.idle_bytes : 0;
}

size_t ws_caller_idle_bytes(int device)
{
    const Allocator a = caller_allocator();
    return a.idle ? a.idle(device) : 0;
}

size_t ws_limit(size_t total_bytes)
{
    return caller_allocator().alloc ? total_bytes / 16 : kIdle;
}

Workspace::Workspace(hipStream_t stream, hipStream_t owner_stream) : st(stream), owner(owner_stream)
{
    (void)hipGetDevice(&device);
}

Workspace::~Workspace()
{
    if (ptrs.empty()) return;
    const bool idle = hipStreamSynchronize(st) == hipSuccess;
    for (void *p : ptrs) ws_free(device, p, idle);
}

hub_status Workspace::alloc(void **p, size_t bytes, bool spare)
{
    *p = nullptr;
    try {
        ptrs.push_back(nullptr);
    } catch (const std::bad_alloc &) {
        return no_memory(bytes, "host allocation failed");
    }
    bool external = false;
    const hub_status r = ws_alloc(p, bytes, owner, spare, external);
    ptrs.back() = *p;
    if (r != HUB_OK || !external || owner == st) return r;
    // what used the block before is queued on the owner's stream
    hipEvent_t e;
    HUB_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    const bool ok = hipEventRecord(e, owner) == hipSuccess && hipStreamWaitEvent(st, e, 0) == hipSuccess;
    (void)hipEventDestroy(e);
    if (ok) return HUB_OK;
    set_error("workspace: ordering after the caller's stream failed");
    return HUB_ERR_DEVICE;
}

}  // namespace hub

using namespace hub;

extern "C" {

hub_status hub_set_allocator(hub_alloc_fn alloc, hub_release_fn release, hub_idle_fn idle, hub_trim_fn trim)
{
    if ((alloc == nullptr) != (release == nullptr)) {
        set_error("hub_set_allocator: alloc and release go together");
        return HUB_ERR_INVALID_ARG;
    }
    Lists &l = lists();
    std::lock_guard<std::mutex> lk(l.mu);
    l.caller = Allocator{alloc, release, idle, trim};
    return HUB_OK;
}

hub_status hub_workspace_trim(int64_t *bytes)
{
    try {
        const size_t n = trim_all();
        if (bytes) *bytes = (int64_t)n;
    } catch (const std::bad_alloc &) {
        return no_memory(0, "host allocation failed");
    }
    return HUB_OK;
}

}  // extern "C"
