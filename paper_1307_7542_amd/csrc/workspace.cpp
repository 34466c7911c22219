// Device memory for the duration of one call.  Blocks go back to a per-device
// list instead of to the driver, because memory that the driver takes back is
// wiped before it can be allocated again: a solve that allocates 18 GB for its
// vectors waits about 25 ms per GB for that once fresh memory has run out (ring
// M=14 FP64 solve: 516 ms per call without the list, 38 ms with it).
//
// The list is bounded (a sixteenth of the device memory while any sector lives
// on the device, 256 MB when none does, no block of 256 MB or more while less than
// an eighth of the device memory is free), is emptied before any allocation of the library is
// reported as failed, and hands a block to one caller at a time under a lock;
// blocks come back only after the caller's stream has been waited for, so they
// may be used on any other stream next.
#include <algorithm>
#include <map>
#include <mutex>
#include <unordered_map>

#include "internal.h"

namespace hub {
namespace {

struct DeviceList {
    std::multimap<size_t, void *> idle;  // by size
    size_t idle_bytes = 0;
    size_t limit = 0;  // while sectors live
    int sectors = 0;
};

struct Lists {
    std::mutex mu;
    std::map<int, DeviceList> dev;
    std::unordered_map<void *, size_t> size;  // every block handed out or idle
};

// never destroyed: the HIP runtime may end before static destructors run
Lists &lists()
{
    static Lists *l = new Lists();
    return *l;
}

constexpr size_t kKeepUnused = (size_t)256 << 20;
constexpr size_t kAskFrom = (size_t)256 << 20;

DeviceList &device_list(Lists &l, int device)
{
    DeviceList &d = l.dev[device];
    if (d.limit == 0) {
        size_t free_b = 0, total_b = 0;
        if (hipMemGetInfo(&free_b, &total_b) == hipSuccess) d.limit = total_b / 16;
        d.limit = std::max(d.limit, kKeepUnused);
    }
    return d;
}

// Takes idle blocks off the list until at most `keep` bytes are left, largest first.
std::vector<void *> trim(Lists &l, DeviceList &d, size_t keep)
{
    std::vector<void *> out;
    while (d.idle_bytes > keep && !d.idle.empty()) {
        auto it = std::prev(d.idle.end());
        d.idle_bytes -= it->first;
        l.size.erase(it->second);
        out.push_back(it->second);
        d.idle.erase(it);
    }
    return out;
}

void free_all(const std::vector<void *> &p)
{
    for (void *q : p) (void)hipFree(q);
}

}  // namespace

hipError_t device_alloc(void **p, size_t bytes)
{
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipSuccess) return e;
    (void)hipGetLastError();
    ws_trim();
    return hipMalloc(p, bytes);
}

hub_status ws_alloc(void **p, size_t bytes)
{
    *p = nullptr;
    const size_t unit = bytes < ((size_t)1 << 20) ? 256 : (size_t)1 << 20;
    bytes = (std::max<size_t>(bytes, 1) + unit - 1) / unit * unit;
    int device = 0;
    HUB_HIP(hipGetDevice(&device));
    Lists &l = lists();
    {
        std::lock_guard<std::mutex> lk(l.mu);
        DeviceList &d = device_list(l, device);
        auto it = d.idle.lower_bound(bytes);
        if (it != d.idle.end() && it->first <= bytes + bytes / 4) {
            *p = it->second;
            d.idle_bytes -= it->first;
            d.idle.erase(it);
            return HUB_OK;
        }
    }
    hipError_t e = device_alloc(p, bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        *p = nullptr;
        set_error(std::string("workspace hipMalloc(") + std::to_string(bytes) + "): " + hipGetErrorString(e));
        return (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation) ? HUB_ERR_OOM : HUB_ERR_DEVICE;
    }
    std::lock_guard<std::mutex> lk(l.mu);
    l.size[*p] = bytes;
    return HUB_OK;
}

void ws_free(int device, void *p, bool reusable)
{
    if (!p) return;
    Lists &l = lists();
    size_t bytes = 0;
    {
        std::lock_guard<std::mutex> lk(l.mu);
        auto it = l.size.find(p);
        if (it != l.size.end()) bytes = it->second;
    }
    // no large block is kept on a device that is nearly full (the query takes 40 us)
    size_t free_b = 0, total_b = 0;
    if (reusable && bytes >= kAskFrom && hipMemGetInfo(&free_b, &total_b) == hipSuccess && free_b < total_b / 8)
        reusable = false;
    {
        std::lock_guard<std::mutex> lk(l.mu);
        DeviceList &d = l.dev[device];
        const size_t limit = d.sectors > 0 ? d.limit : kKeepUnused;
        if (reusable && bytes > 0 && d.idle_bytes + bytes <= limit) {
            d.idle.emplace(bytes, p);
            d.idle_bytes += bytes;
            return;
        }
        l.size.erase(p);
    }
    (void)hipFree(p);
}

size_t ws_idle_bytes(int device)
{
    Lists &l = lists();
    std::lock_guard<std::mutex> lk(l.mu);
    return l.dev[device].idle_bytes;
}

size_t ws_limit(int device)
{
    Lists &l = lists();
    std::lock_guard<std::mutex> lk(l.mu);
    return device_list(l, device).limit;
}

void ws_trim()
{
    int device = 0;
    if (hipGetDevice(&device) != hipSuccess) return;
    Lists &l = lists();
    std::vector<void *> out;
    {
        std::lock_guard<std::mutex> lk(l.mu);
        out = trim(l, l.dev[device], 0);
    }
    free_all(out);
}

void ws_sectors(int device, int delta)
{
    Lists &l = lists();
    std::vector<void *> out;
    {
        std::lock_guard<std::mutex> lk(l.mu);
        DeviceList &d = l.dev[device];
        d.sectors += delta;
        if (d.sectors <= 0) out = trim(l, d, kKeepUnused);
    }
    free_all(out);
}

Workspace::Workspace(hipStream_t stream) : st(stream) { (void)hipGetDevice(&device); }

Workspace::~Workspace()
{
    if (ptrs.empty()) return;
    const bool idle = hipStreamSynchronize(st) == hipSuccess;
    for (void *p : ptrs) ws_free(device, p, idle);
}

hub_status Workspace::alloc(void **p, size_t bytes)
{
    HUB_TRY(ws_alloc(p, bytes));
    ptrs.push_back(*p);
    return HUB_OK;
}

}  // namespace hub
