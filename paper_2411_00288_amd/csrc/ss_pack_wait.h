// What a compression waits with (host code): a word of pinned host memory in which the kernel's last workgroup leaves the verdict, and one of the
// device's kSlots sets of ticket counters.  A call that finds all of those in use has an event instead, given to the launch, that completes with
// the kernel.  Handed out one per call in flight and kept for the next, in an array: nothing here may throw through the C entry.
#ifndef SS_PACK_WAIT_H_
#define SS_PACK_WAIT_H_
#include <hip/hip_runtime_api.h>
#include <mutex>
#include <stdint.h>

namespace ss {

constexpr int kSlots = 16;                        // calls in flight on a device that have counters; further ones wait for an event
struct Verdict {                                  // pinned host memory, zero before the call
    uint32_t done, bad;                           // all is packed (with slot >= 0); a block's mask is invalid
};

struct Waiter {
    Verdict *verdict = nullptr;
    hipEvent_t done = nullptr;        // slot < 0
    int device = -1, slot = -1;
    void clear() const
    {
        __atomic_store_n(&verdict->done, 0u, __ATOMIC_RELAXED);
        __atomic_store_n(&verdict->bad, 0u, __ATOMIC_RELAXED);
    }
};

constexpr int kSlotDevices = 64, kKeptOthers = 64;
constexpr int kKeptWaiters = kSlotDevices * kSlots + kKeptOthers;      // every waiter that has counters, and some that have not
static std::mutex waiter_mutex;
static Waiter kept_waiters[kKeptWaiters];
static int n_kept_waiters = 0, n_kept_others = 0;
static uint32_t slots_given[kSlotDevices];        // per device, a bit for each set of counters that a waiter has

// One of the device's kept waiters, with counters if there is one (the caller holds the mutex).
static bool take_kept(Waiter *w, int dev, bool with_counters_only)
{
    int pick = -1;
    for (int i = n_kept_waiters; i-- > 0 && (pick < 0 || kept_waiters[pick].slot < 0);)
        if (kept_waiters[i].device == dev) pick = i;
    if (pick < 0 || (with_counters_only && kept_waiters[pick].slot < 0)) return false;
    *w = kept_waiters[pick];
    kept_waiters[pick] = kept_waiters[--n_kept_waiters];
    if (w->slot < 0) n_kept_others--;
    w->clear();
    return true;
}

static bool take_waiter(Waiter *w)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    {
        const std::lock_guard<std::mutex> lock(waiter_mutex);
        const uint32_t left = dev >= 0 && dev < kSlotDevices ? ~slots_given[dev] & ((1u << kSlots) - 1) : 0u;
        if (take_kept(w, dev, left != 0)) return true;
        w->slot = -1;
        if (left != 0) {
            w->slot = __builtin_ctz(left);
            slots_given[dev] |= 1u << w->slot;
        }
    }
    void *page = nullptr;
    bool ok = hipHostMalloc(&page, 64, hipHostMallocDefault) == hipSuccess;
    if (ok && w->slot < 0 && hipEventCreateWithFlags(&w->done, hipEventDisableTiming) != hipSuccess) {
        (void)hipHostFree(page);
        ok = false;
    }
    if (!ok) {                                    // no waiter has the counters then: they go to a later call
        const std::lock_guard<std::mutex> lock(waiter_mutex);
        if (w->slot >= 0) slots_given[dev] &= ~(1u << w->slot);
        return take_kept(w, dev, false);
    }
    w->verdict = static_cast<Verdict *>(page);
    w->device = dev;
    w->clear();
    return true;
}

// After a call that waited to its end, or whose kernel was never launched.  (A kernel that may still run keeps its waiter: it would write into
// the next call's.)
static void give_waiter(const Waiter &w)
{
    {
        const std::lock_guard<std::mutex> lock(waiter_mutex);
        if (w.slot >= 0 || n_kept_others < kKeptOthers) {
            if (w.slot < 0) n_kept_others++;
            kept_waiters[n_kept_waiters++] = w;
            return;
        }
    }
    (void)hipEventDestroy(w.done);
    (void)hipHostFree(w.verdict);
}

}  // namespace ss

#endif
