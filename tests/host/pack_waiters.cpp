// The packing calls' waiters (ss_pack_wait.h) against a runtime whose allocations fail on request.
#include "../../paper_2411_00288_amd/csrc/ss_pack_wait.h"
#include <cstdio>
#include <cstdlib>
#include <vector>

static bool no_memory, no_events;
static int device, pages, events;
extern "C" {
hipError_t hipGetDevice(int *d) { *d = device; return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { if (no_memory) return hipErrorOutOfMemory; *p = malloc(n); pages++; return hipSuccess; }
hipError_t hipHostFree(void *p) { free(p); pages--; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { if (no_events) return hipErrorOutOfMemory; *e = reinterpret_cast<hipEvent_t>(malloc(1)); events++; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { free(reinterpret_cast<void *>(e)); events--; return hipSuccess; }
}
using namespace ss;
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)

// Takes `n` waiters at once; how many of them have counters (each a set of its own).
static int with_counters(int n, std::vector<Waiter> *out)
{
    uint32_t seen = 0;
    int found = 0;
    for (int i = 0; i < n; i++) {
        Waiter w;
        if (!take_waiter(&w) || w.device != device || w.verdict->done || w.verdict->bad) return -1;
        if (w.slot >= 0) {
            if (seen >> w.slot & 1) return -1;
            seen |= 1u << w.slot;
            found++;
        } else if (w.done == nullptr) {
            return -1;
        }
        out->push_back(w);
    }
    return found;
}
static void give_all(std::vector<Waiter> *v)
{
    for (const Waiter &w : *v) {
        w.verdict->done = w.verdict->bad = 1;      // (what a call leaves behind)
        give_waiter(w);
    }
    v->clear();
}

int main()
{
    std::vector<Waiter> taken;
    // allocations that fail take no counters with them
    no_memory = true;
    for (int i = 0; i < 3 * kSlots; i++) {
        Waiter w;
        CHECK(!take_waiter(&w));
    }
    no_memory = false;
    CHECK(with_counters(kSlots + 5, &taken) == kSlots && pages == kSlots + 5 && events == 5);
    give_all(&taken);
    CHECK(with_counters(kSlots + 5, &taken) == kSlots && pages == kSlots + 5 && events == 5);      // all of them kept
    // one more than there are, and no event for it
    no_events = true;
    Waiter w;
    CHECK(!take_waiter(&w) && pages == kSlots + 5);
    no_events = false;
    // with counters first
    give_all(&taken);
    CHECK(take_waiter(&w) && w.slot >= 0);
    give_waiter(w);
    // another device: counters of its own; where memory for them fails while one without counters is kept, that one serves
    device = 3;
    CHECK(with_counters(kSlots + 1, &taken) == kSlots);
    Waiter last = taken[0];
    taken.erase(taken.begin());
    give_all(&taken);
    slots_given[3] &= ~(1u << last.slot);          // (as after an allocation that failed)
    CHECK(with_counters(kSlots, &taken) == kSlots);
    no_memory = true;
    slots_given[3] &= ~1u;
    CHECK(take_waiter(&w) && w.slot < 0 && w.done != nullptr);
    // waiters without counters: 64 are kept over all devices, the others given up
    no_memory = false;
    device = 0;
    give_waiter(w);                                // (device 3's)
    CHECK(with_counters(kSlots + kKeptOthers + 9, &taken) == kSlots);
    give_all(&taken);
    CHECK(events == kKeptOthers);
    std::printf("waiter checks passed\n");
    return 0;
}
