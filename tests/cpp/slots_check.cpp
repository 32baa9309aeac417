// Host check of the slots in which calls find their totals
// (paper_2009_09500_amd/csrc/vox_slots.h): a call gives its slot back however it
// ends unless a kernel may still write it, no slot has two owners, and without a
// page, or with every slot taken, a call gets none.  Built and run by
// tests/test_slots.py (CPU only).  Prints "ok" or the first failure.
#include <cstdio>
#include <cstdlib>
#include <thread>
#include <vector>

#include "vox_slots.h"

using vox::HostSlots;
using vox::SlotUse;

static int allocations = 0;
static HostSlots::Slot* page() {
    ++allocations;
    return static_cast<HostSlots::Slot*>(calloc(HostSlots::kSlots, sizeof(HostSlots::Slot)));
}
static HostSlots::Slot* no_page() {
    ++allocations;
    return nullptr;
}
static bool idle(void*) { return true; }
static bool stuck(void*) { return false; }

#define CHECK(x)                                   \
    do {                                           \
        if (!(x)) {                                \
            printf("line %d: %s\n", __LINE__, #x); \
            return 1;                              \
        }                                          \
    } while (0)

int main() {
    {
        HostSlots pool(page);
        CHECK(pool.take(false) == nullptr && allocations == 0);
        for (int i = 0; i < 1000; ++i) {  // calls that fail between taking and waiting, and calls that end well
            SlotUse use(pool, pool.take(true), idle, nullptr);
            CHECK(use);
            if (i % 3 == 0) use.done();
        }
        CHECK(allocations == 1);
        for (int i = 0; i < 10; ++i) SlotUse use(pool, pool.take(true), stuck, nullptr);
        std::vector<HostSlots::Slot*> rest;
        while (HostSlots::Slot* s = pool.take(false)) rest.push_back(s);
        CHECK(rest.size() == HostSlots::kSlots - 10);
        SlotUse none(pool, pool.take(true), idle, nullptr);
        CHECK(!none);
        for (HostSlots::Slot* s : rest) pool.give_back(s);
        CHECK(pool.take(false) != nullptr);
    }
    {
        HostSlots pool(no_page);
        allocations = 0;
        for (int i = 0; i < 3; ++i) CHECK(pool.take(true) == nullptr);
        CHECK(allocations == 1);
    }
    {
        HostSlots pool(page);
        std::atomic<int> wrong{0};
        std::vector<std::thread> threads;
        for (int t = 0; t < 8; ++t)
            threads.emplace_back([&, t] {
                for (int i = 0; i < 20000; ++i) {
                    SlotUse use(pool, pool.take(true), idle, nullptr);
                    if (!use) {
                        ++wrong;
                        continue;
                    }
                    use->total = t * 100000 + i;
                    if (use->status++ != 0) ++wrong;
                    if (use->total != t * 100000 + i) ++wrong;
                    --use->status;
                    if (i % 2) use.done();
                }
            });
        for (std::thread& t : threads) t.join();
        CHECK(wrong == 0);
    }
    printf("ok\n");
    return 0;
}
