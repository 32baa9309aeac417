// Slots of host memory through which calls learn what a kernel computed
// (vox_api.cpp).  Host only, and without HIP, so that a host check runs the code.
#pragma once

#include <stdint.h>

#include <atomic>
#include <mutex>

namespace vox {

// One page for the process, allocated (once, whether or not that succeeds) by the
// first call that may; a call takes a slot of its own for as long as it lasts, and
// none when none is free.
class HostSlots {
  public:
    struct Slot {
        int64_t status, total, pad[6];
    };
    static constexpr int kSlots = 64;

    explicit HostSlots(Slot* (*allocate)()) : allocate_(allocate) {}

    Slot* take(bool may_allocate) {
        Slot* page = page_.load(std::memory_order_acquire);
        if (page == nullptr && may_allocate) page = allocate();
        if (page == nullptr) return nullptr;
        uint64_t used = used_.load(std::memory_order_relaxed);
        while (used != ~uint64_t(0)) {
            const int i = __builtin_ctzll(~used);
            if (used_.compare_exchange_weak(used, used | uint64_t(1) << i, std::memory_order_acquire)) return page + i;
        }
        return nullptr;
    }
    void give_back(Slot* s) {
        used_.fetch_and(~(uint64_t(1) << (s - page_.load(std::memory_order_relaxed))), std::memory_order_release);
    }

  private:
    Slot* allocate() {
        std::lock_guard<std::mutex> lk(mu_);
        if (!tried_) {
            tried_ = true;
            page_.store(allocate_(), std::memory_order_release);
        }
        return page_.load(std::memory_order_relaxed);
    }
    Slot* (*allocate_)();
    std::atomic<Slot*> page_{nullptr};
    std::atomic<uint64_t> used_{0};
    std::mutex mu_;
    bool tried_ = false;
};

// A call's slot, given back at its end however it ends: when done() says that
// the kernels have ended, or else once idle(of) does, which waits for them.  Where
// that fails a kernel may still write the slot, and it stays taken.
class SlotUse {
  public:
    SlotUse(HostSlots& pool, HostSlots::Slot* slot, bool (*idle)(void*), void* of)
        : pool_(pool), slot_(slot), idle_(idle), of_(of) {}
    ~SlotUse() {
        if (slot_ && (done_ || idle_(of_))) pool_.give_back(slot_);
    }
    SlotUse(const SlotUse&) = delete;
    SlotUse& operator=(const SlotUse&) = delete;
    explicit operator bool() const { return slot_ != nullptr; }
    HostSlots::Slot* operator->() const { return slot_; }
    void done() { done_ = true; }

  private:
    HostSlots& pool_;
    HostSlots::Slot* slot_;
    bool (*idle_)(void*);
    void* of_;
    bool done_ = false;
};

}  // namespace vox
