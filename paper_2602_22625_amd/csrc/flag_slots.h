// Slots of pinned host memory for the contexts' error flags: host logic only, with no HIP types, so
// the same code is exercised by a CPU test against a simulated allocator.
//
// Pinned memory of its own costs a context more than it saves: with 40 of them, 65 us to create one
// and 240 to destroy it, 20 and 2 with these slots, and a check saves 20. So a page is shared by up
// to 64 contexts of a device. A page is released once it is empty and another empty one is at hand: at
// most one page (4 KB) more than the live contexts need is kept, for the life of the process. Every
// call takes the pool's lock.
#pragma once

#include <limits.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>

#include <mutex>
#include <vector>

namespace dbmp {

struct FlagSlot {
    int *host = nullptr;  // null: none
    int *dev = nullptr;   // the device's address of it
};

// Ops supplies the memory operations (the ints are 0 on success, else an error code):
//   int acquire(void **p, size_t bytes);     pinned host memory
//   void release(void *p);
//   bool device_address(void *p, void **d);  false if the memory is no longer there (the device
//                                            was reset): it is then forgotten, not released
class FlagSlots {
public:
    static constexpr size_t SLOT = 64, PAGE = 4096, PER_PAGE = PAGE / SLOT;

    static constexpr int NO_ADDRESS = INT_MIN;  // take: the new memory has no device address

    template <class Ops>
    int take(FlagSlot *out, Ops &ops)
    {
        std::lock_guard<std::mutex> lk(mu_);
        *out = FlagSlot{};
        void *d = nullptr;
        size_t i = 0;
        while (i < pages_.size()) {
            if (~pages_[i].used == 0) {
                ++i;
            } else if (!ops.device_address(pages_[i].p, &d)) {
                pages_.erase(pages_.begin() + (long)i);
            } else {
                break;
            }
        }
        if (i == pages_.size()) {
            pages_.reserve(i + 1);
            Page pg;
            void *p = nullptr;
            const int rc = ops.acquire(&p, PAGE);
            if (rc) return rc;
            pg.p = (char *)p;
            if (!ops.device_address(p, &d)) {
                ops.release(p);
                return NO_ADDRESS;
            }
            pages_.push_back(pg);
        }
        Page &pg = pages_[i];
        const int s = __builtin_ctzll(~pg.used);
        pg.used |= 1ull << s;
        out->host = (int *)(pg.p + s * SLOT);
        out->dev = (int *)((char *)d + s * SLOT);
        memset((void *)out->host, 0, SLOT);
        return 0;
    }

    // No kernel may write the slot any more.
    template <class Ops>
    void give(FlagSlot *slot, Ops &ops)
    {
        std::lock_guard<std::mutex> lk(mu_);
        char *h = (char *)slot->host;
        *slot = FlagSlot{};
        size_t empty = 0, mine = pages_.size();
        for (size_t i = 0; h && i < pages_.size(); ++i) {
            if (h >= pages_[i].p && h < pages_[i].p + PAGE) {
                pages_[i].used &= ~(1ull << ((size_t)(h - pages_[i].p) / SLOT));
                mine = i;
            }
            empty += pages_[i].used == 0;
        }
        if (mine == pages_.size() || pages_[mine].used != 0 || empty < 2) return;
        ops.release(pages_[mine].p);
        pages_.erase(pages_.begin() + (long)mine);
    }

private:
    struct Page {
        char *p = nullptr;
        uint64_t used = 0;
    };
    static_assert(PER_PAGE == 64, "one bit per slot");
    std::mutex mu_;
    std::vector<Page> pages_;
};

}  // namespace dbmp
