// Host-logic checks of the pinned slots for the contexts' flags (csrc/flag_slots.h), run on the CPU
// against a simulated allocator that counts, can refuse, and can lose its memory (a device reset).
#include "flag_slots.h"

#include <stdio.h>
#include <stdlib.h>

#include <atomic>
#include <set>
#include <thread>
#include <vector>

namespace {

constexpr ptrdiff_t DEV = 1 << 20;  // the simulated device address is the host's plus this

struct Ops {
    std::atomic<int> acquired{0}, released{0};
    bool refuse = false;
    std::set<void *> lost;
    int acquire(void **p, size_t bytes)
    {
        if (refuse) return -7;
        ++acquired;
        *p = aligned_alloc(4096, bytes);
        memset(*p, 0xAB, bytes);  // recycled memory is never zero
        return 0;
    }
    void release(void *p)
    {
        ++released;
        free(p);
    }
    bool device_address(void *p, void **d)
    {
        if (lost.count(p)) return false;
        *d = (void *)((uintptr_t)p + DEV);
        return true;
    }
};

int failures = 0;
#define CHECK(cond)                                                                  \
    do {                                                                             \
        if (!(cond)) {                                                               \
            fprintf(stderr, "FAILED line %d: %s\n", __LINE__, #cond);                \
            ++failures;                                                              \
        }                                                                            \
    } while (0)

bool zero(const dbmp::FlagSlot &s)
{
    for (size_t i = 0; i < dbmp::FlagSlots::SLOT / 4; ++i)
        if (s.host[i]) return false;
    return true;
}

}  // namespace

int main()
{
    using dbmp::FlagSlot;
    using dbmp::FlagSlots;
    {  // one context after the other: one page, once; an unread flag does not reach the next owner
        FlagSlots f;
        Ops ops;
        for (int i = 0; i < 100; ++i) {
            FlagSlot s;
            CHECK(f.take(&s, ops) == 0);
            CHECK(zero(s) && ((uintptr_t)s.host & 63) == 0);
            CHECK((uintptr_t)s.dev == (uintptr_t)s.host + DEV);
            s.host[i % 16] = 1;
            f.give(&s, ops);
            CHECK(s.host == nullptr);
        }
        CHECK(ops.acquired == 1 && ops.released == 0);
    }
    {  // many alive: distinct slots, a page per 64, all but one page given back at the end; a context
       // created and destroyed at a full page does not allocate each time
        FlagSlots f;
        Ops ops;
        std::vector<FlagSlot> v(200);
        std::set<int *> seen;
        for (FlagSlot &s : v) {
            CHECK(f.take(&s, ops) == 0);
            CHECK(zero(s));
            seen.insert(s.host);
        }
        CHECK(seen.size() == 200 && ops.acquired == 4);
        for (size_t i = 128; i < 200; ++i) f.give(&v[i], ops);
        CHECK(ops.released == 1);
        for (int i = 0; i < 50; ++i) {
            FlagSlot s;
            CHECK(f.take(&s, ops) == 0);
            f.give(&s, ops);
        }
        CHECK(ops.acquired == 4 && ops.released == 1);
        for (size_t i = 0; i < 128; ++i) f.give(&v[i], ops);
        CHECK(ops.released == 3);
        f.give(&v[0], ops);  // an empty slot: nothing
        CHECK(ops.released == 3);
    }
    {  // refused memory is reported; lost memory is forgotten, and its owners may still give it back
        FlagSlots f;
        Ops ops;
        FlagSlot s, t;
        ops.refuse = true;
        CHECK(f.take(&s, ops) == -7 && s.host == nullptr);
        ops.refuse = false;
        CHECK(f.take(&s, ops) == 0);
        ops.lost.insert((void *)((uintptr_t)s.host & ~(uintptr_t)4095));
        CHECK(f.take(&t, ops) == 0 && ops.acquired == 2);
        CHECK(((uintptr_t)t.host & ~(uintptr_t)4095) != ((uintptr_t)s.host & ~(uintptr_t)4095));
        f.give(&s, ops);
        CHECK(ops.released == 0 && zero(t));
        f.give(&t, ops);
    }
    {  // threads
        FlagSlots f;
        Ops ops;
        std::atomic<int> bad{0};
        std::vector<std::thread> th;
        for (int k = 1; k <= 8; ++k)
            th.emplace_back([&, k] {
                for (int i = 0; i < 2000; ++i) {
                    FlagSlot a, b;
                    if (f.take(&a, ops) || f.take(&b, ops)) ++bad;
                    if (!zero(a) || !zero(b) || a.host == b.host) ++bad;
                    a.host[0] = b.host[0] = k;
                    std::this_thread::yield();
                    if (a.host[0] != k || b.host[0] != k) ++bad;
                    f.give(&a, ops);
                    f.give(&b, ops);
                }
            });
        for (std::thread &t : th) t.join();
        CHECK(bad == 0 && ops.acquired == 1 && ops.released == 0);
    }
    if (failures) return 1;
    printf("flag slot checks passed\n");
    return 0;
}
