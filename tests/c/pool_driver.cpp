// When a kept device block may be handed out without a wait (pool.hpp).
// Prints "pool driver ok" and exits 0 when every check holds.
#include <cstdio>
#include <cstring>

#include "../../paper_2209_06478_amd/csrc/pool.hpp"

using dsm::BlockPool;

static int fails = 0;
#define CHECK(c)                                                         \
    do {                                                                 \
        if (!(c)) {                                                      \
            std::printf("FAILED %s:%d: %s\n", __FILE__, __LINE__, #c);   \
            fails++;                                                     \
        }                                                                \
    } while (0)

static char mem[16];
static int handle[2];

int main() {
    BlockPool::Block b;
    bool wait = false;
    const BlockPool::Stream null = nullptr, s0 = &handle[0], s1 = &handle[1], per = BlockPool::per_thread(),
                            any = BlockPool::unknown();
    // freed on a row, wanted on a column: a wait unless both are one known stream
    const BlockPool::Stream st[5] = {null, s0, s1, per, any};
    for (int i = 0; i < 5; i++)
        for (int j = 0; j < 5; j++) {
            BlockPool p;
            p.put(mem, 256, st[i]);
            CHECK(p.bytes() == 256 && !p.take(512, st[j], &b, &wait));
            CHECK(p.take(256, st[j], &b, &wait) && b.p == mem && p.bytes() == 0);
            CHECK(wait == !(i == j && st[i] != per && st[i] != any));
        }
    // a device-wide wait serves the frees before it, not those after
    for (BlockPool::Stream s : st) {
        BlockPool p;
        p.put(mem, 256, s);
        p.waited(p.frees());
        p.put(mem + 1, 256, any);
        CHECK(p.take(256, any, &b, &wait) && b.p == mem && !wait);
        CHECK(p.take(256, any, &b, &wait) && b.p == mem + 1 && wait);
    }
    // an idle block goes before an older one that is not; the oldest goes back first
    {
        BlockPool p;
        p.put(mem, 256, s0);
        p.put(mem + 1, 256, s1);
        p.put(mem + 2, 512, s1);
        CHECK(p.take(256, s1, &b, &wait) && b.p == mem + 1 && !wait);
        CHECK(p.take_oldest(&b) && b.p == mem && p.take_oldest(&b) && b.p == mem + 2 && !p.take_oldest(&b));
        CHECK(p.bytes() == 0 && p.frees() == 3);
        p.waited(2);
        p.waited(1);  // (waits end in any order)
        p.put(mem, 256, any);
        CHECK(p.take(256, any, &b, &wait) && wait);
    }
    // put back after a device-wide wait: idle at once, whatever is freed later
    {
        BlockPool p;
        p.put(mem, 256, any, true);
        p.put(mem + 1, 256, any);
        CHECK(p.take(256, any, &b, &wait) && b.p == mem && !wait);
        CHECK(p.take(256, any, &b, &wait) && wait);
    }
    // a device with room for the bytes, but not for their class, before or after kept blocks go back
    for (size_t bytes : {(size_t)1, (size_t)256, (size_t)4097, (size_t)100000, ((size_t)1 << 34) + 1})
        for (bool budget : {false, true}) {
            const size_t cls = dsm::block_class(bytes, budget);
            CHECK(cls >= bytes && cls % 256 == 0 && cls - bytes <= (budget ? 255 : bytes / 8 + 255));
            CHECK(budget || dsm::block_class(cls, false) == cls);
            for (size_t room : {bytes - 1, bytes, cls - 1, cls})
                for (size_t kept : {(size_t)0, cls}) {
                    if (room < bytes - 1) continue;
                    size_t left = room - (room < kept ? 0 : kept), tries = 0;
                    bool tight = false, back = false;
                    auto obtain = [&](size_t n) -> void * {
                        tries++;
                        return n <= left ? mem : nullptr;
                    };
                    void *p = dsm::new_block(bytes, cls, obtain, [&] { left = room; back = true; }, &tight);
                    CHECK((p != nullptr) == (room >= bytes));
                    CHECK(!p || tight == (room < cls));
                    CHECK(tries <= 3 && (back || left >= cls));
                }
        }
    if (!fails) std::printf("pool driver ok\n");
    return fails != 0;
}
