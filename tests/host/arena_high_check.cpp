// Host-side checks of the arena's blocks taken from the top of a region, built
// with the sanitizers by tests/test_host_sanitized.py (no GPU call is made).
#include "workspace.hip"

#include <cstdio>
#include <cstdlib>
#include <random>

using namespace rrt;

#define CHECK(cond)                                                                 \
    do {                                                                            \
        if (!(cond)) {                                                              \
            std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #cond); \
            std::exit(1);                                                           \
        }                                                                           \
    } while (0)

static bool disjoint(const Ctx& c)
{
    const auto& b = c.arena.blocks;
    for (size_t i = 0; i < b.size(); ++i)
        for (size_t j = i + 1; j < b.size(); ++j)
            if (b[i].region == b[j].region && b[i].off < b[j].off + b[j].size &&
                b[j].off < b[i].off + b[i].size)
                return false;
    return true;
}

int main()
{
    constexpr uint64_t kCap = 65536 + 100;      // not a multiple of the alignment
    static char ws[1 << 20], pb[kCap];
    Ctx c;
    int2* none = nullptr;
    CHECK(ws_alloc(c, &none, 1, kRegionPath, true) == hipErrorOutOfMemory);
    c.arena.base[kRegionWs] = ws;
    c.arena.cap[kRegionWs] = sizeof ws;
    c.arena.base[kRegionPath] = pb;
    c.arena.cap[kRegionPath] = kCap;
    // below the region's (aligned) end, then below the block above; what is freed
    // there leaves the room after the lower blocks in one piece
    int2 *base = nullptr, *h1 = nullptr, *h2 = nullptr, *low = nullptr;
    CHECK(ws_alloc(c, &base, 1000, kRegionPath) == hipSuccess);
    CHECK(ws_alloc(c, &h1, 100, kRegionPath, true) == hipSuccess);
    CHECK(reinterpret_cast<char*>(h1) == pb + 65536 - 1024);
    CHECK(ws_alloc(c, &h2, 100, kRegionPath, true) == hipSuccess);
    CHECK(reinterpret_cast<char*>(h2) == pb + 65536 - 2048);
    CHECK(ws_alloc(c, &low, 32, kRegionPath) == hipSuccess);
    CHECK(reinterpret_cast<char*>(low) == pb + 8192 && disjoint(c));
    CHECK(ws_alloc(c, &h1, kCap, kRegionPath, true) == hipErrorOutOfMemory);
    CHECK(h1 == nullptr && c.arena.short_region == kRegionPath);
    ws_free(c, &h2);
    ws_free(c, &low);
    CHECK(ws_largest_gap(c, kRegionPath) >= 65536 - 8192);
    // a gap that fits exactly, and one block more
    int2* all = nullptr;
    CHECK(ws_alloc(c, &all, (65536 - 8192) / sizeof(int2), kRegionPath, true) == hipSuccess);
    CHECK(reinterpret_cast<char*>(all) == pb + 8192 && disjoint(c));
    CHECK(ws_alloc(c, &low, 1, kRegionPath) == hipErrorOutOfMemory);
    ws_free(c, &all);
    // the highest gap that is large enough, not the highest
    CHECK(ws_alloc(c, &h1, 100, kRegionPath, true) == hipSuccess);
    CHECK(ws_alloc(c, &h2, 32, kRegionPath, true) == hipSuccess);
    CHECK(ws_alloc(c, &low, 100, kRegionPath, true) == hipSuccess);
    ws_free(c, &h2);                            // a hole of 256 bytes
    CHECK(ws_alloc(c, &all, 64, kRegionPath, true) == hipSuccess);
    CHECK(reinterpret_cast<char*>(all) < reinterpret_cast<char*>(low) && disjoint(c));
    CHECK(ws_alloc(c, &h2, 32, kRegionPath, true) == hipSuccess);
    CHECK(reinterpret_cast<char*>(h2) == pb + 65536 - 1024 - 256);
    // random churn from both ends: blocks stay disjoint and inside their regions
    std::mt19937 rng(11);
    std::vector<void*> slots(48, nullptr);
    for (int it = 0; it < 20000; ++it) {
        void** o = &slots[rng() % slots.size()];
        if (rng() % 3 == 0) {
            ws_free(c, o);
            continue;
        }
        const size_t bytes = 1 + rng() % 40000;
        const int region = (int)(rng() % 2);
        if (ws_alloc(c, o, bytes, region, rng() % 2 == 0) == hipSuccess) {
            char* q = static_cast<char*>(*o);
            CHECK(q >= c.arena.base[region] &&
                  q + bytes <= c.arena.base[region] + c.arena.cap[region]);
            q[0] = 1;
            q[bytes - 1] = 2;
        } else {
            CHECK(*o == nullptr);
        }
        if (it % 97 == 0) CHECK(disjoint(c));
    }
    CHECK(disjoint(c));
    std::printf("arena checks from the top passed\n");
    return 0;
}
