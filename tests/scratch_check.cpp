// Host check of the scratch memory (bc_scratch.h) against a stand-in for the
// device allocator: what each part of the device side may rely on.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>
#include <random>

#include "bc_scratch.h"

// ---- the device: sizes only, one memory per device -------------------------
static int cur_dev = 0;
static uint64_t dev_size[2] = {~0ull, ~0ull}, dev_used[2], n_malloc, n_sync;
struct Mem {
    uint64_t size;
    int dev;
};
static std::map<void *, Mem> live;
static uintptr_t next_addr = 1ull << 40;

extern "C" hipError_t hipMalloc(void **p, size_t n)
{
    ++n_malloc;
    if (n > dev_size[cur_dev] - dev_used[cur_dev]) return hipErrorOutOfMemory;
    *p = (void *)next_addr;
    next_addr += (n + 0xfffff) & ~0xfffffull;
    live[*p] = {n, cur_dev};
    dev_used[cur_dev] += n;
    return hipSuccess;
}
extern "C" hipError_t hipFree(void *p)
{
    auto it = live.find(p);
    if (it == live.end()) abort();
    dev_used[it->second.dev] -= it->second.size;
    live.erase(it);
    return hipSuccess;
}
extern "C" hipError_t hipStreamSynchronize(hipStream_t)
{
    ++n_sync;
    return hipSuccess;
}
extern "C" hipError_t hipGetLastError(void) { return hipSuccess; }

// host memory that runs out when told to
static bool host_full = false;
void *operator new(size_t n)
{
    void *p = host_full ? nullptr : malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }

static int bad = 0;
#define CHECK(x)                                             \
    do {                                                     \
        if (!(x)) {                                          \
            printf("line %d: %s\n", __LINE__, #x);           \
            ++bad;                                           \
        }                                                    \
    } while (0)

// ---- a capped call holds at most its cap, and counts what it holds ---------
static void check_cap()
{
    std::mt19937_64 rng(7);
    auto size = [&] { return 1 + rng() % (1ull << (8 + rng() % 18)); };
    for (int t = 0; t < 2000; ++t) {
        const uint64_t cap = (1ull << 20) + rng() % (64ull << 20);
        std::vector<uint64_t> want;
        uint64_t sum = 0;
        for (int i = 0; i < 40; ++i) {
            const uint64_t n = size(), r = (n + 255) & ~255ull;
            if (sum + r > cap) break;
            sum += r;
            want.push_back(n);
        }
        // all these requests fit the cap: the call or, where blocks were larger
        // than asked for, its second run on exact blocks gets them
        bool ok = true, padded = false;
        for (int run = 0; run < 2; ++run) {
            DevAlloc mem(nullptr, 0, nullptr);
            mem.cap = cap;
            mem.exact = run == 1;
            ok = true;
            for (uint64_t n : want) {
                void *p;
                ok = ok && mem.raw(&p, n) == hipSuccess;
                uint64_t held = 0;
                for (const auto &o : mem.ptrs) held += live.at(o.p).size;
                CHECK(held <= cap && held == mem.total);
            }
            padded = mem.padded;
            if (ok) break;
            CHECK(run == 0 && padded);
        }
        CHECK(ok);
        if (t % 3 == 0) {   // uncapped calls between them
            DevAlloc mem(nullptr, 0, nullptr);
            void *p;
            for (int i = 0; i < 10; ++i) CHECK(mem.raw(&p, size()) == hipSuccess);
        }
    }
}

// ---- what is kept is kept per device ---------------------------------------
static uint64_t kept_on(int dev) { return dev_used[dev]; }   // (no call is running)

static void check_devices()
{
    const uint64_t block = 6ull << 30;
    auto fill = [&](int dev) {
        cur_dev = dev;
        DevAlloc mem(nullptr, dev, nullptr);
        void *p;
        for (int i = 0; i < 5; ++i) CHECK(mem.raw(&p, block) == hipSuccess);
    };
    // each keeps its 30 GiB: less than kKeep on either, more on both
    fill(0);
    fill(1);
    CHECK(kept_on(0) == 5 * block && kept_on(1) == 5 * block);
    // a shortage on one device leaves the other's blocks alone
    dev_size[0] = 6 * block;
    {
        cur_dev = 0;
        DevAlloc mem(nullptr, 0, nullptr);
        void *p;
        CHECK(mem.raw(&p, 6 * block) == hipSuccess);   // only when all of device 0's are given back
        CHECK(dev_used[0] == 6 * block && kept_on(1) == 5 * block);
    }
    // above kKeep the longest unused go, on that device
    CHECK(kept_on(0) == 0 && kept_on(1) == 5 * block);
    ScratchCache::get().trim(1, block);
    CHECK(kept_on(1) == block);
    fill(0);
    ScratchCache::get().trim_all(0);
    CHECK(kept_on(0) == 0 && kept_on(1) == 0 && live.empty());
}

// ---- a call that ends with no host memory left still ends ------------------
static void check_host_full()
{
    {
        DevAlloc mem(nullptr, 0, nullptr);
        void *p;
        for (int i = 0; i < 40; ++i) CHECK(mem.raw(&p, 600ull << 20) == hipSuccess);
        host_full = true;   // its blocks find no room in the list of kept ones
    }
    ScratchCache::get().trim_all(0);
    host_full = false;
    CHECK(live.empty());
}

int main(int argc, char **argv)
{
    const char *what = argc > 1 ? argv[1] : "";
    if (!strcmp(what, "cap")) check_cap();
    else if (!strcmp(what, "devices")) check_devices();
    else if (!strcmp(what, "host_full")) check_host_full();
    else return 2;
    printf("%s: bad %d, %llu mallocs\n", what, bad, (unsigned long long)n_malloc);
    return bad != 0;
}
