// Device scratch of the calls: blocks kept between calls, and one call's
// allocations out of them.
#pragma once

#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstdint>
#include <mutex>
#include <new>
#include <vector>

#include "bc.h"

namespace {

// Device memory that earlier calls have finished with, kept for the next ones:
// on each device at most kKeep bytes (kKeepIdle when the process's last graph
// goes), the longest unused given back first, all of a device's when an
// allocation on it fails and when a service sizes its budget there.  A block is put here only when nothing on the
// device uses it any more, so any thread and stream may take it.
//
// (The runtime's own stream-ordered pool, which held this scratch before, gave
// blocks of hundreds of MiB back to the driver and took them again within a run
// of like calls, 0.5 to 1 ms each and now and then hundreds of ms: 40k edges
// (6,2) 0.74 against 1.8 ms a call, 50k edges (3,3) 0.51 against 1.37 ms, and
// 6 to 7 ms from some 400 calls on.)
class ScratchCache {
public:
    static constexpr uint64_t kKeep = 32ull << 30, kKeepIdle = 1ull << 30;
    static ScratchCache &get()
    {
        static ScratchCache *c = new ScratchCache;   // outlives every static object that may hold a graph
        return *c;
    }
    // a block of at least bytes and, if a kept one serves, at most `most`;
    // *size is what it has
    hipError_t take(int device, uint64_t bytes, uint64_t most, void **p, uint64_t *size)
    {
        {
            std::lock_guard<std::mutex> g(mu);
            size_t best = kept.size();
            for (size_t i = 0; i < kept.size(); ++i)
                if (kept[i].device == device && kept[i].size >= bytes && kept[i].size <= most &&
                    (best == kept.size() || kept[i].size <= kept[best].size))
                    best = i;
            if (best != kept.size()) {
                *p = kept[best].p;
                *size = kept[best].size;
                kept.erase(kept.begin() + (ptrdiff_t)best);
                return hipSuccess;
            }
        }
        *size = bytes;
        hipError_t e = hipMalloc(p, bytes);
        if (e == hipSuccess) return e;
        (void)hipGetLastError();
        trim(device, 0);
        e = hipMalloc(p, bytes);
        if (e != hipSuccess) (void)hipGetLastError();
        return e;
    }
    void put(int device, void *p, uint64_t size)
    {
        bool listed = true;
        {
            std::lock_guard<std::mutex> g(mu);
            try {   // (called from a destructor, under C entries)
                kept.push_back({p, size, device});
            } catch (const std::bad_alloc &) {
                listed = false;
            }
        }
        if (listed) trim(device, kKeep);
        else (void)hipFree(p);
    }
    // gives a device's blocks back until at most `most` bytes of it are kept
    void trim(int device, uint64_t most)
    {
        for (;;) {
            void *p = nullptr;
            {
                std::lock_guard<std::mutex> g(mu);
                uint64_t total = 0;
                size_t first = kept.size();
                for (size_t i = kept.size(); i-- > 0;)
                    if (kept[i].device == device) {
                        total += kept[i].size;
                        first = i;
                    }
                if (total <= most) return;
                p = kept[first].p;
                kept.erase(kept.begin() + (ptrdiff_t)first);
            }
            (void)hipFree(p);
        }
    }
    // the same on every device
    void trim_all(uint64_t most)
    {
        int last = -1;
        {
            std::lock_guard<std::mutex> g(mu);
            for (const Block &b : kept) last = std::max(last, b.device);
        }
        for (int device = 0; device <= last; ++device) trim(device, most);
    }

private:
    struct Block {
        void *p;
        uint64_t size;
        int device;
    };
    std::mutex mu;
    std::vector<Block> kept;   // the longest unused first
};

// Device scratch of one call, released when the call ends.  Three sources:
// blocks of the cache above (default), the caller's allocator hook, or a fixed
// device region carved by bumping an offset (the no-allocation entry point;
// nothing is allocated or freed).  Every request is rounded up to 256 bytes.  A
// failed request returns hipErrorOutOfMemory.
//
// Uncapped requests to the cache share blocks, each twice the one before
// (kChunk, up to kMostChunk; larger requests are rounded up to an eighth of
// their power of two), so that calls on graphs of a few sizes find each
// other's.  Capped ones take blocks of their own, at most a quarter larger than
// that, and all of a block counts against the cap; a call that runs out of room
// for it (padded) is run again on blocks of exactly what it asks for.
struct DevAlloc {
    static constexpr uint64_t kChunk = 32ull << 20, kMostChunk = 512ull << 20;
    uint64_t next_chunk = kChunk;
    uint8_t *chunk = nullptr;
    uint64_t chunk_left = 0;
    struct Owned {
        void *p;
        uint64_t size;
    };
    std::vector<Owned> ptrs;
    hipStream_t st;
    int device = 0;
    const bc_allocator *hook = nullptr;
    uint8_t *fixed = nullptr;
    uint64_t fixed_cap = 0, fixed_used = 0;
    bool fixed_short = false;    // a request did not fit the fixed region
    uint64_t cap = 0;            // nonzero: at most this many bytes in all (other sources)
    bool exact = false;          // capped: blocks of the size asked for only
    bool padded = false;         // capped: some block was larger
    uint64_t total = 0;          // bytes taken so far (nothing is released before the end)
    DevAlloc(hipStream_t s, int dev, const bc_allocator *h) : st(s), device(dev), hook(h) {}
    DevAlloc(hipStream_t s, void *region, uint64_t cap) : st(s), fixed((uint8_t *)region), fixed_cap(cap) {}
    ~DevAlloc()
    {
        // (an error may have left work behind; with none this returns at once)
        if (!hook && !ptrs.empty()) (void)hipStreamSynchronize(st);
        for (const Owned &o : ptrs) {
            if (hook) hook->free(hook->ctx, o.p, st);
            else ScratchCache::get().put(device, o.p, o.size);
        }
    }
    // bytes left in the fixed region or under the cap (else unbounded)
    uint64_t room() const
    {
        if (fixed) return fixed_cap - fixed_used;
        return cap ? (cap > total ? cap - total : 0) : ~0ull;
    }
    hipError_t raw(void **p, uint64_t bytes)
    {
        bytes = (std::max<uint64_t>(bytes, 1) + 255) & ~255ull;
        *p = nullptr;
        if (fixed) {
            if (bytes > fixed_cap - fixed_used) {
                fixed_short = true;
                return hipErrorOutOfMemory;
            }
            *p = fixed + fixed_used;
            fixed_used += bytes;
            total += bytes;
            return hipSuccess;
        }
        if (cap && bytes > room()) return hipErrorOutOfMemory;
        void *v = nullptr;
        if (hook) {
            v = hook->alloc(hook->ctx, bytes, st);
            if (!v) return hipErrorOutOfMemory;
            ptrs.push_back({v, bytes});
        } else if (bytes <= chunk_left) {
            v = chunk;
            chunk += bytes;
            chunk_left -= bytes;
        } else {
            uint64_t size = bytes, got = 0;
            const bool share = !cap && bytes <= kMostChunk;
            if (share) {
                while (next_chunk < bytes) next_chunk *= 2;
                size = next_chunk;
            } else if (!exact) {
                const uint64_t step = 1ull << (60 - __builtin_clzll(bytes));
                size = std::min((bytes + step - 1) / step * step, room());
            }
            ScratchCache &cache = ScratchCache::get();
            const uint64_t most = exact ? size : std::min(cap ? size + size / 4 : 2 * size, room());
            hipError_t e = cache.take(device, size, most, &v, &got);
            if (e != hipSuccess && size != bytes)   // memory is short: no more than what is asked for
                e = cache.take(device, bytes, cap ? bytes : 2 * bytes, &v, &got);
            if (e != hipSuccess) return e;
            ptrs.push_back({v, got});
            if (cap) {
                padded = padded || got > bytes;
                bytes = got;
            }
            if (share && got > bytes) {
                chunk = (uint8_t *)v + bytes;
                chunk_left = got - bytes;
                next_chunk = std::min(2 * next_chunk, kMostChunk);
            }
        }
        total += bytes;
        *p = v;
        return hipSuccess;
    }
    // gives back what was taken since the mark (no queued work may use it)
    struct Mark {
        size_t n_ptrs;
        uint8_t *chunk;
        uint64_t chunk_left, next_chunk, fixed_used, total;
    };
    Mark mark() const { return {ptrs.size(), chunk, chunk_left, next_chunk, fixed_used, total}; }
    void rollback(const Mark &m)
    {
        for (; ptrs.size() > m.n_ptrs; ptrs.pop_back()) {
            if (hook) hook->free(hook->ctx, ptrs.back().p, st);
            else ScratchCache::get().put(device, ptrs.back().p, ptrs.back().size);
        }
        chunk = m.chunk;
        chunk_left = m.chunk_left;
        next_chunk = m.next_chunk;
        fixed_used = m.fixed_used;
        total = m.total;
        fixed_short = false;
    }
    template <typename T>
    hipError_t get(T **p, uint64_t count)
    {
        void *v = nullptr;
        hipError_t e = raw(&v, count * sizeof(T));
        *p = (T *)v;
        return e;
    }
};

}  // namespace
