// Host check of the candidate pass's row storage: whatever the roots and the
// order in which the blocks meet them, rows that add up to w words all find room
// in a pool of row_pool_words(w, blocks).
#include <cstdio>
#include <random>
#include <vector>

#include "bc_device.h"

using namespace bcdev;

int main()
{
    std::mt19937_64 rng(3);
    unsigned bad = 0, roots = 0;
    for (int t = 0; t < 3000; ++t) {
        const uint64_t w = 1 + rng() % (1ull << (8 + rng() % 14));
        const uint32_t n_blocks = 1 + (uint32_t)(rng() % (t % 5 ? 40 : 1792));
        // lengths that leave the most behind: just past half, an eighth, a small part of a chunk
        const uint64_t lens[] = {kRowChunk / 2 + 1, kRowChunk / 8, kRowChunk / 8 + 1, kRowChunk / 8 - 1, 1, 3, kRowChunk, 5000};
        std::vector<RowChunk> c(n_blocks, RowChunk{0, 0});
        const uint64_t cap = row_pool_words(w, n_blocks);
        uint64_t head = 0, used = 0;
        std::vector<uint8_t> taken(cap, 0);
        for (uint32_t x = 0; used < w; ++x) {
            uint64_t need = t & 1 ? lens[rng() % 8] : 1 + rng() % (1 + rng() % 600);
            need = std::min(need, w - used);
            const uint64_t at = take_rows(c[t % 3 ? rng() % n_blocks : x % n_blocks], need, kRowChunk, cap, [&](uint64_t n) {
                head += n;
                return head - n;
            });
            used += need;
            ++roots;
            if (at == ~0ull || at + need > cap) {
                ++bad;
                continue;
            }
            for (uint64_t i = at; i < at + need; ++i) bad += taken[i]++;
        }
        // no chunks where the pool is limited: what is asked for, to the last word
        RowChunk one{0, 0};
        uint64_t h = 0;
        auto bump = [&](uint64_t n) { h += n; return h - n; };
        bad += take_rows(one, w, 0, w, bump) != 0 || take_rows(one, 1, 0, w, bump) != ~0ull;
    }
    printf("roots %u bad %u\n", roots, bad);
    return bad != 0;
}
