// Where a batch's counters and descriptors lie: see test_batch_layout.py.
#include <cstdint>
#include <cstdio>

#include "aes_batch.h"

using namespace aesgpu;

// The three counters, each alone on a 128-byte line, all inside kCounterBytes.
static_assert(kQueueStride * 4 % 128 == 0 && kExitWord * 4 % 128 == 0);
static_assert(kExitWord / 32 != kQueueStride / 32 && kExitWord / 32 != 0);
static_assert(kCounterBytes % 128 == 0 && (kExitWord + 1) * 4 <= kCounterBytes);
static_assert(kCounterBytes <= 512, "nothing but the counters");

int main() {
    const size_t counts[] = {0, 1, 15, 16, 17, 63, 257, 65536};
    for (size_t m : counts)
        for (size_t f : counts)
            for (size_t i : counts)
                for (size_t g : {size_t(0), size_t(1), size_t(33)}) {
                    const BatchLayout at(m, f, i, g, 16 * g);
                    const size_t part[][2] = {{at.counters, kCounterBytes},
                                              {at.msgs, m * sizeof(DevMsg)},
                                              {at.tiles[0], f * sizeof(Tile)},
                                              {at.tiles[1], i * sizeof(Tile)},
                                              {at.cbc_groups, g * sizeof(Tile)},
                                              {at.cbc_dummy, 16},
                                              {at.cbc_list, 16 * g * sizeof(uint32_t)}};
                    size_t end = 0;
                    for (const auto &p : part) {
                        if (p[0] % 256 != 0 || p[0] < end) return 1;
                        end = p[0] + p[1];
                    }
                    if (at.total != end) return 2;
                }
    std::printf("counters %zu bytes, descriptors from %zu\n", kCounterBytes, BatchLayout::msgs);
    return 0;
}
