// Plans a batch while there is no memory for a second copy of its tiles: the plan
// must come out all the same, in the same order (see test_tile_order_no_memory.py).
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

#include "aes_batch.h"

static size_t refused_from = ~size_t(0), refused_to = 0, refused = 0;

static void *get(size_t n) {
    if (n >= refused_from && n <= refused_to) {
        ++refused;
        return nullptr;
    }
    return std::malloc(n ? n : 1);
}
static void *get_aligned(size_t n, std::align_val_t a) {
    if (n >= refused_from && n <= refused_to) {
        ++refused;
        return nullptr;
    }
    return std::aligned_alloc(size_t(a), (n + size_t(a) - 1) / size_t(a) * size_t(a));
}
static void *or_throw(void *p) { return p ? p : throw std::bad_alloc(); }
void *operator new(size_t n) { return or_throw(get(n)); }
void *operator new[](size_t n) { return or_throw(get(n)); }
void *operator new(size_t n, std::align_val_t a) { return or_throw(get_aligned(n, a)); }
void *operator new[](size_t n, std::align_val_t a) { return or_throw(get_aligned(n, a)); }
void *operator new(size_t n, const std::nothrow_t &) noexcept { return get(n); }
void *operator new[](size_t n, const std::nothrow_t &) noexcept { return get(n); }
void *operator new(size_t n, std::align_val_t a, const std::nothrow_t &) noexcept {
    return get_aligned(n, a);
}
void *operator new[](size_t n, std::align_val_t a, const std::nothrow_t &) noexcept {
    return get_aligned(n, a);
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete[](void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }
void operator delete[](void *p, size_t) noexcept { std::free(p); }
void operator delete(void *p, std::align_val_t) noexcept { std::free(p); }
void operator delete[](void *p, std::align_val_t) noexcept { std::free(p); }
void operator delete(void *p, size_t, std::align_val_t) noexcept { std::free(p); }
void operator delete[](void *p, size_t, std::align_val_t) noexcept { std::free(p); }

using namespace aesgpu;

int main() {
    const size_t m = 3000;   // one tile each; not a size that a growing vector asks for
    std::vector<aesgpu_msg> msgs(m);
    for (size_t i = 0; i < m; ++i) {
        std::memset(&msgs[i], 0, sizeof msgs[i]);
        msgs[i].n_bytes = 16 * (1 + i * 2654435761u % 4096);
        msgs[i].key_bits = 128;
    }
    std::vector<DevMsg> dm;
    std::vector<Tile> tiles[2], want[2];
    std::vector<uint32_t> cbc_list;
    std::vector<Tile> cbc_groups;
    BatchTotals tot;
    if (build_tiles(msgs.data(), m, 4096, dm, want, cbc_list, cbc_groups, tot) != AESGPU_OK) return 2;
    // A copy of the tiles, and some bytes that an array of them may take more.
    refused_from = m * sizeof(Tile);
    refused_to = m * sizeof(Tile) + 64;
    int st;
    try {
        st = build_tiles(msgs.data(), m, 4096, dm, tiles, cbc_list, cbc_groups, tot);
    } catch (const std::bad_alloc &) {
        std::printf("an exception left the planner\n");
        return 3;
    }
    refused_from = ~size_t(0);
    if (st != AESGPU_OK) return 4;
    if (!refused) return 5;   // nothing asked for it: this test tests nothing
    for (int q = 0; q < 2; ++q) {
        if (tiles[q].size() != want[q].size()) return 6;
        for (size_t i = 0; i < want[q].size(); ++i)
            if (tiles[q][i].msg != want[q][i].msg || tiles[q][i].n_blocks != want[q][i].n_blocks)
                return 7;
    }
    std::printf("%zu requests refused, the same order\n", refused);
    return 0;
}
