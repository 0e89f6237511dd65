// Plans messages through build_tiles() and compares the order of the tiles with
// a stable comparison sort of the same tiles, longest first.
//   tile_order <messages> <tile_blocks> <longest message, blocks>
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#include "aes_batch.h"
#include "aes_internal.h"
#include "aesgpu.h"

using namespace aesgpu;

int main(int argc, char **argv) {
    if (argc != 4) return 2;
    const size_t m = std::strtoul(argv[1], nullptr, 10);
    const uint32_t tile_blocks = uint32_t(std::strtoul(argv[2], nullptr, 10));
    const uint64_t longest = std::strtoull(argv[3], nullptr, 10);
    std::mt19937_64 rng(m * 31 + tile_blocks);
    std::vector<aesgpu_msg> msgs(m);
    uint64_t at = 0;
    for (auto &x : msgs) {
        std::memset(&x, 0, sizeof x);
        // Whole tiles, single blocks and lengths between.
        const uint64_t pick = rng() % 4;
        const uint64_t blocks = pick == 0 ? 1 : pick == 1 ? longest : 1 + rng() % longest;
        x.in_off = x.out_off = at;
        x.n_bytes = 16 * blocks;
        x.key_bits = 128;
        x.mode = AESGPU_MODE_ECB;
        x.dir = uint32_t(rng() % 2);
        at += x.n_bytes;
    }
    std::vector<DevMsg> dm;
    std::vector<Tile> tiles[2];
    std::vector<uint32_t> cbc_list;
    std::vector<Tile> cbc_groups;
    BatchTotals tot;
    if (build_tiles(msgs.data(), m, tile_blocks, dm, tiles, cbc_list, cbc_groups, tot) != AESGPU_OK)
        return 3;
    for (int set = 0; set < 2; ++set) {
        std::vector<Tile> want;
        for (size_t i = 0; i < m; ++i) {
            if ((msgs[i].dir == AESGPU_DIR_DECRYPT) != (set == 1)) continue;
            const uint64_t n = msgs[i].n_bytes / 16;
            for (uint64_t f = 0; f < n; f += tile_blocks)
                want.push_back(Tile{uint32_t(i), uint32_t(std::min<uint64_t>(tile_blocks, n - f)), f});
        }
        std::stable_sort(want.begin(), want.end(),
                         [](const Tile &a, const Tile &b) { return a.n_blocks > b.n_blocks; });
        if (want.size() != tiles[set].size()) return 4;
        for (size_t i = 0; i < want.size(); ++i) {
            const Tile &a = want[i], &b = tiles[set][i];
            if (a.msg != b.msg || a.n_blocks != b.n_blocks || a.first_block != b.first_block) return 5;
        }
        std::printf("set %d: %zu tiles\n", set, want.size());
    }
    return 0;
}
