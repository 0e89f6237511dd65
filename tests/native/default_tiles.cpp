// The planner's own choice of tile size, on 256 CUs.
#include <cstdio>
#include <cstring>
#include <vector>

#include "aes_batch.h"

using namespace aesgpu;

static void add(std::vector<aesgpu_msg> &v, size_t m, uint64_t n_bytes, int mode, int dir) {
    aesgpu_msg x;
    std::memset(&x, 0, sizeof x);
    x.n_bytes = n_bytes;
    x.key_bits = 128;
    x.mode = uint8_t(mode);
    x.dir = uint8_t(dir);
    v.insert(v.end(), m, x);
}

static uint32_t chosen(const std::vector<aesgpu_msg> &v) {
    return default_tile_blocks(256, v.data(), v.size());
}

static int check(const char *what, uint32_t got, uint32_t want) {
    std::printf("%s: %u\n", what, got);
    return got == want ? 0 : 1;
}

int main() {
    const int enc = AESGPU_DIR_ENCRYPT, dec = AESGPU_DIR_DECRYPT;
    const uint64_t waves = 256 * 16;   // tiles of t blocks for two a wave: 2 * waves * t blocks
    int bad = 0;
    std::vector<aesgpu_msg> v;
    bad += check("no messages", chosen(v), 256);
    // 23 MB in tiles: the same with or without CBC encryption beside it.
    add(v, 256, 90000 / 16 * 16, AESGPU_MODE_ECB, enc);
    bad += check("23 MB of ECB", chosen(v), 256);
    add(v, 10000, 15504, AESGPU_MODE_CBC, enc);
    bad += check("23 MB of ECB, 155 MB of CBC encryption", chosen(v), 256);
    add(v, 60000, 16384, AESGPU_MODE_CBC, enc);
    bad += check("23 MB of ECB, 1.1 GB of CBC encryption", chosen(v), 256);
    // CBC decryption is cut into tiles like the other modes, in either direction of CTR.
    for (int mode : {AESGPU_MODE_ECB, AESGPU_MODE_CTR, AESGPU_MODE_CBC}) {
        v.clear();
        add(v, 2 * waves, 16 * 1024, mode, dec);
        bad += check("two tiles of 1024 blocks a wave", chosen(v), 1024);
    }
    // A partial block is a block of its message's last tile.
    v.clear();
    add(v, 2 * waves, 16 * 1024 - 15, AESGPU_MODE_CTR, enc);
    bad += check("the same of odd length", chosen(v), 1024);
    add(v, 1, 1, AESGPU_MODE_CTR, enc);
    bad += check("and one byte more", chosen(v), 1024);
    add(v, 2 * waves, 1, AESGPU_MODE_CTR, enc);
    bad += check("and single bytes, a block each", chosen(v), 1280);
    v.clear();
    add(v, 65536, uint64_t(1) << 20, AESGPU_MODE_ECB, enc);
    bad += check("64 GiB", chosen(v), 4096);
    v.clear();
    add(v, 3, ~uint64_t(0), AESGPU_MODE_ECB, enc);   // refused later; no overflow here
    bad += check("impossible lengths", chosen(v), 4096);
    return bad;
}
