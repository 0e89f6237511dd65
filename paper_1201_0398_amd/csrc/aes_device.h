// Device-side building blocks shared by the AES kernels: LDS table layout,
// table lookups, and the rounds of the paper's section 2.1 (Eq. (1)).
//
// LDS image (byte addresses; c = lane % 32 is the lane's private copy, so the
// bank of every lookup is fixed by the lane whatever the data):
//    T_t[x], copy c:      (t >> 1) * 65536 + x * 256 + (t & 1) * 128 + 4c   (128 KiB)
//    (InvS[x] | S[x]<<8): 131072 + x * 128 + 4c      (inverse set only, 32 KiB)
// The forward set holds T0..T3, the inverse set Td0..Td3 plus the S-box word.
// One v_perm_b32 forms a T address: byte k of the state word goes to bits
// 8..15 and the lane's per-table base supplies bits 0..7 and 16..23.
#pragma once

#include <hip/hip_runtime.h>

#include "aes_internal.h"

namespace aesgpu {
namespace dev {

constexpr int kWG = 1024;
constexpr uint32_t kFwdWords = 32768;      // replicated T0..T3 (or Td0..Td3)
constexpr uint32_t kInvSWords = 8192;      // replicated InvS
constexpr uint32_t kInvSByte = 4 * kFwdWords;

struct Bases {
    uint32_t t[4];  // byte address of this lane's copy of T_t[0]
    uint32_t invs;  // byte address of this lane's copy of InvS[0]
};

__device__ __forceinline__ Bases lane_bases() {
    const uint32_t c4 = (threadIdx.x & 31u) * 4u;
    return {{c4, c4 + 128u, c4 + 65536u, c4 + 65536u + 128u}, kInvSByte + c4};
}

// a ^ b ^ c in one v_bitop3_b32 (truth table 0x96 is symmetric in its inputs).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ uint32_t lds_at(const uint32_t *lds, uint32_t byte_addr) {
    return *reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(lds) + byte_addr);
}

// T lookup indexed by byte K of `word`, in the table whose lane base is `base`.
template <int K>
__device__ __forceinline__ uint32_t tlook(const uint32_t *lds, uint32_t word, uint32_t base) {
    // v_perm_b32: result bytes {base.b0, word.bK, base.b2, 0}.
    const uint32_t addr = __builtin_amdgcn_perm(word, base, 0x0C020000u | ((4u + K) << 8));
    return lds_at(lds, addr);
}

// InvS lookup indexed by byte K of `word`: InvS in byte 0, S in byte 1.
template <int K>
__device__ __forceinline__ uint32_t islook(const uint32_t *lds, uint32_t word, uint32_t base) {
    const uint32_t x = (word >> (8 * K)) & 0xFFu;
    return lds_at(lds, (x << 7) + base);
}

// Byte 0 of v0, byte 1 of v1, byte 2 of v2 and byte 3 of v3, XORed with k.
// The two halves have disjoint bytes, so OR-ing them is the same as XOR.
__device__ __forceinline__ uint32_t merge4_xor(uint32_t v0, uint32_t v1, uint32_t v2, uint32_t v3,
                                               uint32_t k) {
    const uint32_t lo = __builtin_amdgcn_perm(v1, v0, 0x0C0C0500u);
    const uint32_t hi = __builtin_amdgcn_perm(v3, v2, 0x07020C0Cu);
    return xor3(lo, hi, k);
}

// Byte 0 of each of v0..v3 into bytes 0..3 of the result, XORed with k.
__device__ __forceinline__ uint32_t merge4_low_xor(uint32_t v0, uint32_t v1, uint32_t v2,
                                                   uint32_t v3, uint32_t k) {
    const uint32_t lo = __builtin_amdgcn_perm(v1, v0, 0x0C0C0400u);
    const uint32_t hi = __builtin_amdgcn_perm(v3, v2, 0x04000C0Cu);
    return xor3(lo, hi, k);
}

// Rounds of NB blocks held by a lane.  Every function makes the lookups of block
// j + 1 before it combines those of block j, and all 16 of a block before it
// combines any.  The compiler's scheduler finds such an order by itself only
// where it keeps within its register limits from the start; where it does not,
// it goes back to the order written here, and with each output word's four
// lookups followed by its XORs a wave had only 3 to 5 reads in flight.
template <bool kInv>
__device__ __forceinline__ void mid_lookups(const uint32_t *lds, const Bases &b,
                                            const uint32_t (&s)[4], uint32_t (&v)[4][4]) {
    // One middle round, Eq. (1).  Forward: output word c reads byte k of word
    // (c + k) mod 4.  Inverse (equivalent inverse cipher): word (c - k) mod 4.
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        v[c][0] = tlook<0>(lds, s[c], b.t[0]);
        v[c][1] = tlook<1>(lds, s[(kInv ? c + 3 : c + 1) & 3], b.t[1]);
        v[c][2] = tlook<2>(lds, s[(c + 2) & 3], b.t[2]);
        v[c][3] = tlook<3>(lds, s[(kInv ? c + 1 : c + 3) & 3], b.t[3]);
    }
}

template <bool kInv>
__device__ __forceinline__ void last_lookups(const uint32_t *lds, const Bases &b,
                                             const uint32_t (&s)[4], uint32_t (&v)[4][4]) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        if constexpr (kInv) {
            // InvSubBytes + InvShiftRows.
            v[c][0] = islook<0>(lds, s[c], b.invs);
            v[c][1] = islook<1>(lds, s[(c + 3) & 3], b.invs);
            v[c][2] = islook<2>(lds, s[(c + 2) & 3], b.invs);
            v[c][3] = islook<3>(lds, s[(c + 1) & 3], b.invs);
        } else {
            // SubBytes + ShiftRows.  The S-box byte is taken from the T
            // tables: T2 holds S(x) in byte 0, T3 in byte 1, T0 in byte 2 and
            // T1 in byte 3.
            v[c][0] = tlook<0>(lds, s[c], b.t[2]);
            v[c][1] = tlook<1>(lds, s[(c + 1) & 3], b.t[3]);
            v[c][2] = tlook<2>(lds, s[(c + 2) & 3], b.t[0]);
            v[c][3] = tlook<3>(lds, s[(c + 3) & 3], b.t[1]);
        }
    }
}

// One middle round.
template <bool kInv, int NB>
__device__ __forceinline__ void mid_round(const uint32_t *lds, const Bases &b, uint32_t (&s)[NB][4],
                                          const uint32_t *k) {
    uint32_t v[NB][4][4];
    mid_lookups<kInv>(lds, b, s[0], v[0]);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        if (j + 1 < NB) mid_lookups<kInv>(lds, b, s[(j + 1) % NB], v[(j + 1) % NB]);
#pragma unroll
        for (int c = 0; c < 4; ++c)
            s[j][c] = xor3(xor3(v[j][c][0], v[j][c][1], v[j][c][2]), v[j][c][3], k[c]);
    }
}

// The last round (no MixColumns), with AddRoundKey.
template <bool kInv, int NB>
__device__ __forceinline__ void last_round(const uint32_t *lds, const Bases &b,
                                           uint32_t (&s)[NB][4], const uint32_t *k) {
    uint32_t v[NB][4][4];
    last_lookups<kInv>(lds, b, s[0], v[0]);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        if (j + 1 < NB) last_lookups<kInv>(lds, b, s[(j + 1) % NB], v[(j + 1) % NB]);
#pragma unroll
        for (int c = 0; c < 4; ++c)
            s[j][c] = kInv ? merge4_low_xor(v[j][c][0], v[j][c][1], v[j][c][2], v[j][c][3], k[c])
                           : merge4_xor(v[j][c][0], v[j][c][1], v[j][c][2], v[j][c][3], k[c]);
    }
}

// Copies the table set into the LDS image; tid is the thread's index in the
// workgroup.  Needs blockDim.x == WG.  Each table word is loaded once per
// workgroup and its thread writes all 32 copies, four to a ds_write_b128: at
// step i the lane takes copies 4 * ((i + tid) % 8) .. + 3, so eight
// neighbouring lanes (neighbouring entries, 256 bytes apart) cover all the
// banks and the writes run at the LDS's 128 bytes per clock.  What bounds it
// is then that rate: 128 KiB are 1024 clocks.  With each thread loading every
// one of the 32 words that it wrote, a 4 MiB ECB call took 7.98 us instead of
// 7.58, a 24 MiB CBC decryption 23.6 instead of 23.2.
template <bool kInv, int WG = kWG>
struct TableWords {
    uint32_t v[1024 / WG];
    uint32_t s;   // inverse S-box word
};

template <bool kInv, int WG = kWG>
__device__ __forceinline__ TableWords<kInv, WG> load_tables(const uint32_t *__restrict__ g,
                                                            uint32_t tid) {
    static_assert(1024 % WG == 0 && WG % 256 == 0, "workgroup size");
    const uint32_t *src = g + (kInv ? kTd : kTe);
    TableWords<kInv, WG> w{};
#pragma unroll
    for (int k = 0; k < 1024 / WG; ++k) w.v[k] = src[tid + uint32_t(k) * WG];
    if constexpr (kInv) w.s = g[kInvSS + (tid & 255u)];
    return w;
}

template <bool kInv, int WG>
__device__ __forceinline__ void write_tables(uint32_t *lds, const TableWords<kInv, WG> &w,
                                             uint32_t tid) {
#pragma unroll
    for (int k = 0; k < 1024 / WG; ++k) {
        const uint32_t e = tid + uint32_t(k) * WG, t = e >> 8, x = e & 255u;
        uint32_t *row = lds + (t >> 1) * 16384u + x * 64u + (t & 1u) * 32u;
#pragma unroll
        for (uint32_t i = 0; i < 8; ++i)
            *reinterpret_cast<uint4 *>(row + 4u * ((i + tid) & 7u)) =
                make_uint4(w.v[k], w.v[k], w.v[k], w.v[k]);
    }
    if constexpr (kInv) {
        // The inverse S-box words: WG / 256 threads share an entry's copies.
        constexpr uint32_t kEach = 8 / (WG / 256);
        uint32_t *row = lds + kFwdWords + (tid & 255u) * 32u;
#pragma unroll
        for (uint32_t i = 0; i < kEach; ++i)
            *reinterpret_cast<uint4 *>(row + 4u * (((tid >> 8) * kEach + i + tid) & 7u)) =
                make_uint4(w.s, w.s, w.s, w.s);
    }
    __syncthreads();
}

template <bool kInv, int WG = kWG>
__device__ __forceinline__ void stage_tables(uint32_t *lds, const uint32_t *__restrict__ g) {
    write_tables(lds, load_tables<kInv, WG>(g, threadIdx.x), threadIdx.x);
}

// The next share (or tile) for this wave: lane 0 adds one to the workgroup's count in
// LDS and the old count goes to every lane.  The exec mask is narrowed inside
// the asm block, which also waits for the result, so the tile loop has no
// branch.  The count is kept in the high half of its word (with the inverse
// tables the low half holds an InvS table entry, which the add leaves as it
// is).  Needs all 64 lanes of the wave active.  No memory clobber: the only
// LDS data the add shares a word with is read-only, and with the clobber the
// compiler kept only about five table reads in flight in AES-256 encryption.
__device__ __forceinline__ uint32_t claim_share(uint32_t *count) {
    uint32_t old = 0;
    uint64_t exec_save;
    const uint32_t addr = uint32_t(reinterpret_cast<uintptr_t>(count));   // LDS offset
    asm volatile(
        "s_mov_b64 %1, exec\n\t"
        "s_mov_b64 exec, 1\n\t"
        "ds_add_rtn_u32 %0, %2, %3\n\t"
        "s_waitcnt lgkmcnt(0)\n\t"
        "s_mov_b64 exec, %1\n\t"
        "s_nop 4"
        : "+v"(old), "=&s"(exec_save)
        : "v"(addr), "v"(0x10000u));
    return uint32_t(__builtin_amdgcn_readfirstlane(old)) >> 16;
}

__device__ __forceinline__ uint32_t bswap32(uint32_t v) {
    return __builtin_amdgcn_perm(v, v, 0x00010203u);
}

// Raw buffer accesses.  The hardware checks each offset against the
// resource's range: past it a load reads zero and a store writes nothing.
// Kernels use them for block loads and stores so that no lane needs a branch
// and the compiler can count the outstanding memory operations exactly.
using rsrc_t = __amdgpu_buffer_rsrc_t;
using u32x4 = uint32_t __attribute__((ext_vector_type(4)));
constexpr int kRawBufferWord3 = 0x00020000;   // gfx9 raw buffer, 32-bit data format

__device__ __forceinline__ rsrc_t buffer_rsrc(const void *base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, int(bytes),
                                             kRawBufferWord3);
}

// Their cache policy: kCached (the default) where what is written may be read
// again from the caches; kStreamed (nt) for buffers too large for that;
// kCoherent (sc1, agent-coherent) for a kernel that runs while others produce
// its inputs and use its outputs, and must see and publish them device-wide
// without L2 invalidations or write-backs.
constexpr int kCached = 0;
constexpr int kStreamed = 2;
constexpr int kCoherent = 16;

template <int kPolicy>
__device__ __forceinline__ uint4 buffer_load16(rsrc_t r, uint32_t offset) {
    const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(r, offset, 0, kPolicy);
    return make_uint4(x[0], x[1], x[2], x[3]);
}

template <int kPolicy>
__device__ __forceinline__ void buffer_store16(rsrc_t r, uint32_t offset, const uint4 &v) {
    const u32x4 x = {v.x, v.y, v.z, v.w};
    __builtin_amdgcn_raw_buffer_store_b128(x, r, offset, 0, kPolicy);
}

// Pointers into the constant address space: a load through one with a
// wave-uniform address is a scalar load through the scalar cache.  Only for
// memory that no kernel in flight writes.
template <class T>
__device__ __forceinline__ const T __attribute__((address_space(4))) *as_const(const T *p) {
    return (const T __attribute__((address_space(4))) *)p;
}

}  // namespace dev
}  // namespace aesgpu
