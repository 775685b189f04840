// Device-side readers of the bit-packed offsets, shared by the products and the
// unpack kernel.
//
// Section 4.2 stores the position of a block's kept weight in log2 b bits.  The
// packed form used here: inside one block-size group (log2 b = l) the retained
// weights are numbered j = 0, 1, ... in storage order and cut into runs of 32;
// run j / 32 is l consecutive 32-bit words, and weight j's index is bits
// (j % 32) * l ... (j % 32) * l + l - 1 of its run read as one little-endian bit
// string.  Groups follow each other in ascending block size; a group with l = 0
// (b = 1: every index is 0) has no words.  A run never straddles a group, so any
// slice of consecutive weights that starts at a multiple of 4, 8 or 16 inside
// its group lies inside one run.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace darb {

// The packed offsets of one group.  `words` must be a readable device address
// even for l = 0 (the readers then load one word and mask it to nothing).
struct PackedGroup {
    const uint32_t *words;   // the group's first word
    int l;                   // log2 b
    int lc;                  // max(l, 1): words a run spans, for index clamping
    uint32_t mask;           // (1 << l) - 1
};

__device__ __forceinline__ PackedGroup packed_group(const uint32_t *words, int64_t first_word,
                                                    int l) {
    return PackedGroup{words + first_word, l, l > 0 ? l : 1, (1u << l) - 1u};
}

// The indices of weights j, j + 1, ... as loaded.  Global loads need no alignment on
// gfx950, so a load starts at any byte, and none leaves its run (lc words): 4 bytes for up
// to 4 indices (j a multiple of their number: at most 28 bits from bit 0 or 4 of the first
// byte, or 14 bits from any), from the byte that holds weight j's first bit or as much
// earlier as it takes to end inside the run; two loads of 4 bytes for 8 indices (an octet:
// l whole bytes), its first 4 and, where it is longer, its last 4.  Every index of an octet
// lies wholly in one of the two.  What a load starts earlier follows from l and the octet's
// place in its run, so nothing is kept for it.  SpMV of 65536 rows, 4 to 6 % kept, us, with
// whole words (two or three loads), with the two loads and their shifts kept, which spilled
// at 6 and 8 vectors per lane, and so:
//   fp16 values, 9216 columns, x fp32 / fp16     20.2 / 22.9   22.2 / 25.2   18.8 / 22.3
//   fp16 values, x fp32, 8192 columns            40.0          42.8          34.0
//   fp32, 9216 columns, 2304 weights a row       57.2          38.5          38.2
//   INT8 codes, x fp32, 9216 / 8192 columns      18.1 / 25.2   17.6 / 31.5   17.7 / 26.2
typedef uint32_t PackedU32 __attribute__((aligned(1)));

struct Packed4 { uint32_t w; int sh; };
struct Packed8 { uint32_t lo, hi; };

__device__ __forceinline__ Packed4 packed_load4(const PackedGroup &pg, int64_t j) {
    const int bit = int(j & 31) * pg.l;
    const int last = 4 * pg.lc - 4;
    const int byte = (bit >> 3) < last ? bit >> 3 : last;
    const char *run = reinterpret_cast<const char *>(pg.words) + (j >> 5) * (4 * pg.l);
    return Packed4{*reinterpret_cast<const PackedU32 *>(run + byte), bit - 8 * byte};
}

// Bytes by which the first load of an octet starts before it: octet `oct` of a run of 4 l
// bytes starts at l oct, a load at 4 l - 4 or earlier.  0 from l = 4 on.
__device__ __forceinline__ constexpr int packed_back(int l, int oct) {
    const int over = l > 0 ? oct * l - (4 * l - 4) : 0;
    return over > 0 ? over : 0;
}

// The octet of weights 8 (v + i), ... where `at` is the byte of weight 8 v (its group's
// words + v l; runs are 4 octets each, so octets follow each other l bytes apart).
__device__ __forceinline__ Packed8 packed_load8(const PackedGroup &pg, const char *at, int v,
                                                int i) {
    const char *p = at + i * pg.l - packed_back(pg.l, (v + i) & 3);
    return Packed8{*reinterpret_cast<const PackedU32 *>(p),
                   *reinterpret_cast<const PackedU32 *>(p + (pg.l > 4 ? pg.l - 4 : 0))};
}
__device__ __forceinline__ const char *packed_octet(const PackedGroup &pg, int64_t v) {
    return reinterpret_cast<const char *>(pg.words) + v * pg.l;
}

// Enough bits for 4 indices.
__device__ __forceinline__ uint32_t packed_bits32(const Packed4 &p) { return p.w >> p.sh; }

// An octet's 8 indices as one bit string, and index q of it for a block size fixed at
// compile time (lo already starts at the octet).
__device__ __forceinline__ uint64_t packed_bits64(const Packed8 &p, const PackedGroup &pg, int oct) {
    const uint32_t lo = p.lo >> (8 * packed_back(pg.l, oct));
    return pg.l > 4 ? lo | (uint64_t(p.hi) << (8 * (pg.l - 4))) : lo;
}
template <int LB> __device__ __forceinline__ int packed_field_c(const Packed8 &p, int q) {
    if ((q + 1) * LB <= 32) return int((p.lo >> (q * LB)) & ((1u << LB) - 1u));
    return int((p.hi >> ((q * LB - 8 * (LB - 4)) & 31)) & ((1u << LB) - 1u));
}

// Index q of a bit string that starts at an index boundary.
template <typename Bits>
__device__ __forceinline__ int packed_field(Bits bits, int q, const PackedGroup &pg) {
    return int(uint32_t(bits >> (q * pg.l)) & pg.mask);
}

}  // namespace darb
