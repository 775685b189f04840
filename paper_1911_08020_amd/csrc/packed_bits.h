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
// gfx950, so a load starts at the byte that holds weight j's first bit, or as much earlier
// as it takes to end inside the run (lc words): 4 bytes for up to 4 indices (j a multiple
// of their number: at most 28 bits from bit 0 or 4 of the first byte, or 14 bits from any),
// twice 4 bytes for 8 (they are l whole bytes).  Whole words took two and three loads: the
// INT8 SpMV of 65536 x 9216, 21.5 us -> 20.4.  (One 8-byte load where the run is long
// enough, behind a uniform branch: the compiler waited for each, 31 us.)
typedef uint32_t PackedU32 __attribute__((aligned(1)));

struct Packed4 { uint32_t w; int sh; };
struct Packed8 { uint32_t lo, hi; int sh_lo, sh_hi; };

__device__ __forceinline__ Packed4 packed_load4(const PackedGroup &pg, int64_t j) {
    const int bit = int(j & 31) * pg.l;
    const int last = 4 * pg.lc - 4;
    const int byte = (bit >> 3) < last ? bit >> 3 : last;
    const char *run = reinterpret_cast<const char *>(pg.words) + (j >> 5) * (4 * pg.l);
    return Packed4{*reinterpret_cast<const PackedU32 *>(run + byte), bit - 8 * byte};
}

// Weights 8 v + 8 i, ... where `at` is the byte of weight 8 v (its group's words + v l; runs
// are 4 l bytes of 4 such octets each, so octets follow each other l bytes apart).
__device__ __forceinline__ Packed8 packed_load8(const PackedGroup &pg, const char *at, int v,
                                                int i) {
    const int in_run = ((v + i) & 3) * pg.l;
    const int over = in_run - (4 * pg.lc - 4);           // past the run's last 4 bytes
    const int back_lo = over > 0 ? over : 0;
    const int back_hi = over + 4 > 0 ? over + 4 : 0;
    const char *p = at + i * pg.l;
    return Packed8{*reinterpret_cast<const PackedU32 *>(p - back_lo),
                   *reinterpret_cast<const PackedU32 *>(p + 4 - back_hi), 8 * back_lo,
                   8 * back_hi};
}
__device__ __forceinline__ const char *packed_octet(const PackedGroup &pg, int64_t v) {
    return reinterpret_cast<const char *>(pg.words) + v * pg.l;
}

// Enough bits for 4 indices.
__device__ __forceinline__ uint32_t packed_bits32(const Packed4 &p) { return p.w >> p.sh; }

// Enough bits for 8 indices (the upper half matters for l > 4 only, where it moves by less
// than 32).
__device__ __forceinline__ uint64_t packed_bits64(const Packed8 &p) {
    return (uint64_t(p.hi >> (p.sh_hi & 31)) << 32) | (p.lo >> p.sh_lo);
}

// Index q of a bit string that starts at an index boundary.
template <typename Bits>
__device__ __forceinline__ int packed_field(Bits bits, int q, const PackedGroup &pg) {
    return int(uint32_t(bits >> (q * pg.l)) & pg.mask);
}

}  // namespace darb
