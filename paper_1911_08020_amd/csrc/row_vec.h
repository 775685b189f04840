// 16 bytes of a row at any element address: global loads need no alignment on gfx950, so a
// row that does not start on 16 bytes (an odd N, an offset view) still takes one load
// instruction per vector.
#pragma once

#include <cstdint>

namespace darb {

template <typename Bits> struct RowVec;
template <> struct RowVec<uint32_t> {
    typedef uint32_t T __attribute__((ext_vector_type(4), aligned(4)));
};
template <> struct RowVec<uint16_t> {
    typedef uint32_t T __attribute__((ext_vector_type(4), aligned(2)));
};

}  // namespace darb
