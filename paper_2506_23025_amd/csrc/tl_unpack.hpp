// The pieces of the device unpacker that lie across the end of a row, in plain integer code: the kernel runs it, and a
// host program checks it.
#pragma once
#include <cstdint>

#if defined(__HIPCC__)
#define TL_UNPACK_FN __host__ __device__ __forceinline__
#else
#define TL_UNPACK_FN inline
#endif

namespace tl {

// The 16 two-bit codes of a piece whose first `left` (1 .. 15) are the last ones of a row of K codes, given in the low bits of
// c (the bits above may hold anything).  next(i) gives the 16 codes from the start of the i-th row after it, which may be fewer,
// with anything above them; it is asked for the rows the piece reaches, and for no other.
template <class Next>
TL_UNPACK_FN uint32_t join_rows(uint32_t c, uint32_t left, uint32_t K, Next&& next)
{
    uint32_t bits = 2u * left;
    c = (c & ((1u << bits) - 1u)) | (next(1) << bits);
    const uint32_t row = 2u * (K < 16u ? K : 16u);        // a row's bits, held at a piece's: twice a long row's K does not fit 32 bits
    for (int i = 2; (bits += row) < 32u; ++i) c = (c & ((1u << bits) - 1u)) | (next(i) << bits);
    return c;
}

}  // namespace tl
