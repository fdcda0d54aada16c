// shapes.hpp -- index rules that kernels and host code share: plain integer
// arithmetic that a host compiler builds too.
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define OGM_HD __host__ __device__ __forceinline__
#else
#define OGM_HD inline
#endif

namespace ogm {

// f(record, piece) for the items of `kept` records of `pieces` pieces each
// that thread t of T takes, kept and T at most 256.  The pieces go in tiles of
// 2^20, so that an item's number in a tile fits 32 bits however wide the records
// are (one number over all of them passes 2^32 at 256 records of 2^24 pieces).
constexpr uint32_t kPieceTile = 1u << 20;

template <class F>
OGM_HD void record_items(uint32_t kept, uint32_t pieces, uint32_t t, uint32_t T, F f) {
    for (uint64_t p0 = 0; p0 < pieces; p0 += kPieceTile) {
        const uint32_t first = (uint32_t)p0, n = pieces - first < kPieceTile ? pieces - first : kPieceTile;
        for (uint32_t k = t; k < kept * n; k += T) {
            const uint32_t j = k / n;
            f(j, first + (k - j * n));
        }
    }
}

}  // namespace ogm
