// shapes.hpp -- index rules that kernels and host code share: plain integer
// arithmetic that a host compiler builds too.
#pragma once

#include <math.h>
#include <stdint.h>

#ifdef __HIPCC__
#define OGM_HD __host__ __device__ __forceinline__
#else
#define OGM_HD inline
#endif

namespace ogm {

// f(record, piece) for the items of `kept` records of `pieces` pieces each
// that thread t of T takes, kept at most 256 and T at most 2^31.  The pieces go in
// tiles of 2^20, so that an item's number in a tile fits 32 bits however wide the
// records are (one number over all of them passes 2^32 at 256 records of 2^24
// pieces).
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

// Workgroups that share the copying of a compaction's blocks of rows (`blocks` of
// them, at most 256 rows at a time), records of rw words: as many as fill the
// chip while each thread has kCopyItems pieces (16 bytes, or a word of ragged
// records) to move.  Records of a one-hot ID are as wide as the table has rows
// / 32, so a table of few blocks may hold megabytes: with one workgroup a block,
// secFetch of 2,000 records of 500 words, all kept, took 254 us, of 70 of 2,000
// words 245; 46 and 23 now (1,024 or 2,048 workgroups, 4 or 8 pieces: the same;
// 100,003 of 21 words 64 us either way).
constexpr uint32_t kCopyGroups = 1024, kCopyItems = 4;

OGM_HD uint32_t compact_copiers(uint32_t blocks, uint64_t nrows, uint32_t rw) {
    const uint64_t pieces = rw & 3u ? rw : rw >> 2, rows = nrows < 256 ? nrows : 256;
    const uint64_t most = (rows * pieces + 256 * kCopyItems - 1) / (256 * kCopyItems);
    const uint64_t want = (kCopyGroups + blocks - 1) / blocks;
    const uint64_t y = want < most ? want : most;
    return y ? (uint32_t)y : 1u;
}

// Whether a single shuffle runs in one workgroup, where its one launch beats the
// three that rank and mask over the chip: up to kAloneRows rows, and up to 128 of
// at most 256 slices in all (one pass of a workgroup's quads), or 320 with the open
// and the compaction behind it (one launch against six).  One workgroup against
// the launches, microseconds, shuffle and (fetch): records of 64 bytes, 64 rows
// 9.0 / 14.9 (12.1 / 22.1), 128 rows 11.6 / 14.9 (16.1 / 22.3), 160 rows 15.1 / 14.7
// (20.0 / 22.3), 300 rows 28 / 15 (35 / 22); 96 rows of 33 words 17.5 / 15.4 (21.8 /
// 22.9), 96 of 64 18.6 / 15.3 (23.7 / 22.6).
constexpr uint32_t kAloneRows = 64;

OGM_HD bool one_workgroup(uint64_t nrows, uint32_t nwords, bool fetch) {
    return nrows <= kAloneRows || (nrows <= 128 && nrows * (((uint64_t)nwords + 15) / 16) <= (fetch ? 320 : 256));
}

// Where slice b of row l lies in the two tables that a shuffle's final round
// gathers (word offsets of its X1 and V words, len of each): interleaved slice by
// slice where `whole`, one after the other otherwise.  16 * b is a word of a
// record and fits 32 bits; 32 * b does not from 2^31 words a record on, so the
// doubling is in 64.
struct XvOffsets {
    uint64_t x1, v;
    OGM_HD XvOffsets(bool whole, uint64_t l, uint32_t b, uint32_t len, uint64_t nrows, uint32_t nwords)
        : x1((l * nwords + 16 * b) << (whole ? 1 : 0)), v(whole ? x1 + len : x1 + nrows * nwords) {}
};

// How a secAccess selection over ncand posting lists splits the lists among the
// workgroups of each slot l < lmax, given nrec, the lists' records in all, which
// only the device has.
//
// How many lists reach slot l is taken to be ncand (l + 1)^-b, with the b that
// gives nrec in all: b = 0 for lists of one length; 1 where nrec is ncand times
// the sum h of 1 / (l + 1); between and beyond, on the line through both in ln nrec.
//
// A workgroup adds its sums to the output by 3 M wx / 2 atomics (M calls, records
// of wx words), after adding its threads' partial sums (V words each) in LDS, where
// 64 V / wx lanes meet in a word.  The two cost as much as streaming about 8 M and
// 1000 M V^2 / wx^2 records, so a workgroup is given several times that, or 1 /
// kSelLarge of the records where that is more; but no more than 1 / kSelFill of
// them, which fills the chip, nor more than kSelMost candidates.
// Measured, whole calls: eight over 30,011 skewed lists of 1,000-byte records, 24 M,
// 32 M, 48 M and 64 M records a workgroup, 173, 172, 164 and 166 us; eight over 3,000
// lists of 24 records of 94 words, 1 / 512, 1 / 640 and 1 / 768 of the records, 80,
// 79 and 79 us, over 20,000 lists of 16 of 4 words 79, 91 and 94; one over 20,000
// lists of 16 of 47 words, 1 / 1024, 1 / 2048 and 1 / 4096, 75, 77 and 91 us, over
// 30,011 lists of 24 of 32 words 82, 78 and 75.
constexpr uint32_t kSelMost = 2048, kSelFill = 512, kSelLarge = 2048;

struct SelRule {
    float ncand, lmax;      // base-2 logarithms
    float slope;            // b / log2(lmax / mean length)
    float records;          // a workgroup's records, for the cost of its end
    uint32_t least;         // workgroups a slot, at least
};

inline SelRule sel_rule(uint64_t ncand, uint32_t lmax, uint32_t M, uint32_t V, uint32_t wx) {
    const double n = (double)ncand, L = (double)lmax, h = log(L) + 0.5772 + 0.5 / L;
    return SelRule{(float)log2(n), (float)log2(L), lmax > 1 ? (float)(1.0 / log2(L / h)) : 0.0f,
                   (float)(48.0 * M + 4000.0 * M * V * V / ((double)wx * wx)),
                   (uint32_t)((ncand + kSelMost - 1) / kSelMost)};
}

OGM_HD uint32_t sel_chunks(const SelRule& r, uint32_t most, uint32_t l, uint32_t nrec) {
    const float n = (float)(nrec ? nrec : 1u), fill = n * (1.0f / kSelFill) + 1.0f;
    const float shorter = r.lmax + r.ncand - log2f(n);                      // log2(lmax / mean length)
    const float lists = exp2f(r.ncand - (shorter > 0.0f ? shorter : 0.0f) * r.slope * log2f((float)(l + 1)));
    const float large = n * (1.0f / kSelLarge), some = large > r.records ? large : r.records;
    const float want = lists / (fill < some ? fill : some) + 1.0f;
    const uint32_t c = want < (float)most ? (uint32_t)want : most;
    return c > r.least ? c : r.least;
}

// Waves of a workgroup in a launch of `tiles` wave tiles, `wgs` workgroups at a
// time: as few as spread the tiles over the chip, but at least four, because the
// workgroup fills 64 KiB of tables first.  One wave alone takes 3 us for it, so
// the shortest walks (64 rows, 8-bit domains) took 7.7 us where workgroups of 16
// waves had taken 6.3; with four waves 4.9 (eight: 4.5, but six launches of a small
// query in turn 121 us instead of 120).
OGM_HD uint64_t tile_waves(uint64_t tiles, uint64_t wgs) {
    const uint64_t w = (tiles + wgs - 1) / wgs;
    return w < 4 ? 4 : w > 16 ? 16 : w;
}

// Numbers the tiles of a batch's descriptors.  A launch numbers its tiles with 32
// bits, so a batch of more (2^32 tiles are 2^37 rows of ranges) takes several
// launches: a descriptor whose tiles no longer fit starts the next one.
constexpr uint64_t kLaunchTiles = 0xFFFFFFF0ull;

struct LaunchTiles {
    uint64_t total = 0;      // of the launch so far
    OGM_HD bool fits(uint64_t tiles) const { return total + tiles <= kLaunchTiles; }
    // first tile of the next descriptor in its launch
    OGM_HD uint32_t add(uint64_t tiles) {
        if (!fits(tiles)) total = 0;
        const uint32_t first = (uint32_t)total;
        total += tiles;
        return first;
    }
};

}  // namespace ogm
