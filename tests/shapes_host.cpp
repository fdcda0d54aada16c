// The library's index rules (csrc/shapes.hpp) built by the host compiler, for test_shapes.py.
#include "../paper_2209_03526_amd/csrc/shapes.hpp"

extern "C" {

// Items that thread t of T takes, at most `most` of them counted, and a sum over their numbers.
uint64_t items_of(uint32_t kept, uint32_t pieces, uint32_t t, uint32_t T, uint64_t* sum, uint8_t* seen) {
    uint64_t n = 0;
    *sum = 0;
    ogm::record_items(kept, pieces, t, T, [&](uint32_t j, uint32_t p) {
        n++;
        *sum += (uint64_t)j * pieces + p;
        if (seen) seen[(uint64_t)j * pieces + p]++;
    });
    return n;
}

void xv_offsets(int32_t whole, uint64_t l, uint32_t b, uint32_t len, uint64_t nrows, uint32_t nwords, uint64_t* to) {
    const ogm::XvOffsets at(whole != 0, l, b, len, nrows, nwords);
    to[0] = at.x1;
    to[1] = at.v;
}

// First tiles of n descriptors, and whether each starts a launch.
void number_tiles(uint32_t n, const uint64_t* tiles, uint32_t* first, uint8_t* starts) {
    ogm::LaunchTiles L;
    for (uint32_t i = 0; i < n; i++) {
        starts[i] = i == 0 || !L.fits(tiles[i]);
        first[i] = L.add(tiles[i]);
    }
}

uint32_t copiers(uint32_t blocks, uint64_t nrows, uint32_t rw) { return ogm::compact_copiers(blocks, nrows, rw); }

uint32_t slot_groups(uint64_t ncand, uint32_t lmax, uint32_t M, uint32_t V, uint32_t wx, uint32_t most, uint32_t l, uint32_t nrec) {
    return ogm::sel_chunks(ogm::sel_rule(ncand, lmax, M, V, wx), most, l, nrec);
}

int32_t alone(uint64_t nrows, uint32_t nwords, int32_t fetch) { return ogm::one_workgroup(nrows, nwords, fetch != 0); }

uint64_t waves(uint64_t tiles, uint64_t wgs) { return ogm::tile_waves(tiles, wgs); }

}
