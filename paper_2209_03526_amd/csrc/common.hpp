// common.hpp -- host-side helpers shared by the library's translation units.
#pragma once

#include <stdint.h>

#include <string>

#include "aes_gfx950.hpp"

namespace ogm {

std::string& last_error();                                            // thread-local message
int fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
int check_launch(const char* what);                                   // FSS_EDEVICE on a launch error
RoundKeys seed_key(uint64_t seed);   // AES-128 schedule of LE64(seed) || "OBLIVGM1"
int shuffle_release();               // the shuffle's own streams (shuffle.hip), for fss_shutdown

// Calls side by side in one launch (a call's numbers ride in the kernel's
// arguments, so at most kSideCalls per launch; these functions launch again
// for the rest).
constexpr uint32_t kSideCalls = 64;

// The re-share of rss_reshare (fss_lib.hip) for `calls` tables of nwords whole
// words each, call c at word c * nwords of x and z and under counters[c] + add;
// x may be z.
int reshare_calls(uint32_t calls, uint64_t nwords, const uint32_t* const x[3], const uint64_t prf_keys[3],
                  const uint32_t* counters, uint32_t add, uint32_t* const z[3], void* stream);

// Shuffles of small tables (shuffle.hip), a workgroup each: call c is rows
// row0[c] .. row0[c + 1] (host array) of g under seeds[3 c .. 3 c + 2], its
// shares to the same rows of out.  compact: 0, or 1 (secFetch's open) or 2 (the
// secAccess filter's), and then the kept records of call c go to kept from row
// row0[c] on, their positions to rows_out + row0[c], their number to count[c].
// xv: 2 * nwords words a row.
bool small_shuffle_fits(uint64_t nrows, uint32_t nwords);
int small_shuffles(uint32_t calls, const uint32_t* row0, uint32_t nwords, const uint32_t* const g[3],
                   const uint64_t* seeds, uint32_t* xv, uint32_t* const out[3], uint32_t compact,
                   uint32_t* const kept[3], uint32_t* rows_out, uint32_t* count, void* stream);

}  // namespace ogm
