// access.hip -- the paper's graph encoding with k-groups (Alg. 1) and secure
// neighbouring-vertex access (Alg. 6) over it.
//
//   rss_group_k            host: Alg. 1's degree protection (padded lengths)
//   k_place_ids,
//   k_split_records        one-hot posting records in CSR order, split into
//                          binary RSS with the ChaCha12 PRF     (HBM stream)
//   k_csr_select           P_m[l] = XOR_c id_m[c] AND id_{c,l}, for up to eight
//                          matched vertices m at once           (HBM stream, XOR atomics)
//   k_attr_select          d = XOR_x id[x] AND d_x per kept ID  (HBM stream, XOR atomics)
// rss_sec_access chains the selection, the RSS re-share, the shuffle with the
// parity open and compaction (shuffle.hip) and the attribute selection.
//
// Selections: a block takes a run of candidates and a tile of record words on
// consecutive threads (coalesced); the partials of one word meet in LDS and
// one atomicXor per word and share goes to the zeroed output.  XOR is
// order-free, so results do not depend on scheduling.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <numeric>
#include <vector>

#include "../../include/oblivgm_fss.h"
#include "chacha_gfx950.hpp"
#include "common.hpp"
#include "shapes.hpp"

using namespace ogm;

namespace {

constexpr int kSelBlock = 256;

unsigned blocks_for(uint64_t n, unsigned block, uint64_t cap) {
    uint64_t g = (n + block - 1) / block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (unsigned)g;
}

__global__ void k_fill(uint64_t n, uint32_t v, uint32_t* __restrict__ p) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += stride) p[k] = v;
}

// rec_id[off[v] + slot[e]] = adj[e] for the true IDs e of vertex v (a slot
// outside the padded list, or an ID outside [0, x_bits), is skipped).
__global__ void k_place_ids(uint64_t n, uint32_t x_bits, const uint32_t* __restrict__ adj_off,
                            const uint32_t* __restrict__ adj, const uint32_t* __restrict__ slot,
                            const uint32_t* __restrict__ off, uint32_t* __restrict__ rec_id) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
        const uint32_t len = off[v + 1] - off[v];
        for (uint32_t e = adj_off[v]; e < adj_off[v + 1]; e++)
            if (slot[e] < len && adj[e] < x_bits) rec_id[off[v] + slot[e]] = adj[e];
    }
}

// Thread m owns words 4m .. 4m+3 of the record table (row-major), lane m & 3
// of the quad that makes PRF block m / 4 of both split keys; share 1 and 2
// are those PRF words, share 3 the one-hot record ^ both.  VEC: the record
// width is a multiple of four words and the shares are 16-byte aligned, so a
// thread's four words lie in one record (one division, one ID read) and go
// out as one 16-byte store per share.
template <bool VEC>
__global__ __launch_bounds__(256) void k_split_records(uint64_t nwords_total, uint32_t wx,
                                                       const uint32_t* __restrict__ rec_id, ChachaKey ka,
                                                       ChachaKey kb, uint32_t counter, uint32_t* __restrict__ s0,
                                                       uint32_t* __restrict__ s1, uint32_t* __restrict__ s2) {
    const uint64_t m = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint4 fa = chacha_quad(ka, (uint32_t)(m >> 2), counter, 0u, 0u);
    const uint4 fb = chacha_quad(kb, (uint32_t)(m >> 2), counter, 0u, 0u);
    if constexpr (VEC) {
        if (4 * m >= nwords_total) return;
        const uint64_t r = 4 * m / wx;
        const uint32_t w0 = (uint32_t)(4 * m - r * wx), x = rec_id[r];
        const uint32_t d = (x >> 5) - w0, bit = x != 0xFFFFFFFFu && d < 4u ? 1u << (x & 31u) : 0u;
        const uint4 plain = make_uint4(d == 0 ? bit : 0u, d == 1 ? bit : 0u, d == 2 ? bit : 0u, d == 3 ? bit : 0u);
        ((uint4*)s0)[m] = fa;
        ((uint4*)s1)[m] = fb;
        ((uint4*)s2)[m] = make_uint4(plain.x ^ fa.x ^ fb.x, plain.y ^ fa.y ^ fb.y, plain.z ^ fa.z ^ fb.z,
                                     plain.w ^ fa.w ^ fb.w);
    } else {
        const uint32_t a[4] = {fa.x, fa.y, fa.z, fa.w}, b[4] = {fb.x, fb.y, fb.z, fb.w};
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const uint64_t g = 4 * m + q;
            if (g >= nwords_total) break;
            const uint64_t r = g / wx;
            const uint32_t w = (uint32_t)(g - r * wx), x = rec_id[r];
            const uint32_t plain = (x != 0xFFFFFFFFu && (x >> 5) == w) ? 1u << (x & 31u) : 0u;
            s0[g] = a[q];
            s1[g] = b[q];
            s2[g] = plain ^ a[q] ^ b[q];
        }
    }
}

// Three-out-of-three product of one word: x_i r_i ^ x_i r_j ^ x_j r_i, j = i + 1.
__device__ __forceinline__ void rss_product(const uint32_t m[3], const uint32_t r[3], uint32_t acc[3]) {
#pragma unroll
    for (int i = 0; i < 3; i++) {
        const int j = (i + 1) % 3;
        acc[i] ^= (r[i] & m[i]) ^ (r[j] & m[i]) ^ (r[i] & m[j]);
    }
}

// Partials of the threads of a tile (tw words, `lanes` candidate lanes) meet
// in LDS; one atomicXor per word and share.
__device__ __forceinline__ void reduce_out(uint32_t (*part)[kSelBlock], const uint32_t acc[3], uint32_t tw,
                                           uint32_t lanes, uint32_t* const out[3], uint64_t base) {
    const uint32_t t = threadIdx.x;
#pragma unroll
    for (int i = 0; i < 3; i++) part[i][t] = acc[i];
    __syncthreads();
    if (t < tw) {
#pragma unroll
        for (int i = 0; i < 3; i++) {
            uint32_t v = 0;
            for (uint32_t k = 0; k < lanes; k++) v ^= part[i][k * tw + t];
            if (v) atomicXor(&out[i][base + t], v);
        }
    }
    __syncthreads();
}

struct Shares3 {
    const uint32_t* p[3];
};
struct Out3 {
    uint32_t* p[3];
};

// Slot l = blockIdx.y of the fetched lists of M calls (call0 = blockIdx.z * M):
// XOR over this block's candidates c with l < len_c of id_m[c] AND record
// (off_c + l), into out[.][call * lmax * wx + l * wx + w].  First the block
// lists in LDS the candidates whose (public, padded) list reaches slot l, with
// the three mask bits of each call; then its threads stream those records, V
// words per load and two records per step, and add each to the sums of all M
// calls: with the calls one by one the posting lists, the bulk of the bytes,
// were read once per call (8 calls over 30,011 candidates and 1,000-byte
// records: 8 x 52 us, now 105 us).  With t_i = r_i ^ r_j, j = i + 1, a product
// x_i r_i ^ x_i r_j ^ x_j r_i is (t_i & x_i) ^ (r_i & x_j): two three-input
// operations a word.  The threads' sums meet in LDS by XOR atomics, then go to
// the zeroed output by 8-byte XOR atomics, 3 M wx / 2 a block.  Those bound a
// grid of many blocks (86, 171 and 341 blocks a slot, 4-byte atomics: 109, 182
// and 323 us), so each slot takes only as many as its lists want (sel_chunks):
// blocks beyond leave at once, so what they evaluate of the rule is kept short
// (in 64-bit integers from two loads it cost 8 of 166 us).  With 1 / (l + 1) of
// slot 0's blocks in slot l, whatever the lists, a secAccess over 3,000 lists of 24
// records of 94 words took 83 us and eight took 161, now 54 and 76.
constexpr int kSelThreads = 512;
constexpr uint32_t kSelCand = 1024;       // candidates listed at a time
static_assert(kSelMost == 2 * kSelCand, "a block lists its candidates in two steps at most");
constexpr uint32_t kSelTile = 256;        // record words per pass
// Records of up to so many words are loaded word by word by a single call, whose
// threads then meet in more words of the LDS sums.  Words against 16 bytes: 20,000
// skewed lists over 100 IDs (4 words) 38 / 70 us, over 1,200 (38) 45 / 48, over 4,000
// (125) 59.1 / 60.6.
constexpr uint32_t kSelNarrow = 128;

struct IdmSet {
    const uint32_t* p[kSideCalls][3];
};

template <int V>
__device__ __forceinline__ void load_words(uint32_t (&r)[V], const uint32_t* __restrict__ p, uint32_t left) {
    if (left >= V) {
        __builtin_memcpy(r, p, 4 * V);
    } else {
#pragma unroll
        for (uint32_t q = 0; q < V; q++) r[q] = q < left ? p[q] : 0u;
    }
}

template <int M, int V>
__device__ __forceinline__ void sel_add(uint32_t (&acc)[M][3][V], const uint32_t (&r)[3][V], uint32_t bits) {
    uint32_t t[3][V];
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int q = 0; q < V; q++) t[i][q] = r[i][q] ^ r[(i + 1) % 3][q];
#pragma unroll
    for (int m = 0; m < M; m++) {
        uint32_t x[3];
#pragma unroll
        for (int i = 0; i < 3; i++) x[i] = (uint32_t)__builtin_amdgcn_sbfe((int)bits, 3 * m + i, 1);
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int q = 0; q < V; q++) {
                const uint32_t a = __builtin_amdgcn_bitop3_b32(acc[m][i][q], t[i][q], x[i], 0x78);   // a ^ (b & c)
                acc[m][i][q] = __builtin_amdgcn_bitop3_b32(a, r[i][q], x[(i + 1) % 3], 0x78);
            }
    }
}

template <int M, int V>
__global__ __launch_bounds__(kSelThreads) void k_csr_select(uint64_t ncand, uint32_t wx, uint32_t ncalls, uint64_t tw,
                                                            SelRule rule, IdmSet idm, const uint32_t* __restrict__ off,
                                                            Shares3 post, Out3 out) {
    __shared__ uint32_t rec[kSelCand];
    __shared__ uint32_t msk[kSelCand];
    __shared__ uint32_t nsel;
    __shared__ uint32_t sum[M * 3][kSelTile];
    const uint32_t l = blockIdx.y, call0 = blockIdx.z * M;
    const uint32_t nm = min(ncalls - call0, (uint32_t)M);
    const uint32_t t = threadIdx.x;
    const uint64_t chunks = sel_chunks(rule, gridDim.x, l, off[ncand]);
    if (blockIdx.x >= chunks) return;
    const uint64_t per = (ncand + chunks - 1) / chunks;
    const uint64_t c1 = min((blockIdx.x + 1) * per, ncand);
    for (uint64_t c0 = blockIdx.x * per; c0 < c1; c0 += kSelCand) {
        if (t == 0) nsel = 0;
        __syncthreads();
        const uint64_t ce = min(c0 + kSelCand, c1);
        for (uint64_t c = c0 + t; c < ce; c += kSelThreads) {
            const uint32_t o = off[c];
            if (l >= off[c + 1] - o) continue;              // the list ends before slot l
            uint32_t bits = 0;
#pragma unroll
            for (int m = 0; m < M; m++)
                if ((uint32_t)m < nm)
#pragma unroll
                    for (int i = 0; i < 3; i++)
                        bits |= ((idm.p[call0 + m][i][c >> 5] >> (c & 31)) & 1u) << (3 * m + i);
            const uint32_t k = atomicAdd(&nsel, 1u);         // order-free: the products are XORed
            rec[k] = o + l;
            msk[k] = bits;
        }
        __syncthreads();
        const uint32_t n = nsel;
        for (uint32_t w0 = 0; n && w0 < wx; w0 += kSelTile) {
            const uint32_t words = min(wx - w0, kSelTile);
            const uint32_t nv = (words + V - 1) / V;         // loads per record
            const uint32_t lanes = kSelThreads / nv;
            const uint32_t v = t % nv, g = t / nv;
            const uint32_t left = words - v * V;
            for (uint32_t k = t; k < M * 3 * kSelTile; k += kSelThreads) (&sum[0][0])[k] = 0u;
            __syncthreads();
            if (g < lanes) {
                uint32_t acc[M][3][V] = {};
                const uint32_t* src[3];
#pragma unroll
                for (int i = 0; i < 3; i++) src[i] = post.p[i] + w0 + v * V;
                uint32_t k = g;
                for (; k + lanes < n; k += 2 * lanes) {
                    const uint64_t a = (uint64_t)rec[k] * wx, b = (uint64_t)rec[k + lanes] * wx;
                    uint32_t ra[3][V], rb[3][V];
#pragma unroll
                    for (int i = 0; i < 3; i++) {
                        load_words<V>(ra[i], src[i] + a, left);
                        load_words<V>(rb[i], src[i] + b, left);
                    }
                    sel_add<M, V>(acc, ra, msk[k]);
                    sel_add<M, V>(acc, rb, msk[k + lanes]);
                }
                if (k < n) {
                    uint32_t ra[3][V];
#pragma unroll
                    for (int i = 0; i < 3; i++) load_words<V>(ra[i], src[i] + (uint64_t)rec[k] * wx, left);
                    sel_add<M, V>(acc, ra, msk[k]);
                }
#pragma unroll
                for (int m = 0; m < M; m++)
#pragma unroll
                    for (int i = 0; i < 3; i++)
#pragma unroll
                        for (int q = 0; q < V; q++)
                            if (v * V + q < words) atomicXor(&sum[3 * m + i][v * V + q], acc[m][i][q]);
            }
            __syncthreads();
            // pairs of words at multiples of 8 bytes, with the odd word at either end on its own
            const uint32_t items = words / 2 + 1;
            for (uint32_t k = t; k < 3 * nm * items; k += kSelThreads) {
                const uint32_t mi = k / items, m = mi / 3;
                uint32_t* to = out.p[mi - 3 * m] + (call0 + m) * tw + (uint64_t)l * wx + w0;
                const uint32_t odd = ((uintptr_t)to >> 2) & 1u;
                const int w = 2 * (int)(k - mi * items) - (int)odd;     // -1: word 0 alone
                const uint32_t lo = w >= 0 && w < (int)words ? sum[mi][w] : 0u;
                const uint32_t hi = w + 1 < (int)words ? sum[mi][w + 1] : 0u;
                if (w >= 0 && w + 1 < (int)words)
                    atomicXor((unsigned long long*)(to + w), (unsigned long long)lo | ((unsigned long long)hi << 32));
                else if (w >= 0 && w < (int)words)
                    atomicXor(to + w, lo);
                else if (w + 1 < (int)words)
                    atomicXor(to + w + 1, hi);
            }
            __syncthreads();
        }
        __syncthreads();                                     // the list is free again
    }
}

// Kept ID k = blockIdx.y of call blockIdx.z (exits when k >= its count): XOR
// over this block's attribute rows x < x_bits of bit x of the kept record AND
// row x.
__global__ __launch_bounds__(kSelBlock) void k_attr_select(uint32_t x_bits, uint32_t wx, uint32_t wd,
                                                           const uint32_t* __restrict__ count, Shares3 ids,
                                                           Shares3 attr, Out3 out) {
    __shared__ uint32_t part[3][kSelBlock];
    if (blockIdx.y >= count[blockIdx.z]) return;                  // uniform over the block
    const uint64_t k = (uint64_t)blockIdx.z * gridDim.y + blockIdx.y;
    const uint32_t* id[3] = {ids.p[0] + k * wx, ids.p[1] + k * wx, ids.p[2] + k * wx};
    const uint64_t per = ((uint64_t)x_bits + gridDim.x - 1) / gridDim.x;
    const uint64_t x0 = (uint64_t)blockIdx.x * per;
    const uint64_t x1 = x0 + per < x_bits ? x0 + per : x_bits;
    const uint32_t t = threadIdx.x;
    for (uint32_t w0 = 0; w0 < wd; w0 += kSelBlock) {
        const uint32_t tw = wd - w0 < kSelBlock ? wd - w0 : kSelBlock;
        const uint32_t lanes = kSelBlock / tw;
        const uint32_t w = t % tw, g = t / tw;
        uint32_t acc[3] = {0, 0, 0};
        if (g < lanes) {
            for (uint64_t x = x0 + g; x < x1; x += lanes) {
                uint32_t m[3], r[3];
#pragma unroll
                for (int i = 0; i < 3; i++) {
                    m[i] = 0u - ((id[i][x >> 5] >> (x & 31)) & 1u);
                    r[i] = attr.p[i][x * wd + w0 + w];
                }
                rss_product(m, r, acc);
            }
        }
        reduce_out(part, acc, tw, lanes, out.p, k * wd + w0);
    }
}

// secEval, the re-share and secFetch's table {x || id || d} of several groups of
// candidates in one launch (blockIdx.x = group, blockIdx.y = a block of its
// rows): a wave takes a row, its lanes the record's words.  Group c's rows are
// rows src[c] .. of the one-hot records and rows row0[c] .. row0[c + 1] of the
// table.  Server s's share of a row's bit is the parity of (ea_s & d_s) ^
// (eb_s & d_{s+1}); the row's bit of the group's zero sharing (bit r % 32 of
// word r / 32 of F(k_i, counter) ^ F(k_{i-1}, counter)) makes it RSS.  Small
// groups are launch-bound: five launches each for 196 groups of 1 to 40 rows.
constexpr uint32_t kGroupRows = 16;       // rows per block of four waves
constexpr uint32_t kGroupMost = 1024;     // rows of a group, at most (32 words of bits)

struct GroupTable {
    ChachaKey prf[3];
    const uint32_t* eval[6];        // ea_1, eb_1, ea_2, eb_2, ea_3, eb_3
    const uint32_t* ids[3];
    const uint32_t* vals[3];
    uint32_t* out[3];
    uint32_t wi, wv;
    uint32_t src[kSideCalls];
    uint32_t row0[kSideCalls + 1];
    uint32_t counter[kSideCalls];
};

__global__ __launch_bounds__(256) void k_group_table(GroupTable A) {
    __shared__ uint32_t f[3][32];
    const uint32_t call = blockIdx.x, t = threadIdx.x, lane = t & 63u;
    const uint32_t row0 = A.row0[call], n = A.row0[call + 1] - row0;
    if (blockIdx.y * kGroupRows >= n) return;            // the whole block leaves
    if (t < 64) {                                        // six PRF blocks: two of each key
        const uint32_t q = t >> 2, k = q % 3, blk = q / 3;
        const uint4 o = chacha_quad(A.prf[k], blk, A.counter[call], 0u, 0u);
        if (q < 6) {
            uint32_t* to = &f[k][16 * blk + 4 * (t & 3u)];
            to[0] = o.x, to[1] = o.y, to[2] = o.z, to[3] = o.w;
        }
    }
    __syncthreads();
    const uint32_t W = 1 + A.wi + A.wv;
    for (uint32_t j = t >> 6; j < kGroupRows; j += 4) {
        const uint32_t r = blockIdx.y * kGroupRows + j;
        if (r >= n) break;                               // whole waves
        const uint64_t from = (uint64_t)A.src[call] + r, to = (uint64_t)(row0 + r) * W;
        uint32_t acc[3] = {0u, 0u, 0u};
        for (uint32_t w = lane; w < A.wv; w += 64) {
            uint32_t d[3];
#pragma unroll
            for (int i = 0; i < 3; i++) {
                d[i] = A.vals[i][from * A.wv + w];
                A.out[i][to + 1 + A.wi + w] = d[i];
            }
#pragma unroll
            for (int i = 0; i < 3; i++) acc[i] ^= (A.eval[2 * i][w] & d[i]) ^ (A.eval[2 * i + 1][w] & d[(i + 1) % 3]);
        }
        for (uint32_t w = lane; w < A.wi; w += 64)
#pragma unroll
            for (int i = 0; i < 3; i++) A.out[i][to + 1 + w] = A.ids[i][from * A.wi + w];
#pragma unroll
        for (int i = 0; i < 3; i++) {
            const uint64_t odd = __ballot(__builtin_popcount(acc[i]) & 1);
            const uint32_t z = (f[i][r >> 5] ^ f[(i + 2) % 3][r >> 5]) >> (r & 31u);
            if (lane == 0) A.out[i][to] = ((uint32_t)__builtin_popcountll(odd) ^ z) & 1u;
        }
    }
}

struct Carve {
    uint8_t* base;
    uint64_t size, used = 0;
    bool ok = true;
    uint32_t* take(uint64_t words) {
        const uint64_t bytes = (words * 4 + 255) & ~255ull;
        if (used + bytes > size) {
            ok = false;
            return nullptr;
        }
        uint32_t* p = (uint32_t*)(base + used);
        used += bytes;
        return p;
    }
};

uint64_t rnd(uint64_t words) { return (words * 4 + 255) & ~255ull; }

}  // namespace

extern "C" {

int rss_group_k_lists(uint64_t n, uint32_t nlists, const uint32_t* lengths, const uint32_t* types, uint32_t k,
                      uint32_t* padded, uint32_t* group) {
    last_error().clear();
    if (n == 0) return FSS_OK;
    if (!lengths || !types || !padded) return fail(FSS_EINVAL, "rss_group_k: NULL argument");
    if (k == 0) return fail(FSS_EINVAL, "rss_group_k: k must be at least 1");
    if (nlists == 0) return fail(FSS_EINVAL, "rss_group_k: no list types");
    auto len = [&](uint32_t l, uint64_t v) { return lengths[(uint64_t)l * n + v]; };
    std::vector<uint64_t> order(n);
    std::iota(order.begin(), order.end(), 0);
    // by type, then the vector of list lengths (list type 0 first), then vertex ID
    std::sort(order.begin(), order.end(), [&](uint64_t a, uint64_t b) {
        if (types[a] != types[b]) return types[a] < types[b];
        for (uint32_t l = 0; l < nlists; l++)
            if (len(l, a) != len(l, b)) return len(l, a) < len(l, b);
        return a < b;
    });
    uint32_t gid = 0;
    for (uint64_t s = 0; s < n;) {
        uint64_t e = s;
        while (e < n && types[order[e]] == types[order[s]]) e++;     // [s, e): one type
        const uint64_t m = e - s;
        const uint64_t ngroups = m / k > 0 ? m / k : 1;
        for (uint64_t g = 0; g < ngroups; g++) {
            const uint64_t lo = s + g * k, hi = g + 1 < ngroups ? lo + k : e;   // the last takes the rest
            for (uint32_t l = 0; l < nlists; l++) {
                uint32_t mx = 0;
                for (uint64_t i = lo; i < hi; i++) mx = std::max(mx, len(l, order[i]));
                for (uint64_t i = lo; i < hi; i++) padded[(uint64_t)l * n + order[i]] = mx;
            }
            if (group)
                for (uint64_t i = lo; i < hi; i++) group[order[i]] = gid;
            gid++;
        }
        s = e;
    }
    return FSS_OK;
}

int rss_group_k(uint64_t n, const uint32_t* lengths, const uint32_t* types, uint32_t k, uint32_t* padded,
                uint32_t* group) {
    return rss_group_k_lists(n, 1, lengths, types, k, padded, group);
}

int rss_enc_posting_lists(uint64_t n, uint32_t x_bits, const uint32_t* d_adj_off, const uint32_t* d_adj,
                          const uint32_t* d_slot, const uint32_t* d_off, uint64_t nrec, const uint64_t split_keys[2],
                          uint32_t counter, uint32_t* const d_out[3], void* d_work, uint64_t work_bytes,
                          void* stream) {
    last_error().clear();
    if (x_bits == 0) return fail(FSS_EINVAL, "rss_enc_posting_lists: x_bits is 0");
    if (n == 0 || nrec == 0) return FSS_OK;
    if (!d_adj_off || !d_adj || !d_slot || !d_off || !split_keys || !d_out || !d_out[0] || !d_out[1] || !d_out[2])
        return fail(FSS_EINVAL, "rss_enc_posting_lists: NULL argument");
    const uint32_t wx = (x_bits + 31) / 32;
    if (nrec > 0xFFFFFFFFull || nrec * wx / 16 > 0xFFFFFFFFull)
        return fail(FSS_EUNSUPPORTED, "rss_enc_posting_lists: table too large");
    if (!d_work || work_bytes < nrec * 4)
        return fail(FSS_ENOMEM, "rss_enc_posting_lists: workspace needs %llu bytes", (unsigned long long)(nrec * 4));
    hipStream_t s = (hipStream_t)stream;
    uint32_t* rec_id = (uint32_t*)d_work;
    hipLaunchKernelGGL(k_fill, dim3(blocks_for(nrec, 256, 4096)), dim3(256), 0, s, nrec, 0xFFFFFFFFu, rec_id);
    hipLaunchKernelGGL(k_place_ids, dim3(blocks_for(n, 256, 4096)), dim3(256), 0, s, n, x_bits, d_adj_off, d_adj,
                       d_slot, d_off, rec_id);
    const uint64_t total = nrec * wx, quads = (total + 3) / 4;
    const bool vec = wx % 4 == 0 && ((uintptr_t)d_out[0] | (uintptr_t)d_out[1] | (uintptr_t)d_out[2]) % 16 == 0;
    const ChachaKey ka = chacha_key(split_keys[0], 5), kb = chacha_key(split_keys[1], 5);
    if (vec)
        hipLaunchKernelGGL(k_split_records<true>, dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, s, total, wx,
                           rec_id, ka, kb, counter, d_out[0], d_out[1], d_out[2]);
    else
        hipLaunchKernelGGL(k_split_records<false>, dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, s, total, wx,
                           rec_id, ka, kb, counter, d_out[0], d_out[1], d_out[2]);
    return check_launch("rss_enc_posting_lists");
}

uint64_t rss_sec_access_workspace_bytes(uint32_t lmax, uint32_t x_bits, uint32_t attr_words) {
    const uint64_t wx = (x_bits + 31) / 32, l = lmax ? lmax : 1;
    return 6 * rnd(l * wx) + 3 * rnd(l * attr_words) + rss_fetch_many_workspace_bytes(l, (uint32_t)wx) + 256;
}

// Whether one workgroup shuffles a group of n rows of W words.
static bool group_fits(uint32_t n, uint32_t W) { return n <= kGroupMost && small_shuffle_fits(n, W); }

uint64_t rss_sec_fetch_groups_workspace_bytes(uint32_t ngroups, const uint32_t* n, uint32_t npos, uint32_t id_words) {
    const uint32_t W = 1 + id_words + (npos + 31) / 32;
    uint64_t most = 0;
    for (uint32_t c = 0; n && c < ngroups;) {
        if (!group_fits(n[c], W)) {
            most = std::max(most, 6 * rnd((n[c] + 31) / 32) + 3 * rnd((uint64_t)n[c] * W) +
                                      rss_fetch_many_workspace_bytes(n[c], W));
            c++;
            continue;
        }
        uint64_t rows = 0;
        for (uint32_t m = 0; m < kSideCalls && c < ngroups && group_fits(n[c], W); m++) rows += n[c++];
        most = std::max(most, 8 * rnd(rows * W));       // the tables, their shuffle's two and three
    }
    return most + 256;
}

int rss_sec_fetch_groups(uint32_t ngroups, const uint32_t* src, const uint32_t* n, uint32_t npos,
                         const uint32_t* const d_eval[6], uint32_t id_words, const uint32_t* const d_ids[3],
                         const uint32_t* const d_vals[3], const uint64_t prf_keys[3], uint32_t counter,
                         const uint64_t* seeds, uint32_t* const d_out[3], uint32_t* d_rows_out, uint32_t* d_count,
                         void* d_work, uint64_t work_bytes, void* stream) {
    last_error().clear();
    const char* who = "rss_sec_fetch_groups";
    if (ngroups == 0) return FSS_OK;
    if (npos == 0) return fail(FSS_EINVAL, "%s: no positions", who);
    if (!src || !n || !d_eval || !d_vals || (id_words && !d_ids) || !prf_keys || !seeds || !d_out || !d_rows_out ||
        !d_count)
        return fail(FSS_EINVAL, "%s: NULL argument", who);
    const uint32_t wv = (npos + 31) / 32;
    for (int i = 0; i < 6; i++)
        if (!d_eval[i]) return fail(FSS_EINVAL, "%s: NULL evaluation %d", who, i);
    for (int i = 0; i < 3; i++)
        if (!d_vals[i] || (id_words && !d_ids[i]) || !d_out[i]) return fail(FSS_EINVAL, "%s: NULL share %d", who, i);
    if ((uint64_t)id_words + wv + 1 > 65535)
        return fail(FSS_EUNSUPPORTED, "%s: more than 65535 words per record", who);
    const uint32_t W = 1 + id_words + wv;
    uint64_t all = 0;
    for (uint32_t c = 0; c < ngroups; c++) all += n[c];
    if (all > 0x7FFFFFFFull) return fail(FSS_EUNSUPPORTED, "%s: more than 2^31 rows", who);
    if (!d_work || work_bytes < rss_sec_fetch_groups_workspace_bytes(ngroups, n, npos, id_words))
        return fail(FSS_ENOMEM, "%s: workspace needs %llu bytes", who,
                    (unsigned long long)rss_sec_fetch_groups_workspace_bytes(ngroups, n, npos, id_words));
    hipStream_t s = (hipStream_t)stream;
    // runs of consecutive groups that one workgroup each can shuffle go together
    uint64_t row = 0;
    for (uint32_t c0 = 0; c0 < ngroups;) {
        Carve ws{(uint8_t*)d_work, work_bytes};
        uint32_t* out[3] = {d_out[0] + row * (W - 1), d_out[1] + row * (W - 1), d_out[2] + row * (W - 1)};
        if (group_fits(n[c0], W)) {
            GroupTable A{};
            uint32_t m = 0, most = 0;
            for (; m < kSideCalls && c0 + m < ngroups && group_fits(n[c0 + m], W); m++) {
                A.src[m] = src[c0 + m];
                A.row0[m + 1] = A.row0[m] + n[c0 + m];
                A.counter[m] = counter + c0 + m;
                most = std::max(most, n[c0 + m]);
            }
            const uint64_t tw = (uint64_t)A.row0[m] * W;
            uint32_t* table[3] = {ws.take(tw), ws.take(tw), ws.take(tw)};
            uint32_t* xv = ws.take(2 * tw);
            uint32_t* sh[3] = {ws.take(tw), ws.take(tw), ws.take(tw)};
            if (!ws.ok) return fail(FSS_ENOMEM, "%s: workspace too small", who);
            for (int i = 0; i < 3; i++) {
                A.prf[i] = chacha_key(prf_keys[i], 5);
                A.ids[i] = id_words ? d_ids[i] : nullptr;
                A.vals[i] = d_vals[i];
                A.out[i] = table[i];
            }
            for (int i = 0; i < 6; i++) A.eval[i] = d_eval[i];
            A.wi = id_words, A.wv = wv;
            if (most) {
                hipLaunchKernelGGL(k_group_table, dim3(m, (most + kGroupRows - 1) / kGroupRows), dim3(256), 0, s, A);
                if (const int rc = check_launch("k_group_table")) return rc;
            }
            const uint32_t* g[3] = {table[0], table[1], table[2]};
            const int rc = small_shuffles(m, A.row0, W, g, seeds + 3 * (uint64_t)c0, xv, sh, 1u, out, d_rows_out + row,
                                          d_count + c0, stream);
            if (rc) return rc;
            row += A.row0[m];
            c0 += m;
            continue;
        }
        // a larger group, step by step
        const uint64_t rows = n[c0], bw = (rows + 31) / 32;
        uint32_t* x3[3] = {ws.take(bw), ws.take(bw), ws.take(bw)};
        uint32_t* z3[3] = {ws.take(bw), ws.take(bw), ws.take(bw)};
        uint32_t* table[3] = {ws.take(rows * W), ws.take(rows * W), ws.take(rows * W)};
        const uint64_t fws = rss_fetch_many_workspace_bytes(rows, W);
        uint32_t* fwork = ws.take((fws + 3) / 4);
        if (!ws.ok) return fail(FSS_ENOMEM, "%s: workspace too small", who);
        const uint32_t *ids[3], *vals[3];
        for (int i = 0; i < 3; i++) {
            ids[i] = id_words ? d_ids[i] + (uint64_t)src[c0] * id_words : nullptr;
            vals[i] = d_vals[i] + (uint64_t)src[c0] * wv;
        }
        for (int i = 0; i < 3; i++) {
            const int rc = rss_sec_eval_records(rows, npos, d_eval[2 * i], d_eval[2 * i + 1], vals[i], vals[(i + 1) % 3],
                                                x3[i], stream);
            if (rc) return rc;
        }
        const uint32_t* xc[3] = {x3[0], x3[1], x3[2]};
        int rc = rss_reshare(rows, xc, prf_keys, counter + c0, z3, stream);
        const uint32_t* zc[3] = {z3[0], z3[1], z3[2]};
        if (!rc) rc = rss_fetch_table(rows, zc, id_words, ids, wv, vals, table, stream);
        const uint32_t* tc[3] = {table[0], table[1], table[2]};
        if (!rc)
            rc = rss_fetch_many(rows, W, tc, seeds + 3 * (uint64_t)c0, out, d_rows_out + row, d_count + c0, fwork, fws,
                                stream);
        if (rc) return rc;
        row += rows;
        c0++;
    }
    return FSS_OK;
}

// Whether `words` words from p on meet the `n` words from `from` on.
static bool meets(const uint32_t* p, uint64_t words, const uint32_t* from, uint64_t n) {
    return (uintptr_t)p < (uintptr_t)(from + n) && (uintptr_t)from < (uintptr_t)(p + words);
}

// The calls of a secAccess batch, as many side by side as the workspace holds
// single calls (each step one launch for all of them), the rest after them.  A
// call that reads an output of one before it (a matched ID that is a kept one)
// starts a new group: side by side the selections of all run first.
static int sec_access_calls(uint32_t count, uint64_t ncand, uint32_t x_bits, const uint32_t* const* d_idm,
                            const uint32_t* d_off, uint32_t lmax, const uint32_t* const* d_post, uint32_t attr_words,
                            const uint32_t* const* d_attr, const uint64_t* prf_keys, const uint32_t* counters,
                            const uint64_t* seeds, uint32_t* const* d_ids, uint32_t* const* d_attrs,
                            uint32_t* d_rows_out, uint32_t* d_count, void* d_work, uint64_t work_bytes, void* stream,
                            const char* who) {
    if (x_bits == 0 || attr_words == 0) return fail(FSS_EINVAL, "%s: empty IDs or attribute records", who);
    if (lmax == 0 || lmax > 65535) return fail(FSS_EINVAL, "%s: lmax %u outside 1..65535", who, lmax);
    if (!d_off || !d_post || !d_attr || !prf_keys) return fail(FSS_EINVAL, "%s: NULL argument", who);
    for (int i = 0; i < 3; i++)
        if (!d_post[i] || !d_attr[i]) return fail(FSS_EINVAL, "%s: NULL share %d", who, i);
    if (ncand > 0xFFFFFFFFull) return fail(FSS_EUNSUPPORTED, "%s: more than 2^32 candidates", who);
    const uint32_t wx = (x_bits + 31) / 32, wd = attr_words;
    const uint64_t single = rss_sec_access_workspace_bytes(lmax, x_bits, wd);
    if (!d_work || work_bytes < single)
        return fail(FSS_ENOMEM, "%s: workspace needs %llu bytes", who, (unsigned long long)single);
    hipStream_t s = (hipStream_t)stream;
    const uint64_t tw = (uint64_t)lmax * wx, ta = (uint64_t)lmax * wd;
    if (std::max(tw, ta) > 1ull << 36)      // the re-shares' PRF block numbers are 32-bit: 16 words a block
        return fail(FSS_EUNSUPPORTED, "%s: more than 2^36 words of fetched records", who);
    // side by side: tables that one workgroup shuffles
    const bool small = small_shuffle_fits(lmax, wx);
    const uint32_t most = small ? (uint32_t)std::min<uint64_t>(std::min<uint64_t>(count, kSideCalls), work_bytes / single)
                                : 1u;
    uint32_t row0[kSideCalls + 1];         // most is at most kSideCalls
    for (uint32_t c = 0; c <= most; c++) row0[c] = c * lmax;
    const uint64_t mw = (ncand + 31) / 32;             // words of a matched ID's share
    for (uint32_t c0 = 0, n; c0 < count; c0 += n) {
        auto reads_earlier = [&](uint32_t c) {          // an output of the calls c0 .. c - 1
            const uint64_t k = c - c0;
            for (int j = 0; j < 3; j++) {
                const uint32_t* p = d_idm[3 * (uint64_t)c + j];
                for (int i = 0; i < 3; i++)
                    if (meets(p, mw, d_ids[i] + c0 * tw, k * tw) || meets(p, mw, d_attrs[i] + c0 * ta, k * ta)) return true;
                if (meets(p, mw, d_rows_out + (uint64_t)c0 * lmax, k * lmax) || meets(p, mw, d_count + c0, k)) return true;
            }
            return false;
        };
        for (n = 1; n < most && c0 + n < count && !reads_earlier(c0 + n);) n++;
        Carve ws{(uint8_t*)d_work, work_bytes};
        uint32_t* zeroed = ws.take(3 * n * (tw + ta));
        uint32_t* add[3] = {zeroed, zeroed + n * tw, zeroed + 2 * n * tw};
        uint32_t* att[3];
        for (int i = 0; i < 3; i++) att[i] = zeroed + 3 * n * tw + i * n * ta;
        uint32_t* rss[3] = {ws.take(n * tw), ws.take(n * tw), ws.take(n * tw)};
        if (!ws.ok) return fail(FSS_ENOMEM, "%s: workspace too small", who);
        uint32_t *ids[3], *attrs[3];
        for (int i = 0; i < 3; i++) {
            ids[i] = d_ids[i] + c0 * tw;
            attrs[i] = d_attrs[i] + c0 * ta;
        }
        // 1. P_m[l] = XOR_c id_m[c] AND id_{c,l}: additive shares
        hipLaunchKernelGGL(k_fill, dim3(blocks_for(3 * n * (tw + ta), 256, 4096)), dim3(256), 0, s, 3 * n * (tw + ta), 0u,
                           zeroed);
        if (ncand) {
            IdmSet idm{};
            for (uint32_t c = 0; c < n; c++)
                for (int i = 0; i < 3; i++) idm.p[c][i] = d_idm[3 * (uint64_t)(c0 + c) + i];
            // blocks of slot 0, the most of any slot: enough to fill the chip over lmax slots
            const uint64_t chunks = std::max((ncand + kSelMost - 1) / kSelMost,
                                             std::min<uint64_t>((ncand + 63) / 64, 4096 / lmax + 1));
            const uint32_t m = n > 4 ? 8 : n > 1 ? 4 : 1;      // calls per pass over the lists
            const dim3 grid((unsigned)chunks, lmax, (n + m - 1) / m);
            const Shares3 post{{d_post[0], d_post[1], d_post[2]}};
            const Out3 o{{add[0], add[1], add[2]}};
            const uint32_t v = m == 8 ? 2 : m == 1 && wx <= kSelNarrow ? 1 : 4;      // words a load
            auto k = m == 8 ? k_csr_select<8, 2> : m == 4 ? k_csr_select<4, 4> : v == 1 ? k_csr_select<1, 1> : k_csr_select<1, 4>;
            hipLaunchKernelGGL(k, grid, dim3(kSelThreads), 0, s, ncand, wx, n, tw, sel_rule(ncand, lmax, m, v, wx), idm,
                               d_off, post, o);
        }
        int rc = check_launch("k_csr_select");
        if (rc) return rc;
        // ... re-shared into RSS
        const uint32_t* a3[3] = {add[0], add[1], add[2]};
        rc = reshare_calls(n, tw, a3, prf_keys, counters + c0, 0, rss, stream);
        if (rc) return rc;
        // 2. shuffle, open the parity of each record, keep the valid IDs
        const uint32_t* r3[3] = {rss[0], rss[1], rss[2]};
        if (small) {
            uint32_t* sh[3] = {ws.take(n * tw), ws.take(n * tw), ws.take(n * tw)};
            uint32_t* xv = ws.take(2 * n * tw);
            if (!ws.ok) return fail(FSS_ENOMEM, "%s: workspace too small", who);
            rc = small_shuffles(n, row0, wx, r3, seeds + 3 * (uint64_t)c0, xv, sh, 2u, ids,
                                d_rows_out + (uint64_t)c0 * lmax, d_count + c0, stream);
        } else {
            const uint64_t cws = rss_fetch_many_workspace_bytes(lmax, wx);
            uint32_t* cwork = ws.take((cws + 3) / 4);
            if (!ws.ok) return fail(FSS_ENOMEM, "%s: workspace too small", who);
            rc = rss_compact_valid(lmax, wx, r3, seeds + 3 * (uint64_t)c0, ids, d_rows_out + (uint64_t)c0 * lmax,
                                   d_count + c0, cwork, cws, stream);
        }
        if (rc) return rc;
        // 3. the attribute record of every kept ID, then one re-share of them all
        const uint64_t xchunks = std::max<uint64_t>(1, std::min<uint64_t>((x_bits + 255) / 256, 2048 / lmax + 1));
        hipLaunchKernelGGL(k_attr_select, dim3((unsigned)xchunks, lmax, n), dim3(kSelBlock), 0, s, x_bits, wx, wd,
                           d_count + c0, Shares3{{ids[0], ids[1], ids[2]}}, Shares3{{d_attr[0], d_attr[1], d_attr[2]}},
                           Out3{{att[0], att[1], att[2]}});
        rc = check_launch("k_attr_select");
        if (rc) return rc;
        const uint32_t* t3[3] = {att[0], att[1], att[2]};
        rc = reshare_calls(n, ta, t3, prf_keys, counters + c0, 1, attrs, stream);
        if (rc) return rc;
    }
    return FSS_OK;
}

int rss_sec_access(uint64_t ncand, uint32_t x_bits, const uint32_t* const d_idm[3], const uint32_t* d_off,
                   uint32_t lmax, const uint32_t* const d_post[3], uint32_t attr_words,
                   const uint32_t* const d_attr[3], const uint64_t prf_keys[3], uint32_t counter,
                   const uint64_t seeds[3], uint32_t* const d_ids[3], uint32_t* const d_attrs[3],
                   uint32_t* d_rows_out, uint32_t* d_count, void* d_work, uint64_t work_bytes, void* stream) {
    last_error().clear();
    const char* who = "rss_sec_access";
    if (!d_idm || !seeds || !d_ids || !d_attrs || !d_rows_out || !d_count)
        return fail(FSS_EINVAL, "%s: NULL argument", who);
    for (int i = 0; i < 3; i++)
        if (!d_idm[i] || !d_ids[i] || !d_attrs[i]) return fail(FSS_EINVAL, "%s: NULL share %d", who, i);
    return sec_access_calls(1, ncand, x_bits, d_idm, d_off, lmax, d_post, attr_words, d_attr, prf_keys, &counter, seeds,
                            d_ids, d_attrs, d_rows_out, d_count, d_work, work_bytes, stream, who);
}

int rss_sec_access_batch(uint32_t count, uint64_t ncand, uint32_t x_bits, const uint32_t* const* d_idm,
                         const uint32_t* d_off, uint32_t lmax, const uint32_t* const d_post[3], uint32_t attr_words,
                         const uint32_t* const d_attr[3], const uint64_t prf_keys[3], const uint32_t* counters,
                         const uint64_t* seeds, uint32_t* const d_ids[3], uint32_t* const d_attrs[3],
                         uint32_t* d_rows_out, uint32_t* d_count, void* d_work, uint64_t work_bytes, void* stream) {
    last_error().clear();
    const char* who = "rss_sec_access_batch";
    if (count == 0) return FSS_OK;
    if (!d_idm || !counters || !seeds || !d_ids || !d_attrs || !d_rows_out || !d_count)
        return fail(FSS_EINVAL, "%s: NULL argument", who);
    for (uint64_t k = 0; k < 3ull * count; k++)
        if (!d_idm[k]) return fail(FSS_EINVAL, "%s: NULL matched-ID share %llu", who, (unsigned long long)k);
    for (int i = 0; i < 3; i++)
        if (!d_ids[i] || !d_attrs[i]) return fail(FSS_EINVAL, "%s: NULL output share %d", who, i);
    return sec_access_calls(count, ncand, x_bits, d_idm, d_off, lmax, d_post, attr_words, d_attr, prf_keys, counters,
                            seeds, d_ids, d_attrs, d_rows_out, d_count, d_work, work_bytes, stream, who);
}

}  // extern "C"
