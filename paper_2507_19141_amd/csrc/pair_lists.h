// Pair lists: how the tiled table scatter finds the updates of each tile.
//
// A query updates 16 corner rows of a level, taken as 8 x-pairs (same y, z, t; lower and
// upper x).  A pre-pass sorts the pairs of each chunk of queries by tile (a counting sort
// in LDS) and writes one 16-bit entry per pair: the query's number in its chunk, the pair
// and, where a query has two corner sets (Eq. 11), which of them.  A tile workgroup then
// reads exactly its own pairs, one per lane, in query order, so that neighbouring lanes'
// loads of positions and gradients share cache lines.
//
// A chunk's entries fill at most one region of kListEntries (a level's only chunk's is as short
// as its queries allow); chunk c of list level l starts at entry list_entry[l] + c
// kListEntries, and heads[list_head[l] + list * chunks + c] holds the first
// entry and the count of the list's run in it (one list per tile, but see dense).
//
// Tiles of a list level (make_tile_map):
//  - hashed, tight: 2^tile_shift consecutive rows.  pi_1 = 1 and T a power of two keep the
//    two rows of a pair within 2 N_s rows of each other, inside one tile.
//  - dense: the level's x-lines (runs of N_s + 1 rows, same y, z, t) are dealt to
//    2^tile_shift tiles in turn, line h P + k of P lines going to tile k + 11 h mod P, so
//    that queries crowded into a few cells (every query at one timestamp, a clustered
//    cloud) still spread over all tiles.  A pair lies in one line, hence in one tile.  A
//    level of more than kListTiles tiles has kListTiles lists, each for 2^share_shift
//    neighbouring tiles, which walk it and add the rows of their own lines.
//  - loose (hashed, T no power of two or 2 N_s above the tile's rows): consecutive rows,
//    but a pair may straddle two tiles.  Such a pair has an entry in both, and the
//    scatter adds the rows that lie in its own tile.
#pragma once

#include "h4d_device.h"

namespace h4d {

constexpr uint32_t kListQMask = 2047;  // bits 0..10: query in its chunk
constexpr int kListPShift = 11;        // bits 11..13: pair
constexpr int kListKShift = 14;        // bits 14..15: kind (corner sets, see tile_pre_lists)

// Tile of x-line `line` of a dense list level with 2^b tiles; its inverse: the line in slot
// h of tile t; and the line's list where 2^share tiles have one (line_tile >> share).  Each
// round of 2^b lines is dealt 11 tiles further on, so that lines 2^b apart (the next z or t)
// lie in different tiles: one timestamp's step 375 us, 380 without, 379 and 374 with 1 and 5;
// random times and the batched plan within 2 % for all of them.
__device__ __forceinline__ uint32_t line_tile(uint32_t line, int b) { return (line + 11u * (line >> b)) & ((1u << b) - 1u); }
__device__ __forceinline__ uint32_t tile_line(uint32_t h, uint32_t t, int b) {
    return (h << b) + ((t - 11u * h) & ((1u << b) - 1u));
}
__device__ __forceinline__ uint32_t line_list(uint32_t line, int b, int share) {
    return __builtin_amdgcn_ubfe(line + 11u * (line >> b), (uint32_t)share, (uint32_t)(b - share));
}

__device__ __forceinline__ uint32_t cell_line(const Cell& c, uint32_t S, uint32_t p) {
    return ((uint32_t)c.iy + (p & 1u)) + S * (((uint32_t)c.iz + ((p >> 1) & 1u)) + S * ((uint32_t)c.it + ((p >> 2) & 1u)));
}

// Lists of the 8 pairs (one byte each, pairs 0-3 in t[0]); tight and dense levels.
__device__ __forceinline__ void pair_tiles(const DevGrid& g, const TileMap& tm, int l, const Cell& c, uint32_t (&t)[2]) {
    uint32_t b[8];
    const int sh = tm.tile_shift[l];
    if ((g.dense_bits >> l) & 1u) {
        const uint32_t S = (uint32_t)g.res_s[l] + 1u;
        const uint32_t line = cell_line(c, S, 0u);
        const int share = tm.share_shift[l];
#pragma unroll
        for (int p = 0; p < 8; ++p) b[p] = line_list(line + (p & 1) + ((p >> 1) & 1) * S + (p >> 2) * S * S, sh, share);
    } else {  // the x term lies below the tile's row bits
        const uint32_t hy0 = (uint32_t)c.iy * g.prime[1], hy1 = hy0 + g.prime[1];
        const uint32_t hz0 = (uint32_t)c.iz * g.prime[2], hz1 = hz0 + g.prime[2];
        const uint32_t ht0 = (uint32_t)c.it * g.prime[3], ht1 = ht0 + g.prime[3];
#pragma unroll
        for (int p = 0; p < 8; ++p)
            b[p] = ((((p & 1) ? hy1 : hy0) ^ ((p & 2) ? hz1 : hz0) ^ ((p & 4) ? ht1 : ht0)) & g.tmask) >> sh;
    }
    t[0] = b[0] | (b[1] << 8) | (b[2] << 16) | (b[3] << 24);
    t[1] = b[4] | (b[5] << 8) | (b[6] << 16) | (b[7] << 24);
}

// The same of the lower and of the upper corners; loose levels.  Returns the pairs
// (a bit each) whose corners lie in different tiles.
__device__ __forceinline__ uint32_t corner_tiles(const DevGrid& g, const TileMap& tm, int l, const Cell& c,
                                                 uint32_t (&lo)[2], uint32_t (&hi)[2]) {
    uint32_t row[16];
    level_rows(g, l, c, row);
    const int sh = tm.tile_shift[l];
    const uint32_t off = g.off[l];
    lo[0] = lo[1] = hi[0] = hi[1] = 0u;
    uint32_t apart = 0u;
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        const uint32_t a = (row[2 * p] - off) >> sh, b = (row[2 * p + 1] - off) >> sh;
        lo[p >> 2] |= a << (8 * (p & 3));
        hi[p >> 2] |= b << (8 * (p & 3));
        apart |= (uint32_t)(a != b) << p;
    }
    return apart;
}

__device__ __forceinline__ int level_lists(const TileMap& tm, int l) {
    return (tm.tile_start[l + 1] - tm.tile_start[l]) >> tm.share_shift[l];
}

// ---- the pre-pass: one workgroup sorts one chunk of one level ----
// Bound by its LDS atomics (one per entry, about 15 clocks a wavefront) and the passes over
// the chunk in LDS: 34 us for 200k queries at 16 levels, 58 us with two corner sets.
// 1024 threads at eight wavefronts per SIMD (64 registers) with one corner set per query
// (512 threads: 36 us); two sets need more registers, where 512 threads are faster (58
// against 79 us).
constexpr int pre_block(bool pair) { return pair ? 512 : 1024; }
constexpr int pre_waves_per_eu(bool pair) { return pair ? 4 : 8; }

template <bool PAIR>
struct PreShared {
    static constexpr int kPreWaves = pre_block(PAIR) / 64;
    union {
        uint8_t tiles[kListEntries];     // tile of every entry, query by query
        uint16_t sorted[kListEntries];
    };
    uint8_t valid[kListEntries / 8];     // per query and set of 8: which entries exist
    uint32_t cnt[kPreWaves * kListTiles];
    uint32_t wsum[kPreWaves];
};

// x + eps, rounded in FP32.
__device__ __forceinline__ float4 perturbed(float4 x, float4 e) {
    return make_float4(__fadd_rn(x.x, e.x), __fadd_rn(x.y, e.y), __fadd_rn(x.z, e.z), __fadd_rn(x.w, e.w));
}

// Entries are numbered query by query (8 per query and corner set).  One lane per query
// finds its entries' tiles and stores them as bytes; then one lane per entry counts it:
// every wavefront counts its own consecutive queries (cnt[wavefront][tile]), 8 queries to
// an instruction, and the LDS atomic that counts an entry also gives its rank.  So inside
// a tile's run the entries stay in query order, and the scatter's neighbouring lanes load
// positions and gradients from the same 128-byte lines: a gather costs a clock per line
// that neighbouring lanes do not share (entries of 64 queries pair by pair: 4.75e7 L1
// accesses in the scatter of 200k queries; in query order 3.25e7).
// PAIR: pos(q, x, xp) gives two positions; both in one cell give one entry per pair (kind
// 2: both weights at the same two rows), else 8 entries of kind 0 (x) and 8 of kind 1
// (xp).  Without PAIR every entry is of kind 0.
template <bool PAIR, bool LOOSE, typename Pos>
__device__ __forceinline__ void tile_pre_lists(const DevGrid& g, const TileMap& tm, int l, int chunk, int n, Pos pos,
                                               uint16_t* __restrict__ region, uint32_t* __restrict__ heads,
                                               int nchunks, PreShared<PAIR>& sh) {
    constexpr int kPreBlock = pre_block(PAIR), kPreWaves = kPreBlock / 64;
    constexpr int kSets = (PAIR ? 2 : 1) * (LOOSE ? 2 : 1);
    constexpr int kChunk = 1 << list_chunk_log(PAIR, LOOSE), kWaveQueries = kChunk / kPreWaves;
    constexpr int kPer = kWaveQueries / 64;  // queries per thread, 64 apart
    static_assert(kPer >= 1 && kChunk * 8 * kSets == kListEntries, "a chunk's entries fill its region");
    constexpr int kWaveEntries = kListEntries / kPreWaves, kEach = kWaveEntries / 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int P = level_lists(tm, l);
    const int q0 = chunk << list_chunk_log(PAIR, LOOSE);
    for (int i = threadIdx.x; i < kPreWaves * P; i += kPreBlock) sh.cnt[i] = 0u;
    float4 xs[kPer], xp[kPer];  // every load in flight before the first use
#pragma unroll
    for (int i = 0; i < kPer; ++i) pos(min(q0 + wave * kWaveQueries + i * 64 + lane, n - 1), xs[i], xp[i]);
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int ql = wave * kWaveQueries + i * 64 + lane;
        uint32_t t[kSets][2], v[kSets];
        const uint32_t all = q0 + ql < n ? 0xffu : 0u;
        const Cell c0 = level_cell(g, l, xs[i]);
        v[0] = all;
        if constexpr (LOOSE) v[1] = all & corner_tiles(g, tm, l, c0, t[0], t[1]);
        else pair_tiles(g, tm, l, c0, t[0]);
        if constexpr (PAIR) {
            constexpr int k = kSets / 2;
            const Cell c1 = level_cell(g, l, xp[i]);
            const bool same = c0.ix == c1.ix && c0.iy == c1.iy && c0.iz == c1.iz && c0.it == c1.it;
            v[k] = same ? 0u : all;
            if constexpr (LOOSE) v[k + 1] = v[k] & corner_tiles(g, tm, l, c1, t[k], t[k + 1]);
            else pair_tiles(g, tm, l, c1, t[k]);
        }
#pragma unroll
        for (int k = 0; k < kSets; ++k) {
            *reinterpret_cast<uint2*>(&sh.tiles[(ql * kSets + k) * 8]) = make_uint2(t[k][0], t[k][1]);
            if constexpr (kSets > 1) sh.valid[ql * kSets + k] = (uint8_t)v[k];
        }
    }
    __syncthreads();
    uint32_t* mine = sh.cnt + wave * P;
    uint32_t key[kEach];  // tile << 16 | rank; a wavefront has at most 2^11 entries
    auto count = [&](int j) {
        const int k = wave * kWaveEntries + j * 64 + lane;
        const uint32_t t = sh.tiles[k];
        key[j] = (t << 16) | atomicAdd(&mine[t], 1u);
    };
    if (kSets == 1 && q0 + kChunk <= n) {  // every entry exists
#pragma unroll
        for (int j = 0; j < kEach; ++j) count(j);
    } else {
#pragma unroll
        for (int j = 0; j < kEach; ++j) {
            const int k = wave * kWaveEntries + j * 64 + lane;
            key[j] = ~0u;
            if (kSets > 1 ? (sh.valid[k >> 3] >> (k & 7)) & 1u : q0 + (k >> 3) < n) count(j);
        }
    }
    __syncthreads();
    // exclusive scan of the counts, tile by tile and wavefront by wavefront inside a tile
    constexpr int kPerThread = kPreWaves * kListTiles / kPreBlock;
    uint32_t v[kPerThread], sum = 0u;
    const int per = (kPreWaves * P + kPreBlock - 1) / kPreBlock;
    auto counter = [&](int k) -> uint32_t& {
        const int i = (int)threadIdx.x * per + k;
        return sh.cnt[(i % kPreWaves) * P + i / kPreWaves];
    };
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
        v[k] = k < per && (int)threadIdx.x * per + k < kPreWaves * P ? counter(k) : 0u;
        sum += v[k];
    }
    uint32_t incl = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t a = __shfl_up(incl, d);
        if (lane >= d) incl += a;
    }
    if (lane == 63) sh.wsum[wave] = incl;
    __syncthreads();
    uint32_t run = incl - sum, total = 0u;
#pragma unroll
    for (int w = 0; w < kPreWaves; ++w) {
        if (w < wave) run += sh.wsum[w];
        total += sh.wsum[w];
    }
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
        if (k < per && (int)threadIdx.x * per + k < kPreWaves * P) counter(k) = run;
        run += v[k];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kEach; ++j) {
        if (key[j] == ~0u) continue;
        const uint32_t k = (uint32_t)(wave * kWaveEntries + j * 64 + lane);
        const uint32_t ql = k / (8 * kSets), set = (k >> 3) % kSets;
        uint32_t kind = 0u;
        if constexpr (PAIR)
            kind = sh.valid[ql * kSets + kSets / 2] == 0 ? 2u : set < kSets / 2 ? 0u : 1u;
        sh.sorted[mine[key[j] >> 16] + (key[j] & 0xffffu)] =
            (uint16_t)(ql | ((k & 7u) << kListPShift) | (kind << kListKShift));
    }
    for (int t = threadIdx.x; t < P; t += kPreBlock) {
        const uint32_t first = sh.cnt[t], next = t + 1 < P ? sh.cnt[t + 1] : total;
        heads[(int64_t)t * nchunks + chunk] = first | ((next - first) << 16);
    }
    __syncthreads();
    uint4* dst = reinterpret_cast<uint4*>(region);
    const uint4* src = reinterpret_cast<const uint4*>(sh.sorted);
    const int quads = ((int)total + 7) / 8;
    for (int i = threadIdx.x; i < quads; i += kPreBlock) dst[i] = src[i];
}

// One workgroup of the pre-pass: chunk `chunk` of level l, its lists or (levels with masks,
// chunks of kMaskChunk queries) its tile masks.  tm's list offsets count chunk0 +
// chunk as the chunk of a longer run (segments of one scene); heads and regions are the
// run's.
template <bool PAIR, typename Pos>
__device__ __forceinline__ void tile_pre(const DevGrid& g, const TileMap& tm, int l, int chunk, int chunk0,
                                         int nchunks, int n, Pos pos, uint32_t* __restrict__ mask,
                                         uint16_t* __restrict__ lists, uint32_t* __restrict__ heads, PreShared<PAIR>& sh) {
    if ((tm.lists >> l) & 1u) {
        uint16_t* region = lists + tm.list_entry[l] + (int64_t)(chunk0 + chunk) * kListEntries;
        uint32_t* h = heads + tm.list_head[l] + chunk0;
        if ((tm.loose >> l) & 1u) tile_pre_lists<PAIR, true>(g, tm, l, chunk, n, pos, region, h, nchunks, sh);
        else tile_pre_lists<PAIR, false>(g, tm, l, chunk, n, pos, region, h, nchunks, sh);
        return;
    }
    uint32_t* lm = mask + (int64_t)__popc(tm.masks & ((1u << l) - 1u)) * mask_stride(n);
    for (int i = 0; i < kMaskChunk / pre_block(PAIR); ++i) {
        const int q = chunk * kMaskChunk + i * pre_block(PAIR) + (int)threadIdx.x;
        if (q >= n) return;
        float4 x, xp;
        pos(q, x, xp);
        uint32_t m = corner_tile_mask(g, tm, l, x);
        if constexpr (PAIR) m |= corner_tile_mask(g, tm, l, xp);
        lm[q] = m;
    }
}

// Chunks of level l's pre-pass over n queries.
__host__ __device__ constexpr int pre_chunk_log(const TileMap& tm, int l, bool pair) {
    return (tm.lists >> l) & 1u ? list_chunk_log(pair, (tm.loose >> l) & 1u) : kMaskChunkLog;
}
__host__ __device__ constexpr int pre_chunks(int n, int log) { return (int)(((int64_t)n + (1 << log) - 1) >> log); }

// ---- one tile of a list level in the scatter ----
// Where a tile's rows lie: rows [first, first + cnt) of the level, or (dense) its lines.
struct TileRows {
    uint32_t tile;        // in the level
    uint32_t first, cnt;  // cnt: rows held in LDS
    bool dense;           // lines dealt in turn
    uint32_t copies;      // copies of the tile in LDS (a power of two), and their distance
    uint32_t stride;      // in values
};

// Copies of a list tile of cnt rows.  Lanes of one wavefront that update the same row
// retry their swaps one after the other, so where queries crowd into few cells a tile
// that leaves LDS free keeps several copies, lane i adding to copy i mod copies.  At most
// 16, no more than fit, and no more rows in all than the tile's expected share of the 8 n
// pairs (clearing and summing the copies would cost more than the retries).  A training step
// in us with at most 1 / 4 / 16 / 64 copies: 4096 queries 47.5 / 46.2 / 42.0 / 41.3, 200k 469 /
// 428 / 433 / 432, one timestamp 427 / 373 / 375 / 373.
template <typename G, int F>
__device__ __forceinline__ void set_copies(TileRows& r, int tiles, int64_t n) {
    r.stride = r.cnt * F + 2u;  // a row's copies lie in different banks
    const int64_t share = n * 8 / tiles;
    r.copies = 1u;
    while (r.copies < 16u && 2u * r.copies * r.stride * sizeof(G) <= (uint32_t)kTileBytes &&
           (int64_t)(2u * r.copies * r.cnt) <= share)
        r.copies *= 2u;
}

__device__ __forceinline__ TileRows tile_rows(const DevGrid& g, const TileMap& tm, int l, uint32_t tile) {
    TileRows r;
    r.copies = 1u;
    r.tile = tile;
    r.dense = ((tm.lists & g.dense_bits) >> l) & 1u;
    if (r.dense) {
        const uint32_t S = (uint32_t)g.res_s[l] + 1u, lines = (uint32_t)tm.level_rows[l] / S;
        r.first = 0u;
        r.cnt = ((lines + (1u << tm.tile_shift[l]) - 1u) >> tm.tile_shift[l]) * S;
    } else {
        r.first = tile << tm.tile_shift[l];
        r.cnt = min(1u << tm.tile_shift[l], (uint32_t)tm.level_rows[l] - r.first);
    }
    return r;
}

// Zero the first `values` values of the tile (whose buffer is a whole number of 16-byte
// units).
template <int BLOCK, typename G>
__device__ __forceinline__ void zero_tile(G* tile, uint32_t values) {
    uint4* t = reinterpret_cast<uint4*>(tile);
    const uint32_t quads = (values * (uint32_t)sizeof(G) + 15u) / 16u;
    for (uint32_t i = threadIdx.x; i < quads; i += BLOCK) t[i] = make_uint4(0u, 0u, 0u, 0u);
}

// put(i, at) for every value i < cnt F of the tile held in LDS; at: its index in the
// level's values (row F + feature).  Slots past the level's last line hold no row.
template <int F, int BLOCK, typename Put>
__device__ __forceinline__ void each_tile_value(const DevGrid& g, const TileMap& tm, int l, const TileRows& tr, Put put) {
    if (tr.dense) {
        const uint32_t W = ((uint32_t)g.res_s[l] + 1u) * F, total = (uint32_t)tm.level_rows[l] * F;
        for (uint32_t i = threadIdx.x; i < tr.cnt * F; i += BLOCK) {
            const uint32_t h = i / W, line = tile_line(h, tr.tile, tm.tile_shift[l]);
            const uint32_t v = line * W + (i - h * W);
            if (v < total) put(i, v);
        }
    } else {
        for (uint32_t i = threadIdx.x; i < tr.cnt * F; i += BLOCK) put(i, tr.first * F + i);
    }
}

// What a tile's visits need of their level, in scalar registers.
struct ListLevel {
    float Ns, Nt;         // resolutions
    uint32_t py, pz, pt;  // hashed: primes
    uint32_t S;           // dense: rows of a line
    int shift;            // dense: log2 of the tiles
    uint32_t rmask, tmask, T, px;
    uint32_t first, cnt;
    uint32_t tile;        // dense
    bool dense, own;      // own: only the rows in the tile are added (loose, or a shared list)
};

__device__ __forceinline__ ListLevel list_level(const DevGrid& g, const TileMap& tm, int l, const TileRows& tr) {
    ListLevel c;
    c.Ns = (float)g.res_s[l];
    c.Nt = (float)g.res_t[l];
    c.px = g.prime[0];
    c.py = g.prime[1];
    c.pz = g.prime[2];
    c.pt = g.prime[3];
    c.S = (uint32_t)g.res_s[l] + 1u;
    c.shift = tm.tile_shift[l];
    c.rmask = (1u << c.shift) - 1u;
    c.tmask = g.tmask;
    c.T = g.T;
    c.first = tr.first;
    c.cnt = tr.cnt;
    c.dense = tr.dense;
    c.tile = tr.tile;
    c.own = ((tm.loose >> l) & 1u) || tm.share_shift[l] > 0;
    return c;
}

// level_cell with the lower vertex kept in FP32 (exact: resolutions are at most 2^24).
struct FCell {
    float ix, iy, iz, it, fx, fy, fz, ft;
};

__device__ __forceinline__ void fcell_1d(float x, float N, float& i, float& fr) {
#pragma clang fp contract(off)
    const float pos = clamp_unit(x) * N;
    i = fminf(floorf(pos), N - 1.0f);
    fr = pos - i;
}

__device__ __forceinline__ FCell list_cell(const ListLevel& lv, float4 x) {
    FCell c;
    fcell_1d(x.x, lv.Ns, c.ix, c.fx);
    fcell_1d(x.y, lv.Ns, c.iy, c.fy);
    fcell_1d(x.z, lv.Ns, c.iz, c.fz);
    fcell_1d(x.w, lv.Nt, c.it, c.ft);
    return c;
}

// Bits of the pair of entry e as masks: 0 or -1 per axis.
struct PairMask {
    int y, z, t;
};
__device__ __forceinline__ PairMask pair_mask(uint32_t e) {
    return PairMask{(int)(e << (31 - kListPShift)) >> 31, (int)(e << (30 - kListPShift)) >> 31,
                    (int)(e << (29 - kListPShift)) >> 31};
}

// frac where the mask is set, 1 - frac where it is not: |(1 or 0) - frac|, the same
// rounding as the two forms, the absolute value being free on a product's operand.
template <typename G>
__device__ __forceinline__ G axis_weight(float frac, int mask) {
    if constexpr (sizeof(G) == 4) return fabsf(__uint_as_float(0x3f800000u & ~(uint32_t)mask) - frac);
    else return mask ? G(frac) : G(1) - G(frac);
}

template <typename G>
struct PairWeights {
    G w0, w1;
};

// Weights of the lower and upper corner of a pair, times scale.
template <typename G>
__device__ __forceinline__ PairWeights<G> pair_weights(const FCell& c, const PairMask& m, G scale) {
    const G w = ((axis_weight<G>(c.fy, m.y) * axis_weight<G>(c.fz, m.z)) * axis_weight<G>(c.ft, m.t)) * scale;
    return PairWeights<G>{(G(1) - G(c.fx)) * w, G(c.fx) * w};
}

// Rows of a pair of cell c in the tile.  OWN: a row outside the tile is at or above cnt.
template <bool OWN>
__device__ __forceinline__ void pair_rows(const ListLevel& lv, const FCell& c, const PairMask& m, uint32_t& r0,
                                          uint32_t& r1) {
    const uint32_t ix = (uint32_t)c.ix, iy = (uint32_t)((int)c.iy - m.y), iz = (uint32_t)((int)c.iz - m.z),
                   it = (uint32_t)((int)c.it - m.t);
    if (OWN && lv.dense) {
        const uint32_t line = iy + lv.S * (iz + lv.S * it);
        r0 = line_tile(line, lv.shift) == lv.tile ? (line >> lv.shift) * lv.S + ix : ~1u;
        r1 = r0 + 1u;
    } else if constexpr (OWN) {
        const uint32_t H = (iy * lv.py) ^ (iz * lv.pz) ^ (it * lv.pt), hx = ix * lv.px;
        const uint32_t h0 = hx ^ H, h1 = (hx + lv.px) ^ H;
        r0 = (lv.tmask ? h0 & lv.tmask : h0 % lv.T) - lv.first;
        r1 = (lv.tmask ? h1 & lv.tmask : h1 % lv.T) - lv.first;
    } else if (lv.dense) {
        r0 = ((iy + lv.S * (iz + lv.S * it)) >> lv.shift) * lv.S + ix;
        r1 = r0 + 1u;
    } else {
        // tiles are aligned powers of two of at most 2^15 rows, so a row's place in its
        // tile is its low bits, which 24-bit products give (full rate, unlike 32-bit ones)
        const uint32_t H = __umul24(iy, lv.py) ^ __umul24(iz, lv.pz) ^ __umul24(it, lv.pt);
        r0 = (ix ^ H) & lv.rmask;  // pi_1 = 1
        r1 = ((ix + 1u) ^ H) & lv.rmask;
    }
}

// Add a at the lower and b at the upper corner of a pair (OWN: where they lie in the tile).
template <typename G, int F, bool OWN>
__device__ __forceinline__ void add_pair(G* tile, uint32_t cnt, uint32_t r0, const G (&a)[F], uint32_t r1, const G (&b)[F]) {
    if constexpr (OWN) {
        if (r0 < cnt) lds_add_values<G, F>(tile + r0 * F, a);
        if (r1 < cnt) lds_add_values<G, F>(tile + r1 * F, b);
    } else if constexpr (sizeof(G) == 4 && F == 2) {
        lds_add2_two(tile + r0 * 2, a[0], a[1], tile + r1 * 2, b[0], b[1]);
    } else {
        lds_add_values<G, F>(tile + r0 * F, a);
        lds_add_values<G, F>(tile + r1 * F, b);
    }
}

// Visit every pair entry of one tile: run(load(round, cq, e)) for every entry e of every
// chunk c < nchunks, in chunk order; heads[c] = first entry | entries << 16 inside region
// c of lists.  Called by the whole workgroup; lds holds kWalkLds ints.
//
// Chunks are taken kWalkChunks at a time (a round).  The tile's entries in them are cut
// into batches of 64 (a chunk's last one may be partial), and each wavefront takes one
// contiguous range of the batches, all ranges equally long.  Lane i finds batch i of the
// next 64 of its wavefront's range (its chunk by a binary search over the chunks' batch
// counts), so that per batch only two values are read from a lane, and scalar work, which
// is issued at the same rate as vector work, stays a few instructions.
//
// While a wavefront adds a batch, the data of the next two (load) and the entries of the
// two after those are in flight.  Every lane loads (lanes
// past a batch's end repeat its last entry, a batch past the range's end the range's last
// batch), so the loop has no branch around a load.
//
// load's cq = first query of the entry's chunk, counted from the round's first query
// (below 2^21); the first round's queries start at query 0 of the run.
constexpr int kWalkChunks = 1024;
constexpr int kWalkLds = 2 * kWalkChunks + 16;

// A wavefront holds the descriptions of batches base .. base + 63 of its range, which ends
// before batch b1.  It reads on past the end; base may then lie there too, and every lane
// describes the last batch.
__host__ __device__ constexpr int walk_lane(int next, int base, int b1) {
    const int i = (next < b1 ? next : b1 - 1) - base;
    return i > 0 ? i : 0;
}
constexpr bool walk_lanes_exist(int b1) {
    for (int next = 0, base = 0; next < b1 + 6; ++next) {
        if (next - base >= 64) base = next;
        const int batch = base + walk_lane(next, base, b1), want = next < b1 ? next : b1 - 1;
        if (walk_lane(next, base, b1) < 0 || walk_lane(next, base, b1) > 63 || (batch < b1 ? batch : b1 - 1) != want)
            return false;
    }
    return true;
}
static_assert(walk_lanes_exist(1) && walk_lanes_exist(2) && walk_lanes_exist(62) && walk_lanes_exist(63) &&
                  walk_lanes_exist(64) && walk_lanes_exist(65) && walk_lanes_exist(127) && walk_lanes_exist(128),
              "ranges of whole sets of 64 batches and next to them");

template <int BLOCK, typename Load, typename Run>
__device__ __forceinline__ void walk_pair_lists(int nchunks, int chunk_log, const uint32_t* __restrict__ heads,
                                                const uint16_t* __restrict__ lists, int* lds, Load load, Run run) {
    static_assert(BLOCK == kWalkChunks, "one thread per chunk head");
    constexpr int kWaves = BLOCK / 64;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    uint32_t* lhead = reinterpret_cast<uint32_t*>(lds);
    int* lbefore = lds + kWalkChunks;             // batches before each chunk
    int* wtot = lbefore + kWalkChunks;            // batches per wavefront of heads
    for (int cb = 0; cb < nchunks; cb += kWalkChunks) {
        const int nc = min(kWalkChunks, nchunks - cb);
        const int c = (int)threadIdx.x;
        const uint32_t head = c < nc ? heads[cb + c] : 0u;
        const int nb = (int)((head >> 16) + 63u) >> 6;
        int incl = nb;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int a = __shfl_up(incl, d);
            if (lane >= d) incl += a;
        }
        __syncthreads();  // the previous round's reads are done
        lhead[c] = head;
        if (lane == 63) wtot[wave] = incl;
        __syncthreads();
        int before = incl - nb, total = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const int t = wtot[w];
            if (w < wave) before += t;
            total += t;
        }
        lbefore[c] = before;
        __syncthreads();
        const int b0 = (int)((int64_t)total * wave / kWaves), b1 = (int)((int64_t)total * (wave + 1) / kWaves);
        if (b0 == b1) continue;
        const uint16_t* rl = lists + (int64_t)cb * kListEntries;
        // batch dbase + lane: its first entry in the round's regions, and its chunk and
        // entry count
        int dbase = 0;
        uint32_t doff = 0u, dcn = 0u;
        auto describe = [&](int b) {
            dbase = b;
            const int i = min(b + lane, b1 - 1);
            int lo = 0;
#pragma unroll
            for (int step = kWalkChunks / 2; step > 0; step >>= 1)  // the last chunk with at most i batches before it
                if (lbefore[lo + step] <= i) lo += step;
            const uint32_t h = lhead[lo];
            const uint32_t at = 64u * (uint32_t)(i - lbefore[lo]);
            doff = (uint32_t)lo * (kListEntries * 2u) + 2u * ((h & 0xffffu) + at);
            dcn = ((uint32_t)lo << 8) | min(64u, (h >> 16) - at);
        };
        struct Batch {
            uint32_t cn;    // chunk << 8 | entries (wavefront-uniform)
            uint32_t e;     // this lane's entry
        };
        int next = b0;
        auto fetch = [&](Batch& b) {  // the next batch of the range, none past its end
            if (next - dbase >= 64) describe(next);
            const int i = walk_lane(next, dbase, b1);
            b.cn = (uint32_t)__builtin_amdgcn_readlane((int)dcn, i);
            const uint32_t off = (uint32_t)__builtin_amdgcn_readlane((int)doff, i);
            b.e = *reinterpret_cast<const uint16_t*>(reinterpret_cast<const char*>(rl) +
                                                     (off + 2u * min((uint32_t)lane, (b.cn & 0xffu) - 1u)));
            if (next >= b1) b.cn &= ~0xffu;
            ++next;
        };
        using Data = decltype(load(0, 0u, 0u));
        struct Item {
            Data d;
            uint32_t n;     // entries (wavefront-uniform)
        };
        auto data = [&](const Batch& b) { return Item{load(cb, (b.cn >> 8) << chunk_log, b.e), b.cn & 0xffu}; };
        describe(b0);
        if constexpr (sizeof(Data) > 128) {
            // two corner sets of eight FP64 features: three batches in flight spill 338
            // registers (50k queries of 8 levels: 718 us, one at a time 590)
            Batch q[2];
            fetch(q[0]);
            for (int b = b0; b < b1; b += 2) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const Item d = data(q[j]);
                    fetch(q[1 - j]);
                    if ((uint32_t)lane < d.n) run(d.d);
                }
            }
            continue;
        }
        Batch q[3];
        Item d[3];
        fetch(q[0]);
        fetch(q[1]);
        d[0] = data(q[0]);
        d[1] = data(q[1]);
        fetch(q[2]);
        fetch(q[0]);
        for (int b = b0; b < b1; b += 3) {
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                d[(j + 2) % 3] = data(q[(j + 2) % 3]);
                fetch(q[(j + 1) % 3]);
                if ((uint32_t)lane < d[j].n) run(d[j].d);
            }
        }
    }
}

}  // namespace h4d
