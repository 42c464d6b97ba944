// 4D hash encoder forward and backward kernels (DASH Section 4.2, Eqs. 8-9).
//
// Forward: one thread per (query, level).  Work items (level, 64 queries) are
// placed on XCDs level by level (xcd_item), so each XCD's L2 holds mostly one
// level's slice of the table (4 MiB FP32 / 2 MiB BF16 for a 2^19-row, F = 2 level)
// instead of every XCD streaming the whole table through its L2.
#include <limits.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <type_traits>

#include "pair_lists.h"

namespace h4d {

constexpr int kEncodeBlock = 64;  // small: a workgroup's wavefronts then end one by one (256: 2 us slower at 200k)

template <typename TT, int F, bool WIDE>
__global__ __launch_bounds__(kEncodeBlock) void k_encode(DevGrid g, const TT* __restrict__ table,
                                                         const float4* __restrict__ xyzt, int n,
                                                         typename AccOf<TT>::type* __restrict__ out,
                                                         int64_t lstride, int64_t qstride) {
    using A = typename AccOf<TT>::type;
    const int chunks = (n + kEncodeBlock - 1) / kEncodeBlock;
    int l, chunk;
    if (!xcd_item(g.L * chunks, chunks, l, chunk)) return;
    const int q = chunk * kEncodeBlock + threadIdx.x;
    const Cell c = level_cell(g, l, xyzt[min(q, n - 1)]);  // every lane takes part in the gather
    A acc[F];
    interpolate<TT, F, WIDE>(g, l, table, c, acc);
    if (q >= n) return;
    A* o = out + (int64_t)l * lstride + (int64_t)q * qstride;
    if constexpr (F == 2 && sizeof(A) == 4) {
        *reinterpret_cast<float2*>(o) = make_float2(acc[0], acc[1]);
    } else {
#pragma unroll
        for (int f = 0; f < F; ++f) o[f] = acc[f];
    }
}

// ------------------------------------------------------ tiled table scatter ----
// Device-scope FP32 atomics on MI355X complete at a fixed rate of about 2e10 per
// second whatever the footprint (they are not executed in the XCD-local L2), so
// the scatter avoids them altogether.  Owner computes: one workgroup per (level,
// tile of 2^tile_shift consecutive table rows of that level; about 32 tiles per
// level) keeps the tile's gradient in LDS, adds w_c g for the corners of the
// level's queries that fall in its tile with compare-and-swap LDS adds (lds_add2),
// and finally adds the tile to d_table with plain loads and stores (no other
// workgroup owns those rows).
//
// A pre-pass tells each tile which queries reach it: pair lists (pair_lists.h), or, on
// hashed levels of more than kListTiles tiles (and where the workspace does not hold one level's
// lists), a 32-bit mask per (query, level) of the tiles the query's corners touch (tile t sets bit t >>
// bit_shift); a tile workgroup reads the masks of its level, compacts the queries whose
// bit is set into per-wavefront LDS queues and runs the corner work on full wavefronts of
// those queries only.
// PAIR: each query also subtracts the same gradient at the corners of x + eps (the
// second term of Eq. 11).
//
// Dense levels of more than kListTiles tiles share lists among neighbouring tiles rather
// than scan masks: where queries crowd (one timestamp), a mask form's tiles of consecutive
// rows get most of a level's updates.  200k queries at one timestamp, one level: 4.1M rows
// of 4 features 698 -> 127 us, 2M of 8 1076 -> 213, 32M of 2 (2048 tiles) 1505 -> 187; at
// random times 195 -> 87, 258 -> 115, 500 -> 203.
//
// The lists are why a tile's time follows its own updates: with the masks alone every tile
// streams its level's mask array and gathers whole queries for one pair each.  200k queries
// of the 16-level, 2^19-row scene: scatter 224 -> 128 us, the passes before it 26 -> 34 us;
// 123k queries of one timestamp 254 -> 173 us (and no pass over tiles split among
// workgroups); two corner sets 558 -> 230 us.  What bounds it now, at four wavefronts per
// SIMD (the tile fills the LDS): vector instructions 59 % of the time, LDS 54 %, L1 fills
// 56 %, none of them alone.  Doubles in the tile with the hardware's FP64 adds, which need
// no retry, were no faster (the tile then holds half the rows: 431 -> 511 us for a step).

// The pre-pass.  Grid (chunks of the level with the most, L, or L + 1 with a sum); levels without tiles belong
// to another pass (scatter_plan).
//
// With PAIR a workgroup past the last level adds up the smoothness loss's partial sums: one
// FP32 atomic per workgroup of 256 queries in order of arrival (12.5k of them for 200k
// queries of 16 levels) left the step's outputs 7.3e-7 from the 64-bit ones, this order
// 2.2e-7.  A launch of its own made calls of 1000 queries 2 us longer (33 us).
template <typename A>
__device__ __forceinline__ void add_fixed_sum(const FixedSum& f) {
    constexpr int kBlock = pre_block(true);
    __shared__ double part[kBlock / 64];
    const A* __restrict__ sums = static_cast<const A*>(f.sums);
    double t = 0.0;
#pragma unroll 8
    for (int i = threadIdx.x; i < f.count; i += kBlock) t += (double)sums[i];
    for (int s = 32; s > 0; s >>= 1) t += __shfl_xor(t, s, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
        t = 0.0;
        for (int w = 0; w < kBlock / 64; ++w) t += part[w];
        atomic_add(static_cast<A*>(f.out), (A)(f.scale * t));  // calls on other streams may add to it too
    }
}

template <bool PAIR>
__global__ __launch_bounds__(pre_block(PAIR)) __attribute__((amdgpu_waves_per_eu(pre_waves_per_eu(PAIR)))) void k_tile_pre(DevGrid g, TileMap tm, const float4* __restrict__ xyzt,
                                                        const float4* __restrict__ eps, int n,
                                                        uint32_t* __restrict__ mask, uint16_t* __restrict__ lists,
                                                        uint32_t* __restrict__ heads, FixedSum sum) {
    __shared__ __align__(16) PreShared<PAIR> sh;
    if constexpr (PAIR) {
        if ((int)blockIdx.y == g.L) {
            if (blockIdx.x > 0) return;
            if (sum.f64) add_fixed_sum<double>(sum);
            else add_fixed_sum<float>(sum);
            return;
        }
    }
    const int l = blockIdx.y, nchunks = pre_chunks(n, pre_chunk_log(tm, l, PAIR));
    if ((int)blockIdx.x >= nchunks || !(((tm.lists | tm.masks) >> l) & 1u)) return;
    tile_pre<PAIR>(g, tm, l, (int)blockIdx.x, 0, nchunks, n,
                   [&](int q, float4& x, float4& xp) {
                       x = xyzt[q];
                       if constexpr (PAIR) xp = perturbed(x, eps[q]);
                   },
                   mask, lists, heads, sh);
}

// 1024 threads share each tile: the 128 KiB of LDS allows one workgroup per CU, and
// sixteen wavefronts (four per SIMD) keep the query loads in flight.
constexpr int kScatterBlock = 1024;

// With PAIR, a second feature gradient (the decoder's) that joins the first at x's
// corners only: a training step with Eq. 11 then scatters both in one pass.
template <typename G>
struct MainGrad {
    const G* src;  // nullptr: none
    int64_t lstride, qstride;
    G scale;
};

// What the scatter loads per queued query: position, gradient (and perturbation).
template <typename G, int F, bool PAIR>
struct TileQuery {
    float4 x;
    float4 e;     // used when PAIR
    G gv[F];
    G gmain[F];   // used when PAIR with a MainGrad
};

// Query q0 + dq (dq below 2^21): the addresses are those of q0, in scalar registers where
// q0 is uniform, plus 32-bit offsets (a query has at most H4D_MAX_LEVELS * 8 features).
template <typename G, int F, bool PAIR>
__device__ __forceinline__ TileQuery<G, F, PAIR> tile_load(int l, const float4* __restrict__ xyzt,
                                                           const float4* __restrict__ eps, const G* __restrict__ src,
                                                           int64_t lstride, int64_t qstride, const MainGrad<G>& mg,
                                                           int q0, uint32_t dq) {
    TileQuery<G, F, PAIR> t;
    auto row = [&](const G* base, int64_t ls, int64_t qs) {
        const char* p = reinterpret_cast<const char*>(base + ((int64_t)l * ls + (int64_t)q0 * qs));
        return reinterpret_cast<const G*>(p + (uint32_t)__umul24(dq, (uint32_t)qs * (uint32_t)sizeof(G)));
    };
    auto quad = [&](const float4* base) {
        return *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(base + q0) + dq * 16u);
    };
    const G* gp = row(src, lstride, qstride);
#pragma unroll
    for (int f = 0; f < F; ++f) t.gv[f] = gp[f];
    t.x = quad(xyzt);
    if constexpr (PAIR) {
        t.e = quad(eps);
        if (mg.src) {
            const G* mp = row(mg.src, mg.lstride, mg.qstride);
#pragma unroll
            for (int f = 0; f < F; ++f) t.gmain[f] = mp[f];
        }
    }
    return t;
}

template <typename G, int F, bool PAIR>
__device__ __forceinline__ void tile_run(const DevGrid& g, const TileMap& tm, int l, const TileQuery<G, F, PAIR>& t,
                                         G scale, const MainGrad<G>& mg, uint32_t base, uint32_t cnt, G* tile) {
    G gv[F];
#pragma unroll
    for (int f = 0; f < F; ++f) gv[f] = t.gv[f] * scale;
    if constexpr (PAIR) {
        G gx[F], gm[F];
#pragma unroll
        for (int f = 0; f < F; ++f) {
            gx[f] = mg.src ? gv[f] + t.gmain[f] * mg.scale : gv[f];
            gm[f] = -gv[f];
        }
        tile_contrib<G, F>(g, tm, l, t.x, gx, base, cnt, tile);
        const float4 x = t.x, e = t.e;
        const float4 xp = make_float4(__fadd_rn(x.x, e.x), __fadd_rn(x.y, e.y), __fadd_rn(x.z, e.z),
                                      __fadd_rn(x.w, e.w));
        tile_contrib<G, F>(g, tm, l, xp, gm, base, cnt, tile);
    } else {
        tile_contrib<G, F>(g, tm, l, t.x, gv, base, cnt, tile);
    }
}

// What the scatter loads per list entry: the query's position and gradient (and, with
// PAIR, its perturbation and main gradient) and the entry's pair and kind.
template <typename G, int F, bool PAIR>
struct ListQuery {
    TileQuery<G, F, PAIR> t;
    uint32_t e;
};

// One tile of a list level.
template <typename G, int F, bool PAIR>
__device__ __forceinline__ void scatter_lists(const DevGrid& g, const TileMap& tm, int l, const TileRows& tr,
                                              const float4* __restrict__ xyzt, const float4* __restrict__ eps, int n,
                                              const uint32_t* __restrict__ heads, const uint16_t* __restrict__ lists,
                                              const G* __restrict__ src, int64_t lstride, int64_t qstride, G scale,
                                              const MainGrad<G>& mg, int* lds, G* tile) {
    const int log = pre_chunk_log(tm, l, PAIR), nchunks = pre_chunks(n, log);
    const ListLevel lv = list_level(g, tm, l, tr);
    auto walk = [&](auto own) {
        constexpr bool kOwn = decltype(own)::value;
        walk_pair_lists<kScatterBlock>(
            nchunks, log, heads + tm.list_head[l] + (int64_t)(tr.tile >> tm.share_shift[l]) * nchunks,
            lists + tm.list_entry[l], lds,
            [&](int round, uint32_t cq, uint32_t e) {
                ListQuery<G, F, PAIR> q;
                q.t = tile_load<G, F, PAIR>(l, xyzt, eps, src, lstride, qstride, mg, round << log,
                                            cq | (e & kListQMask));
                q.e = e;
                return q;
            },
            [&](const ListQuery<G, F, PAIR>& q) {
                const PairMask m = pair_mask(q.e);
                G a[F], b[F];
                uint32_t r0, r1;
                if constexpr (!PAIR) {
                    const FCell c = list_cell(lv, q.t.x);
                    const PairWeights<G> w = pair_weights<G>(c, m, scale);
#pragma unroll
                    for (int f = 0; f < F; ++f) {
                        a[f] = w.w0 * q.t.gv[f];
                        b[f] = w.w1 * q.t.gv[f];
                    }
                    pair_rows<kOwn>(lv, c, m, r0, r1);
                } else {
                    // kind 0: x's pair, +(gradients); kind 1: xp's pair, -(smoothness
                    // gradient); kind 2: both at the same rows
                    const uint32_t kind = q.e >> kListKShift;
                    const float4 xp = perturbed(q.t.x, q.t.e);
                    const FCell c = list_cell(lv, kind == 1u ? xp : q.t.x);
                    const PairWeights<G> w = pair_weights<G>(c, m, G(1));
#pragma unroll
                    for (int f = 0; f < F; ++f) {
                        G v = q.t.gv[f] * scale;
                        v = kind == 1u ? -v : mg.src ? v + q.t.gmain[f] * mg.scale : v;
                        a[f] = w.w0 * v;
                        b[f] = w.w1 * v;
                    }
                    if (kind == 2u) {
                        const PairWeights<G> wp = pair_weights<G>(list_cell(lv, xp), m, scale);
#pragma unroll
                        for (int f = 0; f < F; ++f) {
                            a[f] -= wp.w0 * q.t.gv[f];
                            b[f] -= wp.w1 * q.t.gv[f];
                        }
                    }
                    pair_rows<kOwn>(lv, c, m, r0, r1);
                }
                add_pair<G, F, kOwn>(tile, tr.cnt, r0, a, r1, b);
            });
    };
    if (lv.own) walk(std::true_type{});
    else walk(std::false_type{});
}

// *counter += the non-finite values the wavefront's lanes counted (one atomic per
// wavefront that has any).  Called by every lane of the wavefront.
__device__ __forceinline__ void add_count(int* counter, int bad) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) bad += __shfl_xor(bad, d, 64);
    if ((threadIdx.x & 63) == 0 && bad) atomicAdd(counter, bad);
}

// Tiles of one run of the scatter's XCD placement (16 runs).
__host__ __device__ constexpr int scatter_run(int tiles) { return (tiles + 2 * kXcds - 1) / (2 * kXcds); }

// The tile's rows have no other owner: add them to d_table, or with overwrite set write
// every row (the tiles of the levels cover all E rows); count the non-finite values
// written if asked.
template <typename G, int F>
__device__ __forceinline__ void flush_tile(const DevGrid& g, const TileMap& tm, int l, const TileRows& tr, const G* tile,
                                           G* __restrict__ d_table, int overwrite, int* __restrict__ nonfinite) {
    G* out = d_table + (size_t)g.off[l] * F;
    auto value = [&](uint32_t i) {
        G v = tile[i];
        for (uint32_t k = 1; k < tr.copies; ++k) v += tile[k * tr.stride + i];
        return v;
    };
    int bad = 0;
    if (overwrite) {
        each_tile_value<F, kScatterBlock>(g, tm, l, tr, [&](uint32_t i, uint32_t at) {
            const G v = value(i);
            out[at] = v;
            bad += !__builtin_isfinite(v);
        });
    } else {
        each_tile_value<F, kScatterBlock>(g, tm, l, tr, [&](uint32_t i, uint32_t at) {
            const G v = value(i);
            if (v != G(0)) {
                const G r = out[at] + v;
                out[at] = r;
                bad += !__builtin_isfinite(r);
            }
        });
    }
    if (nonfinite) add_count(nonfinite, bad);
}

// Tile of workgroup blockIdx.x, false if none.  XCD placement: the level-ordered tiles are
// cut into 16 equal runs, XCD x working on runs x and 15 - x, so its L2 holds the lists
// and gradients of two or three levels instead of every XCD fetching every level's, and
// every XCD gets one coarse and one fine run: the coarse levels' tiles take longer where
// queries share cells, the fine ones' where a query's two corner sets differ.
__device__ __forceinline__ bool scatter_tile(const DevGrid& g, const TileMap& tm, int& l, uint32_t& tile) {
    const int tiles = tm.tile_start[g.L];
    const int per = scatter_run(tiles);
    const int x = (int)blockIdx.x % kXcds, i0 = (int)blockIdx.x / kXcds;
    const int tix = i0 < per ? x * per + i0 : (2 * kXcds - 1 - x) * per + i0 - per;
    if (tix >= tiles) return false;
    l = 0;
    while (l + 1 < g.L && tix >= tm.tile_start[l + 1]) ++l;
    tile = (uint32_t)(tix - tm.tile_start[l]);
    return true;
}

// Tiles of the list levels.
template <typename G, int F, bool PAIR>
__global__ __launch_bounds__(kScatterBlock) void k_scatter_tiled(DevGrid g, TileMap tm, const float4* __restrict__ xyzt,
                                                                const float4* __restrict__ eps, int n,
                                                                const uint16_t* __restrict__ lists,
                                                                const uint32_t* __restrict__ heads,
                                                                const G* __restrict__ src, int64_t lstride,
                                                                int64_t qstride, G scale, G* __restrict__ d_table,
                                                                int overwrite, MainGrad<G> mg,
                                                                int* __restrict__ nonfinite) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int walk[kWalkLds];
    G* tile = reinterpret_cast<G*>(smem);
    int l;
    uint32_t t;
    if (!scatter_tile(g, tm, l, t) || !((tm.lists >> l) & 1u)) return;
    TileRows tr = tile_rows(g, tm, l, t);
    set_copies<G, F>(tr, tm.tile_start[l + 1] - tm.tile_start[l], n);
    zero_tile<kScatterBlock>(tile, tr.copies > 1u ? tr.copies * tr.stride : tr.cnt * F);
    __syncthreads();
    scatter_lists<G, F, PAIR>(g, tm, l, tr, xyzt, eps, n, heads, lists, src, lstride, qstride, scale, mg, walk,
                              tile + (threadIdx.x & (tr.copies - 1u)) * tr.stride);
    __syncthreads();
    flush_tile<G, F>(g, tm, l, tr, tile, d_table, overwrite, nonfinite);
}

// Tiles of the levels with masks.
template <typename G, int F, bool PAIR>
__global__ __launch_bounds__(kScatterBlock) void k_scatter_masked(DevGrid g, TileMap tm, const float4* __restrict__ xyzt,
                                                                 const float4* __restrict__ eps, int n,
                                                                 const uint32_t* __restrict__ mask,
                                                                 const G* __restrict__ src, int64_t lstride,
                                                                 int64_t qstride, G scale, G* __restrict__ d_table,
                                                                 int overwrite, MainGrad<G> mg,
                                                                 int* __restrict__ nonfinite) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int queue[2 * kScatterBlock];  // 128 entries per wavefront
    G* tile = reinterpret_cast<G*>(smem);
    int l;
    uint32_t t;
    if (!scatter_tile(g, tm, l, t) || !((tm.masks >> l) & 1u)) return;
    const TileRows tr = tile_rows(g, tm, l, t);
    zero_tile<kScatterBlock>(tile, tr.cnt * F);
    __syncthreads();
    masked_queue_loop<kScatterBlock>(
        n, mask + (int64_t)__popc(tm.masks & ((1u << l) - 1u)) * mask_stride(n), tile_bit(tm, l, tr.first), queue,
        [&](int q) { return tile_load<G, F, PAIR>(l, xyzt, eps, src, lstride, qstride, mg, q, 0u); },
        [&](const TileQuery<G, F, PAIR>& q) {
            tile_run<G, F, PAIR>(g, tm, l, q, scale, mg, g.off[l] + tr.first, tr.cnt, tile);
        });
    __syncthreads();
    flush_tile<G, F>(g, tm, l, tr, tile, d_table, overwrite, nonfinite);
}

__global__ __launch_bounds__(kEncodeBlock) void k_corner_indices(DevGrid g, const float4* __restrict__ xyzt, int n,
                                                                 int32_t* __restrict__ rows, float* __restrict__ w) {
    const int l = blockIdx.y;
    const int q = blockIdx.x * kEncodeBlock + threadIdx.x;
    if (q >= n) return;
    const Cell c = level_cell(g, l, xyzt[q]);
    uint32_t row[16];
    level_rows(g, l, c, row);
    float wt[16];
    level_weights<float>(c, wt);
    const int64_t base = ((int64_t)q * g.L + l) * 16;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        if (rows) rows[base + k] = (int32_t)row[k];
        if (w) w[base + k] = wt[k];
    }
}

// ---------------------------------------------------------------- launchers ----
static dim3 level_major_grid(int n, int L) { return dim3((unsigned)((n + kEncodeBlock - 1) / kEncodeBlock), (unsigned)L); }

template <typename TT>
static hipError_t encode_t(const DevGrid& g, const void* table, const float* xyzt, int n, void* out,
                           int64_t ls, int64_t qs, hipStream_t s) {
    using A = typename AccOf<TT>::type;
    const int chunks = (n + kEncodeBlock - 1) / kEncodeBlock;
    const dim3 grid((unsigned)(kXcds * xcd_items_per(g.L * chunks))), block(kEncodeBlock);
    const TT* t = static_cast<const TT*>(table);
    const float4* x = reinterpret_cast<const float4*>(xyzt);
    A* o = static_cast<A*>(out);
#define H4D_ENC(FF, WW) hipLaunchKernelGGL((k_encode<TT, FF, WW>), grid, block, 0, s, g, t, x, n, o, ls, qs)
    switch (g.F) {
        case 1:
            if (can_widen<TT, 1>(table, g.rows)) H4D_ENC(1, true);
            else H4D_ENC(1, false);
            break;
        case 2:
            if (can_widen<TT, 2>(table, g.rows)) H4D_ENC(2, true);
            else H4D_ENC(2, false);
            break;
        case 4: H4D_ENC(4, false); break;
        case 8: H4D_ENC(8, false); break;
        default: return hipErrorInvalidValue;
    }
#undef H4D_ENC
    return hipGetLastError();
}

hipError_t launch_encode(const DevGrid& g, h4d_dtype dt, const void* table, const float* xyzt, int n, void* out,
                         int64_t ls, int64_t qs, hipStream_t s) {
    switch (dt) {
        case H4D_F32: return encode_t<float>(g, table, xyzt, n, out, ls, qs, s);
        case H4D_BF16: return encode_t<bf16_t>(g, table, xyzt, n, out, ls, qs, s);
        case H4D_F64: return encode_t<double>(g, table, xyzt, n, out, ls, qs, s);
    }
    return hipErrorInvalidValue;
}

// Tiles of at most 128 KiB of LDS; tile_start is the first tile of each level.
TileMap make_tile_map(const DevGrid& g, const int64_t* level_rows, int F, int gbytes, int n, int segs, bool pair,
                      uint32_t levels, uint32_t listed) {
    TileMap tm;
    memset(&tm, 0, sizeof tm);
    tm.max_rows = kTileBytes / (F * gbytes);  // a power of two: F and gbytes are
    int tiles[H4D_MAX_LEVELS], line_shift[H4D_MAX_LEVELS];
    uint32_t can = 0u;  // levels that can have lists
    for (int l = 0; l < g.L; ++l) {
        const int64_t rows = level_rows[l];
        tm.level_rows[l] = (int32_t)rows;
        const int64_t want = (rows + kTilesPerLevel - 1) / kTilesPerLevel;
        int sh = 8;  // at least 256 rows per tile
        while ((1 << sh) < tm.max_rows && ((int64_t)1 << sh) < want) ++sh;
        tm.tile_shift[l] = sh;
        tiles[l] = (int)((rows + (1 << sh) - 1) >> sh);
        if ((g.dense_bits >> l) & 1u) {
            // 32 tiles of x-lines (fewer where there are fewer lines), more if 32 do not fit.
            // The only level of a grid: 256, which fill the CUs.  200k queries in one hundredth
            // of the cube, 31^3 x 17 vertices: 645 us with 32, 237 with 256 (uniform 77 and 37).
            // Two levels or more gain nothing (within 1 %), three lose (384 tiles: 71 -> 98 us).
            const int64_t S = (int64_t)g.res_s[l] + 1, lines = rows / S;
            int b = g.L == 1 ? 8 : 5;
            while (b > 0 && ((int64_t)1 << b) > lines) --b;
            while (((int64_t)1 << b) < lines && ((lines + (1 << b) - 1) >> b) * S > tm.max_rows) ++b;
            line_shift[l] = b;
            if (((lines + (1 << b) - 1) >> b) * S <= tm.max_rows) can |= 1u << l;
        } else {
            if (g.tmask != 0u && g.prime[0] == 1u && rows >= ((int64_t)1 << sh) &&
                2 * (int64_t)g.res_s[l] <= ((int64_t)1 << sh))
                tm.pair_cotiled |= 1u << l;
            if (tiles[l] <= kListTiles) can |= 1u << l;
        }
    }
    tm.lists = levels & listed & can;
    tm.masks = levels & ~tm.lists;
    int t = 0;
    int64_t entry = 0, head = 0;
    for (int l = 0; l < g.L; ++l) {
        if (!((levels >> l) & 1u)) {
            tiles[l] = 0;
        } else if ((tm.lists >> l) & 1u) {
            if ((g.dense_bits >> l) & 1u) {
                tm.tile_shift[l] = line_shift[l];
                tiles[l] = 1 << line_shift[l];
                while ((tiles[l] >> tm.share_shift[l]) > kListTiles) ++tm.share_shift[l];
            } else if (!((tm.pair_cotiled >> l) & 1u)) {
                tm.loose |= 1u << l;
            }
        }
        tm.tile_start[l] = t;
        tm.list_entry[l] = entry;
        tm.list_head[l] = head;
        if ((tm.lists >> l) & 1u) {
            const int log = pre_chunk_log(tm, l, pair), per_seg = pre_chunks(n, log);
            const int64_t chunks = (int64_t)segs * per_seg;
            entry += chunks == 1 ? (int64_t)(kListEntries >> log) * n : chunks * kListEntries;
            head += chunks * (tiles[l] >> tm.share_shift[l]);
        } else if ((tm.masks >> l) & 1u) {
            while (((tiles[l] - 1) >> tm.bit_shift[l]) >= 32) ++tm.bit_shift[l];
        }
        t += tiles[l];
    }
    tm.tile_start[g.L] = t;
    tm.list_entry[g.L] = entry;
    tm.list_head[g.L] = head;
    return tm;
}

// One pass of the tiled scatter (a pre-pass and a launch over some of the levels), and what
// it takes of the workspace, each part 256-byte aligned: pair lists | list heads |
// masks [mask level][stride] u32.
struct ScatterPass {
    size_t heads, masks, total;
    TileMap tm;
};

static size_t align256(size_t b) { return (b + 255) / 256 * 256; }

static ScatterPass scatter_pass(const DevGrid& g, const int64_t* level_rows, int n, int gbytes, bool pair,
                                uint32_t levels, uint32_t listed) {
    ScatterPass w;
    w.tm = make_tile_map(g, level_rows, g.F, gbytes, n, 1, pair, levels, listed);
    w.heads = align256((size_t)w.tm.list_entry[g.L] * sizeof(uint16_t));
    w.masks = w.heads + align256((size_t)w.tm.list_head[g.L] * sizeof(uint32_t));
    w.total = w.masks + align256((size_t)mask_stride(n) * __builtin_popcount(w.tm.masks) * sizeof(uint32_t));
    return w;
}

// How a workspace of `avail` bytes is used that does not hold the lists of all levels: by
// passes over runs of levels, one after the other in the same memory.  The runs have
// equal numbers of levels or about equal bytes, whichever fits with fewer rounds of
// workgroups over the CUs (a tile fills one): 16 levels of 2^14 rows at 200k queries take
// 173 us in passes of 256 tiles, 217 us where one has 11 levels.  Masks on the levels that
// do not fit cost far more (250k queries: 203 us in two passes, 336 us with masks), so only
// a level whose own lists do not fit has them.
struct ScatterPlan {
    int passes;
    uint32_t listed;
    uint32_t levels[H4D_MAX_LEVELS];  // of each pass
};
constexpr int kCus = 256;

static ScatterPlan scatter_plan(const DevGrid& g, const int64_t* level_rows, int n, int gbytes, bool pair,
                                size_t avail) {
    ScatterPlan best;
    memset(&best, 0, sizeof best);
    best.listed = level_bits(g.L);
    auto pass = [&](uint32_t levels) { return scatter_pass(g, level_rows, n, gbytes, pair, levels, best.listed); };
    size_t level[H4D_MAX_LEVELS], total = 0;
    for (int l = 0; l < g.L; ++l) {
        if (pass(1u << l).total > avail) best.listed &= ~(1u << l);
        total += level[l] = pass(1u << l).total;
    }
    int least = INT_MAX;  // rounds; the last try, a level each, always fits
    for (int passes = 1; passes <= g.L && passes < least; ++passes)
        for (int by_bytes = 0; by_bytes < 2; ++by_bytes) {
            ScatterPlan p = best;
            memset(p.levels, 0, sizeof p.levels);
            p.passes = passes;
            size_t before = 0;
            for (int l = 0; l < g.L; before += level[l++])  // by the middle of the level's bytes
                p.levels[by_bytes ? (before + level[l] / 2) * passes / total : (size_t)(l * passes / g.L)] |= 1u << l;
            int rounds = 0;
            for (int i = 0; i < passes && rounds < least; ++i) {
                const ScatterPass w = pass(p.levels[i]);
                rounds = w.total <= avail ? rounds + (w.tm.tile_start[g.L] + kCus - 1) / kCus : least;
            }
            if (rounds < least) {
                best = p;
                least = rounds;
            }
        }
    return best;
}

// The size that versions without pair lists reported: 12 bytes per (query, level), the
// queries per tile of each chunk of 1024, and two partial tiles for each of up to 96
// workgroups.  A caller may hold a workspace of that size, and the calls that
// hash4d_encode_backward_noalloc takes were settled by it: both are still taken.
static size_t former_ws_bytes(const DevGrid& g, const int64_t* level_rows, int n) {
    size_t slot = 0;
    int tiles = 0;
    for (int gbytes = 4; gbytes <= 8; gbytes += 4) {
        const TileMap tm = make_tile_map(g, level_rows, g.F, gbytes, n, 1, false, level_bits(g.L), 0u);
        tiles = std::max(tiles, tm.tile_start[g.L]);
        for (int l = 0; l < g.L; ++l)
            slot = std::max(slot, (size_t)std::min((int64_t)1 << tm.tile_shift[l], level_rows[l]) * g.F * gbytes);
    }
    const size_t chunks = ((size_t)n + 1023) / 1024, extra = std::min(96, std::max(8, tiles / 4));
    return align256((size_t)mask_stride(n) * g.L * 4) + align256((size_t)mask_stride(n) * g.L * 8) +
           align256((size_t)g.L * chunks * 128) + align256((tiles + extra) * 16) + 256 + align256(extra * 4) +
           2 * extra * slot;
}

// All levels in one pass.  One corner set: the static workspace's size where that is less
// and its entry point takes the call, since that takes exactly the calls for which no more
// is reported; such a call runs in two passes or more, with a workspace of its own too
// unless it brings more.  Never less for more queries: either size and the rule only grow.
size_t scatter_ws_bytes(const DevGrid& g, const int64_t* level_rows, int n, bool pair) {
    const uint32_t all = level_bits(g.L);
    const size_t bytes = std::max(scatter_pass(g, level_rows, n, 4, pair, all, all).total,
                                  scatter_pass(g, level_rows, n, 8, pair, all, all).total);
    return !pair && bytes > kStaticScratchBytes && former_ws_bytes(g, level_rows, n) <= kStaticScratchBytes
               ? kStaticScratchBytes
               : bytes;
}

size_t scatter_ws_least(const DevGrid& g, const int64_t* level_rows, int n, bool pair, size_t more) {
    return std::min(scatter_ws_bytes(g, level_rows, n, pair) + more, former_ws_bytes(g, level_rows, n));
}

struct ScatterBufs {
    uint16_t* lists;
    uint32_t* heads;
    uint32_t* mask;
};

template <typename G, int F, bool PAIR>
static hipError_t tiled_f(const DevGrid& g, const TileMap& tm, const float* xyzt, const float* eps, int n,
                          const ScatterBufs& b, const void* src, int64_t ls, int64_t qs, double scale, void* d_table,
                          bool overwrite, const MainGradArg& main, int32_t* nonfinite, hipStream_t s) {
    const size_t lds = (size_t)tm.max_rows * F * sizeof(G);
    const dim3 grid((unsigned)(2 * kXcds * scatter_run(tm.tile_start[g.L]))), block(kScatterBlock);
    const float4* x = reinterpret_cast<const float4*>(xyzt);
    const float4* ep = reinterpret_cast<const float4*>(eps);
    const G* gr = static_cast<const G*>(src);
    G* out = static_cast<G*>(d_table);
    const MainGrad<G> mg{static_cast<const G*>(main.src), main.lstride, main.qstride, (G)main.scale};
    hipError_t e = hipSuccess;
    if (tm.lists) {
        auto kern = k_scatter_tiled<G, F, PAIR>;
        e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, grid, block, lds, s, g, tm, x, ep, n, b.lists, b.heads, gr, ls, qs, (G)scale, out,
                           overwrite ? 1 : 0, mg, nonfinite);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (tm.masks) {
        auto kern = k_scatter_masked<G, F, PAIR>;
        e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, grid, block, lds, s, g, tm, x, ep, n, b.mask, gr, ls, qs, (G)scale, out,
                           overwrite ? 1 : 0, mg, nonfinite);
        e = hipGetLastError();
    }
    return e;
}

template <typename G, bool PAIR>
static hipError_t tiled_g(const DevGrid& g, const int64_t* level_rows, const float* xyzt, const float* eps, int n,
                          const void* src, int64_t ls, int64_t qs, double scale, void* d_table, void* ws,
                          size_t ws_bytes, bool overwrite, const MainGradArg& main, int32_t* nonfinite,
                          const FixedSum& sum, hipStream_t s) {
    const uint32_t all = level_bits(g.L);
    ScatterPass w = scatter_pass(g, level_rows, n, (int)sizeof(G), PAIR, all, all);
    const bool whole = w.total <= ws_bytes;
    const ScatterPlan plan = whole ? ScatterPlan{1, all, {all}}
                                   : scatter_plan(g, level_rows, n, (int)sizeof(G), PAIR, ws_bytes);
    if (plan.passes == 0) return hipErrorInvalidValue;  // less than the least workspace
    for (int i = 0; i < plan.passes; ++i) {
        const uint32_t levels = plan.levels[i];
        if (!levels) continue;
        if (!whole) w = scatter_pass(g, level_rows, n, (int)sizeof(G), PAIR, levels, plan.listed);
        const TileMap& tm = w.tm;
        char* at = static_cast<char*>(ws);
        const ScatterBufs b{reinterpret_cast<uint16_t*>(at), reinterpret_cast<uint32_t*>(at + w.heads),
                            reinterpret_cast<uint32_t*>(at + w.masks)};
        int chunks = 0;
        for (int l = 0; l < g.L; ++l)
            if ((levels >> l) & 1u) chunks = std::max(chunks, pre_chunks(n, pre_chunk_log(tm, l, PAIR)));
        hipLaunchKernelGGL(k_tile_pre<PAIR>, dim3((unsigned)chunks, (unsigned)(g.L + (PAIR && sum.count > 0 && i == 0 ? 1 : 0))),
                           dim3(pre_block(PAIR)), 0, s, g, tm,
                           reinterpret_cast<const float4*>(xyzt), reinterpret_cast<const float4*>(eps), n, b.mask,
                           b.lists, b.heads, sum);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
#define H4D_SCATTER(FF) tiled_f<G, FF, PAIR>(g, tm, xyzt, eps, n, b, src, ls, qs, scale, d_table, overwrite, main, nonfinite, s)
        switch (g.F) {
            case 1: e = H4D_SCATTER(1); break;
            case 2: e = H4D_SCATTER(2); break;
            case 4: e = H4D_SCATTER(4); break;
            case 8: e = H4D_SCATTER(8); break;
            default: e = hipErrorInvalidValue;
        }
#undef H4D_SCATTER
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_scatter_tiled(const DevGrid& g, const int64_t* level_rows, h4d_dtype grad_dt, const float* xyzt,
                                const float* eps, int n, const void* src, int64_t ls, int64_t qs, double scale,
                                void* d_table, void* ws, size_t ws_bytes, hipStream_t s, bool overwrite,
                                const MainGradArg& main, int32_t* nonfinite, const FixedSum& sum) {
    if ((main.src || sum.count) && !eps) return hipErrorInvalidValue;  // these ride on the pair form only
#define H4D_SCATTER(GG, PP) \
    tiled_g<GG, PP>(g, level_rows, xyzt, eps, n, src, ls, qs, scale, d_table, ws, ws_bytes, overwrite, main, nonfinite, \
                    sum, s)
    if (grad_dt == H4D_F64) return eps ? H4D_SCATTER(double, true) : H4D_SCATTER(double, false);
    return eps ? H4D_SCATTER(float, true) : H4D_SCATTER(float, false);
#undef H4D_SCATTER
}

// ------------------------------------------ static workspace (no allocation) ----
// The pair lists of hash4d_encode_backward_noalloc live in this file-scope array:
// each GPU holds its own copy from module load until the process ends, and every
// call on that GPU shares it.  On the host the array's name is only a stand-in, not
// a device address: its address on the current device is looked up once per device
// with hipGetSymbolAddress and cached, and only that address is ever passed on.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

hipError_t static_scratch(void** ptr) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void* addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return hipSuccess;
}

hipError_t launch_corner_indices(const DevGrid& g, const float* xyzt, int n, int32_t* rows, float* w, hipStream_t s) {
    hipLaunchKernelGGL(k_corner_indices, level_major_grid(n, g.L), dim3(kEncodeBlock), 0, s, g,
                       reinterpret_cast<const float4*>(xyzt), n, rows, w);
    return hipGetLastError();
}

}  // namespace h4d
