// Spatio-temporal smoothness regulariser (DASH Section 4.3, Eq. 11), first pass:
//   L_r = lam / n * sum_q || G(x_q) - G(clamp(x_q + eps_q)) ||^2
// and, when asked, the per-(query, level) difference d = G(x) - G(x~) written
// level-major for the table-gradient pass (the tiled scatter with the pair of
// corner sets, scaled by 2 lam / n).  Both encodes are recomputed per (query,
// level); when x and x~ fall in the same hypervoxel (the coarse levels for a small
// eps) their 16 corners coincide and one gather per corner gives d with the weight
// difference w - w~.  Work items (level, 256 queries) are placed on XCDs level by
// level, and neighbouring lanes gather corners together, both as in the encoder.
#include "h4d_device.h"

namespace h4d {

constexpr int kSmoothBlock = 256;

template <typename TT, int F, bool WIDE>
__global__ __launch_bounds__(kSmoothBlock) void k_smooth(DevGrid g, const TT* __restrict__ table,
                                                         const float4* __restrict__ xyzt,
                                                         const float4* __restrict__ eps, int n,
                                                         typename AccOf<TT>::type lam_over_n,
                                                         typename AccOf<TT>::type* __restrict__ loss,
                                                         typename AccOf<TT>::type* __restrict__ sums,
                                                         typename AccOf<TT>::type* __restrict__ d_out) {
    using A = typename AccOf<TT>::type;
    __shared__ A red[kSmoothBlock / 64];
    const int chunks = (n + kSmoothBlock - 1) / kSmoothBlock;
    int l, chunk;
    if (!xcd_item(g.L * chunks, chunks, l, chunk)) return;
    const int q = chunk * kSmoothBlock + threadIdx.x;
    A part = A(0);
    {   // every lane takes part in the gathers
        const float4 x = xyzt[min(q, n - 1)];
        const float4 e = eps[min(q, n - 1)];
        const float4 xp = make_float4(__fadd_rn(x.x, e.x), __fadd_rn(x.y, e.y), __fadd_rn(x.z, e.z), __fadd_rn(x.w, e.w));
        const Cell c0 = level_cell(g, l, x);
        const Cell c1 = level_cell(g, l, xp);
        const bool same = c0.ix == c1.ix && c0.iy == c1.iy && c0.iz == c1.iz && c0.it == c1.it;
        const CornerWeights<A, (kPairGroup<TT, F> < 8)> w0(c0), w1(c1);
        A d[F], a0[F];
#pragma unroll
        for (int f = 0; f < F; ++f) d[f] = a0[f] = A(0);
        each_pair<TT, F, WIDE>(g, l, table, c0, [&](int p, const A (&lo)[F], const A (&hi)[F]) {
            A l0, h0, l1, h1;
            w0.pair(p, l0, h0);
            w1.pair(p, l1, h1);
            const A dl = l0 - l1, dh = h0 - h1;
#pragma unroll
            for (int f = 0; f < F; ++f) {
                d[f] += dl * lo[f];
                a0[f] += l0 * lo[f];
            }
#pragma unroll
            for (int f = 0; f < F; ++f) {
                d[f] += dh * hi[f];
                a0[f] += h0 * hi[f];
            }
        });
        // the second cell's corners, where it differs in either lane of the pair
        const bool other = lane_swap(same ? 0u : 1u) != 0u;
        if (!same || other) {
            A a1[F];
            interpolate<TT, F, WIDE>(g, l, table, c1, a1);
            if (!same) {
#pragma unroll
                for (int f = 0; f < F; ++f) d[f] = a0[f] - a1[f];
            }
        }
        if (q < n) {
#pragma unroll
        for (int f = 0; f < F; ++f) part += d[f] * d[f];
        if (d_out) {
            A* o = d_out + ((int64_t)l * n + q) * F;
#pragma unroll
            for (int f = 0; f < F; ++f) o[f] = d[f];
        }
        }
    }
    // sum of the workgroup's squared differences: into its place in sums, or (no memory for
    // them) added to the loss with an atomic
    for (int s = 32; s > 0; s >>= 1) part += __shfl_xor(part, s, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = part;
    __syncthreads();
    if (threadIdx.x == 0) {
        A b = A(0);
        for (int w = 0; w < kSmoothBlock / 64; ++w) b += red[w];
        if (sums) sums[(int64_t)l * chunks + chunk] = b;
        else if (b != A(0)) atomic_add(loss, lam_over_n * b);
    }
}

template <typename TT>
static hipError_t smooth_t(const DevGrid& g, const void* table, const float* xyzt, const float* eps, int n, double lam,
                           void* loss, void* d_out, void* sums, FixedSum* rest, hipStream_t s) {
    using A = typename AccOf<TT>::type;
    const int chunks = (n + kSmoothBlock - 1) / kSmoothBlock;
    const dim3 grid((unsigned)(kXcds * xcd_items_per(g.L * chunks))), block(kSmoothBlock);
    const TT* t = static_cast<const TT*>(table);
    const float4* x = reinterpret_cast<const float4*>(xyzt);
    const float4* e = reinterpret_cast<const float4*>(eps);
    const A c = (A)(lam / (double)n);
    A* lo = static_cast<A*>(loss);
    A* dd = static_cast<A*>(d_out);
    A* su = static_cast<A*>(sums);
#define H4D_SMOOTH(FF, WW) hipLaunchKernelGGL((k_smooth<TT, FF, WW>), grid, block, 0, s, g, t, x, e, n, c, lo, su, dd)
    switch (g.F) {
        case 1:
            if (can_widen<TT, 1>(table, g.rows)) H4D_SMOOTH(1, true);
            else H4D_SMOOTH(1, false);
            break;
        case 2:
            if (can_widen<TT, 2>(table, g.rows)) H4D_SMOOTH(2, true);
            else H4D_SMOOTH(2, false);
            break;
        case 4: H4D_SMOOTH(4, false); break;
        case 8: H4D_SMOOTH(8, false); break;
        default: return hipErrorInvalidValue;
    }
#undef H4D_SMOOTH
    if (sums) {
        rest->sums = sums;
        rest->out = loss;
        rest->scale = lam / (double)n;
        rest->count = g.L * chunks;
        rest->f64 = sizeof(A) == 8;
    }
    return hipGetLastError();
}

size_t smoothness_sum_bytes(int L, int n) {
    return (size_t)L * (((size_t)n + kSmoothBlock - 1) / kSmoothBlock) * sizeof(double);
}

hipError_t launch_smoothness(const DevGrid& g, h4d_dtype dt, const void* table, const float* xyzt, const float* eps,
                             int n, double lam, void* loss, void* d_out, void* sums, FixedSum* rest, hipStream_t s) {
    switch (dt) {
        case H4D_F32: return smooth_t<float>(g, table, xyzt, eps, n, lam, loss, d_out, sums, rest, s);
        case H4D_BF16: return smooth_t<bf16_t>(g, table, xyzt, eps, n, lam, loss, d_out, sums, rest, s);
        case H4D_F64: return smooth_t<double>(g, table, xyzt, eps, n, lam, loss, d_out, sums, rest, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace h4d
