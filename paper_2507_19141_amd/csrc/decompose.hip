// Self-supervised dynamic-static split (DASH Section 4.1, Eqs. 4-5): the step that
// decides which Gaussians the 4D hash path deforms.
//
// Keys: the FP32 squared motion magnitude s = (dx^2 + dy^2) + dz^2 of each
// Gaussian's linear-motion vector dp, rounded step by step (no fused multiply-add)
// and ordered by its bit pattern (s >= 0, so the bits order like the values; NaN
// ranks above +Inf).  The threshold tau is the (n_d + 1)-th largest key, found by an
// exact radix select (four passes over 8-bit digits, most significant first); a
// Gaussian is dynamic iff its key is strictly greater than tau.  The dynamic indices
// are then written in ascending order (a stable compaction), and the static ones get
// the static constraint lam_s / N_s * sum ||dp|| and its gradient.
#include "h4d_device.h"

namespace h4d {

constexpr int kDecBlock = 256;

// (x^2 + y^2) + z^2 in FP32, each product and sum rounded on its own: contraction is
// off in this block, so no step becomes a fused multiply-add.
__device__ __forceinline__ uint32_t motion_key(const float* __restrict__ dp, int64_t i) {
#pragma clang fp contract(off)
    const float x = dp[3 * i], y = dp[3 * i + 1], z = dp[3 * i + 2];
    const float s = (x * x + y * y) + z * z;
    return __float_as_uint(s);
}

// A pass reads 12 bytes per Gaussian, so the launches were what the split took its time
// for: 11 of them, 42 us for 200k Gaussians.  Now each kernel starts with the reduction
// that its predecessor left, every workgroup for itself (the pick of a digit from 256
// bins; the sums of the block counts): 7 launches, 28 us.  Letting the workgroup that
// ends a pass last pick its digit took 8.5 us per pass, against 4.0 + 2.3 in two launches:
// every workgroup's release writes its L2 back.

// What a pass knows of the sought key: its digits so far, the rank still sought among the
// keys with that prefix (ascending, 0-based), and 1 in `all` when there is no threshold
// (every Gaussian dynamic).  State p is the one before digit p, state kDigits the threshold.
struct SelectState {
    uint32_t prefix, rank, all, pad;
};
constexpr int kDigits = 4;

__global__ __launch_bounds__(kDecBlock) void k_select_init(SelectState* st, uint32_t* hist, int words, int64_t n,
                                                           int64_t n_d) {
    if (threadIdx.x == 0)  // the (n_d + 1)-th largest, counted from below
        st[0] = SelectState{0u, n_d >= n ? 0u : (uint32_t)(n - n_d - 1), n_d >= n ? 1u : 0u, 0u};
    for (int j = threadIdx.x; j < words; j += kDecBlock) hist[j] = 0u;
}

// State p (> 0) from the one before and that digit's histogram: the bucket holding the
// sought rank extends the prefix.  Called by all threads; workgroup 0 stores the state
// for the next launch.
__device__ __forceinline__ SelectState pick_digit(SelectState* __restrict__ st, const uint32_t* __restrict__ hist,
                                                  int p) {
    __shared__ uint32_t wsum[kDecBlock / 64];
    __shared__ SelectState found;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const SelectState cur = st[p - 1];
    const uint32_t v = hist[threadIdx.x];
    uint32_t c = v;  // inclusive scan
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t a = (uint32_t)__shfl_up((int)c, d, 64);
        if (lane >= d) c += a;
    }
    if (lane == 63) wsum[wave] = c;
    __syncthreads();
    for (int w = 0; w < wave; ++w) c += wsum[w];
    if (c - v <= cur.rank && cur.rank < c) {  // exactly one bucket: the rank exists
        found = SelectState{cur.prefix | (uint32_t)threadIdx.x << (32 - 8 * p), cur.rank - (c - v), cur.all, 0u};
        if (blockIdx.x == 0) st[p] = found;
    }
    __syncthreads();
    return found;
}

// The pick as a launch of its own, where the workspace holds one histogram only: it is
// cleared for the next digit.
__global__ __launch_bounds__(kDecBlock) void k_select_pick(SelectState* __restrict__ st, uint32_t* __restrict__ hist,
                                                           int p) {
    pick_digit(st, hist, p);
    hist[threadIdx.x] = 0u;
}

// Histogram of digit p over the keys whose higher digits equal the prefix; state p is
// picked from `prev`, the last digit's histogram, unless that is NULL.
__global__ __launch_bounds__(kDecBlock) void k_select_hist(const float* __restrict__ dp, int64_t n,
                                                           SelectState* __restrict__ st, int p,
                                                           const uint32_t* __restrict__ prev,
                                                           uint32_t* __restrict__ hist) {
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0u;
    const uint32_t prefix = prev ? pick_digit(st, prev, p).prefix : st[p].prefix;
    __syncthreads();
    const int shift = 24 - 8 * p;
    const uint32_t hi_mask = p == 0 ? 0u : ~((1u << (shift + 8)) - 1u);
    for (int64_t i = (int64_t)blockIdx.x * kDecBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kDecBlock) {
        const uint32_t k = motion_key(dp, i);
        if ((k & hi_mask) == prefix) atomicAdd(&h[(k >> shift) & 255u], 1u);
    }
    __syncthreads();
    if (h[threadIdx.x]) atomicAdd(&hist[threadIdx.x], h[threadIdx.x]);
}

__device__ __forceinline__ bool is_dynamic(uint32_t key, const SelectState& s) { return s.all || key > s.prefix; }

// Per workgroup: dynamic count and the sum of the static magnitudes (FP32 norm) of `per`
// runs of kDecBlock Gaussians.  The threshold is picked from `prev` unless that is NULL.
__global__ __launch_bounds__(kDecBlock) void k_split_count(const float* __restrict__ dp, int64_t n, int per,
                                                           SelectState* __restrict__ st,
                                                           const uint32_t* __restrict__ prev,
                                                           uint32_t* __restrict__ counts, float* __restrict__ sums) {
    __shared__ uint32_t wc[kDecBlock / 64];
    __shared__ float ws[kDecBlock / 64];
    const SelectState s = prev ? pick_digit(st, prev, kDigits) : st[kDigits];
    uint32_t c = 0u;
    float mag = 0.f;
    for (int r = 0; r < per; ++r) {
        const int64_t i = ((int64_t)blockIdx.x * per + r) * kDecBlock + threadIdx.x;
        bool dyn = false;
        if (i < n) {
            dyn = is_dynamic(motion_key(dp, i), s);
            if (!dyn) {
                const float x = dp[3 * i], y = dp[3 * i + 1], z = dp[3 * i + 2];
                mag += sqrtf(x * x + y * y + z * z);
            }
        }
        c += (uint32_t)__popcll(__ballot(dyn));
    }
    for (int o = 32; o > 0; o >>= 1) mag += __shfl_xor(mag, o, 64);
    if ((threadIdx.x & 63) == 0) {
        wc[threadIdx.x >> 6] = c;
        ws[threadIdx.x >> 6] = mag;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t tc = 0;
        float ts = 0.f;
        for (int w = 0; w < kDecBlock / 64; ++w) {
            tc += wc[w];
            ts += ws[w];
        }
        counts[blockIdx.x] = tc;
        sums[blockIdx.x] = ts;
    }
}

// Dynamic: index written at its ascending position.  Static: the constraint's gradient.
// Each workgroup adds up the counts before its own and all of them (integers: every one
// gets the same total); workgroup 0 adds the static constraint to *loss, the sums in a
// fixed order and in 64 bits.
__global__ __launch_bounds__(kDecBlock) void k_split_write(const float* __restrict__ dp, int64_t n, int per,
                                                           const SelectState* __restrict__ st,
                                                           const uint32_t* __restrict__ counts,
                                                           const float* __restrict__ sums, float lam_s,
                                                           int32_t* __restrict__ dyn_idx,
                                                           int32_t* __restrict__ n_dynamic,
                                                           uint8_t* __restrict__ is_dyn, float* __restrict__ loss,
                                                           float* __restrict__ d_dp) {
    constexpr int kWaves = kDecBlock / 64;
    __shared__ uint32_t wb[kWaves], wt[kWaves], wc[kWaves];
    __shared__ double wf[kWaves];
    const SelectState s = st[kDigits];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nb = (int)gridDim.x, b = (int)blockIdx.x;
    uint32_t before = 0u, total = 0u;
    for (int j = threadIdx.x; j < nb; j += kDecBlock) {
        const uint32_t c = counts[j];
        total += c;
        if (j < b) before += c;
    }
    double f = 0.0;
    if (b == 0 && loss)
        for (int j = threadIdx.x; j < nb; j += kDecBlock) f += (double)sums[j];
    for (int o = 32; o > 0; o >>= 1) {
        before += (uint32_t)__shfl_xor((int)before, o, 64);
        total += (uint32_t)__shfl_xor((int)total, o, 64);
        if (b == 0) f += __shfl_xor(f, o, 64);
    }
    if (lane == 0) {
        wb[wave] = before;
        wt[wave] = total;
        wf[wave] = f;
    }
    __syncthreads();
    uint32_t pos0 = 0u, n_dyn = 0u;
    for (int w = 0; w < kWaves; ++w) {
        pos0 += wb[w];
        n_dyn += wt[w];
    }
    const int64_t n_s = n - (int64_t)n_dyn;
    if (b == 0 && threadIdx.x == 0) {
        if (n_dynamic) *n_dynamic = (int32_t)n_dyn;
        if (loss && n_s > 0) *loss += lam_s / (float)n_s * (float)(((wf[0] + wf[1]) + wf[2]) + wf[3]);
    }
    for (int r = 0; r < per; ++r) {
        const int64_t i = ((int64_t)b * per + r) * kDecBlock + threadIdx.x;
        const bool dyn = i < n && is_dynamic(motion_key(dp, i), s);
        const uint64_t bal = __ballot(dyn);
        if (r > 0) __syncthreads();  // the last run's counts are read
        if (lane == 0) wc[wave] = (uint32_t)__popcll(bal);
        __syncthreads();
        uint32_t pos = pos0 + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
        for (int w = 0; w < kWaves; ++w) {
            if (w < wave) pos += wc[w];
            pos0 += wc[w];
        }
        if (i >= n) continue;
        if (is_dyn) is_dyn[i] = dyn ? 1 : 0;
        if (dyn) {
            if (dyn_idx) dyn_idx[pos] = (int32_t)i;
        } else if (d_dp) {
            const float x = dp[3 * i], y = dp[3 * i + 1], z = dp[3 * i + 2];
            const float mag = sqrtf(x * x + y * y + z * z);
            if (mag > 0.f) {
                const float c = lam_s / (float)n_s / mag;
                d_dp[3 * i] += c * x;
                d_dp[3 * i + 1] += c * y;
                d_dp[3 * i + 2] += c * z;
            }
        }
    }
}

// Small splits in one launch of one workgroup: every Gaussian's key stays in a register of
// its thread (up to 16 of them), so nothing but the outputs leaves the CU.  1000 Gaussians
// 40 -> 10 us, 16000 38 -> 27 us, a microsecond more per 1000: one CU's loads and LDS
// atomics.  Past 16 keys a thread would read them again for each digit, and near 30k it
// would take as long as the launches.
constexpr int kSmallBlock = 1024, kSmallRuns = 16;

// Inclusive sums over the first 256 threads' values; called by all threads, with barriers.
__device__ __forceinline__ uint32_t scan256(uint32_t v, uint32_t* wsum) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t c = v;
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t a = (uint32_t)__shfl_up((int)c, d, 64);
        if (lane >= d) c += a;
    }
    if (lane == 63 && wave < 4) wsum[wave] = c;
    __syncthreads();
    for (int w = 0; w < 4; ++w)
        if (w < wave) c += wsum[w];
    __syncthreads();
    return c;
}

__global__ __launch_bounds__(kSmallBlock) void k_split_small(const float* __restrict__ dp, int n, int64_t n_d,
                                                             float lam_s, int32_t* __restrict__ dyn_idx,
                                                             int32_t* __restrict__ n_dynamic,
                                                             uint8_t* __restrict__ is_dyn, float* __restrict__ loss,
                                                             float* __restrict__ d_dp) {
    constexpr int kWaves = kSmallBlock / 64;
    __shared__ uint32_t h[256], wsum[4], total;
    __shared__ uint32_t found[2];              // the key's digits so far, the rank sought among them
    __shared__ uint32_t place[kSmallRuns * kWaves];
    __shared__ float wf[kWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t k[kSmallRuns];
#pragma unroll
    for (int r = 0; r < kSmallRuns; ++r) {
        const int i = r * kSmallBlock + tid;
        k[r] = i < n ? motion_key(dp, i) : 0u;
    }
    const bool all = n_d >= n;
    if (tid == 0) {  // the (n_d + 1)-th largest, counted from below
        found[0] = 0u;
        found[1] = all ? 0u : (uint32_t)(n - n_d - 1);
    }
    for (int shift = 24; shift >= 0; shift -= 8) {
        if (tid < 256) h[tid] = 0u;
        __syncthreads();
        const uint32_t prefix = found[0], rank = found[1];
        const uint32_t hi_mask = shift == 24 ? 0u : ~((1u << (shift + 8)) - 1u);
#pragma unroll
        for (int r = 0; r < kSmallRuns; ++r)
            if (r * kSmallBlock + tid < n && (k[r] & hi_mask) == prefix) atomicAdd(&h[(k[r] >> shift) & 255u], 1u);
        __syncthreads();
        const uint32_t v = tid < 256 ? h[tid] : 0u;
        const uint32_t c = scan256(v, wsum);
        if (tid < 256 && c - v <= rank && rank < c) {  // exactly one bucket: the rank exists
            found[0] = prefix | (uint32_t)tid << shift;
            found[1] = rank - (c - v);
        }
        __syncthreads();
    }
    const uint32_t tau = found[0];
    float mag = 0.f;
#pragma unroll
    for (int r = 0; r < kSmallRuns; ++r) {
        const int i = r * kSmallBlock + tid;
        const bool dyn = i < n && (all || k[r] > tau);
        const uint64_t bal = __ballot(dyn);
        if (lane == 0) place[r * kWaves + wave] = (uint32_t)__popcll(bal);
        if (i < n && !dyn) {
            const float x = dp[3 * i], y = dp[3 * i + 1], z = dp[3 * i + 2];
            mag += sqrtf(x * x + y * y + z * z);
        }
    }
    for (int o = 32; o > 0; o >>= 1) mag += __shfl_xor(mag, o, 64);
    if (lane == 0) wf[wave] = mag;
    __syncthreads();
    const uint32_t v = tid < 256 ? place[tid] : 0u;
    const uint32_t c = scan256(v, wsum);
    if (tid < 256) place[tid] = c - v;
    if (tid == 255) total = c;
    __syncthreads();
    const uint32_t n_dyn = total;
    const int n_s = n - (int)n_dyn;
    if (tid == 0) {
        if (n_dynamic) *n_dynamic = (int32_t)n_dyn;
        if (loss && n_s > 0) {
            double f = 0.0;
            for (int w = 0; w < kWaves; ++w) f += (double)wf[w];
            *loss += lam_s / (float)n_s * (float)f;
        }
    }
#pragma unroll
    for (int r = 0; r < kSmallRuns; ++r) {
        const int i = r * kSmallBlock + tid;
        const bool dyn = i < n && (all || k[r] > tau);
        const uint64_t bal = __ballot(dyn);
        if (i >= n) continue;
        if (is_dyn) is_dyn[i] = dyn ? 1 : 0;
        if (dyn) {
            if (dyn_idx) dyn_idx[place[r * kWaves + wave] + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull))] = i;
        } else if (d_dp) {
            const float x = dp[3 * i], y = dp[3 * i + 1], z = dp[3 * i + 2];
            const float m = sqrtf(x * x + y * y + z * z);
            if (m > 0.f) {
                const float g = lam_s / (float)n_s / m;
                d_dp[3 * i] += g * x;
                d_dp[3 * i + 1] += g * y;
                d_dp[3 * i + 2] += g * z;
            }
        }
    }
}

// 256 bytes of states, and words for one histogram and three per kDecBlock Gaussians.
size_t decompose_workspace_bytes(int64_t n) {
    const int64_t nb = (n + kDecBlock - 1) / kDecBlock;
    return 256 + 256 * 4 + (size_t)nb * 4 * 3;
}

// What lies in the workspace: histograms, and the counts and sums of the split's
// workgroups, each of which covers `per` runs of kDecBlock Gaussians.
struct SplitPlan {
    int hists;   // 1, or kDigits from 256 runs on, where they fit
    int blocks, per;
    int counts;  // word of the first count; the sums follow the counts
};
static SplitPlan split_plan(int64_t n) {
    const int64_t runs = (n + kDecBlock - 1) / kDecBlock;
    constexpr int kHist = 256;
    SplitPlan p;
    p.hists = runs >= 256 ? kDigits : 1;
    // every workgroup of k_split_write reads all the counts, so at most 2048 of them; below
    // 3 * 256 runs the counts lie over the histograms of the digits before the last
    const bool over = p.hists == kDigits && runs < 3 * kHist;
    const int64_t most = over ? (kDigits - 1) * kHist / 2 : 2048;
    p.per = (int)((runs + most - 1) / most);
    p.blocks = (int)((runs + p.per - 1) / p.per);
    p.counts = over ? 0 : p.hists * kHist;
    return p;
}

hipError_t launch_decompose(const float* dp, int64_t n, double k_percent, float lam_s, int32_t* dyn_idx,
                            int32_t* n_dynamic, uint8_t* is_dyn, float* loss, float* d_dp, void* ws, hipStream_t s) {
    const int64_t n_d = (int64_t)floor(k_percent / 100.0 * (double)n);
    if (n <= kSmallBlock * kSmallRuns) {
        hipLaunchKernelGGL(k_split_small, dim3(1), dim3(kSmallBlock), 0, s, dp, (int)n, n_d, lam_s, dyn_idx, n_dynamic,
                           is_dyn, loss, d_dp);
        return hipGetLastError();
    }
    const SplitPlan pl = split_plan(n);
    SelectState* st = static_cast<SelectState*>(ws);
    uint32_t* hist = reinterpret_cast<uint32_t*>(static_cast<char*>(ws) + 256);
    uint32_t* counts = hist + pl.counts;
    float* sums = reinterpret_cast<float*>(counts + pl.blocks);
    hipLaunchKernelGGL(k_select_init, dim3(1), dim3(kDecBlock), 0, s, st, hist, pl.hists * 256, n, n_d);
    // 256 device atomics per workgroup and pass
    const int hist_blocks = (int)std::min<int64_t>((n + kDecBlock - 1) / kDecBlock, 256);
    const uint32_t* prev = nullptr;
    for (int p = 0; p < kDigits; ++p) {
        uint32_t* h = pl.hists == 1 ? hist : hist + p * 256;
        hipLaunchKernelGGL(k_select_hist, dim3(hist_blocks), dim3(kDecBlock), 0, s, dp, n, st, p, prev, h);
        if (pl.hists == 1)
            hipLaunchKernelGGL(k_select_pick, dim3(1), dim3(kDecBlock), 0, s, st, h, p + 1);
        else
            prev = h;
    }
    hipLaunchKernelGGL(k_split_count, dim3((unsigned)pl.blocks), dim3(kDecBlock), 0, s, dp, n, pl.per, st, prev, counts,
                       sums);
    hipLaunchKernelGGL(k_split_write, dim3((unsigned)pl.blocks), dim3(kDecBlock), 0, s, dp, n, pl.per, st, counts, sums,
                       lam_s, dyn_idx, n_dynamic, is_dyn, loss, d_dp);
    return hipGetLastError();
}

}  // namespace h4d
