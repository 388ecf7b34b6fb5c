// Posterior-predictive bands (Sec. 5: 120-day projections from accepted
// samples with the 5th-95th percentile band): per day and compartment, the
// requested quantiles of n recorded trajectories, and its C-ABI entry point
// abc_trajectory_bands. Each quantile interpolates linearly between order
// statistics h = (n - 1) q in float64; the order statistics of few rows are found
// by sorting them in registers, of many by bisection on the value.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.hpp"

namespace abc {

constexpr int BANDS_MAX_N = 8192;
constexpr int BANDS_MAX_Q = 16;

struct BandArgs {
    const int32_t* traj;  // [n][T+1][6]
    int64_t n;
    int32_t T;
    int32_t nq;
    double q[BANDS_MAX_Q];
    float* out;           // [nq][T+1][6]
};

// unsigned image of an int32 that keeps its order
__device__ __forceinline__ uint32_t ordered(int32_t x) { return (uint32_t)x ^ 0x80000000u; }

// Quantile k between the order statistics lo (x) and lo + 1 (y). What the rounding of
// (n - 1) q took away stays in the fraction: (n - 1) q - lo, rounded once.
__device__ __forceinline__ void store_quantile(const BandArgs& a, int k, int day, int c, int lo, uint32_t x, uint32_t y)
{
    const double t = fma((double)(a.n - 1), a.q[k], -(double)lo);
    const double p = (double)(int32_t)(x ^ 0x80000000u), q = (double)(int32_t)(y ^ 0x80000000u);
    a.out[((int64_t)k * (a.T + 1) + day) * 6 + c] = (float)fma(q - p, t, p);
}

constexpr int BANDS_CAND = 4;  // values per lane once few are left

// values up to mid of a wavefront's V per lane
template <int V>
__device__ __forceinline__ int count_up_to(const uint32_t (&v)[V], uint32_t mid)
{
    uint32_t own = 0;
#pragma unroll
    for (int e = 0; e < V; ++e) own += v[e] <= mid ? 1u : 0u;
    int cnt = 0;
#pragma unroll
    for (int b = 0; (V >> b) > 0; ++b) cnt += __popcll(__ballot((own >> b) & 1u)) << b;
    return cnt;
}

template <int V>
__device__ __forceinline__ uint32_t least_above(const uint32_t (&v)[V], uint32_t x)
{
    uint32_t y = 0xFFFFFFFFu;
#pragma unroll
    for (int e = 0; e < V; ++e) y = min(y, v[e] > x ? v[e] : 0xFFFFFFFFu);
#pragma unroll
    for (int off = 32; off; off >>= 1) y = min(y, (uint32_t)__shfl_xor((int)y, off, 64));
    return y;
}

// A workgroup takes half the compartments of a day, four wavefronts each. A
// wavefront holds the n values in registers, V per lane, and finds the order
// statistics of one quantile at a time by bisection on the value: a step counts
// the values up to the middle, two instructions per 64 values, with no barrier
// and no memory. Once 256 values or fewer lie in the interval they alone are
// kept. Counted values bound it beyond some 2000 rows, below that the loads: a
// row's three compartments are one load, since every row is a line of its own.
// 121 days, three quantiles, 1000 / 2048 / 8192 rows: 10 / 15 / 51 us; sorting
// each (day, compartment) in LDS took 38 / 78 / 358 us.
template <int V>
__global__ __launch_bounds__(768) void k_bands(BandArgs a)
{
    __shared__ uint32_t vs[3][V * 64];
    __shared__ uint32_t cand[12][64 * BANDS_CAND];
    const int day = blockIdx.x, half = blockIdx.y;
    const int n = (int)a.n, lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = wv >> 2;
    {
        const int32_t* src = a.traj + (int64_t)day * 6 + half * 3;
        constexpr int E = (V * 64 + 767) / 768;
        int32_t x[E][3];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int r = e * 768 + threadIdx.x;
            const int32_t* q = src + (int64_t)(r < n ? r : 0) * (a.T + 1) * 6;
            x[e][0] = q[0]; x[e][1] = q[1]; x[e][2] = q[2];
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int r = e * 768 + threadIdx.x;
            if (r < V * 64)
#pragma unroll
                for (int k = 0; k < 3; ++k) vs[k][r] = r < n ? ordered(x[e][k]) : 0xFFFFFFFFu;
        }
    }
    __syncthreads();
    if (4 * (int)blockIdx.z + (wv & 3) >= a.nq) return;
    uint32_t v[V], vmin = 0xFFFFFFFFu, vmax = 0u;
#pragma unroll
    for (int e = 0; e < V; ++e) {
        v[e] = vs[c][e * 64 + lane];
        vmin = min(vmin, v[e]);
        vmax = max(vmax, e * 64 + lane < n ? v[e] : 0u);
    }
#pragma unroll
    for (int off = 32; off; off >>= 1) {
        vmin = min(vmin, (uint32_t)__shfl_xor((int)vmin, off, 64));
        vmax = max(vmax, (uint32_t)__shfl_xor((int)vmax, off, 64));
    }
    vmin = __builtin_amdgcn_readfirstlane(vmin);
    vmax = __builtin_amdgcn_readfirstlane(vmax);
    for (int k = 4 * blockIdx.z + (wv & 3); k < a.nq; k += 4 * gridDim.z) {
        const double h = (double)(a.n - 1) * a.q[k];
        int lo = (int)floor(h);
        if (lo > n - 1) lo = n - 1;
        const int hi = lo + 1 < n ? lo + 1 : lo;
        // the smallest value x with more than lo values up to it lies in
        // [x, top]; below values lie under x, upto are no larger than top
        uint32_t x = vmin, top = vmax;
        int below = 0, upto = n;
        while (x < top && upto - below > 64 * BANDS_CAND) {
            const uint32_t mid = x + ((top - x) >> 1);
            const int cnt = count_up_to(v, mid);
            if (cnt > lo) { top = mid; upto = cnt; }
            else { x = mid + 1u; below = cnt; }
        }
        uint32_t y = x;  // the order statistic after it
        if (x < top) {
            uint32_t* own = cand[wv];
            int m = 0;
#pragma unroll
            for (int e = 0; e < V; ++e) {
                const bool in = v[e] >= x && v[e] <= top && e * 64 + lane < n;
                const uint64_t b = __ballot(in);
                if (in) own[m + (int)mask_rank(b)] = v[e];
                m += __popcll(b);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            const uint32_t last = top;
            uint32_t u[BANDS_CAND];
#pragma unroll
            for (int e = 0; e < BANDS_CAND; ++e) u[e] = e * 64 + lane < m ? own[e * 64 + lane] : 0xFFFFFFFFu;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            while (x < top) {
                const uint32_t mid = x + ((top - x) >> 1);
                if (below + count_up_to(u, mid) > lo) top = mid; else x = mid + 1u;
            }
            // ranks of values below `last` are counted among the kept ones
            const int cnt = x < last ? below + count_up_to(u, x) : upto;
            if (cnt > hi) y = x;
            else y = cnt < upto ? least_above(u, x) : least_above(v, x);
        } else if (upto <= hi) {
            y = least_above(v, x);
        }
        if (lane == 0) {
            store_quantile(a, k, day, half * 3 + c, lo, x, y);
        }
    }
}

// Ascending bitonic sort of a wavefront's 64 V values; value e of lane l is number
// 64 e + l.
template <int V>
__device__ __forceinline__ void sort_values(uint32_t (&v)[V], int lane)
{
#pragma unroll
    for (int k = 2; k <= 64 * V; k <<= 1)
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1)
#pragma unroll
            for (int e = 0; e < V; ++e) {
                const bool up = k < 64 ? (lane & k) == 0 : (e & (k >> 6)) == 0;
                if (j >= 64) {
                    const int p = e | (j >> 6);
                    if (p != e) {
                        const uint32_t x = min(v[e], v[p]), y = max(v[e], v[p]);
                        v[e] = up ? x : y;
                        v[p] = up ? y : x;
                    }
                } else {
                    const uint32_t o = (uint32_t)__shfl_xor((int)v[e], j, 64);
                    v[e] = ((lane & j) == 0) == up ? min(v[e], o) : max(v[e], o);
                }
            }
}

// Few rows: a wavefront sorts the values of a (day, compartment) in its registers,
// without a barrier, and a lane forms each quantile. Bisection is a search a
// quantile: of 121 days, with 1 / 3 / 16 quantiles, the whole call, 10 rows took
// 29 / 29 / 44 us, now 26; 256 rows 29 / 29 / 45, now 26; 512 rows 34 / 34 / 61, now
// 30 (from 1000 on bisection is ahead with few quantiles).
template <int V>
__global__ __launch_bounds__(192) void k_bands_few(BandArgs a)
{
    __shared__ uint32_t sorted[3][64 * V];
    const int day = blockIdx.x, half = blockIdx.y;
    const int n = (int)a.n, lane = threadIdx.x & 63;
    const int c = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int32_t* src = a.traj + (int64_t)day * 6 + half * 3 + c;
    uint32_t v[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
        const int r = e * 64 + lane;
        v[e] = ordered(src[(int64_t)(r < n ? r : 0) * (a.T + 1) * 6]);
    }
#pragma unroll
    for (int e = 0; e < V; ++e) v[e] = e * 64 + lane < n ? v[e] : 0xFFFFFFFFu;
    sort_values(v, lane);
#pragma unroll
    for (int e = 0; e < V; ++e) sorted[c][e * 64 + lane] = v[e];
    wave_lds_sync();
    if (lane < a.nq) {
        const double h = (double)(a.n - 1) * a.q[lane];
        int lo = (int)floor(h);
        if (lo > n - 1) lo = n - 1;
        store_quantile(a, lane, day, half * 3 + c, lo, sorted[c][lo], sorted[c][lo + 1 < n ? lo + 1 : lo]);
    }
}

template <int V>
static void launch_bands_few(const BandArgs& a, hipStream_t s)
{
    hipLaunchKernelGGL((k_bands_few<V>), dim3(a.T + 1, 2), dim3(192), 0, s, a);
}

template <int V>
static void launch_bands(const BandArgs& a, hipStream_t s)
{
    // more than four quantiles: workgroups of their own, unless the values fill half
    // a CU's LDS (16 quantiles of 1000 rows 63 -> 56 us, of 8192 rows 244 and 322)
    const unsigned z = V <= 32 ? (unsigned)(a.nq + 3) / 4 : 1u;
    hipLaunchKernelGGL((k_bands<V>), dim3(a.T + 1, 2, z), dim3(768), 0, s, a);
}

}  // namespace abc

using namespace abc;

extern "C" abc_status abc_trajectory_bands(const int32_t* traj, int64_t n, int32_t T,
                                           const double* q, int32_t nq, float* out, void* stream)
{
    ABC_REQUIRE(traj && q && out, "NULL argument");
    ABC_REQUIRE(n >= 1 && n <= BANDS_MAX_N, "n must be in [1, %d]", BANDS_MAX_N);
    ABC_REQUIRE(T >= 0 && T <= ABC_T_MAX, "T out of range");
    ABC_REQUIRE(nq >= 1 && nq <= BANDS_MAX_Q, "nq must be in [1, %d]", BANDS_MAX_Q);
    BandArgs a{};
    a.traj = traj;
    a.n = n;
    a.T = T;
    a.nq = nq;
    for (int k = 0; k < nq; ++k) {
        ABC_REQUIRE(q[k] >= 0.0 && q[k] <= 1.0, "quantile %d outside [0, 1]", k);
        a.q[k] = q[k];
    }
    a.out = out;
    const hipStream_t s = as_stream(stream);
    if (n <= 64) launch_bands_few<1>(a, s);
    else if (n <= 64 * 4) launch_bands_few<4>(a, s);
    else if (n <= 64 * 8) launch_bands_few<8>(a, s);
    else if (n <= 64 * 16) launch_bands<16>(a, s);
    else if (n <= 64 * 32) launch_bands<32>(a, s);
    else if (n <= 64 * 64) launch_bands<64>(a, s);
    else launch_bands<BANDS_MAX_N / 64>(a, s);
    return check_launch("k_bands");
}
