// Nearest-k selection: the k samples with the smallest distances, ties to the
// lower sample index, returned in index order (the "keep the k nearest prior
// samples" rule of the single-country workload; the per-run Top-k return of
// Sec. 3.2), and its C-ABI entry points abc_nearest_k (float32 distances of a
// launch) and abc_nearest_k_rows (float64 distances of a small row set).
//
// abc_nearest_k never sorts the n distances. Distances map to order-preserving
// 32-bit keys; then
//   k_nk_minmax   min / max key of the distances below +inf and their count, by
//                 workgroup;
//   k_nk_hist     4096 linear bins over a key range (or, for a run of equal
//                 keys, over the sample index), wavefront-private LDS counts;
//   k_nk_narrow   narrows the range to the bin holding the k-th key until at
//                 most NK_CAP samples lie at or below the threshold (each pass
//                 shrinks the range 4096-fold);
//   k_nk_collect  composite keys (key << 32 | index) of those samples;
//   k_nk_finish   one workgroup orders them (counted ranks, or a bitonic sort in
//                 LDS), keeps the first k in index order and writes the rows.
// Each pass reads the distances once (4 B per sample). The host launches all of
// them with one histogram pass and synchronises once, for the count of finite
// distances; a range that needs more passes costs a synchronisation each.
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "common.hpp"
#include "model.hpp"

namespace abc {

constexpr int NK_BINS = 4096;
constexpr int NK_CAP = 16384;
constexpr int NK_MAX_K = 4096;
constexpr int NK_GRID = 1024;

// IEEE order as unsigned order; -0 maps to +0 (they compare equal) and every
// NaN to the largest key, above +inf.
__device__ __forceinline__ uint32_t order_key(float d)
{
    uint32_t u = __float_as_uint(d);
    if (d != d) return 0xFFFFFFFFu;
    if (u == 0x80000000u) u = 0u;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

constexpr uint32_t KEY_POS_INF = 0xFF800000u;  // order_key(+inf)

// Of the distances below +inf: least and greatest key, and how many.
struct NkRange {
    uint32_t mn, mx;
    unsigned long long cnt;
};

// What the kernels pass on, and the host reads up to hist.
struct NkCtl {
    unsigned long long finite;
    uint64_t lo, hi;     // range of the next histogram pass: keys, or indices of a tie
    uint64_t below;      // rows strictly below it
    uint64_t tidx;       // threshold: rows with key < tkey, or == tkey and index <= tidx
    uint32_t tkey;
    uint32_t mode, tie;  // 0: keys; 1: indices of the rows with key == tie
    int32_t state;       // NK_OPEN: another pass is needed
    uint32_t count;      // collected rows
    uint32_t hist[NK_BINS];
    NkRange part[NK_GRID];  // of the workgroups of k_nk_minmax
};

constexpr int32_t NK_OPEN = 0, NK_FITS = 1, NK_LOST = 2, NK_STUCK = 3;

// The range of a workgroup of 256 threads from the ranges of its threads.
__device__ __forceinline__ NkRange nk_join(NkRange r)
{
    __shared__ NkRange wave[4];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        r.mn = min(r.mn, (uint32_t)__shfl_xor((int)r.mn, off, 64));
        r.mx = max(r.mx, (uint32_t)__shfl_xor((int)r.mx, off, 64));
        r.cnt += __shfl_xor(r.cnt, off, 64);
    }
    if ((threadIdx.x & 63) == 0) wave[threadIdx.x >> 6] = r;
    __syncthreads();
    r = wave[0];
#pragma unroll
    for (int w = 1; w < 4; ++w) {
        r.mn = min(r.mn, wave[w].mn);
        r.mx = max(r.mx, wave[w].mx);
        r.cnt += wave[w].cnt;
    }
    return r;
}

// The range of all distances, from what k_nk_minmax left.
__device__ __forceinline__ NkRange nk_range(const NkCtl* c, int parts)
{
    NkRange r{0xFFFFFFFFu, 0u, 0ull};
    for (int g = threadIdx.x; g < parts; g += 256) {
        const NkRange p = c->part[g];
        r.mn = min(r.mn, p.mn);
        r.mx = max(r.mx, p.mx);
        r.cnt += p.cnt;
    }
    return nk_join(r);
}

// calls f(k, order_key(dist[k])) for this thread's samples of a grid-stride
// pass, four loads at a time; past the end the last sample is read again
template <typename F>
__device__ __forceinline__ void nk_each(const float* dist, int64_t n, F f)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t k0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k0 < n; k0 += 4 * stride) {
        float d[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) d[u] = dist[k0 + u * stride < n ? k0 + u * stride : n - 1];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (k0 + u * stride < n) f(k0 + u * stride, order_key(d[u]));
    }
}

// The range of each workgroup's distances, and a clear histogram. Whoever needs the
// range of all joins the parts, so that no atomics meet and no launch before this one
// sets them up: the 100 nearest of 1e7 distances 152 -> 123 us, of 1e5 65 -> 62. The
// single-country run of 2000 samples, whose simulation and selection come to eight
// commands before the host waits, 272 -> 242 us with seven.
__global__ __launch_bounds__(256) void k_nk_minmax(const float* dist, int64_t n, NkCtl* c)
{
    for (int b = blockIdx.x * 256 + threadIdx.x; b < NK_BINS; b += gridDim.x * 256) c->hist[b] = 0u;
    NkRange r{0xFFFFFFFFu, 0u, 0ull};
    nk_each(dist, n, [&](int64_t, uint32_t key) {
        if (key < KEY_POS_INF) {  // below +inf (NaN and +inf excluded)
            r.mn = min(r.mn, key);
            r.mx = max(r.mx, key);
            ++r.cnt;
        }
    });
    r = nk_join(r);
    if (threadIdx.x == 0) c->part[blockIdx.x] = r;
}

// One histogram pass over the range of the control block (FIRST: all keys):
// mode 0: keys in [lo, hi], bin = (key - lo) / width;
// mode 1: key == tie and index in [lo, hi], bin = (index - lo) / width.
struct HistArgs {
    const float* dist;
    int64_t n;
    int32_t k;
    int32_t parts;  // of the first pass, else 0
    NkCtl* c;
};

__global__ __launch_bounds__(256) void k_nk_hist(HistArgs a)
{
    __shared__ uint32_t h[4][NK_BINS];  // one histogram per wavefront
    NkCtl* c = a.c;
    const int wv = threadIdx.x >> 6;
    uint32_t mode = 0u, tie = 0u;
    uint64_t lo, hi;
    if (a.parts > 0) {
        const NkRange r = nk_range(c, a.parts);
        if (r.cnt < (unsigned long long)a.k) return;  // the host reports it
        lo = r.mn;
        hi = r.mx;
    } else {
        mode = c->mode;
        tie = c->tie;
        lo = c->lo;
        hi = c->hi;
    }
    const uint64_t width = (hi - lo + NK_BINS) / NK_BINS;  // ceil of the span over the bins
    for (int b = threadIdx.x; b < 4 * NK_BINS; b += blockDim.x) (&h[0][0])[b] = 0u;
    __syncthreads();
    // keys and indices are below 2^32, so are the range and its bins
    const uint32_t lo32 = (uint32_t)lo, span32 = (uint32_t)(hi - lo), w32 = (uint32_t)width;
    nk_each(a.dist, a.n, [&](int64_t k, uint32_t key) {
        const uint32_t v = mode == 0 ? key : (uint32_t)k;
        if (v >= lo32 && v - lo32 <= span32 && (mode == 0 || key == tie)) atomicAdd(&h[wv][(v - lo32) / w32], 1u);
    });
    __syncthreads();
    for (int b = threadIdx.x; b < NK_BINS; b += blockDim.x) {
        const uint32_t s = h[0][b] + h[1][b] + h[2][b] + h[3][b];
        if (s) atomicAdd(&c->hist[b], s);
    }
}

// What the counts of a pass leave: the threshold, or the range of the next pass, from
// the bin with the k-th row. A launch of its own: narrowing in the histogram's
// last workgroup takes two fences of every workgroup, each of which writes back and
// invalidates an L2 (1e7 distances 198 us, here 153; 1e3 to 1e5 alike).
__global__ __launch_bounds__(256) void k_nk_narrow(HistArgs a)
{
    __shared__ uint32_t wave_tot[4];
    NkCtl* c = a.c;
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint32_t mode = 0u, tie = 0u;
    uint64_t lo, hi, below = 0;
    if (a.parts > 0) {
        const NkRange r = nk_range(c, a.parts);
        if (threadIdx.x == 0) {
            c->finite = r.cnt;
            c->below = 0;
            c->mode = 0u;
            c->tie = 0u;
            c->state = NK_OPEN;
            c->count = 0u;
        }
        if (r.cnt < (unsigned long long)a.k) return;
        lo = r.mn;
        hi = r.mx;
    } else {
        mode = c->mode;
        tie = c->tie;
        lo = c->lo;
        hi = c->hi;
        below = c->below;
    }
    const uint64_t width = (hi - lo + NK_BINS) / NK_BINS;
    // thread t holds bins 16 t .. 16 t + 15; the first bin whose running sum
    // reaches k
    uint32_t x[NK_BINS / 256], own = 0;
#pragma unroll
    for (int q = 0; q < NK_BINS / 256; ++q) {
        x[q] = c->hist[threadIdx.x * (NK_BINS / 256) + q];
        own += x[q];
    }
    uint32_t incl = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
    }
    if (lane == 63) wave_tot[wv] = incl;
    __syncthreads();  // and what the range was is read, and the start written, before the next is
    uint32_t excl = incl - own, total = 0;
    for (int w = 0; w < 4; ++w) {
        if (w < wv) excl += wave_tot[w];
        total += wave_tot[w];
    }
    const uint64_t want = (uint64_t)a.k;
    if (threadIdx.x == 0 && below + total < want) c->state = NK_LOST;
    if (below + excl < want && want <= below + excl + own) {
        uint64_t cum = below + excl;
        int q = 0;
        while (cum + x[q] < want) cum += x[q++];
        const uint64_t blo = lo + (uint64_t)(threadIdx.x * (NK_BINS / 256) + q) * width;
        const uint64_t bhi = blo + width - 1 < hi ? blo + width - 1 : hi;
        c->tkey = mode == 0 ? (uint32_t)bhi : tie;
        c->tidx = mode == 0 ? UINT64_MAX : bhi;
        if (cum + x[q] <= (uint64_t)NK_CAP) {
            c->state = NK_FITS;
        } else {
            c->below = cum;
            if (width == 1 && mode == 0) {
                // a run of equal keys: continue on the sample index
                c->mode = 1u;
                c->tie = (uint32_t)blo;
                c->lo = 0;
                c->hi = (uint64_t)a.n - 1;
            } else if (width == 1) {
                c->state = NK_STUCK;
            } else {
                c->lo = blo;
                c->hi = bhi;
            }
        }
    }
}

__global__ __launch_bounds__(256) void k_nk_clear_hist(NkCtl* c)
{
    for (int b = threadIdx.x; b < NK_BINS; b += blockDim.x) c->hist[b] = 0u;
}

// rows with key < tkey, or key == tkey and index <= tidx
__global__ __launch_bounds__(256) void k_nk_collect(const float* dist, int64_t n, NkCtl* c, uint64_t* out)
{
    if (c->state != NK_FITS) return;
    const uint32_t tkey = c->tkey;
    const uint64_t tidx = c->tidx;
    const int lane = threadIdx.x & 63;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t b0 = (int64_t)blockIdx.x * blockDim.x; b0 < n; b0 += 4 * stride) {
        const int64_t k0 = b0 + threadIdx.x;
        float d[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) d[u] = dist[k0 + u * stride < n ? k0 + u * stride : n - 1];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t k = k0 + u * stride;
            const uint32_t key = order_key(d[u]);
            const bool sel = k < n && (key < tkey || (key == tkey && (uint64_t)k <= tidx));
            const uint64_t m = __ballot(sel);
            if (m == 0ull) continue;
            uint32_t base = 0;
            if (lane == 0) base = atomicAdd(&c->count, (uint32_t)__popcll(m));
            base = (uint32_t)__shfl((int)base, 0, 64);
            if (sel) {
                const uint32_t r = base + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
                if (r < (uint32_t)NK_CAP) out[r] = ((uint64_t)key << 32) | (uint64_t)k;
            }
        }
    }
}

__device__ void bitonic_u64(uint64_t* v, int npow)
{
    for (int k = 2; k <= npow; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int t = threadIdx.x; t < npow; t += blockDim.x) {
                const int p = t ^ j;
                if (p > t) {
                    const bool up = (t & k) == 0;
                    const uint64_t x = v[t], y = v[p];
                    if ((x > y) == up) {
                        v[t] = y;
                        v[p] = x;
                    }
                }
            }
            __syncthreads();
        }
}

struct FinishArgs {
    const uint64_t* cand;
    const NkCtl* c;
    int32_t k;
    const float* dist;
    const float* theta;  // or null: re-draw from the prior
    float lo[8], width[8];
    Key key;
    uint32_t domain, series;
    uint64_t first;
    int64_t* out_idx;
    float* out_theta;
    float* out_dist;
    float* out_kth;
};

__device__ __forceinline__ float key_to_float(uint32_t key)
{
    return __uint_as_float((key & 0x80000000u) ? (key & 0x7FFFFFFFu) : ~key);
}

__device__ __forceinline__ void finish_row(const FinishArgs& a, int r, int64_t loc)
{
    const uint64_t i = a.first + (uint64_t)loc;
    a.out_idx[r] = (int64_t)i;
    if (a.out_dist) a.out_dist[r] = a.dist[loc];
    if (a.out_theta) {
        float th[8];
        if (a.theta) {
#pragma unroll
            for (int j = 0; j < 8; ++j) th[j] = a.theta[8 * loc + j];
        } else {
            prior_draw(a.key, i, a.series, a.domain, a.lo, a.width, th);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) a.out_theta[8 * r + j] = th[j];
    }
}

// Up to this many rows are ranked by counting the smaller ones (110 rows: 6 us);
// the two sorts of more rows are 20 or more barriers each (110 rows: 14 us).
constexpr int NK_RANK_MAX = 512;

__global__ __launch_bounds__(1024) void k_nk_finish(FinishArgs a)
{
    extern __shared__ uint64_t v[];  // [NK_CAP]
    __shared__ uint32_t chosen[NK_RANK_MAX];  // indices of the first k, else all ones
    if (a.c->state != NK_FITS) return;
    const int cnt = (int)min(a.c->count, (uint32_t)NK_CAP);
    if (cnt <= NK_RANK_MAX) {
        const int t = threadIdx.x;
        const uint64_t own = t < cnt ? a.cand[t] : 0ull;
        if (t < cnt) v[t] = own;
        __syncthreads();
        int r = 0;  // the composite keys are distinct
        if (t < cnt) {
#pragma unroll 8
            for (int j = 0; j < cnt; ++j) r += v[j] < own ? 1 : 0;
            chosen[t] = r < a.k ? (uint32_t)own : 0xFFFFFFFFu;
            if (r == a.k - 1 && a.out_kth) *a.out_kth = key_to_float((uint32_t)(own >> 32));
        }
        __syncthreads();
        if (t < cnt && r < a.k) {
            int pos = 0;
#pragma unroll 8
            for (int j = 0; j < cnt; ++j) pos += chosen[j] < (uint32_t)own ? 1 : 0;
            finish_row(a, pos, (int64_t)(uint32_t)own);
        }
        return;
    }
    int npow = 1;
    while (npow < cnt) npow <<= 1;
    for (int t = threadIdx.x; t < npow; t += blockDim.x) v[t] = t < cnt ? a.cand[t] : ~0ull;
    __syncthreads();
    bitonic_u64(v, npow);
    if (threadIdx.x == 0 && a.out_kth) *a.out_kth = key_to_float((uint32_t)(v[a.k - 1] >> 32));
    // the first k by (key, index); now order them by index
    int kpow = 1;
    while (kpow < a.k) kpow <<= 1;
    uint64_t mine[4];
    int nm = 0;
    for (int t = threadIdx.x; t < kpow; t += blockDim.x) mine[nm++] = t < a.k ? (v[t] & 0xFFFFFFFFull) : ~0ull;
    __syncthreads();
    nm = 0;
    for (int t = threadIdx.x; t < kpow; t += blockDim.x) v[t] = mine[nm++];
    __syncthreads();
    bitonic_u64(v, kpow);
    for (int r = threadIdx.x; r < a.k; r += blockDim.x) finish_row(a, r, (int64_t)v[r]);
}

// ---------------------------------------------------------------------------
// small row sets in float64: rank by (distance, index) in O(n^2)
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool row_less(double da, int64_t ia, double db, int64_t ib)
{
    // NaN sorts after every number (no branches: rows are compared in bulk)
    const bool na = da != da, nb = db != db;
    return (nb & !na) | (da < db) | (((da == db) | (na & nb)) & (ia < ib));
}

__global__ __launch_bounds__(256) void k_rows_rank(const double* d, const int64_t* idx, int64_t n,
                                                   int32_t k, int32_t* rank)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    const double dq = d[q];
    const int64_t iq = idx[q];
    // eight rows' loads in flight at a time (a short row set is latency-bound)
    int64_t r = 0, j = 0;
    for (; j + 8 <= n; j += 8) {
        double dj[8];
        int64_t ij[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            dj[u] = d[j + u];
            ij[u] = idx[j + u];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) r += row_less(dj[u], ij[u], dq, iq) ? 1 : 0;
    }
    for (; j < n; ++j) r += row_less(d[j], idx[j], dq, iq) ? 1 : 0;
    rank[q] = r < k ? (int32_t)r : -1;
}

__global__ __launch_bounds__(256) void k_rows_place(const double* d, const int64_t* idx,
                                                    const float* theta, int64_t n, const int32_t* rank,
                                                    int64_t* out_idx, float* out_theta, double* out_d)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n || rank[q] < 0) return;
    const int64_t iq = idx[q];
    int64_t pos = 0, j = 0;  // selected rows with a smaller sample index
    for (; j + 8 <= n; j += 8) {
        int32_t rj[8];
        int64_t ij[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            rj[u] = rank[j + u];
            ij[u] = idx[j + u];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            pos += (rj[u] >= 0 && (ij[u] < iq || (ij[u] == iq && j + u < q))) ? 1 : 0;
    }
    for (; j < n; ++j) pos += (rank[j] >= 0 && (idx[j] < iq || (idx[j] == iq && j < q))) ? 1 : 0;
    out_idx[pos] = iq;
    if (out_d) out_d[pos] = d[q];
    if (out_theta)
        for (int j = 0; j < 8; ++j) out_theta[8 * pos + j] = theta[8 * q + j];
}

// The same for a set that one workgroup's lanes hold, a row each, from LDS and in
// one launch (114 rows: 11 us; two launches took 11 and 9, each a chain of loads).
constexpr int ROWS_SMALL = 1024;

__global__ __launch_bounds__(ROWS_SMALL) void k_rows_small(const double* d, const int64_t* idx, const float* theta,
                                                           int32_t n, int32_t k, int64_t* out_idx, float* out_theta,
                                                           double* out_d)
{
    // rows past n compare as greater than any: the loops run over whole eights
    __shared__ double ds[ROWS_SMALL];
    __shared__ int64_t is[ROWS_SMALL];
    __shared__ alignas(8) uint8_t keep[ROWS_SMALL];  // 1: one of the k
    const int q = threadIdx.x;
    const double dq = q < n ? d[q] : NAN;
    const int64_t iq = q < n ? idx[q] : INT64_MAX;
    ds[q] = dq;
    is[q] = iq;
    __syncthreads();
    int r = 0;
    if (q < n)
        for (int j = 0; j < n; j += 8) {
            double dj[8];
            int64_t ij[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) { dj[u] = ds[j + u]; ij[u] = is[j + u]; }
#pragma unroll
            for (int u = 0; u < 8; ++u) r += row_less(dj[u], ij[u], dq, iq) ? 1 : 0;
        }
    keep[q] = q < n && r < k ? 1 : 0;
    __syncthreads();
    if (q >= n || r >= k) return;
    int pos = 0;  // selected rows with a smaller sample index
    for (int j = 0; j < n; j += 8) {
        const uint64_t kept = *reinterpret_cast<const uint64_t*>(&keep[j]);
        int64_t ij[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) ij[u] = is[j + u];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            pos += (((kept >> (8 * u)) & 1u) != 0u) & ((ij[u] < iq) | ((ij[u] == iq) & (j + u < q))) ? 1 : 0;
    }
    out_idx[pos] = iq;
    if (out_d) out_d[pos] = dq;
    if (out_theta)
#pragma unroll
        for (int j = 0; j < 8; ++j) out_theta[8 * (int64_t)pos + j] = theta[8 * (int64_t)q + j];
}

// workgroups of the histogram pass: about 16 samples per thread, so a
// short input does not pay for hundreds of LDS histogram clears and merges
static unsigned nk_grid(int64_t n)
{
    const int64_t g = (n + 4095) / 4096;
    return (unsigned)(g < NK_GRID ? (g > 0 ? g : 1) : NK_GRID);
}

// and of the passes without a histogram: four samples per thread
static unsigned nk_grid_light(int64_t n)
{
    const int64_t g = (n + 1023) / 1024;
    return (unsigned)(g < NK_GRID ? (g > 0 ? g : 1) : NK_GRID);
}

}  // namespace abc

using namespace abc;

extern "C" abc_status abc_nearest_k(const float* dist, const float* theta, const abc_prior* prior,
                                    const abc_stream* st, int64_t n, uint64_t first, int32_t k,
                                    int64_t* out_idx, float* out_theta, float* out_dist,
                                    float* out_kth, void* stream)
{
    ABC_REQUIRE(dist && out_idx, "dist/out_idx NULL");
    ABC_REQUIRE(n >= 1 && n < ((int64_t)1 << 32), "n must be in [1, 2^32)");
    ABC_REQUIRE(k >= 1 && k <= NK_MAX_K && k <= n, "k must be in [1, min(n, %d)]", NK_MAX_K);
    FinishArgs fa{};
    if (out_theta && !theta) {
        abc_status rc = prior_lo_width(prior, fa.lo, fa.width);
        if (rc) return rc;
        if ((rc = check_stream_sel(st))) return rc;
        fa.key = make_key(st->seed);
        fa.domain = st->domain;
        fa.series = st->series;
    }
    const hipStream_t s = as_stream(stream);
    void* mem = nullptr;
    const size_t ctl_bytes = (sizeof(NkCtl) + 255) & ~(size_t)255;
    {
        const abc_status rs = stream_scratch(s, ctl_bytes + sizeof(uint64_t) * NK_CAP, &mem);
        if (rs) return rs;
    }
    NkCtl* dc = static_cast<NkCtl*>(mem);
    uint64_t* cand = reinterpret_cast<uint64_t*>(static_cast<char*>(mem) + ctl_bytes);
    constexpr size_t HEAD = offsetof(NkCtl, hist);
    void* pinned = nullptr;
    {
        const abc_status rs = stream_pinned(s, HEAD, &pinned);
        if (rs) return rs;
    }
    const NkCtl* h = static_cast<const NkCtl*>(pinned);  // up to hist
    fa.cand = cand;
    fa.c = dc;
    fa.k = k;
    fa.dist = dist;
    fa.theta = theta;
    fa.first = first;
    fa.out_idx = out_idx;
    fa.out_theta = out_theta;
    fa.out_dist = out_dist;
    fa.out_kth = out_kth;
    HistArgs ha{dist, n, k, 0, dc};
    abc_status rc;
    hipLaunchKernelGGL(k_nk_minmax, dim3(nk_grid_light(n)), dim3(256), 0, s, dist, n, dc);
    for (int pass = 0; pass < 16; ++pass) {
        // narrow the range until the rows at or below the threshold fit; with a
        // pass that leaves it open the last two kernels do nothing
        if (pass > 0) hipLaunchKernelGGL(k_nk_clear_hist, dim3(1), dim3(256), 0, s, dc);
        ha.parts = pass == 0 ? (int32_t)nk_grid_light(n) : 0;
        hipLaunchKernelGGL(k_nk_hist, dim3(nk_grid(n)), dim3(256), 0, s, ha);
        hipLaunchKernelGGL(k_nk_narrow, dim3(1), dim3(256), 0, s, ha);
        hipLaunchKernelGGL(k_nk_collect, dim3(nk_grid_light(n)), dim3(256), 0, s, dist, n, dc, cand);
        hipLaunchKernelGGL(k_nk_finish, dim3(1), dim3(1024), sizeof(uint64_t) * NK_CAP, s, fa);
        if ((rc = check_launch("k_nk_finish"))) return rc;
        ABC_HIP(hipMemcpyAsync(pinned, dc, HEAD, hipMemcpyDeviceToHost, s));
        ABC_HIP(hipStreamSynchronize(s));
        if (h->finite < (unsigned long long)k)
            return set_error(ABC_EINVAL, "only %llu of the %lld distances are finite, fewer than k = %d",
                             h->finite, (long long)n, k);
        if (h->state == NK_FITS) return ABC_OK;
        if (h->state == NK_LOST) return set_error(ABC_EHIP, "nearest-k: histogram lost rows");
        if (h->state == NK_STUCK) return set_error(ABC_EHIP, "nearest-k: index refinement did not converge");
    }
    return set_error(ABC_EHIP, "nearest-k: threshold search did not converge");
}

extern "C" abc_status abc_nearest_k_rows(const double* dist64, const int64_t* idx, const float* theta,
                                         int64_t n, int32_t k, int64_t* out_idx, float* out_theta,
                                         double* out_dist, void* stream)
{
    ABC_REQUIRE(dist64 && idx && out_idx, "dist64/idx/out_idx NULL");
    ABC_REQUIRE(!out_theta || theta, "out_theta needs theta");
    ABC_REQUIRE(n >= 1 && n <= 65536, "n must be in [1, 65536]");
    ABC_REQUIRE(k >= 1 && k <= n, "k must be in [1, n]");
    const hipStream_t s = as_stream(stream);
    if (n <= ROWS_SMALL) {
        hipLaunchKernelGGL(k_rows_small, dim3(1), dim3(ROWS_SMALL), 0, s, dist64, idx, theta, (int32_t)n, k, out_idx,
                           out_theta, out_dist);
        return check_launch("k_rows_small");
    }
    void* mem = nullptr;
    {
        const abc_status rs = stream_scratch(s, sizeof(int32_t) * (size_t)n, &mem);
        if (rs) return rs;
    }
    int32_t* rank = static_cast<int32_t*>(mem);
    const dim3 g((unsigned)((n + 255) / 256)), b(256);
    hipLaunchKernelGGL(k_rows_rank, g, b, 0, s, dist64, idx, n, k, rank);
    abc_status rc = check_launch("k_rows_rank");
    if (rc) return rc;
    hipLaunchKernelGGL(k_rows_place, g, b, 0, s, dist64, idx, theta, n, rank, out_idx, out_theta,
                       out_dist);
    return check_launch("k_rows_place");
}
