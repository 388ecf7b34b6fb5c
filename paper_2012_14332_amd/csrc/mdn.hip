// Learned mixture-density proposal for rejection ABC: training pairs from the
// simulator itself, a 96-256-256-136 GELU network trained with hand-written
// BF16 MFMA kernels (FP32 accumulation) and Adam, and a defensive-mixture
// proposal sampler with importance weights. Not part of the paper, whose
// proposal is the prior (eq. 2); the prior stays both the fallback and the
// reference for the learned posterior.
//
// Network: x (96 = log1p A, R, D at 32 evenly spaced days, standardised per
// feature) -> z1 = x W1 + b1, h1 = gelu(z1) -> z2 = h1 W2 + b2, h2 = gelu(z2)
// -> out = h2 W3 + b3 = (8 logits, 8x8 means, 8x8 log sd clamped to [-7, 3])
// of a diagonal Gaussian mixture over theta standardised by the prior's mean
// and sd. Loss: mean negative log-likelihood. Parameters are float32 master
// copies [W1 96x256 | b1 | W2 256x256 | b2 | W3 256x136 | b3]; the products read
// bfloat16 copies refreshed by the Adam update.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <mutex>
#include <vector>

#include "common.hpp"
#include "model.hpp"
#include "proposal.hpp"

namespace abc {

constexpr int NN_IN = 96, NN_H = 256, NN_K = 8, NN_D = 8, NN_OUT = 136;
constexpr int64_t OFF_W1 = 0, OFF_B1 = OFF_W1 + NN_IN * NN_H, OFF_W2 = OFF_B1 + NN_H,
                  OFF_B2 = OFF_W2 + NN_H * NN_H, OFF_W3 = OFF_B2 + NN_H,
                  OFF_B3 = OFF_W3 + NN_H * NN_OUT, NN_PARAMS = OFF_B3 + NN_OUT;

// The bf16 copies of the weights, one per product that reads them, in the order
// in which v_mfma_f32_16x16x32_bf16 takes them: a fragment is 16 columns by 32
// values of k, lane l holding column l & 15 at k = 8 (l >> 4) + 0..7, so a
// wavefront reads a fragment as 1 KB of consecutive memory. Forward products
// sum over a layer's inputs (F), the input gradients over its outputs (B). The
// 136 outputs are padded with zeros to 144 columns and to 160 values of k.
constexpr int FRAG = 64 * 8;  // elements of a fragment
constexpr int NF_IN = NN_IN / 16, NF_H = NN_H / 16, NF_OUT = 9;  // fragments of columns
constexpr int KF_IN = NN_IN / 32, KF_H = NN_H / 32, KF_OUT = 5;  // fragments of k
constexpr int64_t PB_F1 = 0, PB_F2 = PB_F1 + NF_H * KF_IN * FRAG, PB_F3 = PB_F2 + NF_H * KF_H * FRAG,
                  PB_B3 = PB_F3 + NF_OUT * KF_H * FRAG, PB_B2 = PB_B3 + NF_H * KF_OUT * FRAG,
                  NN_PB = PB_B2 + NF_H * KF_H * FRAG;
constexpr float LOGSIG_LO = -7.0f, LOGSIG_HI = 3.0f;
static_assert(NN_K == MIX_K && NN_D == MIX_D && NN_OUT == MIX_OUT && LOGSIG_LO == MIX_LOGSIG_LO &&
                  LOGSIG_HI == MIX_LOGSIG_HI,
              "network output layout and proposal layout must agree");

typedef uint16_t bf16;

__device__ __forceinline__ bf16 f2bf(float x)
{
    // round to nearest even
    uint32_t u = __float_as_uint(x);
    if ((u & 0x7f800000u) == 0x7f800000u) return (bf16)((u >> 16) | ((u & 0xffff) ? 0x40 : 0));
    u += 0x7fffu + ((u >> 16) & 1u);
    return (bf16)(u >> 16);
}

__device__ __forceinline__ float bf2f(bf16 h) { return __uint_as_float((uint32_t)h << 16); }

// element (column n, k) of an operand with kf fragments of k per 16 columns
__device__ __forceinline__ int frag_pos(int n, int k, int kf)
{
    return (((n >> 4) * kf + (k >> 5)) * 64 + ((k >> 3) & 3) * 16 + (n & 15)) * 8 + (k & 7);
}

// the bf16 copies of parameter e (biases have none)
__device__ __forceinline__ void put_bf16(bf16* pb, int e, float p)
{
    const bf16 h = f2bf(p);
    if (e < OFF_B1) {
        pb[PB_F1 + frag_pos(e % NN_H, e / NN_H, KF_IN)] = h;
    } else if (e >= OFF_W2 && e < OFF_B2) {
        const int q = e - (int)OFF_W2, i = q / NN_H, o = q % NN_H;
        pb[PB_F2 + frag_pos(o, i, KF_H)] = h;
        pb[PB_B2 + frag_pos(i, o, KF_H)] = h;
    } else if (e >= OFF_W3 && e < OFF_B3) {
        const int q = e - (int)OFF_W3, i = q / NN_OUT, o = q % NN_OUT;
        pb[PB_F3 + frag_pos(o, i, KF_H)] = h;
        pb[PB_B3 + frag_pos(i, o, KF_OUT)] = h;
    }
}

// gelu(z) = z (1 + erf(z / sqrt 2)) / 2, and its derivative from the same erf
__device__ __forceinline__ float gelu_f(float z, float& grad)
{
    const float e = 1.0f + erff(z * 0.70710678118654752440f);
    grad = 0.5f * e + z * expf(-0.5f * z * z) * 0.39894228040143267794f;
    return 0.5f * z * e;
}

// ----------------------------------------------------------------------------
// training pairs: theta from the prior, T and P drawn per sample, float32
// simulation, features at the 32 days d_k = 1 + rint(k (T - 1) / 31)
// ----------------------------------------------------------------------------
struct FeatArgs {
    Key key;
    uint32_t domain, series;
    uint64_t first;
    int64_t n;
    float lo[8], width[8];
    int32_t T_lo, T_hi;
    double lp_lo, lp_hi;   // log10 population range
    int32_t A0, R0, D0;
    float* features;       // [n][96] log1p counts (raw)
    float* theta;          // [n][8]
    int32_t* TP;           // [n][2] (T, P) or null
};

// Feature day k = 0..31 of a horizon T: 1 + rint(k (T - 1) / 31), in integers
// (31 is odd, so the quotient is never halfway between two).
__device__ __forceinline__ int feature_day(int T, int k)
{
    return 1 + (2 * k * (T - 1) + 31) / 62;
}

__device__ __forceinline__ int feature_T(const FeatArgs& a, uint32_t w)
{
    const int T = a.T_lo + (int)floor((double)(w >> 8) * 0x1p-24 * (double)(a.T_hi - a.T_lo + 1));
    return T > a.T_hi ? a.T_hi : T;
}

// Order of the samples, longest horizon first and every horizon's samples
// padded to whole wavefronts (order -1: no sample): a wavefront's lanes then
// end together and record their features on the same days. cnt[b] counts
// horizon T_hi - b; start and fill are its first and next free position.
constexpr int FEAT_BINS = ABC_T_MAX;
constexpr int FEAT_BLOCK = 256;
// Samples from which on the ordering pays (four short launches): with T in
// [30, 200], 8192 samples take 183 us without and 90 us with it, 1000 samples
// 179 and 217 us (too few to fill the wavefronts of 171 horizons).
constexpr int64_t FEAT_SORT_MIN = (int64_t)1 << 13;
// And the longest horizon from which on: a trajectory has 32 recorded days, so below it
// lanes in any order record on almost every day alike. 2e4 samples, without / with: T in
// [5, 10] 53 / 68 us, [5, 20] 64 / 71, [5, 40] 83 / 79, [30, 100] 122 / 93.
constexpr int32_t FEAT_SORT_T = 40;

struct FeatOrder {
    uint32_t* cnt;    // [bins]
    uint32_t* fill;   // [bins]
    int32_t* order;   // [n + 63 bins]
    int bins;
    uint32_t* total;  // positions in use
};

__global__ __launch_bounds__(FEAT_BLOCK) void k_feat_count(FeatArgs a, FeatOrder o)
{
    __shared__ uint32_t h[FEAT_BINS];
    for (int b = threadIdx.x; b < o.bins; b += FEAT_BLOCK) h[b] = 0u;
    __syncthreads();
    for (int64_t k = (int64_t)blockIdx.x * FEAT_BLOCK + threadIdx.x; k < a.n; k += (int64_t)gridDim.x * FEAT_BLOCK) {
        const uint4 w = stream_words(a.key, a.first + (uint64_t)k, a.series, ctr_word3(0, a.domain, 2));
        atomicAdd(&h[a.T_hi - feature_T(a, w.x)], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < o.bins; b += FEAT_BLOCK)
        if (h[b]) atomicAdd(&o.cnt[b], h[b]);
}

__global__ __launch_bounds__(FEAT_BINS) void k_feat_scan(FeatOrder o)
{
    __shared__ uint32_t part[FEAT_BINS];
    const int b = threadIdx.x;
    const uint32_t c = b < o.bins ? o.cnt[b] : 0u;
    const uint32_t padded = (c + 63u) & ~63u;
    part[b] = padded;
    __syncthreads();
    for (int off = 1; off < FEAT_BINS; off <<= 1) {
        const uint32_t v = b >= off ? part[b - off] : 0u;
        __syncthreads();
        part[b] += v;
        __syncthreads();
    }
    const uint32_t end = part[b], start = end - padded;
    if (b < o.bins) {
        o.fill[b] = start;
        for (uint32_t q = start + c; q < end; ++q) o.order[q] = -1;
    }
    if (b == FEAT_BINS - 1) *o.total = end;
}

// each workgroup takes its samples' positions with one addition per horizon
__global__ __launch_bounds__(FEAT_BLOCK) void k_feat_place(FeatArgs a, FeatOrder o)
{
    __shared__ uint32_t h[FEAT_BINS];
    constexpr int PER = 8;
    for (int b = threadIdx.x; b < o.bins; b += FEAT_BLOCK) h[b] = 0u;
    __syncthreads();
    const int64_t k0 = (int64_t)blockIdx.x * FEAT_BLOCK * PER + threadIdx.x;
    int bin[PER];
    uint32_t rank[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int64_t k = k0 + (int64_t)q * FEAT_BLOCK;
        if (k >= a.n) break;
        const uint4 w = stream_words(a.key, a.first + (uint64_t)k, a.series, ctr_word3(0, a.domain, 2));
        bin[q] = a.T_hi - feature_T(a, w.x);
        rank[q] = atomicAdd(&h[bin[q]], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < o.bins; b += FEAT_BLOCK)
        if (h[b]) h[b] = atomicAdd(&o.fill[b], h[b]);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int64_t k = k0 + (int64_t)q * FEAT_BLOCK;
        if (k >= a.n) break;
        o.order[h[bin[q]] + rank[q]] = (int32_t)k;
    }
}

// One lane per trajectory. Bound by VALU issue, like the float32 simulation,
// when the lanes of a wavefront share a horizon (order given); eight recorded
// days are kept in LDS and stored together, so that every store fills a 32-byte
// sector (4-byte stores 384 bytes apart, and lanes waiting for the longest
// horizon of 64 with three float64 logarithms on almost every day, took
// 3.8 ms for 1e6 pairs of T in [30, 200]; now 0.65 ms).
constexpr int FEAT_HOLD = 8;

__global__ __launch_bounds__(FEAT_BLOCK) void k_mdn_features(FeatArgs a, const int32_t* order, const uint32_t* total)
{
    __shared__ Math64 tab;
    __shared__ float hold_all[FEAT_BLOCK / 64][3 * FEAT_HOLD][64];
    stage_math64(tab);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    float (*hold)[64] = hold_all[threadIdx.x >> 6];
    int64_t k = (int64_t)blockIdx.x * FEAT_BLOCK + threadIdx.x;
    if (order) {
        if (k >= (int64_t)*total) return;
        k = order[k];
        if (k < 0) return;
    } else if (k >= a.n) {
        return;
    }
    const uint64_t i = a.first + (uint64_t)k;
    float th[8];
    prior_draw(a.key, i, a.series, a.domain, a.lo, a.width, th);
    const uint4 w = stream_words(a.key, i, a.series, ctr_word3(0, a.domain, 2));
    const double uP = (double)(w.y >> 8) * 0x1p-24;
    const int T = feature_T(a, w.x);
    double P = rint(pow(10.0, a.lp_lo + (a.lp_hi - a.lp_lo) * uP));
    if (P > 2147483647.0) P = 2147483647.0;
    const int32_t Pi = (int32_t)P;
    const Theta tt = theta_from(th);
    const RatesF r = rates_f32(tt);
    State s = init_state(tt.ka, Pi, a.A0, a.R0, a.D0);
    const float invP = 1.0f / (float)Pi;
    const float nc = noise_c(1.0f);
    const PhiloxSeries ps = philox_series(a.series, a.key);
    PhiloxDays ph;
    ph.begin(i, ps.u0, a.key);
    float* f = a.features + 96 * k;
    const bool vec = (reinterpret_cast<uintptr_t>(a.features) & 15u) == 0;
    int next = 0, dnext = 1;
    for (int t = 1; t <= T; ++t) {
        const uint4 wd = ph.day(((uint32_t)t << 8) | (a.domain << 4), ps.b1, a.key);
        Noise32 z;
        normals_f32(wd, nc, z);
        day_step_f32<0>(s, r, invP, z);
        if (t != dnext) continue;
        const float v0 = (float)log1p_count_f64(s.A, tab), v1 = (float)log1p_count_f64(s.R, tab),
                    v2 = (float)log1p_count_f64(s.D, tab);
        while (dnext == t) {  // short horizons record a day more than once
            const int j = next & (FEAT_HOLD - 1);
            hold[j][lane] = v0;
            hold[FEAT_HOLD + j][lane] = v1;
            hold[2 * FEAT_HOLD + j][lane] = v2;
            ++next;
            if (j == FEAT_HOLD - 1) {
#pragma unroll
                for (int q = 0; q < 3 * FEAT_HOLD; q += 4) {
                    const float4 x = make_float4(hold[q][lane], hold[q + 1][lane], hold[q + 2][lane], hold[q + 3][lane]);
                    float* to = f + 32 * (q / FEAT_HOLD) + (next - FEAT_HOLD) + q % FEAT_HOLD;
                    if (vec) {
                        *reinterpret_cast<float4*>(to) = x;
                    } else {
                        to[0] = x.x; to[1] = x.y; to[2] = x.z; to[3] = x.w;
                    }
                }
            }
            dnext = next < 32 ? feature_day(T, next) : 0;
        }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) a.theta[8 * k + j] = th[j];
    if (a.TP) {
        a.TP[2 * k] = T;
        a.TP[2 * k + 1] = Pi;
    }
}

// features of an observed series [3][T]
__global__ void k_obs_features(const int32_t* obs, int T, float* out)
{
    const int q = threadIdx.x;
    if (q >= 96) return;
    const int c = q / 32, k = q % 32;
    out[q] = (float)log1p((double)obs[c * T + feature_day(T, k) - 1]);
}

// Per-feature mean and sd in float64: the rows are cut into G contiguous
// ranges (G a function of n alone); a workgroup streams its range, ten rows of
// 24 float4 per step, each thread keeping sums and squares of its four columns
// about a value of the range, the median of three of its rows. What is left of a
// range is its sum and its squares about its own mean, which one workgroup per
// column joins in a fixed order. (Sums about the first of all rows lost up to a
// unit of float32 where that row was the column's only other value: 1e7 rows.)
// Bound by HBM: 1e6 rows (384 MB) take 56 us (one workgroup per column, reading 4
// bytes every 384 twice: 4.4 ms).
constexpr int CS_ROWS = 10, CS_BLOCK = 256, CS_GROUPS = 1024;
static_assert(NN_IN == 96 && CS_ROWS * (NN_IN / 4) <= CS_BLOCK, "a step of the column sums");

static int64_t colstats_groups(int64_t n)
{
    const int64_t g = (n + 8 * CS_ROWS - 1) / (8 * CS_ROWS);
    return g < CS_GROUPS ? g : CS_GROUPS;
}

__device__ __forceinline__ void store_colstats(int c, double m, double squares, int64_t n, float* mean, float* sd)
{
    const double s = sqrt(squares / (double)(n > 1 ? n - 1 : 1));
    mean[c] = (float)m;
    sd[c] = (float)(s > 1e-6 ? s : 1e-6);
}

// Few rows: one workgroup per column, whose threads hold their rows between the sum
// and the squares; one launch (1000 rows: 21 us a call, two launches 24).
constexpr int CS_FEW = 16;  // rows per thread, at most

__global__ __launch_bounds__(CS_BLOCK) void k_colstats_few(const float* x, int n, float* mean, float* sd)
{
    __shared__ double red[2][CS_BLOCK / 64];
    const int c = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    auto total = [&](double v, int k) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
        if (lane == 0) red[k][wave] = v;
        __syncthreads();
        return red[k][0] + red[k][1] + red[k][2] + red[k][3];
    };
    float v[CS_FEW];
#pragma unroll
    for (int q = 0; q < CS_FEW; ++q) {
        const int r = q * CS_BLOCK + threadIdx.x;
        v[q] = x[(int64_t)(r < n ? r : 0) * NN_IN + c];
    }
    double s = 0.0, squares = 0.0;
#pragma unroll
    for (int q = 0; q < CS_FEW; ++q) s += q * CS_BLOCK + (int)threadIdx.x < n ? (double)v[q] : 0.0;
    const double m = total(s, 0) / (double)n;
#pragma unroll
    for (int q = 0; q < CS_FEW; ++q) {
        const double d = (double)v[q] - m;
        squares += q * CS_BLOCK + (int)threadIdx.x < n ? d * d : 0.0;
    }
    squares = total(squares, 1);
    if (threadIdx.x == 0) store_colstats(c, m, squares, n, mean, sd);
}

template <bool VEC>
__global__ __launch_bounds__(CS_BLOCK) void k_colsums(const float* x, int64_t n, double* part)
{
    __shared__ double red[CS_ROWS][2 * NN_IN];
    __shared__ float centre[NN_IN];
    const int c4 = threadIdx.x % (NN_IN / 4), sub = threadIdx.x / (NN_IN / 4);
    const int64_t R = (n + gridDim.x - 1) / gridDim.x;
    const int64_t r0 = (int64_t)blockIdx.x * R, r1 = r0 + R < n ? r0 + R : n;
    if (r0 >= n) return;  // k_colstats counts no row of this range
    auto load = [&](int64_t row, float v[4]) {
        const float* p = x + row * NN_IN + 4 * c4;
        if (VEC) {
            const float4 q = load_stream(reinterpret_cast<const float4*>(p));
            v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = p[j];
        }
    };
    if (sub < CS_ROWS) {
        float c[4], first[4], last[4];
        load(r0, first);
        load(r0 + (r1 - r0) / 2, c);
        load(r1 - 1, last);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            c[j] = fmaxf(fminf(first[j], c[j]), fminf(fmaxf(first[j], c[j]), last[j]));
            c[j] = fabsf(c[j]) < INFINITY ? c[j] : 0.0f;
            if (sub == 0) centre[4 * c4 + j] = c[j];
        }
        double s1[4] = {0.0, 0.0, 0.0, 0.0}, s2[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
        for (int64_t row = r0 + sub; row < r1; row += CS_ROWS) {
            float v[4];
            load(row, v);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const double d = (double)v[j] - (double)c[j];
                s1[j] += d;
                s2[j] += d * d;
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            red[sub][4 * c4 + j] = s1[j];
            red[sub][NN_IN + 4 * c4 + j] = s2[j];
        }
    }
    __syncthreads();
    if (threadIdx.x < NN_IN) {
        const int c = threadIdx.x;
        double s1 = 0.0, s2 = 0.0;
#pragma unroll
        for (int q = 0; q < CS_ROWS; ++q) {
            s1 += red[q][c];
            s2 += red[q][NN_IN + c];
        }
        const double rows = (double)(r1 - r0);
        const double sum = rows * (double)centre[c] + s1, squares = s2 - s1 * s1 / rows;
        part[(int64_t)blockIdx.x * 2 * NN_IN + c] = sum;
        part[(int64_t)blockIdx.x * 2 * NN_IN + NN_IN + c] = squares;
    }
}

__global__ __launch_bounds__(64) void k_colstats(int64_t n, const double* part, int groups, float* mean, float* sd)
{
    constexpr int PER = CS_GROUPS / 64;
    const int c = blockIdx.x, lane = threadIdx.x;
    const int64_t R = (n + groups - 1) / groups;
    double sum[PER], squares[PER], rows[PER], s = 0.0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int g = q * 64 + lane;
        const int64_t r0 = g * R, left = g < groups && r0 < n ? n - r0 : 0;
        rows[q] = (double)(left < R ? left : R);
        sum[q] = left ? part[(int64_t)g * 2 * NN_IN + c] : 0.0;
        squares[q] = left ? part[(int64_t)g * 2 * NN_IN + NN_IN + c] : 0.0;
        s += sum[q];
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
    const double m = s / (double)n;
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if (rows[q] > 0.0) {
            const double d = sum[q] / rows[q] - m;
            v += squares[q] + rows[q] * d * d;
        }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    if (lane == 0) store_colstats(c, m, v, n, mean, sd);
}

// ----------------------------------------------------------------------------
// batch rows: row b of a training step is dataset row (mul (j0 + b) + add) mod n
// of its epoch's affine permutation, j0 = (step mod steps per epoch) batch;
// elsewhere row b itself. Features are standardised per column, (x - mean) / sd,
// and theta by the prior's centre and sd, as they are read.
// ----------------------------------------------------------------------------
struct RowMap {
    const float* features;   // [n][96] raw features
    const float* theta;      // [n][8] or null
    int64_t n, mul, add, j0;
    double inv_n;
    const float* fmean;
    const float* fsd;
    float tc[8], ts[8];
};

__device__ __forceinline__ int64_t map_row(const RowMap& r, int b)
{
    // mul and j0 + b are below n < 2^31: no overflow, and a quotient below 2^31,
    // which the product with 1 / n misses by one at most
    const int64_t x = r.mul * (r.j0 + b) + r.add;
    int64_t m = x - (int64_t)((double)x * r.inv_n) * r.n;
    if (m < 0) m += r.n;
    if (m >= r.n) m -= r.n;
    return m;
}

typedef float float4_t __attribute__((ext_vector_type(4)));
typedef unsigned short us4 __attribute__((ext_vector_type(4)));
typedef unsigned short us8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// ----------------------------------------------------------------------------
// Everything a step computes per row, in one kernel: the batch row, the three
// layers, the mixture negative log-likelihood with its gradient w.r.t. the
// outputs, and the gradients w.r.t. both hidden layers (forward only: the
// outputs). 16 rows per workgroup stay in LDS and registers from the features
// to dZ1; sixteen wavefronts split the columns of a layer, so each weight
// fragment is read by one wavefront, straight from memory into the registers of
// its product and requested a layer ahead.
//
// v_mfma_f32_16x16x32_bf16: lane l supplies row (l & 15) of A and column (l & 15)
// of B at k = 8 (l >> 4) + 0..7 and receives C[4 (l >> 4) + r][l & 15]. Products
// sum over k in ascending steps of 32.
//
// What the weight gradients read (they sum over rows) is written as fragments
// too, 16 columns by 32 rows: this workgroup's 16 rows are half a fragment. Rows
// past the batch are zeros there.
//
// What bounds it: the weights of all products, 456 KB per workgroup from the L2
// (3 us at 64 B a clock), and the error functions and exponentials of two layers
// (4 us of issue on a full chip at a batch of 4096); 16 rows, not 32 or 64, so
// that such a batch is a workgroup for each of the 256 CUs, and sixteen
// wavefronts rather than eight because the error functions branch and their
// chains want company (at least 20 us then, 18.1 so). 19.4 us in the mean at a batch
// of 4096, 12 at 64; with the weight gradients 33.6 us a step, where seven kernels
// with the activations in memory between them took 70.5.
// ----------------------------------------------------------------------------
constexpr int R_ROWS = 16, R_WAVES = 16, R_BLOCK = 64 * R_WAVES;
constexpr int R_LX = NN_IN + 8, R_LH = NN_H + 8, R_LO = NN_OUT + 4, R_LD = 32 * KF_OUT + 8;
static_assert(NF_H == R_WAVES && NF_OUT <= R_WAVES, "one fragment of columns a wavefront");
static_assert(NN_K == 8 && NN_D == 8 && NN_OUT == 136 && NN_H == 256, "output layer layout");

struct RowArgs {
    RowMap rm;
    int n;                // rows of the batch
    const bf16* pb;
    const float *b1, *b2, *b3;
    float* out;           // forward only: [n][136]
    bf16 *X, *H1, *H2, *dOUT, *dZ2, *dZ1;  // fragments, [blocks of 32 rows][columns / 16]
    // Bias gradients: what their sums in the order of 64-row tiles need. Of 32
    // rows, the sums over rows 4 g + 0..3 of the first 16 rows [4][256], then the
    // second 16 rows themselves [16][256]; of the outputs, the sums over 16 rows.
    float *cs1, *cs2, *cs3;
    float* loss;          // the batch's mean NLL is added here (its value only)
};

__device__ __forceinline__ float sum8(float v)  // over the 8 lanes of a row
{
    v += __shfl_xor(v, 1, 64);
    v += __shfl_xor(v, 2, 64);
    v += __shfl_xor(v, 4, 64);
    return v;
}

__device__ __forceinline__ float max8(float v)
{
    v = fmaxf(v, __shfl_xor(v, 1, 64));
    v = fmaxf(v, __shfl_xor(v, 2, 64));
    v = fmaxf(v, __shfl_xor(v, 4, 64));
    return v;
}

__device__ __forceinline__ float sum_rows(float v)  // over the 8 rows (lane bits 3..5)
{
    v += __shfl_xor(v, 8, 64);
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    return v;
}

// fragments nf KF .. nf KF + KF - 1 of an operand, this lane's 16 bytes of each
template <int KF>
__device__ __forceinline__ void load_frags(us8 (&w)[KF], const bf16* base, int nf, int lane)
{
    const us8* p = reinterpret_cast<const us8*>(base) + (nf * KF) * 64 + lane;
#pragma unroll
    for (int k = 0; k < KF; ++k) w[k] = p[k * 64];
}

// one 16 x 16 tile: A from LDS (16 rows of LD elements), B fragments in registers
template <int KF, int LD>
__device__ __forceinline__ float4_t tile(const bf16 (&A)[R_ROWS][LD], const us8 (&w)[KF], int lane, float4_t acc)
{
#pragma unroll
    for (int k = 0; k < KF; ++k) {
        const us8 x = *reinterpret_cast<const us8*>(&A[lane & 15][32 * k + 8 * (lane >> 4)]);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, w[k]),
                                                      acc, 0, 0, 0);
    }
    return acc;
}

// this workgroup's half of fragment nf of its 32 rows: rows 8 q + 0..7, column c
__device__ __forceinline__ bf16* row_frag(bf16* base, int columns16, int nf, int q, int c)
{
    return base + (((int64_t)(blockIdx.x >> 1) * columns16 + nf) * 64 + ((blockIdx.x & 1) * 2 + q) * 16 + c) * 8;
}

// a tile's four rows of column c = 16 nf + (lane & 15), to LDS rows and the fragment
template <int LD>
__device__ __forceinline__ void put_tile(bf16 (&S)[R_ROWS][LD], bf16* base, int nf, const us4& h, int lane)
{
    const int g = lane >> 4, c = lane & 15;
#pragma unroll
    for (int r = 0; r < 4; ++r) S[4 * g + r][16 * nf + c] = h[r];
    if (base) *reinterpret_cast<us4*>(row_frag(base, NF_H, nf, g >> 1, c) + (g & 1) * 4) = h;
}

// columns [0, 16 NF) of the workgroup's 16 rows, from LDS to their half fragments,
// by threads t = 0, 1, ..
template <int NF, int LD>
__device__ __forceinline__ void put_columns(const bf16 (&S)[R_ROWS][LD], bf16* base, int t)
{
    if (t < 0 || t >= NF * 32) return;
    const int q = t / (16 * NF), c = t % (16 * NF);
    us8 x;
#pragma unroll
    for (int r = 0; r < 8; ++r) x[r] = S[8 * q + r][c];
    *reinterpret_cast<us8*>(row_frag(base, NF, c >> 4, q, c & 15)) = x;
}

// the gradient of a hidden layer's pre-activations from its product, for one tile
template <bool LDS, int LD>
__device__ __forceinline__ void put_gradient(const float4_t& acc, const float (&grad)[4], int row0, int n, int nf,
                                             bf16 (&S)[R_ROWS][LD], bf16* base, float* cs, int lane)
{
    const int g = lane >> 4, c = 16 * nf + (lane & 15);
    float v[4], sum = 0.0f;
    us4 h;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        v[r] = row0 + 4 * g + r < n ? acc[r] * grad[r] : 0.0f;
        h[r] = f2bf(v[r]);
        sum += v[r];
    }
    if (LDS) {
        put_tile(S, base, nf, h, lane);
    } else {
        *reinterpret_cast<us4*>(row_frag(base, NF_H, nf, g >> 1, lane & 15) + (g & 1) * 4) = h;
    }
    float* o = cs + (int64_t)(blockIdx.x >> 1) * 20 * NN_H;
    if ((blockIdx.x & 1) == 0) {
        o[g * NN_H + c] = sum;
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) o[(4 + 4 * g + r) * NN_H + c] = v[r];
    }
}

template <bool TRAIN>
__global__ __launch_bounds__(R_BLOCK) void k_rows(RowArgs a)
{
    __shared__ __align__(16) bf16 Xs[R_ROWS][R_LX];
    __shared__ __align__(16) bf16 Ha[R_ROWS][R_LH];
    __shared__ __align__(16) bf16 Hb[R_ROWS][R_LH];
    __shared__ __align__(16) float Os[R_ROWS][R_LO];
    __shared__ __align__(16) bf16 Ds[TRAIN ? R_ROWS : 1][R_LD];
    __shared__ __align__(16) float Ts[TRAIN ? R_ROWS : 1][NN_D];
    __shared__ float part[TRAIN ? 2 : 1][TRAIN ? 2 * NN_D + 2 : 1][64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row0 = blockIdx.x * R_ROWS;
    const int g = lane >> 4;

    us8 w1[KF_IN], w2[KF_H];
    load_frags(w1, a.pb + PB_F1, wv, lane);
    // the rows: a float4 of features per thread, standardised
    constexpr int XV = NN_IN / 4;
    if (tid < R_ROWS * XV) {
        const int r = tid / XV, c = 4 * (tid % XV);
        us4 h = {0, 0, 0, 0};
        if (row0 + r < a.n) {
            const float4 f = *reinterpret_cast<const float4*>(a.rm.features + map_row(a.rm, row0 + r) * NN_IN + c);
            const float4 m = *reinterpret_cast<const float4*>(a.rm.fmean + c), d = *reinterpret_cast<const float4*>(a.rm.fsd + c);
            h[0] = f2bf((f.x - m.x) / d.x);
            h[1] = f2bf((f.y - m.y) / d.y);
            h[2] = f2bf((f.z - m.z) / d.z);
            h[3] = f2bf((f.w - m.w) / d.w);
        }
        *reinterpret_cast<us4*>(&Xs[r][c]) = h;
    } else if (TRAIN && tid >= R_BLOCK - R_ROWS * NN_D) {
        const int t = tid - (R_BLOCK - R_ROWS * NN_D), r = t / NN_D, c = t % NN_D;
        if (row0 + r < a.n) Ts[r][c] = (a.rm.theta[map_row(a.rm, row0 + r) * NN_D + c] - a.rm.tc[c]) / a.rm.ts[c];
        else Ts[r][c] = 0.0f;
    }
    load_frags(w2, a.pb + PB_F2, wv, lane);
    const float bias1 = a.b1[16 * wv + (lane & 15)], bias2 = a.b2[16 * wv + (lane & 15)];
    __syncthreads();

    const float4_t zero = {0.f, 0.f, 0.f, 0.f};
    // derivatives of both activations, where the input gradients need them
    float grad1[4], grad2[4];
    if (TRAIN) put_columns<NF_IN>(Xs, a.X, tid);
    // h1 = gelu(x W1 + b1)
    {
        const float4_t acc = tile(Xs, w1, lane, zero);
        us4 h;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bf16 y = f2bf(gelu_f(acc[r] + bias1, grad1[r]));
            h[r] = row0 + 4 * g + r < a.n ? y : (bf16)0;
        }
        put_tile(Ha, TRAIN ? a.H1 : nullptr, wv, h, lane);
    }
    us8 w3[KF_H];
    float bias3 = 0.0f;
    if (wv < NF_OUT) {
        load_frags(w3, a.pb + PB_F3, wv, lane);
        if (16 * wv + (lane & 15) < NN_OUT) bias3 = a.b3[16 * wv + (lane & 15)];
    }
    __syncthreads();
    // h2 = gelu(h1 W2 + b2)
    {
        const float4_t acc = tile(Ha, w2, lane, zero);
        us4 h;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bf16 y = f2bf(gelu_f(acc[r] + bias2, grad2[r]));
            h[r] = row0 + 4 * g + r < a.n ? y : (bf16)0;
        }
        put_tile(Hb, TRAIN ? a.H2 : nullptr, wv, h, lane);
    }
    us8 w4[KF_OUT];
    if (TRAIN) load_frags(w4, a.pb + PB_B3, wv, lane);
    __syncthreads();
    // out = h2 W3 + b3
    if (wv < NF_OUT) {
        const float4_t acc = tile(Hb, w3, lane, zero);
        if (16 * wv + (lane & 15) < NN_OUT)
#pragma unroll
            for (int r = 0; r < 4; ++r) Os[4 * g + r][16 * wv + (lane & 15)] = acc[r] + bias3;
    }
    if (TRAIN)  // the padding of dOUT's columns
        for (int t = tid; t < R_ROWS * (R_LD - NN_OUT); t += R_BLOCK)
            Ds[t / (R_LD - NN_OUT)][NN_OUT + t % (R_LD - NN_OUT)] = 0;
    __syncthreads();
    if constexpr (!TRAIN) {
        for (int t = tid; t < R_ROWS * NN_OUT; t += R_BLOCK) {
            const int r = t / NN_OUT;
            if (row0 + r < a.n) a.out[(int64_t)(row0 + r) * NN_OUT + t % NN_OUT] = Os[r][t % NN_OUT];
        }
    } else {
        us8 w5[KF_H];
        load_frags(w5, a.pb + PB_B2, wv, lane);
        // The loss: 8 rows in each of the first two wavefronts, lane 8 r + k
        // holding row r's mixture component k (its logit, 8 means, 8 log sds, and
        // the row's 8 targets), so the per-row sums over components are 8-lane
        // shuffles and no lane repeats another's transcendentals.
        const int k = lane & 7;
        if (wv < 2) {
            const int rl = 8 * wv + (lane >> 3);
            const bool live = row0 + rl < a.n;
            const float inv_n = 1.0f / (float)a.n;
            const float* o = &Os[rl][0];
            const float4* mu4 = reinterpret_cast<const float4*>(o + NN_K + NN_D * k);
            const float4* raw4 = reinterpret_cast<const float4*>(o + NN_K + NN_K * NN_D + NN_D * k);
            const float4* t4 = reinterpret_cast<const float4*>(&Ts[rl][0]);
            const float logit = o[k];
            const float4 m0v = mu4[0], m1v = mu4[1], r0v = raw4[0], r1v = raw4[1], t0v = t4[0], t1v = t4[1];
            const float mu[8] = {m0v.x, m0v.y, m0v.z, m0v.w, m1v.x, m1v.y, m1v.z, m1v.w};
            const float raw[8] = {r0v.x, r0v.y, r0v.z, r0v.w, r1v.x, r1v.y, r1v.z, r1v.w};
            const float t[8] = {t0v.x, t0v.y, t0v.z, t0v.w, t1v.x, t1v.y, t1v.z, t1v.w};
            // log-softmax of the row's logits
            const float lmax = max8(logit);
            const float lse_logits = lmax + logf(sum8(expf(logit - lmax)));
            // component k's log density: sum over dimensions of -u^2 / 2 - log sd
            float u[8], si[8], term = 0.0f;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float ls = fminf(fmaxf(raw[j], LOGSIG_LO), LOGSIG_HI);
                si[j] = expf(-ls);
                u[j] = (t[j] - mu[j]) * si[j];
                term += -0.5f * u[j] * u[j] - ls;
            }
            const float Lk = logit - lse_logits - 0.5f * NN_D * 1.83787706640934548356f + term;
            // log-sum-exp over the components
            const float Lmax = max8(Lk);
            const float lse = Lmax + logf(sum8(expf(Lk - Lmax)));
            const float resp = expf(Lk - lse);
            const float gk = live ? (expf(logit - lse_logits) - resp) * inv_n : 0.0f;
            float gmu[8], gls[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                gmu[j] = live ? -resp * u[j] * si[j] * inv_n : 0.0f;
                gls[j] = (live && raw[j] > LOGSIG_LO && raw[j] < LOGSIG_HI) ? -resp * (u[j] * u[j] - 1.0f) * inv_n
                                                                             : 0.0f;
            }
            us8 bm, bl;
#pragma unroll
            for (int j = 0; j < 8; ++j) { bm[j] = f2bf(gmu[j]); bl[j] = f2bf(gls[j]); }
            Ds[rl][k] = f2bf(gk);
            *reinterpret_cast<us8*>(&Ds[rl][NN_K + NN_D * k]) = bm;
            *reinterpret_cast<us8*>(&Ds[rl][NN_K + NN_K * NN_D + NN_D * k]) = bl;
            // of the component, by lane: what is summed over the 16 rows
            float (*own)[64] = part[wv];
            own[0][lane] = gk;
#pragma unroll
            for (int j = 0; j < 8; ++j) { own[1 + j][lane] = gmu[j]; own[1 + NN_D + j][lane] = gls[j]; }
            own[2 * NN_D + 1][lane] = live && k == 0 ? -lse : 0.0f;
        }
        __syncthreads();
        // the output bias's sums over the 16 rows, and the loss
        for (int q = wv; q < 2 * NN_D + 2; q += R_WAVES) {
            const float v = sum_rows(part[0][q][lane] + part[1][q][lane]);
            const int col = q == 0 ? k : (q <= NN_D ? NN_K + NN_D * k + q - 1 : NN_K + NN_K * NN_D + NN_D * k + q - 1 - NN_D);
            if (q == 2 * NN_D + 1) {  // lane 0's rows: the others of a row hold zeros
                if (lane == 0 && a.loss && row0 < a.n) atomicAdd(a.loss, v / (float)a.n);
            } else if (lane < 8) {
                a.cs3[(int64_t)blockIdx.x * NN_OUT + col] = v;
            }
        }
        put_columns<NF_OUT>(Ds, a.dOUT, R_BLOCK - 1 - tid);
        // dZ2 = (dOUT W3^T) gelu'(z2), then dZ1 = (dZ2 W2^T) gelu'(z1)
        put_gradient<true>(tile(Ds, w4, lane, zero), grad2, row0, a.n, wv, Ha, a.dZ2, a.cs2, lane);
        __syncthreads();
        put_gradient<false>(tile(Ha, w5, lane, zero), grad1, row0, a.n, wv, Ha, a.dZ1, a.cs1, lane);
    }
}

// ----------------------------------------------------------------------------
// Weight and bias gradients and, with adam, the update (Kingma & Ba) of the
// float32 master parameters and the bf16 copies of the weights.
//
// A workgroup takes a 32 x 16 tile of one weight gradient over the whole batch:
// dW = A^T B, summed over rows. The rows come in ranges of k_per_split (128 from
// a batch of 512 on), each range a product of its own and the ranges added in
// order; eight wavefronts take the ranges in turn, 32 of them at a time, and the
// partial tiles meet in LDS, where the thread that then updates a parameter adds
// its ranges. Nothing but the parameters goes back to memory. The last
// workgroups add the bias gradients, 16 columns each, in the order of 64-row tiles.
// Bound by the L2: 95 MB of fragments at a batch of 4096 take 13 us with 4 us of
// it for the chain of one range (batch 64: 4.3 us). Partial products in memory,
// as tiles of 64 x 64 need them to fill the chip, were 16 MB each way.
// ----------------------------------------------------------------------------
constexpr int W_BLOCK = 512, W_WAVES = W_BLOCK / 64, W_RANGES = 32;
constexpr int W_TILES1 = NN_IN / 32 * NF_H, W_TILES2 = NN_H / 32 * NF_H, W_TILES3 = NN_H / 32 * NF_OUT;
constexpr int W_TILES = W_TILES1 + W_TILES2 + W_TILES3;
static_assert(NN_H / 32 == 8 && NN_IN / 32 == 3 && NF_H == 16, "the split of the tiles over eight XCDs");
constexpr int W_COLS = 16;  // bias columns of a workgroup
constexpr int W_BIAS_H = NN_H / W_COLS, W_BIAS_OUT = (NN_OUT + W_COLS - 1) / W_COLS;
constexpr int W_GRID = W_TILES + 2 * W_BIAS_H + W_BIAS_OUT;

struct GradArgs {
    const bf16 *X, *H1, *H2, *dOUT, *dZ2, *dZ1;
    const float *cs1, *cs2, *cs3;
    int n, k_per_split;
    float* g;
    int adam;
    float* p;
    float* m;
    float* v;
    bf16* pb;
    int updates;          // of the parameters, this one included
    float lr, b1, b2, eps;
};

__device__ __forceinline__ void finish_param(const GradArgs& a, int e, float gsum, float m0, float v0, float p0,
                                             const float (&power)[2])
{
    a.g[e] = gsum;
    if (!a.adam) return;
    const float m = a.b1 * m0 + (1.0f - a.b1) * gsum;
    const float v = a.b2 * v0 + (1.0f - a.b2) * gsum * gsum;
    a.m[e] = m;
    a.v[e] = v;
    const float mh = m / (1.0f - power[0]);
    const float vh = v / (1.0f - power[1]);
    const float p = p0 - a.lr * mh / (sqrtf(vh) + a.eps);
    a.p[e] = p;
    put_bf16(a.pb, e, p);
}

// STEPS: products of 32 rows in a range
template <int STEPS>
__global__ __launch_bounds__(W_BLOCK) void k_weight_grad(GradArgs a)
{
    __shared__ float part[W_RANGES][W_BLOCK];
    __shared__ float power[2];  // the decay rates to the number of updates
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    int b = blockIdx.x;
    if (a.adam && wv == W_WAVES - 1) {
        const float x = powf((lane & 1) ? a.b2 : a.b1, (float)a.updates);
        if (lane < 2) power[lane] = x;  // read after a barrier of the sums
    }
    if (b < W_TILES) {
        // Workgroups go to the eight XCDs in turn, and what an XCD reads of the
        // fragments comes over the fabric: its tiles share rows and columns.
        const bf16 *A, *B;
        int ca, cb, cols, off, mt, nt;  // fragments per row block of either operand, columns, first parameter, tile
        const int xcd = b & 7, q = b >> 3;
        if (q < W_TILES2 / 8) {
            A = a.H1; B = a.dZ2; ca = NF_H; cb = NF_H; cols = NN_H; off = (int)OFF_W2;
            mt = 4 * (xcd & 1) + (q & 3); nt = 4 * (xcd >> 1) + (q >> 2);
        } else if (q < (W_TILES2 + W_TILES3) / 8) {
            A = a.H2; B = a.dOUT; ca = NF_H; cb = NF_OUT; cols = NN_OUT; off = (int)OFF_W3;
            mt = xcd; nt = q - W_TILES2 / 8;
        } else {
            const int u = q - (W_TILES2 + W_TILES3) / 8;
            A = a.X; B = a.dZ1; ca = NF_IN; cb = NF_H; cols = NN_H; off = (int)OFF_W1;
            mt = u % 3; nt = 2 * xcd + u / 3;
        }
        // thread t holds element t of the tile: C[4 (lane >> 4) + (wv & 3)][lane & 15] of half wv >> 2
        const int col = 16 * nt + (lane & 15);
        const int e = off + (32 * mt + 16 * (wv >> 2) + 4 * (lane >> 4) + (wv & 3)) * cols + col;
        const bool mine = col < cols;
        float m0 = 0.0f, v0 = 0.0f, p0 = 0.0f;
        if (a.adam && mine) { m0 = a.m[e]; v0 = a.v[e]; p0 = a.p[e]; }
        const int nblk = (a.n + 31) / 32;
        const int ranges = (nblk + STEPS - 1) / STEPS;
        // a range in groups of four products at most
        constexpr int GROUP = STEPS < 4 ? STEPS : (STEPS == 6 ? 3 : 4), GROUPS = STEPS / GROUP;
        struct Group { us8 x0[GROUP], x1[GROUP], y[GROUP]; };
        const us8* pa = reinterpret_cast<const us8*>(A) + (2 * mt) * 64;
        const us8* pq = reinterpret_cast<const us8*>(B) + nt * 64;
        float gsum = 0.0f;
        for (int z0 = 0; z0 < ranges; z0 += W_RANGES) {
            const int zn = min(W_RANGES, ranges - z0);
            // this wavefront's ranges wv, wv + 8, .. of the 32, in groups
            const int items = wv < zn ? ((zn - 1 - wv) / W_WAVES + 1) * GROUPS : 0;
            auto first = [&](int t) { return (z0 + wv + W_WAVES * (t / GROUPS)) * STEPS + GROUP * (t % GROUPS); };
            // (blocks past the last are read as block 0, unused, so that no branch
            // stands between a group's loads and the wait for the group before it)
            auto load = [&](int t, Group& f) {
                const int blk0 = first(t);
#pragma unroll
                for (int q = 0; q < GROUP; ++q) {
                    const int blk = blk0 + q < nblk ? blk0 + q : 0;  // uniform
                    f.x0[q] = pa[(int64_t)(blk * ca) * 64 + lane];
                    f.x1[q] = pa[(int64_t)(blk * ca) * 64 + 64 + lane];
                    f.y[q] = pq[(int64_t)(blk * cb) * 64 + lane];
                }
            };
            float4_t acc[2];
            auto multiply = [&](int t, const Group& f) {
                if (t >= items) return;
                const int lim = nblk - first(t);
                if (t % GROUPS == 0) acc[0] = acc[1] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int q = 0; q < GROUP; ++q) {
                    if (q >= lim) break;
                    const bf16x8 yb = __builtin_bit_cast(bf16x8, f.y[q]);
                    acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f.x0[q]), yb, acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f.x1[q]), yb, acc[1], 0, 0, 0);
                }
                if (t % GROUPS == GROUPS - 1)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int r = 0; r < 4; ++r) part[wv + W_WAVES * (t / GROUPS)][(4 * i + r) * 64 + lane] = acc[i][r];
            };
            // two groups in flight
            Group f0, f1;
            load(0, f0);
            for (int t = 0; t < items; t += 2) {
                load(t + 1, f1);
                multiply(t, f0);
                load(t + 2, f0);
                multiply(t + 1, f1);
            }
            __syncthreads();
            int z = 0;
            for (; z + 8 <= zn; z += 8) {
                float p[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) p[q] = part[z + q][tid];
#pragma unroll
                for (int q = 0; q < 8; ++q) gsum += p[q];
            }
            for (; z < zn; ++z) gsum += part[z][tid];
            __syncthreads();
        }
        if (mine) finish_param(a, e, gsum, m0, v0, p0, power);
        return;
    }
    b -= W_TILES;
    // biases: thread (i, c) forms the sum of column c over one 64-row tile
    constexpr int IN = W_BLOCK / W_COLS;  // tiles side by side
    const int c = tid % W_COLS, i = tid / W_COLS;
    const bool hidden = b < 2 * W_BIAS_H;
    const int cols = hidden ? NN_H : NN_OUT;
    const int col0 = W_COLS * (hidden ? b % W_BIAS_H : b - 2 * W_BIAS_H) + c;
    const bool mine = col0 < cols;
    const int col = mine ? col0 : 0;
    const int e = (hidden ? (int)(b < W_BIAS_H ? OFF_B1 : OFF_B2) : (int)OFF_B3) + col;
    const float* cs = b < W_BIAS_H ? a.cs1 : a.cs2;
    float m0 = 0.0f, v0 = 0.0f, p0 = 0.0f;
    if (a.adam && mine && i == 0) { m0 = a.m[e]; v0 = a.v[e]; p0 = a.p[e]; }
    const int tiles = (a.n + 63) / 64, nblk = (a.n + 31) / 32;
    float gsum = 0.0f;
    for (int t0 = 0; t0 < tiles; t0 += IN) {
        const int t = t0 + i;
        // the blocks of 32 rows of the tile; missing ones count as zeros, and are
        // read as block 0 so that all loads are in flight together
        const bool in[2] = {2 * t < nblk, 2 * t + 1 < nblk};
        const int64_t blk[2] = {in[0] ? 2 * t : 0, in[1] ? 2 * t + 1 : 0};
        float sum = 0.0f;
        if (hidden) {
            float s[2][4], x[2][16];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float* o = cs + blk[h] * 20 * NN_H + col;
#pragma unroll
                for (int g = 0; g < 4; ++g) s[h][g] = o[g * NN_H];
#pragma unroll
                for (int r = 0; r < 16; ++r) x[h][r] = o[(4 + r) * NN_H];
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int r = 0; r < 16; ++r) s[h][r >> 2] += x[h][r];
                const float v = (s[h][0] + s[h][1]) + (s[h][2] + s[h][3]);
                sum = h == 0 ? v : sum + (in[1] ? v : 0.0f);
            }
        } else {
            float x[4];
#pragma unroll
            for (int w = 0; w < 4; ++w) x[w] = a.cs3[(2 * blk[w >> 1] + (w & 1)) * NN_OUT + col];
#pragma unroll
            for (int w = 0; w < 4; ++w) sum += in[w >> 1] ? x[w] : 0.0f;
        }
        part[0][tid] = sum;
        __syncthreads();
        if (i == 0) {
            const int tn = min(IN, tiles - t0);
            float p[IN];
#pragma unroll
            for (int q = 0; q < IN; ++q) p[q] = part[0][q * W_COLS + c];
#pragma unroll
            for (int q = 0; q < IN; ++q)
                if (q < tn) gsum += p[q];
        }
        __syncthreads();
    }
    if (mine && i == 0) finish_param(a, e, gsum, m0, v0, p0, power);
}

__global__ void k_zero_f32(float* p, int64_t n)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n) p[e] = 0.0f;
}

__global__ void k_params_bf16(const float* p, bf16* pb)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < NN_PARAMS) put_bf16(pb, (int)e, p[e]);
}

// initialisation (domain 3 stream): W ~ U(-1/sqrt(fan_in), 1/sqrt(fan_in)), b = 0
__global__ void k_mdn_init(float* p, uint64_t seed)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= NN_PARAMS) return;
    int fan_in = 0;
    if (e < OFF_B1) fan_in = NN_IN;
    else if (e >= OFF_W2 && e < OFF_B2) fan_in = NN_H;
    else if (e >= OFF_W3 && e < OFF_B3) fan_in = NN_H;
    float v = 0.0f;
    if (fan_in) {
        const uint4 w = stream_words(make_key(seed), (uint64_t)e, 0, ctr_word3(0, 3, 0));
        const float u = (float)(w.x >> 8) * 0x1p-24f;
        v = (2.0f * u - 1.0f) * rsqrtf((float)fan_in);
    }
    p[e] = v;
}

// ----------------------------------------------------------------------------
// defensive-mixture proposal: with probability lambda a prior draw, else a
// draw from the network's mixture for one series, mapped back to theta units;
// draws outside the prior box are redrawn (attempt a uses day a + 1 of the
// proposal stream). weight = prior density / q, q = (1 - lambda) q_mix +
// lambda prior (q_mix carries the Jacobian of the standardisation). The
// truncation's normalising constant cancels under self-normalised weights.
// ----------------------------------------------------------------------------
struct SampleArgs {
    const float* mix;     // [136] network output for the series
    ProposalBox prop;
    Key key;
    uint32_t domain, series;
    uint64_t first;
    int64_t n;
    float* theta;         // [n][8]
    float* weight;        // [n]
};

__global__ __launch_bounds__(256) void k_mdn_sample(SampleArgs a)
{
    __shared__ float o[NN_OUT];
    __shared__ MixTable tab;
    for (int q = threadIdx.x; q < NN_OUT; q += blockDim.x) o[q] = a.mix[q];
    __syncthreads();
    if (threadIdx.x < MIX_K * MIX_D) mix_table_entry(o, a.prop, threadIdx.x / MIX_D, threadIdx.x % MIX_D, tab);
    __syncthreads();
    if (threadIdx.x == 0) mix_table_finish(o, tab);
    __syncthreads();
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= a.n) return;
    float th[8];
    const float w = proposal_draw(tab, a.prop, a.key, a.first + (uint64_t)k, a.series, a.domain, th);
    for (int j = 0; j < 8; ++j) a.theta[8 * k + j] = th[j];
    a.weight[k] = w;
}

// Rows per range of the weight-gradient products: 128 from a batch of 512 on,
// else ranges of whole 64-row tiles, at most 256 rows each.
static int k_per_split_for(int K)
{
    if (K >= 512) return 128;
    const int tiles = (K + 63) / 64;
    const int splits = (tiles + 3) / 4;
    return ((tiles + splits - 1) / splits) * 64;
}

}  // namespace abc

using namespace abc;

struct abc_mdn {
    float* p = nullptr;
    bf16* pb = nullptr;
    float* m = nullptr;
    float* v = nullptr;
    float* g = nullptr;
    float* fmean = nullptr;
    float* fsd = nullptr;
    float* loss_acc = nullptr;
    double* colpart = nullptr;  // partials of the column sums
    float lo[8], hi[8], tc[8], ts[8];
    int ws = 0;  // workspace: blocks of 32 rows
    bf16* frags = nullptr;  // fragments of X, H1, H2, dOUT, dZ2, dZ1
    float* sums = nullptr;  // bias gradients' partials cs1, cs2, cs3
};

namespace {

constexpr int64_t WS_FRAGS = (int64_t)(NF_IN + 4 * NF_H + NF_OUT) * FRAG;  // of 32 rows
constexpr int64_t WS_SUMS = 2 * 20 * NN_H + 2 * NN_OUT;

void free_ws(abc_mdn* n)
{
    if (n->frags) (void)hipFree(n->frags);
    if (n->sums) (void)hipFree(n->sums);
    n->frags = nullptr;
    n->sums = nullptr;
    n->ws = 0;
}

abc_status ensure_ws(abc_mdn* n, int rows)
{
    const int blocks = (rows + 31) / 32;
    if (blocks <= n->ws) return ABC_OK;
    free_ws(n);
    ABC_HIP(hipMalloc((void**)&n->frags, (size_t)blocks * WS_FRAGS * sizeof(bf16)));
    ABC_HIP(hipMalloc((void**)&n->sums, (size_t)blocks * WS_SUMS * sizeof(float)));
    n->ws = blocks;
    return ABC_OK;
}

// the batch's rows: rows 0..n-1 in order
RowMap row_map(const abc_mdn* net, const float* features, const float* theta, int64_t n)
{
    RowMap r{};
    r.features = features;
    r.theta = theta;
    r.n = n;
    r.mul = 1;
    r.inv_n = 1.0 / (double)n;
    r.fmean = net->fmean;
    r.fsd = net->fsd;
    for (int j = 0; j < 8; ++j) { r.tc[j] = net->tc[j]; r.ts[j] = net->ts[j]; }
    return r;
}

RowArgs row_args(const abc_mdn* net, const RowMap& rm, int n)
{
    RowArgs a{};
    a.rm = rm;
    a.n = n;
    a.pb = net->pb;
    a.b1 = net->p + OFF_B1;
    a.b2 = net->p + OFF_B2;
    a.b3 = net->p + OFF_B3;
    if (net->ws) {
        const int64_t w = net->ws;
        a.X = net->frags;
        a.H1 = a.X + w * NF_IN * FRAG;
        a.H2 = a.H1 + w * NF_H * FRAG;
        a.dOUT = a.H2 + w * NF_H * FRAG;
        a.dZ2 = a.dOUT + w * NF_OUT * FRAG;
        a.dZ1 = a.dZ2 + w * NF_H * FRAG;
        a.cs1 = net->sums;
        a.cs2 = a.cs1 + w * 20 * NN_H;
        a.cs3 = a.cs2 + w * 20 * NN_H;
    }
    return a;
}

// a launch covers whole blocks of 32 rows: rows past the batch are zeros
void launch_rows(const RowArgs& a, bool train, hipStream_t s)
{
    const dim3 grid(2 * ((a.n + 31) / 32)), block(R_BLOCK);
    if (train) hipLaunchKernelGGL(k_rows<true>, grid, block, 0, s, a);
    else hipLaunchKernelGGL(k_rows<false>, grid, block, 0, s, a);
}

GradArgs grad_args(const abc_mdn* net, const RowArgs& r)
{
    GradArgs a{};
    a.X = r.X; a.H1 = r.H1; a.H2 = r.H2; a.dOUT = r.dOUT; a.dZ2 = r.dZ2; a.dZ1 = r.dZ1;
    a.cs1 = r.cs1; a.cs2 = r.cs2; a.cs3 = r.cs3;
    a.n = r.n;
    a.k_per_split = k_per_split_for(r.n);
    a.g = net->g;
    return a;
}

void launch_weight_grad(const GradArgs& a, hipStream_t s)
{
    const dim3 grid(W_GRID), block(W_BLOCK);
    switch (a.k_per_split / 32) {
    case 2: hipLaunchKernelGGL(k_weight_grad<2>, grid, block, 0, s, a); break;
    case 4: hipLaunchKernelGGL(k_weight_grad<4>, grid, block, 0, s, a); break;
    case 6: hipLaunchKernelGGL(k_weight_grad<6>, grid, block, 0, s, a); break;
    default: hipLaunchKernelGGL(k_weight_grad<8>, grid, block, 0, s, a); break;
    }
}

unsigned blocks_for(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

extern "C" int64_t abc_mdn_param_count(void) { return NN_PARAMS; }

extern "C" abc_status abc_mdn_create(const abc_prior* prior, uint64_t init_seed, abc_mdn** out)
{
    ABC_REQUIRE(out != nullptr, "out is NULL");
    float lo[8], width[8];
    abc_status rc = prior_lo_width(prior, lo, width);
    if (rc) return rc;
    for (int j = 0; j < 8; ++j) ABC_REQUIRE(width[j] > 0.0f, "prior box %d has zero width", j);
    abc_mdn* n = new abc_mdn();
    for (int j = 0; j < 8; ++j) {
        n->lo[j] = prior->lo[j];
        n->hi[j] = prior->hi[j];
        n->tc[j] = 0.5f * (prior->lo[j] + prior->hi[j]);
        n->ts[j] = (prior->hi[j] - prior->lo[j]) / 3.46410161513775458705f;  // as proposal_standardiser
    }
    hipError_t e = hipSuccess;
    e = e ? e : hipMalloc((void**)&n->p, NN_PARAMS * sizeof(float));
    e = e ? e : hipMalloc((void**)&n->pb, NN_PB * sizeof(bf16));
    e = e ? e : hipMalloc((void**)&n->m, NN_PARAMS * sizeof(float));
    e = e ? e : hipMalloc((void**)&n->v, NN_PARAMS * sizeof(float));
    e = e ? e : hipMalloc((void**)&n->g, NN_PARAMS * sizeof(float));
    e = e ? e : hipMalloc((void**)&n->fmean, NN_IN * sizeof(float));
    e = e ? e : hipMalloc((void**)&n->fsd, NN_IN * sizeof(float));
    e = e ? e : hipMalloc((void**)&n->loss_acc, sizeof(float));
    e = e ? e : hipMalloc((void**)&n->colpart, sizeof(double) * 2 * NN_IN * CS_GROUPS);
    if (e != hipSuccess) {
        abc_mdn_destroy(n);
        return set_error(ABC_EHIP, "abc_mdn_create: %s", hipGetErrorString(e));
    }
    hipLaunchKernelGGL(k_mdn_init, dim3(blocks_for(NN_PARAMS)), dim3(256), 0, 0, n->p, init_seed);
    static_assert(NN_PB % 2 == 0, "cleared as float32");
    hipLaunchKernelGGL(k_zero_f32, dim3(blocks_for(NN_PB / 2)), dim3(256), 0, 0, reinterpret_cast<float*>(n->pb), NN_PB / 2);
    hipLaunchKernelGGL(k_params_bf16, dim3(blocks_for(NN_PARAMS)), dim3(256), 0, 0, n->p, n->pb);
    hipLaunchKernelGGL(k_zero_f32, dim3(blocks_for(NN_PARAMS)), dim3(256), 0, 0, n->m, NN_PARAMS);
    hipLaunchKernelGGL(k_zero_f32, dim3(blocks_for(NN_PARAMS)), dim3(256), 0, 0, n->v, NN_PARAMS);
    hipLaunchKernelGGL(k_zero_f32, dim3(1), dim3(NN_IN), 0, 0, n->fmean, NN_IN);
    std::vector<float> ones(NN_IN, 1.0f);
    e = hipMemcpy(n->fsd, ones.data(), NN_IN * sizeof(float), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) {
        abc_mdn_destroy(n);
        return set_error(ABC_EHIP, "abc_mdn_create: %s", hipGetErrorString(e));
    }
    *out = n;
    return ABC_OK;
}

extern "C" abc_status abc_mdn_destroy(abc_mdn* n)
{
    if (!n) return ABC_OK;
    free_ws(n);
    void* ptrs[] = {n->p, n->pb, n->m, n->v, n->g, n->fmean, n->fsd, n->loss_acc, n->colpart};
    for (void* q : ptrs)
        if (q) (void)hipFree(q);
    delete n;
    return ABC_OK;
}

extern "C" abc_status abc_mdn_params(abc_mdn* n, float** params, float** grads)
{
    ABC_REQUIRE(n != nullptr, "net is NULL");
    if (params) *params = n->p;
    if (grads) *grads = n->g;
    return ABC_OK;
}

extern "C" abc_status abc_mdn_sync_params(abc_mdn* n, void* stream)
{
    ABC_REQUIRE(n != nullptr, "net is NULL");
    hipLaunchKernelGGL(k_params_bf16, dim3(blocks_for(NN_PARAMS)), dim3(256), 0, as_stream(stream), n->p, n->pb);
    return check_launch("k_params_bf16");
}

extern "C" abc_status abc_mdn_simulate_features(const abc_prior* prior, uint64_t seed,
                                                uint32_t domain, uint32_t series, uint64_t first,
                                                int64_t n, int32_t T_lo, int32_t T_hi,
                                                double log10P_lo, double log10P_hi, int32_t A0,
                                                float* features, float* theta, int32_t* TP,
                                                void* stream)
{
    FeatArgs a{};
    abc_status rc = prior_lo_width(prior, a.lo, a.width);
    if (rc) return rc;
    for (int k = 0; k < 8; ++k) ABC_REQUIRE(prior->lo[k] >= 0.0f, "prior lo[%d] < 0", k);
    ABC_REQUIRE(domain <= 15u, "domain > 15");
    ABC_REQUIRE(n >= 0, "n < 0");
    ABC_REQUIRE(T_lo >= 1 && T_hi >= T_lo && T_hi <= ABC_T_MAX, "need 1 <= T_lo <= T_hi <= %d", ABC_T_MAX);
    ABC_REQUIRE(log10P_lo <= log10P_hi && log10P_hi <= 9.33, "bad population range");
    ABC_REQUIRE(A0 >= 1 && pow(10.0, log10P_lo) >= 4.0 * A0, "P must exceed 4 A0");
    if (n == 0) return ABC_OK;
    ABC_REQUIRE(features && theta, "NULL output");
    a.key = make_key(seed);
    a.domain = domain;
    a.series = series;
    a.first = first;
    a.n = n;
    a.T_lo = T_lo;
    a.T_hi = T_hi;
    a.lp_lo = log10P_lo;
    a.lp_hi = log10P_hi;
    a.A0 = A0;
    a.features = features;
    a.theta = theta;
    a.TP = TP;
    const hipStream_t s = as_stream(stream);
    const int bins = T_hi - T_lo + 1;
    // The order needs scratch, which a captured call must not take (a replay
    // would use it after it was grown or released) and a full device may not
    // have: the samples then go unordered, with the same results. Calls of
    // several threads on one stream share the scratch, so each enqueues its
    // launches before the next one's.
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    bool ordered = n >= FEAT_SORT_MIN && T_hi >= FEAT_SORT_T && n < ((int64_t)1 << 30) && bins > 1;
    if (ordered && (hipStreamIsCapturing(s, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone)) {
        (void)hipGetLastError();
        ordered = false;
    }
    static std::mutex enqueue;
    std::unique_lock<std::mutex> lock(enqueue, std::defer_lock);
    const int64_t room = n + 63 * (int64_t)bins;
    void* mem = nullptr;
    if (ordered) {
        lock.lock();
        if (stream_scratch(s, sizeof(uint32_t) * (2 * (size_t)bins + 1) + sizeof(int32_t) * (size_t)room, &mem, SCRATCH_PAIRS)) {
            (void)hipGetLastError();
            ordered = false;
        }
    }
    if (!ordered) {
        hipLaunchKernelGGL(k_mdn_features, dim3(blocks_for(n)), dim3(FEAT_BLOCK), 0, s, a, nullptr, nullptr);
        return check_launch("k_mdn_features");
    }
    FeatOrder o{};
    o.bins = bins;
    o.cnt = static_cast<uint32_t*>(mem);
    o.fill = o.cnt + bins;
    o.total = o.fill + bins;
    o.order = reinterpret_cast<int32_t*>(o.total + 1);
    hipLaunchKernelGGL(k_zero_f32, dim3((bins + 255) / 256), dim3(256), 0, s, reinterpret_cast<float*>(o.cnt), bins);
    const unsigned count_grid = (unsigned)((n + 8 * FEAT_BLOCK - 1) / (8 * FEAT_BLOCK));
    hipLaunchKernelGGL(k_feat_count, dim3(count_grid < 1024 ? count_grid : 1024), dim3(FEAT_BLOCK), 0, s, a, o);
    hipLaunchKernelGGL(k_feat_scan, dim3(1), dim3(FEAT_BINS), 0, s, o);
    hipLaunchKernelGGL(k_feat_place, dim3(count_grid), dim3(FEAT_BLOCK), 0, s, a, o);
    hipLaunchKernelGGL(k_mdn_features, dim3(blocks_for(room)), dim3(FEAT_BLOCK), 0, s, a, o.order, o.total);
    return check_launch("k_mdn_features");
}

extern "C" abc_status abc_series_features(const abc_series* ser, float* out, void* stream)
{
    abc_status rc;
    if ((rc = check_series(ser, true))) return rc;
    ABC_REQUIRE(out != nullptr, "out is NULL");
    hipLaunchKernelGGL(k_obs_features, dim3(1), dim3(128), 0, as_stream(stream), ser->obs, ser->T, out);
    return check_launch("k_obs_features");
}

extern "C" abc_status abc_mdn_fit_standardizer(abc_mdn* net, const float* features, int64_t n,
                                               void* stream)
{
    ABC_REQUIRE(net && features && n >= 2, "need a net and >= 2 feature rows");
    const hipStream_t s = as_stream(stream);
    if (n <= CS_FEW * CS_BLOCK) {
        hipLaunchKernelGGL(k_colstats_few, dim3(NN_IN), dim3(CS_BLOCK), 0, s, features, (int)n, net->fmean, net->fsd);
        return check_launch("k_colstats_few");
    }
    const int groups = (int)colstats_groups(n);
    if ((reinterpret_cast<uintptr_t>(features) & 15u) == 0)
        hipLaunchKernelGGL((k_colsums<true>), dim3(groups), dim3(CS_BLOCK), 0, s, features, n, net->colpart);
    else
        hipLaunchKernelGGL((k_colsums<false>), dim3(groups), dim3(CS_BLOCK), 0, s, features, n, net->colpart);
    hipLaunchKernelGGL(k_colstats, dim3(NN_IN), dim3(64), 0, s, n, net->colpart, groups, net->fmean, net->fsd);
    return check_launch("k_colstats");
}

extern "C" abc_status abc_mdn_forward(abc_mdn* net, const float* features, int64_t n, float* out,
                                      void* stream)
{
    ABC_REQUIRE(net && features && out && n >= 1 && n <= (1 << 20), "bad forward arguments");
    ABC_REQUIRE((reinterpret_cast<uintptr_t>(features) & 15u) == 0, "features must be 16-byte aligned");
    RowArgs a = row_args(net, row_map(net, features, nullptr, n), (int)n);
    a.out = out;
    launch_rows(a, false, as_stream(stream));
    return check_launch("abc_mdn_forward");
}

extern "C" abc_status abc_mdn_loss_grad(abc_mdn* net, const float* features, const float* theta,
                                        int64_t n, float* loss, float* grad, void* stream)
{
    ABC_REQUIRE(net && features && theta && n >= 1 && n <= (1 << 20), "bad arguments");
    ABC_REQUIRE((reinterpret_cast<uintptr_t>(features) & 15u) == 0, "features must be 16-byte aligned");
    abc_status rc = ensure_ws(net, (int)n);
    if (rc) return rc;
    const hipStream_t s = as_stream(stream);
    hipLaunchKernelGGL(k_zero_f32, dim3(1), dim3(64), 0, s, net->loss_acc, (int64_t)1);
    RowArgs a = row_args(net, row_map(net, features, theta, n), (int)n);
    a.loss = net->loss_acc;
    launch_rows(a, true, s);
    launch_weight_grad(grad_args(net, a), s);
    if (loss) ABC_HIP(hipMemcpyAsync(loss, net->loss_acc, sizeof(float), hipMemcpyDeviceToDevice, s));
    if (grad) ABC_HIP(hipMemcpyAsync(grad, net->g, NN_PARAMS * sizeof(float), hipMemcpyDeviceToDevice, s));
    return check_launch("abc_mdn_loss_grad");
}

extern "C" abc_status abc_mdn_train(abc_mdn* net, const float* features, const float* theta,
                                    int64_t n, int32_t epochs, int32_t batch, float lr,
                                    uint64_t shuffle_seed, float* loss_log, int64_t* steps_out,
                                    float* train_ms, void* stream)
{
    ABC_REQUIRE(net && features && theta, "NULL argument");
    ABC_REQUIRE((reinterpret_cast<uintptr_t>(features) & 15u) == 0, "features must be 16-byte aligned");
    ABC_REQUIRE(n >= batch && batch >= 64 && batch <= 65536 && n < (1ll << 31), "need 64 <= batch <= n < 2^31");
    ABC_REQUIRE(epochs >= 1 && epochs <= 10000, "epochs out of range");
    ABC_REQUIRE(isfinite(lr) && lr > 0.0f, "lr must be positive");
    abc_status rc = ensure_ws(net, batch);
    if (rc) return rc;
    const int spe = (int)(n / batch);  // steps per epoch (the partial batch is dropped)
    const int64_t steps = (int64_t)spe * epochs;
    // affine permutations j -> (a j + c) mod n, one per epoch
    std::vector<int64_t> ab(2 * (size_t)epochs);
    uint64_t st = shuffle_seed * 0x9E3779B97F4A7C15ull + 0x632BE59BD9B4E019ull;
    auto next = [&]() {  // splitmix64
        st += 0x9E3779B97F4A7C15ull;
        uint64_t z = st;
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        return z ^ (z >> 31);
    };
    auto gcd = [](int64_t x, int64_t y) { while (y) { int64_t t = x % y; x = y; y = t; } return x; };
    for (int e = 0; e < epochs; ++e) {
        int64_t a = 0;
        do { a = (int64_t)(next() % (uint64_t)n); } while (a == 0 || gcd(a, n) != 1);
        ab[2 * e] = a;
        ab[2 * e + 1] = (int64_t)(next() % (uint64_t)n);
    }
    const hipStream_t s = as_stream(stream);
    hipEvent_t t0, t1;
    ABC_HIP(hipEventCreate(&t0));
    ABC_HIP(hipEventCreate(&t1));
    struct EF { hipEvent_t a, b; ~EF() { (void)hipEventDestroy(a); (void)hipEventDestroy(b); } } ef{t0, t1};
    if (loss_log) hipLaunchKernelGGL(k_zero_f32, dim3(blocks_for(steps)), dim3(256), 0, s, loss_log, steps);
    hipLaunchKernelGGL(k_zero_f32, dim3(blocks_for(NN_PARAMS)), dim3(256), 0, s, net->m, NN_PARAMS);
    hipLaunchKernelGGL(k_zero_f32, dim3(blocks_for(NN_PARAMS)), dim3(256), 0, s, net->v, NN_PARAMS);

    // Two launches a step. They take longer than their launches, so a graph of
    // them gains nothing over the stream, and its capture took a tenth of a
    // short training run.
    RowArgs r = row_args(net, row_map(net, features, theta, n), batch);
    GradArgs f = grad_args(net, r);
    f.adam = 1;
    f.p = net->p; f.m = net->m; f.v = net->v; f.pb = net->pb;
    f.lr = lr; f.b1 = 0.9f; f.b2 = 0.999f; f.eps = 1e-8f;
    ABC_HIP(hipEventRecord(t0, s));
    for (int64_t k = 0; k < steps; ++k) {
        const int64_t e = k / spe;
        r.rm.mul = ab[2 * e];
        r.rm.add = ab[2 * e + 1];
        r.rm.j0 = (k % spe) * batch;
        r.loss = loss_log ? loss_log + k : nullptr;
        launch_rows(r, true, s);
        f.updates = (int)(k + 1);
        launch_weight_grad(f, s);
    }
    if ((rc = check_launch("abc_mdn_train"))) return rc;
    ABC_HIP(hipEventRecord(t1, s));
    ABC_HIP(hipEventSynchronize(t1));
    float ms = 0.0f;
    ABC_HIP(hipEventElapsedTime(&ms, t0, t1));
    if (train_ms) *train_ms = ms;
    if (steps_out) *steps_out = steps;
    return ABC_OK;
}

extern "C" abc_status abc_mdn_sample(const abc_mdn* net, const float* mix, float lambda,
                                     float inflate, const abc_stream* st, uint64_t first,
                                     int64_t n, float* theta, float* weight, void* stream)
{
    ABC_REQUIRE(isfinite(inflate) && inflate >= 1.0f && inflate <= 100.0f, "inflate must be in [1, 100]");
    ABC_REQUIRE(net && mix, "NULL net or mixture");
    abc_status rc;
    if ((rc = check_stream_sel(st))) return rc;
    ABC_REQUIRE(lambda >= 0.0f && lambda <= 1.0f, "lambda must be in [0, 1]");
    ABC_REQUIRE(n >= 0, "n < 0");
    if (n == 0) return ABC_OK;
    ABC_REQUIRE(theta && weight, "NULL output");
    SampleArgs a{};
    a.mix = mix;
    for (int j = 0; j < 8; ++j) {
        a.prop.lo[j] = net->lo[j]; a.prop.hi[j] = net->hi[j];
        a.prop.tc[j] = net->tc[j]; a.prop.ts[j] = net->ts[j];
    }
    a.prop.lambda = lambda;
    a.prop.log_inflate = logf(inflate);
    a.key = make_key(st->seed);
    a.domain = st->domain;
    a.series = st->series;
    a.first = first;
    a.n = n;
    a.theta = theta;
    a.weight = weight;
    hipLaunchKernelGGL(k_mdn_sample, dim3(blocks_for(n)), dim3(256), 0, as_stream(stream), a);
    return check_launch("k_mdn_sample");
}

extern "C" abc_status abc_mdn_set_params(abc_mdn* net, const float* src, void* stream)
{
    ABC_REQUIRE(net && src, "NULL argument");
    const hipStream_t s = as_stream(stream);
    ABC_HIP(hipMemcpyAsync(net->p, src, NN_PARAMS * sizeof(float), hipMemcpyDeviceToDevice, s));
    hipLaunchKernelGGL(k_params_bf16, dim3(blocks_for(NN_PARAMS)), dim3(256), 0, s, net->p, net->pb);
    return check_launch("abc_mdn_set_params");
}

extern "C" abc_status abc_mdn_get_params(const abc_mdn* net, float* dst, void* stream)
{
    ABC_REQUIRE(net && dst, "NULL argument");
    ABC_HIP(hipMemcpyAsync(dst, net->p, NN_PARAMS * sizeof(float), hipMemcpyDeviceToDevice,
                           as_stream(stream)));
    return ABC_OK;
}

extern "C" abc_status abc_mdn_get_standardizer(const abc_mdn* net, float* mean96, float* sd96,
                                               void* stream)
{
    ABC_REQUIRE(net && mean96 && sd96, "NULL argument");
    const hipStream_t s = as_stream(stream);
    ABC_HIP(hipMemcpyAsync(mean96, net->fmean, NN_IN * sizeof(float), hipMemcpyDeviceToDevice, s));
    ABC_HIP(hipMemcpyAsync(sd96, net->fsd, NN_IN * sizeof(float), hipMemcpyDeviceToDevice, s));
    return ABC_OK;
}
