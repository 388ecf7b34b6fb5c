// Prior sampling, simulate+distance and trajectory recording kernels, and their
// C-ABI entry points (abc_sample_prior, abc_simulate_distance,
// abc_simulate_record).
//
// simulate+distance: one lane per trajectory. The observed series of the
// launch is staged once per workgroup in LDS as rows of one day (log2(1 + O),
// or O for the raw distance), so the day loop touches no global memory at all: per sample the
// kernel reads 32 B of theta (or none when theta is drawn in-kernel) and
// writes 4 B of distance. A sample leaves the day loop as soon as its running
// squared distance passes the early-exit bound.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "bound.hpp"
#include "common.hpp"
#include "model.hpp"

namespace abc {

constexpr int SIM_BLOCK = 256;

struct SimArgs {
    const float* theta;  // [n][8] or null -> prior draw
    float lo[8];
    float width[8];
    float hi[8];         // support check of supplied theta (box != 0)
    int32_t box;
    Key key;
    uint32_t domain;
    uint32_t series;
    uint64_t first;
    int64_t n;
    int32_t P, A0, R0, D0, T;
    const int32_t* obs;  // [3][T]
    float scale;
    float exit_f32;      // squared-distance early-exit bound (float path)
    double exit_f64;     // same, double path
    float* dist;
    double* dist64;
    unsigned long long* days;  // nullable: += sample-days executed
    int32_t* traj;       // record mode: [n][T+1][6]
    int32_t refill_min;  // refill a wave's idle lanes once at least this many are idle
    int32_t lb_ntb;      // future-days bound table: time blocks (0 = no bound)
    int32_t walk_at;     // float64: byte offset of the wavefronts' row arrays in LDS
    int32_t lb_sh;       // days per time block = 2^lb_sh
};

__device__ __forceinline__ void load_or_draw_theta(const SimArgs& a, bool prior, int64_t k,
                                                   uint64_t i, float th[8])
{
    if (prior) {
        prior_draw(a.key, i, a.series, a.domain, a.lo, a.width, th);
    } else {
        const float4* p = reinterpret_cast<const float4*>(a.theta + 8 * k);
        const float4 x = p[0], y = p[1];
        th[0] = x.x; th[1] = x.y; th[2] = x.z; th[3] = x.w;
        th[4] = y.x; th[5] = y.y; th[6] = y.z; th[7] = y.w;
    }
}

// Prior support of a supplied theta (closed box; NaN is outside).
__device__ __forceinline__ bool outside_box(const SimArgs& a, const float th[8])
{
    bool out = false;
#pragma unroll
    for (int j = 0; j < 8; ++j) out |= !(th[j] >= a.lo[j] && th[j] <= a.hi[j]);
    return out;
}

// ---------------------------------------------------------------------------
// float32 simulate + distance with per-wave lane refill
//
// Each wavefront owns a fixed set of 64-sample chunks (chunk c = wave id +
// j * number of waves) and walks through them as a queue. A lane whose
// sample is finished -- early exit or day T reached -- writes its distance
// and takes the next queue position at once, so lanes never idle behind the
// slowest trajectory of the wave. Per-sample constants (rates, I0) are
// produced 64 at a time by the whole wave into a small per-wave LDS ring,
// which keeps the prior draw (two Philox calls) out of the divergent refill
// branch. SPL independent sample slots per lane add instruction-level
// parallelism. The result of each sample depends only on its index and
// theta, never on the launch shape or on which lane ran it.
// ---------------------------------------------------------------------------
// Everything a lane needs to start a sample, prepared by the whole wave so the
// divergent refill branch only copies 48 bytes out of LDS.
struct alignas(16) Slot {
    float a0, al, n, be, ga, de, bh;
    int32_t i0;                   // -1: prior density zero (not simulated)
    uint32_t c1base, g3, h3, f3;  // per-sample part of Philox rounds 1-3
};

template <bool PRIOR>
__device__ __forceinline__ void fill_slot(const SimArgs& a, int64_t k, uint32_t u0, Slot& out)
{
    float thv[8];
    load_or_draw_theta(a, PRIOR, k, a.first + (uint64_t)k, thv);
    const Theta th = theta_from(thv);
    const RatesF r = rates_f32(th);
    const State s0 = init_state(th.ka, a.P, a.A0, a.R0, a.D0);
    PhiloxDays ph;
    ph.begin(a.first + (uint64_t)k, u0, a.key);
    out.a0 = r.a0; out.al = r.al; out.n = r.n; out.be = r.be;
    out.ga = r.ga; out.de = r.de; out.bh = r.bh; out.i0 = s0.I;
    out.c1base = ph.c1base; out.g3 = ph.g3; out.h3 = ph.h3; out.f3 = ph.f3;
    if (!PRIOR && a.box && outside_box(a, thv)) out.i0 = -1;
}

struct Lane {
    StateD s;
    RatesF r;
    PhiloxDays ph;
    int64_t k;     // sample offset within the launch
    uint32_t w;    // fourth counter word of the next day, day << 8 | domain << 4; 0: no sample (idle)
    uint32_t p;    // LDS address of the day's observed row
    float acc, comp;
};

// BOUND: with the future-days bound (log1p distance and an exit bound). With
// one sample per lane the scheduler is asked for 7 wavefronts per SIMD: left
// alone it takes 76 registers (6 wavefronts), asked for 8 it takes 53 and
// orders the day for registers instead of latency; at 62 registers 1e7 samples
// of T = 100 take 908 us against 924 and 1017.
template <int NOISE, int DIST, bool KAHAN, bool PRIOR, int SPL, bool BOUND>
__global__ __launch_bounds__(1024 / SPL, SPL == 1 ? 7 : 1) void k_simulate_f32(SimArgs a)
{
    constexpr int RING = 64;  // one chunk of 64 queue positions
    extern __shared__ float lds_f[];
    const int T = a.T;
    const int obs_words = 4 * T;
    const int ntb = BOUND ? a.lb_ntb : 0;
    float* tab = lds_f + obs_words;  // [ntb][2][LB_Q] future-days bound
    Slot* ring_all = reinterpret_cast<Slot*>(lds_f + obs_words + 2 * LB_Q * ntb);

    // observed rows (obs_row)
    const uint32_t tab_at = lds_address(tab);
    for (int q = threadIdx.x; q < T; q += blockDim.x)
        reinterpret_cast<float4*>(lds_f)[q] =
            obs_row<DIST>(a.obs[q], a.obs[T + q], a.obs[2 * T + q],
                          tab_at + (uint32_t)sizeof(float) * (2 * LB_Q * ((q + 1) >> a.lb_sh)));
    if (BOUND) {
        // b_s of R and D in float64, staged where the ring will live
        double* stage = reinterpret_cast<double*>(ring_all);
        for (int q = threadIdx.x; q < 2 * T; q += blockDim.x)
            stage[q] = log1p((double)a.obs[T + q]) * 1.44269504088896340736;
        __syncthreads();
        build_future_bound(stage, T, a.lb_sh, ntb, (double)a.exit_f32, tab);
    }
    __syncthreads();

    // The float32 waves take issue priority over waves of other kernels
    // sharing the compute unit (the float64 band decision of the previous
    // launch runs beside this one and fills the gaps instead of holding up
    // the waves whose static share of the launch it would delay).
    __builtin_amdgcn_s_setprio(1);
    const int lane = threadIdx.x & 63;
    // the wavefront index is uniform over the wave: kept scalar, so is the
    // queue arithmetic derived from it
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    Slot* ring = ring_all + wv * RING;
    const int64_t wg = (int64_t)blockIdx.x * (blockDim.x >> 6) + wv;
    const int64_t nw = (int64_t)gridDim.x * (blockDim.x >> 6);
    const int64_t nchunks = (a.n + 63) >> 6;
    if (wg >= nchunks) return;
    // queue positions of this wave (fits 32 bits: the host limits n per launch);
    // its j-th chunk is wg + j nw
    const uint32_t Q = __builtin_amdgcn_readfirstlane((uint32_t)(((nchunks - 1 - wg) / nw + 1) << 6));

    const PhiloxSeries ps = philox_series(a.series, a.key);
    const float invP = 1.0f / (float)a.P;
    const float nc = noise_c(a.scale);
    const float dscale = DIST == 0 ? 0.693147180559945309417f : 1.0f;
    const uint32_t w1 = 256u | (a.domain << 4), wend = ((uint32_t)T << 8) | (a.domain << 4);
    const uint32_t row1 = lds_address(lds_f);
    const int32_t room = a.P - (a.A0 + a.R0 + a.D0);

    // the ring holds one chunk: sample offsets cur_base + lane, of which
    // cur_valid exist (fewer than 64 only in the last chunk)
    int64_t cur_base = 0;
    uint32_t cur_valid = 0;
    auto fill = [&](int64_t c) {
        cur_base = c << 6;
        cur_valid = (uint32_t)min(a.n - cur_base, (int64_t)64);
        if ((uint32_t)lane < cur_valid) fill_slot<PRIOR>(a, cur_base + lane, ps.u0, ring[lane]);
    };

    // wave-uniform queue state, kept in scalar registers
    uint32_t qb = 0;               // next queue position
    uint32_t filled = 0xFFFFFFFFu; // chunk currently in the ring
    Lane L[SPL];
#pragma unroll
    for (int j = 0; j < SPL; ++j) {
        L[j] = Lane{};  // idle, with a valid state (no people) and row
        L[j].s = state_d(0, 0, 0, 0, 0);
        L[j].p = row1;
    }
    uint64_t days_done = 0;        // of the whole wavefront

    while (true) {
        // refill every idle slot from the wave queue, in queue order, once at
        // least refill_min lanes are idle; a refill may span the end of one
        // chunk and the start of the next
        uint64_t any = 0;
#pragma unroll
        for (int j = 0; j < SPL; ++j) {
            uint64_t m = __ballot(L[j].w == 0u);
            if (__popcll(m) >= a.refill_min) {
                while (m != 0ull && qb < Q) {
                    const uint32_t jc = qb >> 6;
                    if (jc != filled) {
                        fill(wg + (int64_t)jc * nw);
                        filled = jc;
                    }
                    const uint32_t off = qb & 63u, avail = 64u - off;
                    const uint32_t rank = mask_rank(m);
                    const uint64_t took = m & __ballot(rank < avail);
                    if (in_mask(took) && off + rank < cur_valid) {
                        const Slot sl = ring[off + rank];
                        const int64_t k = cur_base + (int64_t)(off + rank);
                        if (!PRIOR && sl.i0 < 0) {
                            a.dist[k] = INFINITY;
                            if (a.dist64) a.dist64[k] = (double)INFINITY;
                        } else {
                            Lane& l = L[j];
                            l.r = RatesF{sl.a0, sl.al, sl.n, sl.be, sl.ga, sl.de, sl.bh};
                            l.s = state_d(room, a.A0, a.R0, a.D0, sl.i0);
                            l.ph.c1base = sl.c1base; l.ph.g3 = sl.g3; l.ph.h3 = sl.h3; l.ph.f3 = sl.f3;
                            l.k = k;
                            l.w = w1;
                            l.p = row1;
                            l.acc = 0.0f;
                            l.comp = 0.0f;
                        }
                    }
                    qb += (uint32_t)__popcll(took);
                    m &= ~took;  // lanes still without a position
                }
                m = __ballot(L[j].w == 0u);
            }
            any |= ~m;
            days_done += (uint64_t)__popcll(~m);
        }
        if (any == 0ull && qb >= Q) break;

        // One day of every slot. Idle lanes take it too, from the state that their
        // last sample left, and drop it: behind any branch, also one past a
        // wavefront without a sample, the nine values of a day were new
        // registers, copied back each day. Three countries of 1e7 samples: 1.91 ->
        // 1.87 ms, 64 series in rounds (the same loop) 24.7 -> 23.9. Without early
        // exits it gains nothing: there the 16 wide multiplications and 16
        // transcendentals of a day, four times as long as other instructions, bound it.
#pragma unroll
        for (int j = 0; j < SPL; ++j) {
            Lane& l = L[j];
            const bool live = l.w != 0u;
            const float4 ob = lds_row(l.p);
            const uint4 words = l.ph.day(l.w, ps.b1, a.key);
            float lr, ld;
            day_distance_f32<NOISE, DIST, KAHAN>(l.s, l.r, words, invP, nc, ob, l.acc, l.comp, lr, ld);
            float sum = l.acc;
            if (BOUND) sum += future_bound(__float_as_uint(ob.w), lr, ld);
            const bool exited = sum > a.exit_f32;
            const bool done = exited | (l.w == wend);
            if (done & live) {
                const float dd = exited ? INFINITY : finish_distance_f32(l.acc, dscale);
                a.dist[l.k] = dd;
                if (a.dist64) a.dist64[l.k] = (double)dd;
            }
            const bool idle = done | !live;
            l.w = idle ? 0u : l.w + 256u;
            l.p = idle ? row1 : l.p + (uint32_t)sizeof(float4);
        }
    }
    if (a.days && lane == 0) atomicAdd(a.days, (unsigned long long)days_done);
}

// ---------------------------------------------------------------------------
// float64 simulate + distance (precision study, recheck of borderline samples)
// ---------------------------------------------------------------------------

// Lane refill as in the float32 kernel: each wavefront walks its share of the
// 64-sample chunks as a queue, and the idle lanes take the next positions once
// at least F64_REFILL of them are idle. A sample's parameters are drawn (or
// read) by the lane that takes it: two Philox blocks are short beside a
// float64 day. Bound by float64 issue: one day is about 430 instructions of
// four cycles each. With one lane per sample for the whole launch, early exits
// left most lanes idle behind the longest trajectory of their wavefront: 1e6
// samples of T = 100 at the 1e-3 quantile took 3.46 ms (with the library's
// functions), now 0.67 ms.
constexpr int F64_BLOCK = 512;
constexpr int F64_REFILL = 8;
constexpr int F64_BLOCKS_PER_CU = 1;
// A wavefront whose queue is empty and that has few samples left walks those
// again from their first day, four lanes each as the rows of a band decision, if
// that is sooner than their days to come: a day takes a lane 3 us, whose
// instructions wait for each other, and eight rows 0.7. T = 100 at the 1e-3
// quantile, when the walk came: 1e4 samples 310 -> 205 us, 1e5 308 -> 220, 1e6
// 765 -> 715 (the last is 672 now); with four rows 225, 267 and 726, with sixteen
// 196, 224 and 723.
constexpr int F64_WALK_ROWS = 8;

constexpr int F64_WALK_GAIN = 4;  // days of a row in the time of a lane's day

// LDS arrays of a wavefront that walks rows (simulate_rows_f64_wave)
struct RowLds {
    Math64* tab;
    double* lobs;
    double* zs;
    uint64_t* rix;
    int64_t* rq;
    int32_t* xs;
    float* rth;
};

// the arrays of wavefront wv, after each other from base
constexpr size_t F64_WALK_BYTES = sizeof(double) * 5 * ROW_PAIRS + (sizeof(uint64_t) + sizeof(int64_t)) * F64_WALK_ROWS +
                                  sizeof(int32_t) * 4 * ROW_PAIRS + sizeof(float) * 8 * F64_WALK_ROWS;

__device__ __forceinline__ RowLds wave_rows(double* base, int wv, Math64* tab, double* lobs)
{
    RowLds l;
    l.tab = tab;
    l.lobs = lobs;
    l.zs = base + wv * (F64_WALK_BYTES / sizeof(double));
    l.rix = reinterpret_cast<uint64_t*>(l.zs + 5 * ROW_PAIRS);
    l.rq = reinterpret_cast<int64_t*>(l.rix + F64_WALK_ROWS);
    l.xs = reinterpret_cast<int32_t*>(l.rq + F64_WALK_ROWS);
    l.rth = reinterpret_cast<float*>(l.xs + 4 * ROW_PAIRS);
    return l;
}

template <int NOISE, int DIST, bool PRIOR>
__global__ __launch_bounds__(F64_BLOCK) void k_simulate_f64(SimArgs a)
{
#pragma clang fp contract(off)
    // Math64 | [3][T] | future-days bound [ntb][2][LB_Q] f32, then the space that builds it
    extern __shared__ double lds_d[];
    Math64& tab = *reinterpret_cast<Math64*>(lds_d);
    double* lobs = lds_d + sizeof(Math64) / sizeof(double);
    const int ntb = DIST == 0 ? a.lb_ntb : 0;
    double* stage = lobs + 3 * a.T;
    float* lbt = reinterpret_cast<float*>(stage + (ntb > 0 ? 2 * a.T + LB_MAX_SEG * 2 * LB_Q : 0));
    stage_math64(tab);
    __syncthreads();
    stage_obs_f64<DIST>(a.obs, a.T, lobs, tab);
    if (DIST == 0 && ntb > 0) {
        for (int q = threadIdx.x; q < 2 * a.T; q += blockDim.x)
            stage[q] = log1p((double)a.obs[a.T + q]) * 1.44269504088896340736;
        __syncthreads();
        build_future_bound(stage, a.T, a.lb_sh, ntb, (double)a.exit_f32, lbt);
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t wg = (int64_t)blockIdx.x * (F64_BLOCK / 64) + wv;
    const int64_t nw = (int64_t)gridDim.x * (F64_BLOCK / 64);
    const int64_t nchunks = (a.n + 63) >> 6;
    if (wg >= nchunks) return;
    // queue positions of this wave: its j-th chunk is wg + j nw
    const int64_t Q = ((nchunks - 1 - wg) / nw + 1) << 6;
    const int T = a.T;
    const double Pd = (double)a.P, rP = 1.0 / Pd, scale = (double)a.scale;
    const PhiloxSeries ps = philox_series(a.series, a.key);
    constexpr double LOG2E = 1.44269504088896340736;
    const uint32_t lb_at = lds_address(lbt);

    const RowLds walk = wave_rows(lds_d + a.walk_at / sizeof(double), wv, &tab, lobs);
    int64_t qb = 0, k = 0;
    PhiloxDays ph{};
    int t = 0;  // the day simulated next; 0: no sample (idle)
    State s{};
    float thv[8];
    bool mid = true;
    double acc = 0.0;
    int rows = 0;  // gathered for a walk
    auto put_row = [&](int slot, int64_t sample) {
        walk.rq[slot] = sample;
        walk.rix[slot] = a.first + (uint64_t)sample;
#pragma unroll
        for (int j = 0; j < 8; ++j) walk.rth[8 * slot + j] = thv[j];
    };
    auto walk_rows = [&](int nr) {
        wave_lds_sync();
        const double dd = simulate_rows_f64_wave<NOISE, DIST, true>(
            nr, walk.rth, walk.rix, a.key, a.series, a.domain, a.P, a.A0, a.R0, a.D0, T, scale, lobs, tab, walk.zs,
            walk.xs, a.exit_f64);
        if (lane < nr) {
            const int64_t q = walk.rq[lane];
            a.dist[q] = (float)dd;
            if (a.dist64) a.dist64[q] = dd;
        }
    };
    while (true) {
        const uint64_t m = __ballot(t == 0);
        if (qb < Q && __popcll(m) >= F64_REFILL) {
            const int64_t q = qb + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                             __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            const int64_t kk = ((wg + (q >> 6) * nw) << 6) + (q & 63);
            if (t == 0 && q < Q && kk < a.n) {
                k = kk;
                load_or_draw_theta(a, PRIOR, k, a.first + (uint64_t)k, thv);
                if (!PRIOR && a.box && outside_box(a, thv)) {
                    a.dist[k] = INFINITY;
                    if (a.dist64) a.dist64[k] = (double)INFINITY;
                } else {
                    s = init_state(thv[7], a.P, a.A0, a.R0, a.D0);
                    mid = theta_mid(thv) && (PRIOR || !negative_start(thv));
                    ph.begin(a.first + (uint64_t)k, ps.u0, a.key);
                    acc = 0.0;
                    t = 1;
                }
            }
            qb += __popcll(m);
        }
        const uint64_t live = __ballot(t != 0);
        if (live == 0ull) {
            if (qb >= Q) break;
            continue;
        }
        const int nr = __popcll(live);
        if (qb >= Q && nr <= F64_WALK_ROWS) {
            int left = t != 0 ? T - t + 1 : 0;
#pragma unroll
            for (int off = 32; off; off >>= 1) left = max(left, __shfl_xor(left, off, 64));
            if (left * F64_WALK_GAIN > T + F64_WALK_GAIN * 4) {
                if (t != 0) put_row(mask_rank(live), k);
                // where the walk's code stands decides the registers of the days: behind
                // the loop it is 2 to 3 % sooner with given parameters, where many reach the
                // last day; prior draws with exits 1 to 3 % sooner with it here
                if (PRIOR) walk_rows(nr);
                else rows = nr;
                break;
            }
        }
        if (t != 0) {
            const uint4 w = ph.day(ctr_word3((uint32_t)t, a.domain, 0), ps.b1, a.key);
            double z[5];
            normals_f64(w, tab, z);
            day_step_f64<NOISE, !PRIOR>(s, theta_from(thv), mid, Pd, rP, scale, z, tab);
            const int32_t X[3] = {s.A, s.R, s.D};
            double lx[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                lx[c] = DIST == 0 ? log1p_count_f64(X[c], tab) : (double)X[c];
                if (DIST == 0 && !PRIOR && !mid && X[c] < 0) lx[c] = log1p_general((double)X[c]);
                const double d = lx[c] - lobs[c * T + t - 1];
                acc += d * d;
            }
            // the days still to come, bounded below in float32 with its own
            // margins: a sample it ends would have passed the exit bound
            float lb = 0.0f;
            if (DIST == 0 && ntb > 0 && (PRIOR || mid)) {  // (counts of 0 or more)
                lb = future_bound(lb_at + (uint32_t)sizeof(float) * 2 * LB_Q * (uint32_t)(t >> a.lb_sh),
                                  (float)(lx[1] * LOG2E), (float)(lx[2] * LOG2E));
            }
            const bool exited = acc > a.exit_f64 ||
                                (lb > 0.0f && (float)(acc * (LOG2E * LOG2E)) + lb > a.exit_f32);
            if (exited || t == T) {
                const double dd = exited ? (double)INFINITY : sqrt_mid(acc);
                a.dist[k] = (float)dd;
                if (a.dist64) a.dist64[k] = dd;
                t = 0;
            } else {
                ++t;
            }
        }
    }
    if (rows > 0) walk_rows(rows);
}

// Float64 decision for the candidates of a float32 pass (compacted at
// eps (1 + w)): rows whose float32 distance lies above eps (1 - w) are
// simulated again in float64 and decided by that distance; then the kept
// rows are compacted in place, in their original order. One workgroup.
struct RecheckArgs {
    SimArgs sim;
    float eps;
    float band_lo;   // eps (1 - w)
    float band_hi;   // eps (1 + w)
    int64_t capacity;
    int64_t* idx;
    float* theta;
    float* dist;
    float* weight;
    int64_t* count;
    uint8_t* keep;   // scratch [capacity]
    int32_t* rechecked;  // nullable: number of rows simulated in float64
    int32_t scan_min;    // candidates per wavefront at least
    int32_t all_rows;    // 1: every candidate is decided in float64, not only the band
    double* dist64;      // nullable [capacity]: float64 distance of each row so decided
};

// LDS of the float64 row kernels, for up to R rows per wavefront:
// Math64 | obs [3 T] f64 | zs [5 ROW_PAIRS] f64 | rix [R] u64 | rq [R] i64 | xs [4 ROW_PAIRS] i32 | rth [R][8] f32
__device__ __forceinline__ RowLds row_lds(double* base, int T, int R)
{
    RowLds l;
    l.tab = reinterpret_cast<Math64*>(base);
    l.lobs = base + sizeof(Math64) / sizeof(double);
    l.zs = l.lobs + 3 * T;
    l.rix = reinterpret_cast<uint64_t*>(l.zs + 5 * ROW_PAIRS);
    l.rq = reinterpret_cast<int64_t*>(l.rix + R);
    l.xs = reinterpret_cast<int32_t*>(l.rq + R);
    l.rth = reinterpret_cast<float*>(l.xs + 4 * ROW_PAIRS);
    return l;
}

// Pass 1: each wavefront scans a contiguous block of candidates (enough for
// the grid to cover the candidate count, at least scan_min), 64 at a time;
// the in-band ones are gathered, in candidate order, into groups of up to
// ROWS_PER_WAVE_MAX rows that are simulated side by side in float64
// (simulate_rows_f64_wave); the others only get their keep flag. A large
// scan_min packs the in-band rows into few wavefronts, so that they take few
// issue slots from a float32 launch running beside them; ROW_SCAN_ALONE
// gives a wavefront about one of them, for the shortest latency (a quarter of the
// candidates is in the band). Workgroups that meet no in-band row never stage the
// observed series.
template <int NOISE, int DIST>
__device__ __forceinline__ void recheck_group(const RecheckArgs& r, const RowLds& l, int nr,
                                              bool& staged)
{
    const SimArgs& a = r.sim;
    if (!staged) {
        stage_math64(*l.tab);
        __syncthreads();
        stage_obs_f64<DIST>(a.obs, a.T, l.lobs, *l.tab);
        staged = true;
    }
    __syncthreads();
    const double d64 = simulate_rows_f64_wave<NOISE, DIST>(
        nr, l.rth, l.rix, a.key, a.series, a.domain, a.P, a.A0, a.R0, a.D0, a.T, (double)a.scale,
        l.lobs, *l.tab, l.zs, l.xs);
    const int lane = threadIdx.x;
    if (lane < nr) {
        const int64_t qq = l.rq[lane];
        r.keep[qq] = d64 <= (double)r.eps ? 1 : 0;
        r.dist[qq] = (float)d64;
        if (r.dist64) r.dist64[qq] = d64;
    }
    if (lane == 0 && r.rechecked) atomicAdd(r.rechecked, nr);
    __syncthreads();  // the row slots are refilled next
}

template <int NOISE, int DIST>
__global__ __launch_bounds__(64) void k_recheck_flags(RecheckArgs r)
{
    extern __shared__ double lds_r[];
    const int64_t count = *r.count;
    if (count > r.capacity) return;  // overflowed candidate set: left for the caller to rerun
    const RowLds l = row_lds(lds_r, r.sim.T, ROWS_PER_WAVE_MAX);
    int64_t per = (count + gridDim.x - 1) / gridDim.x;
    if (per < r.scan_min) per = r.scan_min;
    const int64_t q0 = (int64_t)blockIdx.x * per;
    if (q0 >= count) return;
    const int64_t q1 = q0 + per < count ? q0 + per : count;
    const int lane = threadIdx.x;
    const uint64_t below = (1ull << lane) - 1ull;
    bool staged = false;
    int nr = 0;  // rows gathered so far (wave-uniform)
    for (int64_t c0 = q0; c0 < q1; c0 += 64) {
        const int64_t q = c0 + lane;
        bool inb = false;
        if (q < q1) {
            const float d = r.dist[q];
            inb = r.all_rows || (d > r.band_lo && d <= r.band_hi);
            if (!inb) r.keep[q] = d <= r.eps ? 1 : 0;
        }
        uint64_t m = __ballot(inb);
        while (m) {
            // the lowest (ROWS_PER_WAVE_MAX - nr) in-band lanes join the group
            uint64_t take = 0;
            for (int room = ROWS_PER_WAVE_MAX - nr; room > 0 && m; --room) {
                const uint64_t b = m & (~m + 1ull);
                take |= b;
                m ^= b;
            }
            if ((take >> lane) & 1ull) {
                const int slot = nr + __popcll(take & below);
                l.rq[slot] = q;
                l.rix[slot] = (uint64_t)r.idx[q];
#pragma unroll
                for (int j = 0; j < 8; ++j) l.rth[8 * slot + j] = r.theta[8 * q + j];
            }
            nr += __popcll(take);
            if (nr == ROWS_PER_WAVE_MAX) {
                recheck_group<NOISE, DIST>(r, l, nr, staged);
                nr = 0;
            }
        }
    }
    if (nr > 0) recheck_group<NOISE, DIST>(r, l, nr, staged);
}

// Pass 2: stable in-place compaction of the kept rows, COMPACT_BLOCK rows at a
// time in one workgroup. Bound by the round trips of a step, so a step takes as
// many rows as a workgroup has lanes; rows before the first dropped one stay
// where they are. Averaged over the chunks of eight SMC generations of 4096: 20 us
// with 256 rows a step, now 11.
constexpr int COMPACT_BLOCK = 1024;

__global__ __launch_bounds__(COMPACT_BLOCK) void k_recheck_compact(RecheckArgs r)
{
    __shared__ int wave_tot[COMPACT_BLOCK / 64];
    const int64_t count = *r.count;
    if (count > r.capacity) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int64_t base = 0;  // rows kept so far
    bool next = (int64_t)threadIdx.x < count && r.keep[threadIdx.x];
    for (int64_t c0 = 0; c0 < count; c0 += COMPACT_BLOCK) {
        const int64_t q = c0 + threadIdx.x;
        const bool kp = next;
        next = q + COMPACT_BLOCK < count && r.keep[q + COMPACT_BLOCK];
        const uint64_t m = __ballot(kp);
        const int rank = __popcll(m & ((1ull << lane) - 1ull));
        if (lane == 0) wave_tot[wave] = __popcll(m);
        __syncthreads();
        int off = 0, tot = 0;
#pragma unroll
        for (int v = 0; v < COMPACT_BLOCK / 64; ++v) {
            const int t = wave_tot[v];
            if (v < wave) off += t;
            tot += t;
        }
        const int64_t dst = base + off + rank;
        const bool move = kp && dst != q;
        int64_t id = 0;
        float th[8], d = 0.0f, w = 0.0f;
        double d64 = 0.0;
        if (move) {
            id = r.idx[q];
#pragma unroll
            for (int j = 0; j < 8; ++j) th[j] = r.theta[8 * q + j];
            d = r.dist[q];
            if (r.weight) w = r.weight[q];
            if (r.dist64) d64 = r.dist64[q];
        }
        __syncthreads();  // every row of this chunk is in registers before any write
        if (move) {
            r.idx[dst] = id;
#pragma unroll
            for (int j = 0; j < 8; ++j) r.theta[8 * dst + j] = th[j];
            r.dist[dst] = d;
            if (r.weight) r.weight[dst] = w;
            if (r.dist64) r.dist64[dst] = d64;
        }
        base += tot;
    }
    if (threadIdx.x == 0) *r.count = base;
}

__global__ void k_zero_i32(int32_t* p)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) *p = 0;
}


// float64 distances of listed rows (sample idx[q], theta[q]), rows_per_wave
// consecutive rows at a time per wavefront, walked side by side in lanes.
struct RowsArgs {
    SimArgs sim;
    const int64_t* idx;
    double* dist64;
    int32_t rows_per_wave;
};

template <int NOISE, int DIST>
__global__ __launch_bounds__(64) void k_rows_f64(RowsArgs r)
{
    extern __shared__ double lds_w[];
    const SimArgs& a = r.sim;
    const int T = a.T, R = r.rows_per_wave;
    const RowLds l = row_lds(lds_w, T, R);
    stage_math64(*l.tab);
    __syncthreads();
    stage_obs_f64<DIST>(a.obs, T, l.lobs, *l.tab);
    const int lane = threadIdx.x;
    for (int64_t q0 = (int64_t)blockIdx.x * R; q0 < a.n; q0 += (int64_t)gridDim.x * R) {
        const int nr = (int)(a.n - q0 < R ? a.n - q0 : R);
        if (lane < nr) {
            l.rix[lane] = (uint64_t)r.idx[q0 + lane];
#pragma unroll
            for (int j = 0; j < 8; ++j) l.rth[8 * lane + j] = a.theta[8 * (q0 + lane) + j];
        }
        __syncthreads();
        const double d64 = simulate_rows_f64_wave<NOISE, DIST>(
            nr, l.rth, l.rix, a.key, a.series, a.domain, a.P, a.A0, a.R0, a.D0, T,
            (double)a.scale, l.lobs, *l.tab, l.zs, l.xs);
        if (lane < nr) r.dist64[q0 + lane] = d64;
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// trajectory recording (float32 or float64 arithmetic)
// ---------------------------------------------------------------------------
__device__ __forceinline__ void store_state(int32_t* row, const State& s)
{
    row[0] = s.S; row[1] = s.I; row[2] = s.A; row[3] = s.R; row[4] = s.D; row[5] = s.Ru;
}

template <int NOISE, bool F64>
__global__ __launch_bounds__(SIM_BLOCK) void k_record(SimArgs a)
{
    __shared__ Math64 tab;
    if (F64) {
        stage_math64(tab);
        __syncthreads();
    }
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= a.n) return;
    const uint64_t i = a.first + (uint64_t)k;
    float thv[8];
    load_or_draw_theta(a, false, k, i, thv);
    const Theta th = theta_from(thv);
    const bool mid = theta_mid(thv) && !negative_start(thv);
    const double rP = 1.0 / (double)a.P;
    State s = init_state(th.ka, a.P, a.A0, a.R0, a.D0);
    int32_t* out = a.traj + (int64_t)6 * (a.T + 1) * k;
    store_state(out, s);
    const RatesF r = rates_f32(th);
    const float invP = 1.0f / (float)a.P;
    const float nc = noise_c(a.scale);
    auto days = [&](auto negative) {
        for (int t = 1; t <= a.T; ++t) {
            const uint4 w = stream_words(a.key, i, a.series, ctr_word3((uint32_t)t, a.domain, 0));
            if (F64) {
                double z[5];
                normals_f64(w, tab, z);
                day_step_f64<NOISE, negative>(s, th, mid, (double)a.P, rP, (double)a.scale, z, tab);
            } else {
                Noise32 z;
                normals_f32(w, nc, z);
                day_step_f32<NOISE>(s, r, invP, z);
            }
            store_state(out + 6 * t, s);
        }
    };
    if (F64 && __ballot(negative_start(thv)) != 0ull) days(std::true_type{});
    else days(std::false_type{});
}

// The float32 recording of few rows. With 64 rows per wavefront a thousand rows
// are 16 wavefronts, each alone on its SIMD, and a day costs what one wavefront
// can issue. The noise needs no state, so a workgroup takes 64 rows: three
// wavefronts draw the noise of a window of days into LDS while the fourth walks
// the window before it, which leaves it about a third of a day's instructions.
// It is bound by that wavefront's issue and the chain of a day. 120 days of
// 1000 rows: 37 -> 25 us.
constexpr int RECORD_DAYS = 6;

template <int NOISE>
__global__ __launch_bounds__(256) void k_record_split(SimArgs a)
{
    __shared__ float4 zs[2][RECORD_DAYS][2][64];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t k = (int64_t)blockIdx.x * 64 + lane;
    const bool live = k < a.n;
    const uint64_t i = a.first + (uint64_t)k;
    const int windows = (a.T + RECORD_DAYS - 1) / RECORD_DAYS;
    const float invP = 1.0f / (float)a.P, nc = noise_c(a.scale);
    RatesF r{};
    State s{};
    int32_t* out = a.traj + (int64_t)6 * (a.T + 1) * k;
    if (wv == 0 && live) {
        float thv[8];
        load_or_draw_theta(a, false, k, i, thv);
        const Theta th = theta_from(thv);
        r = rates_f32(th);
        s = init_state(th.ka, a.P, a.A0, a.R0, a.D0);
        store_state(out, s);
    }
    for (int w = 0; w <= windows; ++w) {
        if (wv > 0) {
            if (w < windows)
                for (int d = wv - 1; d < RECORD_DAYS; d += 3) {
                    const uint4 words = stream_words(a.key, i, a.series, ctr_word3((uint32_t)(w * RECORD_DAYS + d + 1), a.domain, 0));
                    Noise32 z;
                    normals_f32(words, nc, z);
                    zs[w & 1][d][0][lane] = make_float4(z.rr[0], z.rr[1], z.rr[2], z.tr[0]);
                    zs[w & 1][d][1][lane] = make_float4(z.tr[1], z.tr[2], z.tr[3], z.tr[4]);
                }
        } else if (w > 0 && live) {
            const int t0 = (w - 1) * RECORD_DAYS;
            const int days = min(RECORD_DAYS, a.T - t0);
            for (int d = 0; d < days; ++d) {
                const float4 p = zs[(w - 1) & 1][d][0][lane], q = zs[(w - 1) & 1][d][1][lane];
                Noise32 z;
                z.rr[0] = p.x; z.rr[1] = p.y; z.rr[2] = p.z; z.tr[0] = p.w;
                z.tr[1] = q.x; z.tr[2] = q.y; z.tr[3] = q.z; z.tr[4] = q.w;
                day_step_f32<NOISE>(s, r, invP, z);
                store_state(out + 6 * (t0 + d + 1), s);
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// prior sampling
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(SIM_BLOCK) void k_sample_prior(SimArgs a, float* theta)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= a.n) return;
    float th[8];
    prior_draw(a.key, a.first + (uint64_t)k, a.series, a.domain, a.lo, a.width, th);
    float4* p = reinterpret_cast<float4*>(theta + 8 * k);
    p[0] = make_float4(th[0], th[1], th[2], th[3]);
    p[1] = make_float4(th[4], th[5], th[6], th[7]);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
static abc_status fill_series(SimArgs& a, const abc_series* ser, const abc_model* m,
                              const abc_stream* st, uint64_t first, int64_t n)
{
    a.key = make_key(st->seed);
    a.domain = st->domain;
    a.series = st->series;
    a.first = first;
    a.n = n;
    a.P = (int32_t)ser->P;
    a.A0 = ser->A0;
    a.R0 = ser->R0;
    a.D0 = ser->D0;
    a.T = ser->T;
    a.obs = ser->obs;
    a.scale = m->noise_scale;
    return ABC_OK;
}

// float64 row kernels: one wavefront per workgroup, up to R rows side by side
// per wavefront, rows strided over the grid
constexpr int64_t ROW_WAVE_GRID = 2048;
static size_t row_wave_lds_bytes(int T, int R)
{
    return sizeof(Math64) + sizeof(double) * (3 * (size_t)T + 5 * ROW_PAIRS) + sizeof(int32_t) * 4 * ROW_PAIRS +
           (size_t)R * (sizeof(uint64_t) + sizeof(int64_t) + sizeof(float) * 8);
}

static inline unsigned grid_for(int64_t n) { return (unsigned)((n + SIM_BLOCK - 1) / SIM_BLOCK); }

static bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Launch shape of the float32 refill kernel for the calling thread: samples
// per lane, workgroup size and resident workgroups per CU. Until the thread
// sets one (and again after it sets all three to 0) each kernel chooses its
// own from the size of the launch.
struct LaunchConfig : LaunchShape {
    int refill_min = 8;
};
static thread_local LaunchConfig g_launch;

LaunchShape launch_shape() { return g_launch; }

// Resident 512-thread workgroups per CU for a launch of n samples over T days: more
// wavefronts hide more latency, but every wavefront ends on a few trajectories of
// its own, up to T days after its queue is empty, and early exits make its queue
// short. So what a wavefront has to itself (chunks of 64 samples, were there one
// workgroup per CU) is measured against T; raw distances exit late in a
// trajectory, which counts like seven times the samples; without exits every
// trajectory ends on the same day and one chunk each is enough. One / two / three /
// four workgroups per CU, us:
//   T =  49, exits: 1e6 samples 110 / 114 / 118 / 129, 3e6 237 / 220 / 226 / 230, 1e7 699 / 614 / 590 / 590
//   T =  95, exits: 1e6 175 / 181 / 211 / 237, 4e6 479 / 447 / 465 / 481, 2e7 2126 / 1859 / 1812 / 1802
//   T = 200, exits: 2e6 433 / 455 / 500 / 536, 4e6 719 / 706 / 737 / 779, 1e7 1596 / 1461 / 1459 / 1522
//   T = 400, exits: 4e6 997 / 1068 / 1133 / 1207, 1e7 2110 / 1996 / 2076 / 2160
//   T =  49, raw, exits: 3e5 93 / 84 / 85 / 84, 1e6 204 / 200 / 192 / 193
//   T =  49, no exits: 1e6 245 / 229 / 219 / 217
static int refill_blocks_per_cu(int64_t n, int T, bool exits, bool raw)
{
    DeviceInfo info;
    const int64_t num_cu = device_info(&info) == ABC_OK && info.num_cu > 0 ? info.num_cu : 256;
    const double share = (double)((n + 63) / 64) / (double)(num_cu * (512 / 64)) * (exits && raw ? 7.0 : 1.0);
    if (!exits) return share < 2.0 ? 1 : (share >= 4.0 ? 4 : (int)share);
    const double days = T > 50 ? T : 50;
    if (share >= 1.12 * days) return 4;
    if (share >= 0.56 * days) return 3;
    return share >= 14.0 && share >= 0.094 * T ? 2 : 1;
}

// Resident-grid size for the refill kernel: enough workgroups to fill every
// CU several times over, never more than there are 64-sample chunks.
static unsigned refill_grid(int64_t n, int block, int blocks_per_cu)
{
    DeviceInfo info;
    const int num_cu = device_info(&info) == ABC_OK && info.num_cu > 0 ? info.num_cu : 256;
    const int64_t waves_needed = (n + 63) / 64;
    const int64_t per_block = block / 64;
    int64_t g = (int64_t)num_cu * blocks_per_cu;
    const int64_t need = (waves_needed + per_block - 1) / per_block;
    if (g > need) g = need;
    return (unsigned)(g > 0 ? g : 1);
}

// observed series | future-days bound table | ring (which first holds the
// float64 b_s and the segment sums staged for the table)
static size_t refill_lds_bytes(int T, int block, int lb_ntb)
{
    const size_t ring = sizeof(Slot) * 64 * (size_t)(block / 64);
    const size_t stage =
        lb_ntb > 0 ? sizeof(double) * (2 * (size_t)T + (size_t)LB_MAX_SEG * 2 * LB_Q) : 0;
    return sizeof(float) * 4 * (size_t)T + sizeof(float) * 2 * LB_Q * (size_t)lb_ntb +
           (ring > stage ? ring : stage);
}

static size_t max_lds_per_block()
{
    DeviceInfo info;
    return device_info(&info) == ABC_OK && info.max_lds > 0 ? (size_t)info.max_lds : 65536;
}

template <int NOISE, int DIST, bool KAHAN, int SPL, bool BOUND>
static void launch_f32_bound(const SimArgs& a, bool prior, hipStream_t s)
{
    const int block = g_launch.block;
    const size_t lds = refill_lds_bytes(a.T, block, a.lb_ntb);
    const int bpc = g_launch.chosen ? g_launch.blocks_per_cu : refill_blocks_per_cu(a.n, a.T, !isinf(a.exit_f32), DIST == 1);
    const dim3 g(refill_grid(a.n, block, bpc)), b(block);
    if (prior)
        hipLaunchKernelGGL((k_simulate_f32<NOISE, DIST, KAHAN, true, SPL, BOUND>), g, b, lds, s, a);
    else
        hipLaunchKernelGGL((k_simulate_f32<NOISE, DIST, KAHAN, false, SPL, BOUND>), g, b, lds, s, a);
}

template <int NOISE, int DIST, bool KAHAN, int SPL>
static void launch_f32_spl(const SimArgs& a, bool prior, hipStream_t s)
{
    if constexpr (DIST == 0) {
        if (a.lb_ntb > 0) {
            launch_f32_bound<NOISE, DIST, KAHAN, SPL, true>(a, prior, s);
            return;
        }
    }
    launch_f32_bound<NOISE, DIST, KAHAN, SPL, false>(a, prior, s);
}

template <int NOISE, int DIST, bool KAHAN>
static void launch_f32(const SimArgs& a, bool prior, hipStream_t s)
{
    // several samples per lane only for the paper's model and distance
    if constexpr (NOISE == 0 && DIST == 0) {
        switch (g_launch.spl) {
        case 2: launch_f32_spl<NOISE, DIST, KAHAN, 2>(a, prior, s); return;
        case 4: launch_f32_spl<NOISE, DIST, KAHAN, 4>(a, prior, s); return;
        case 8: launch_f32_spl<NOISE, DIST, KAHAN, 8>(a, prior, s); return;
        default: break;
        }
    }
    launch_f32_spl<NOISE, DIST, KAHAN, 1>(a, prior, s);
}

// tables, observed series, the future-days bound and the space that builds it; the
// row arrays of the wavefronts come after them (60 KB together for the longest series
// without the bound)
constexpr size_t F64_WALK_LDS = (F64_BLOCK / 64) * F64_WALK_BYTES;
static size_t f64_lds_bytes(int T, int lb_ntb)
{
    return sizeof(Math64) + sizeof(double) * 3 * (size_t)T +
           (lb_ntb > 0 ? sizeof(double) * (2 * (size_t)T + (size_t)LB_MAX_SEG * 2 * LB_Q) +
                             sizeof(float) * 2 * LB_Q * (size_t)lb_ntb
                       : 0);
}

template <int NOISE, int DIST>
static void launch_f64(const SimArgs& args, bool prior, hipStream_t s)
{
    SimArgs a = args;
    a.walk_at = (int32_t)f64_lds_bytes(a.T, a.lb_ntb);
    const size_t lds = (size_t)a.walk_at + F64_WALK_LDS;
    const dim3 g(refill_grid(a.n, F64_BLOCK, F64_BLOCKS_PER_CU)), b(F64_BLOCK);
    if (prior)
        hipLaunchKernelGGL((k_simulate_f64<NOISE, DIST, true>), g, b, lds, s, a);
    else
        hipLaunchKernelGGL((k_simulate_f64<NOISE, DIST, false>), g, b, lds, s, a);
}

}  // namespace abc

using namespace abc;

extern "C" abc_status abc_sample_prior(const abc_prior* prior, const abc_stream* st,
                                       uint64_t first, int64_t n, float* theta, void* stream)
{
    SimArgs a{};
    abc_status rc = prior_lo_width(prior, a.lo, a.width);
    if (rc) return rc;
    if ((rc = check_stream_sel(st))) return rc;
    ABC_REQUIRE(n >= 0, "n = %lld < 0", (long long)n);
    if (n == 0) return ABC_OK;
    ABC_REQUIRE(theta != nullptr && aligned16(theta), "theta must be a 16-byte aligned device pointer");
    a.key = make_key(st->seed);
    a.domain = st->domain;
    a.series = st->series;
    a.first = first;
    a.n = n;
    hipLaunchKernelGGL(k_sample_prior, dim3(grid_for(n)), dim3(SIM_BLOCK), 0, as_stream(stream),
                       a, theta);
    return check_launch("k_sample_prior");
}

extern "C" abc_status abc_simulate_distance(const abc_series* ser, const abc_model* model,
                                            const abc_stream* st, const float* theta,
                                            const abc_prior* prior, uint64_t first, int64_t n,
                                            float eps_exit, float* dist, double* dist64,
                                            unsigned long long* days, void* stream)
{
    abc_status rc;
    if ((rc = check_series(ser, true))) return rc;
    if ((rc = check_model(model))) return rc;
    if ((rc = check_stream_sel(st))) return rc;
    ABC_REQUIRE(n >= 0 && n <= ((int64_t)1 << 36), "n = %lld outside [0, 2^36]", (long long)n);
    ABC_REQUIRE(!(eps_exit < 0.0f) && !isnan(eps_exit), "eps_exit must be >= 0 (or +INF)");
    if (n == 0) return ABC_OK;
    ABC_REQUIRE(dist != nullptr, "dist is NULL");
    SimArgs a{};
    const bool use_prior = theta == nullptr;
    if (use_prior) {
        if ((rc = prior_lo_width(prior, a.lo, a.width))) return rc;
        for (int k = 0; k < 8; ++k)
            ABC_REQUIRE(prior->lo[k] >= 0.0f, "model rates must be non-negative: prior lo[%d] < 0", k);
    } else {
        ABC_REQUIRE(aligned16(theta), "theta must be 16-byte aligned");
        if (model->flags & ABC_SUPPORT) {
            if ((rc = prior_lo_width(prior, a.lo, a.width))) return rc;
            for (int k = 0; k < 8; ++k) a.hi[k] = prior->hi[k];
            a.box = 1;
        }
    }
    fill_series(a, ser, model, st, first, n);
    a.theta = theta;
    a.dist = dist;
    a.dist64 = dist64;
    a.days = days;
    a.refill_min = g_launch.refill_min;
    // Early-exit bounds with a relative margin that keeps every exited sample
    // strictly above eps_exit after the final square root and rounding.
    const double e2 = (double)eps_exit * (double)eps_exit;
    // the float32 log1p distance accumulates in log2 units: bound / ln(2)^2
    const double unit = (model->flags & ABC_DIST_RAW) ? 1.0 : 2.08136898100560809980;
    a.exit_f32 = isinf(eps_exit) ? INFINITY : (float)(e2 * unit * (1.0 + 0x1p-18));
    a.exit_f64 = isinf(eps_exit) ? (double)INFINITY : e2 * (1.0 + 1e-12);

    const hipStream_t s = as_stream(stream);
    const int noise = (model->flags & ABC_NOISE_LITERAL) ? 1 : 0;
    const int distm = (model->flags & ABC_DIST_RAW) ? 1 : 0;
    // future-days bound for the log1p distance when there is an exit bound;
    // time blocks of 2^sh days keep the table within LB_MAX_BLOCKS rows
    if (distm == 0 && !isinf(eps_exit) && !(model->flags & ABC_NO_BOUND)) {
        int sh = 0;
        while ((a.T >> sh) + 1 > LB_MAX_BLOCKS) ++sh;
        a.lb_sh = sh;
        a.lb_ntb = (a.T >> sh) + 1;
        const size_t need = (model->flags & ABC_FP64) ? f64_lds_bytes(a.T, a.lb_ntb) + F64_WALK_LDS
                                                      : refill_lds_bytes(a.T, g_launch.block, a.lb_ntb);
        if (need > max_lds_per_block()) a.lb_ntb = 0;
    }
    if (model->flags & ABC_FP64) {
        if (noise == 0 && distm == 0) launch_f64<0, 0>(a, use_prior, s);
        else if (noise == 0 && distm == 1) launch_f64<0, 1>(a, use_prior, s);
        else if (noise == 1 && distm == 0) launch_f64<1, 0>(a, use_prior, s);
        else launch_f64<1, 1>(a, use_prior, s);
        return check_launch("k_simulate_f64");
    }
    const size_t lds = refill_lds_bytes(a.T, g_launch.block, a.lb_ntb);
    if (lds > max_lds_per_block())
        return set_error(ABC_EUNSUPPORTED, "T = %d with workgroup size %d needs %zu B of LDS (> %zu)",
                         a.T, g_launch.block, lds, max_lds_per_block());
    const bool kahan = (model->flags & ABC_KAHAN) != 0;
    if (kahan) {
        if (noise == 0 && distm == 0) launch_f32<0, 0, true>(a, use_prior, s);
        else if (noise == 0 && distm == 1) launch_f32<0, 1, true>(a, use_prior, s);
        else if (noise == 1 && distm == 0) launch_f32<1, 0, true>(a, use_prior, s);
        else launch_f32<1, 1, true>(a, use_prior, s);
    } else {
        if (noise == 0 && distm == 0) launch_f32<0, 0, false>(a, use_prior, s);
        else if (noise == 0 && distm == 1) launch_f32<0, 1, false>(a, use_prior, s);
        else if (noise == 1 && distm == 0) launch_f32<1, 0, false>(a, use_prior, s);
        else launch_f32<1, 1, false>(a, use_prior, s);
    }
    return check_launch("k_simulate_f32");
}

extern "C" abc_status abc_simulate_record(const abc_series* ser, const abc_model* model,
                                          const abc_stream* st, const float* theta,
                                          uint64_t first, int64_t n, int32_t* traj, void* stream)
{
    abc_status rc;
    if ((rc = check_series(ser, false))) return rc;
    if ((rc = check_model(model))) return rc;
    if ((rc = check_stream_sel(st))) return rc;
    ABC_REQUIRE(n >= 0, "n = %lld < 0", (long long)n);
    if (n == 0) return ABC_OK;
    ABC_REQUIRE(theta != nullptr && aligned16(theta), "theta must be a 16-byte aligned device pointer");
    ABC_REQUIRE(traj != nullptr, "traj is NULL");
    SimArgs a{};
    fill_series(a, ser, model, st, first, n);
    a.theta = theta;
    a.traj = traj;
    const hipStream_t s = as_stream(stream);
    const bool f64 = (model->flags & ABC_FP64) != 0;
    const int noise = (model->flags & ABC_NOISE_LITERAL) ? 1 : 0;
    const dim3 g(grid_for(n)), b(SIM_BLOCK), gs((unsigned)((n + 63) / 64));
    DeviceInfo info;
    if ((rc = device_info(&info))) return rc;
    // up to two workgroups per CU the split is faster (120 days of 16384 rows 28
    // us against 43, of 32768 46 against 56), from four on it is not (65536: 83, 83)
    if (!f64 && n <= (int64_t)64 * info.num_cu * 2) {
        if (noise) hipLaunchKernelGGL((k_record_split<1>), gs, b, 0, s, a);
        else hipLaunchKernelGGL((k_record_split<0>), gs, b, 0, s, a);
    } else if (f64) {
        if (noise) hipLaunchKernelGGL((k_record<1, true>), g, b, 0, s, a);
        else hipLaunchKernelGGL((k_record<0, true>), g, b, 0, s, a);
    } else {
        if (noise) hipLaunchKernelGGL((k_record<1, false>), g, b, 0, s, a);
        else hipLaunchKernelGGL((k_record<0, false>), g, b, 0, s, a);
    }
    return check_launch("k_record");
}

extern "C" abc_status abc_set_launch_config(int32_t spl, int32_t block, int32_t blocks_per_cu)
{
    const bool chosen = spl != 0 || block != 0 || blocks_per_cu != 0;
    if (spl == 0) spl = 1;
    if (block == 0) block = 512 / spl < 64 ? 64 : 512 / spl;
    if (blocks_per_cu == 0) blocks_per_cu = 2;
    ABC_REQUIRE(spl == 1 || spl == 2 || spl == 4 || spl == 8, "spl must be 1, 2, 4 or 8");
    ABC_REQUIRE(block >= 64 && block <= 1024 / spl && block % 64 == 0,
                "block must be a multiple of 64 in [64, 1024/spl]");
    ABC_REQUIRE(blocks_per_cu >= 1 && blocks_per_cu <= 64, "blocks_per_cu must be in [1, 64]");
    g_launch.spl = spl;
    g_launch.block = block;
    g_launch.blocks_per_cu = blocks_per_cu;
    g_launch.chosen = chosen;
    return ABC_OK;
}

extern "C" abc_status abc_get_launch_config(int32_t* spl, int32_t* block, int32_t* blocks_per_cu)
{
    ABC_REQUIRE(spl && block && blocks_per_cu, "NULL output pointer");
    // what sets the same state again: zeros while the thread has chosen no shape
    *spl = g_launch.chosen ? g_launch.spl : 0;
    *block = g_launch.chosen ? g_launch.block : 0;
    *blocks_per_cu = g_launch.chosen ? g_launch.blocks_per_cu : 0;
    return ABC_OK;
}

namespace abc {
abc_status recheck_band(const abc_series* ser, const abc_model* model, const abc_stream* st,
                        float eps, float band_w, int64_t capacity, int64_t* idx, float* theta,
                        float* dist, float* weight, int64_t* count, int32_t* rechecked,
                        void* stream, int64_t grid_max, int32_t scan_min, double* dist64, bool all_rows)
{
    abc_status rc;
    if ((rc = check_series(ser, true))) return rc;
    if ((rc = check_model(model))) return rc;
    if ((rc = check_stream_sel(st))) return rc;
    ABC_REQUIRE(!isnan(eps) && eps >= 0.0f, "eps must be >= 0 (or +INF)");
    ABC_REQUIRE(isfinite(band_w) && band_w >= 0.0f && band_w < 1.0f, "band_w must be in [0, 1)");
    ABC_REQUIRE(capacity >= 0, "capacity < 0");
    ABC_REQUIRE(count != nullptr, "count is NULL");
    if (capacity == 0) return ABC_OK;
    ABC_REQUIRE(idx && theta && dist, "idx/theta/dist NULL");
    const size_t lds = row_wave_lds_bytes(ser->T, ROWS_PER_WAVE_MAX);
    ABC_REQUIRE(lds <= max_lds_per_block(), "T too long for the float64 recheck");
    const hipStream_t s = as_stream(stream);
    RecheckArgs r{};
    fill_series(r.sim, ser, model, st, 0, 0);
    r.eps = eps;
    r.band_lo = (float)((double)eps * (1.0 - (double)band_w));
    r.band_hi = (float)((double)eps * (1.0 + (double)band_w));
    r.capacity = capacity;
    r.idx = idx;
    r.theta = theta;
    r.dist = dist;
    r.weight = weight;
    r.count = count;
    r.rechecked = rechecked;
    r.scan_min = scan_min < 1 ? 1 : scan_min;
    r.all_rows = all_rows ? 1 : 0;
    r.dist64 = dist64;
    void* scratch = nullptr;
    if ((rc = stream_scratch(s, (size_t)capacity, &scratch))) return rc;
    r.keep = reinterpret_cast<uint8_t*>(scratch);
    const int noise = (model->flags & ABC_NOISE_LITERAL) ? 1 : 0;
    const int distm = (model->flags & ABC_DIST_RAW) ? 1 : 0;
    if (rechecked) hipLaunchKernelGGL(k_zero_i32, dim3(1), dim3(64), 0, s, rechecked);
    const dim3 g((unsigned)(capacity < grid_max ? capacity : grid_max)), b(64);
    if (noise == 0 && distm == 0) hipLaunchKernelGGL((k_recheck_flags<0, 0>), g, b, lds, s, r);
    else if (noise == 0) hipLaunchKernelGGL((k_recheck_flags<0, 1>), g, b, lds, s, r);
    else if (distm == 0) hipLaunchKernelGGL((k_recheck_flags<1, 0>), g, b, lds, s, r);
    else hipLaunchKernelGGL((k_recheck_flags<1, 1>), g, b, lds, s, r);
    rc = check_launch("k_recheck_flags");
    if (rc == ABC_OK) {
        hipLaunchKernelGGL(k_recheck_compact, dim3(1), dim3(COMPACT_BLOCK), 0, s, r);
    }
    if (rc == ABC_OK) rc = check_launch("k_recheck_compact");
    return rc;
}
}  // namespace abc

extern "C" abc_status abc_recheck_band(const abc_series* ser, const abc_model* model,
                                       const abc_stream* st, float eps, float band_w,
                                       int64_t capacity, int64_t* idx, float* theta, float* dist,
                                       float* weight, int64_t* count, int32_t* rechecked,
                                       void* stream)
{
    return recheck_band(ser, model, st, eps, band_w, capacity, idx, theta, dist, weight, count,
                        rechecked, stream, ROW_WAVE_GRID, ROW_SCAN_BESIDE, nullptr, false);
}

extern "C" abc_status abc_simulate_rows_f64(const abc_series* ser, const abc_model* model,
                                            const abc_stream* st, const int64_t* idx,
                                            const float* theta, int64_t n, double* dist64,
                                            void* stream)
{
    abc_status rc;
    if ((rc = check_series(ser, true))) return rc;
    if ((rc = check_model(model))) return rc;
    if ((rc = check_stream_sel(st))) return rc;
    ABC_REQUIRE(n >= 0, "n < 0");
    if (n == 0) return ABC_OK;
    ABC_REQUIRE(idx && theta && dist64, "idx/theta/dist64 NULL");
    // one row per wavefront while each has a CU to itself, then at least four:
    // 1024 wavefronts of one row walk a day in 0.78 us, 256 of four in 0.47
    int64_t want = (n + ROW_WAVE_TARGET - 1) / ROW_WAVE_TARGET;
    if (n > 256 && want < 4) want = 4;
    const int rows = (int)(want < ROWS_PER_WAVE_MAX ? want : ROWS_PER_WAVE_MAX);
    const size_t lds = row_wave_lds_bytes(ser->T, rows);
    ABC_REQUIRE(lds <= max_lds_per_block(), "T too long for the float64 path");
    RowsArgs r{};
    fill_series(r.sim, ser, model, st, 0, n);
    r.sim.theta = theta;
    r.idx = idx;
    r.dist64 = dist64;
    r.rows_per_wave = rows;
    const hipStream_t s = as_stream(stream);
    const int noise = (model->flags & ABC_NOISE_LITERAL) ? 1 : 0;
    const int distm = (model->flags & ABC_DIST_RAW) ? 1 : 0;
    const int64_t waves = (n + rows - 1) / rows;
    const dim3 g((unsigned)(waves < ROW_WAVE_GRID ? waves : ROW_WAVE_GRID)), b(64);
    if (noise == 0 && distm == 0) hipLaunchKernelGGL((k_rows_f64<0, 0>), g, b, lds, s, r);
    else if (noise == 0) hipLaunchKernelGGL((k_rows_f64<0, 1>), g, b, lds, s, r);
    else if (distm == 0) hipLaunchKernelGGL((k_rows_f64<1, 0>), g, b, lds, s, r);
    else hipLaunchKernelGGL((k_rows_f64<1, 1>), g, b, lds, s, r);
    return check_launch("k_rows_f64");
}

extern "C" abc_status abc_set_refill_min(int32_t lanes)
{
    if (lanes == 0) lanes = 8;
    ABC_REQUIRE(lanes >= 1 && lanes <= 64, "lanes must be in [1, 64]");
    g_launch.refill_min = lanes;
    return ABC_OK;
}

extern "C" int32_t abc_get_refill_min(void) { return g_launch.refill_min; }
