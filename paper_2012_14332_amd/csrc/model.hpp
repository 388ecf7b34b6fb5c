// Device-side model of Sec. 2.1 (eqs. 3-5) and the distance of Sec. 2.2.
//
// One lane owns one trajectory: the six compartments live in VGPRs as int32
// (exact for populations below 2^31), the hazards, Gaussian draws and
// distance run in float32 (or float64 for the precision study and the
// recheck of borderline samples). Nothing of the trajectory is written to
// memory; the distance is accumulated day by day.
//
// Day t >= 1 of sample i:
//   M  = A + R + D,  g = alpha0 + alpha / (1 + M^n)                   eq. (4)
//   h  = (g S I / P, gamma I, beta A, delta A, beta eta I)            eq. (5)
//   x_k = h_k + s sd(h_k) z_k with sd = sqrt(h) (or h^(1/4) literally),
//   n_k = floor(x_k) clamped to [0, what the source still holds]: S for n1,
//   I for n2, A for n3, A - n3 for n4, I - n2 for n5 (h order), then
//   S -= n1; I += n1 - n2 - n5; A += n2 - n3 - n4; R += n3; D += n4; Ru += n5.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "math64.hpp"
#include "philox.hpp"

namespace abc {

struct State {
    int32_t S, I, A, R, D, Ru;
};

// Per-sample theta (float32 values as drawn or supplied).
struct Theta {
    float a0, al, n, be, ga, de, et, ka;
};

__device__ __forceinline__ Theta theta_from(const float t[8])
{
    return Theta{t[0], t[1], t[2], t[3], t[4], t[5], t[6], t[7]};
}

// Prior draw (eq. 2): 8 words from blocks 0 and 1 of day 0.
__device__ __forceinline__ void prior_draw(Key key, uint64_t i, uint32_t series, uint32_t domain,
                                           const float* lo, const float* width, float th[8])
{
    const uint4 a = stream_words(key, i, series, ctr_word3(0, domain, 0));
    const uint4 b = stream_words(key, i, series, ctr_word3(0, domain, 1));
    const uint32_t w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const float u = (float)(w[k] >> 8) * 0x1p-24f;  // exact
        th[k] = fmaf(width[k], u, lo[k]);
    }
}

// Day-0 state: Ru = 0, I0 = floor(kappa A0) (computed exactly in double),
// S = P - (A0 + R0 + D0 + I0); I0 is limited so that S >= 0.
__device__ __forceinline__ State init_state(float kappa, int32_t P, int32_t A0, int32_t R0,
                                            int32_t D0)
{
    State s;
    s.A = A0;
    s.R = R0;
    s.D = D0;
    s.Ru = 0;
    const double i0 = floor((double)kappa * (double)A0);
    const int32_t room = P - (A0 + R0 + D0);
    s.I = i0 >= (double)room ? room : (int32_t)i0;
    s.S = room - s.I;
    return s;
}

// The six 21-bit uniforms of one day: u = (f + 1/2) 2^-21, exact in float.
__device__ __forceinline__ void day_fields(uint4 w, uint32_t f[6])
{
    f[0] = w.x >> 11;
    f[1] = w.y >> 11;
    f[2] = w.z >> 11;
    f[3] = w.w >> 11;
    f[4] = ((w.x & 0x7FFu) << 10) | (w.y & 0x3FFu);
    f[5] = ((w.z & 0x7FFu) << 10) | (w.w & 0x3FFu);
}

// ---------------------------------------------------------------------------
// float32 path: hardware transcendentals (v_log_f32 = log2, v_exp_f32 = 2^x,
// v_sqrt_f32, v_rcp_f32, v_sin/v_cos_f32 which take revolutions).
// ---------------------------------------------------------------------------

// Final float32 distance from the squared-sum accumulator: one hardware
// square root (about 1 ulp) times the unit scale (ln 2 for the log2-unit
// log1p distance, 1 for raw counts).
__device__ __forceinline__ float finish_distance_f32(float acc, float scale)
{
    return __builtin_amdgcn_sqrtf(acc) * scale;
}

// The five noise draws of one day in Box-Muller form, kept apart: the squared
// radii scaled by the noise scale s, rr_j = -2 s^2 ln u_{2j} = c log2 u_{2j}
// with c = -2 ln(2) s^2, and the angles' cosines and sines, tr_k, so that
// s z_k = sqrt(rr_j) tr_k. A draw then takes its standard deviation and its
// radius under one square root: sd(h) s z = sqrt(h rr_j) tr_k.
struct Noise32 {
    float rr[3];
    float tr[5];
};

// Uniform (f + 1/2) 2^-21 of the 21-bit field f in the upper bits of x (its
// lower 11 bits are dropped): one funnel shift puts f under the exponent of
// 2^23, and the fma takes the 2^23 away again (exact). A shift, a conversion
// and an fma would be one instruction more.
__device__ __forceinline__ float field_uniform(uint32_t x)
{
    return fmaf(__uint_as_float(__builtin_amdgcn_alignbit(0x258u, x, 11)), 0x1p-21f, 0x1p-22f - 4.0f);
}

__device__ __forceinline__ void normals_f32(uint4 w, float c, Noise32& z)
{
    // the fifth and sixth field: 11 low bits of one word above 10 of the next
    const uint32_t x4 = __builtin_amdgcn_alignbit(w.x, w.y << 22, 11), x5 = __builtin_amdgcn_alignbit(w.z, w.w << 22, 11);
    const float u[6] = {field_uniform(w.x), field_uniform(w.y), field_uniform(w.z),
                        field_uniform(w.w), field_uniform(x4), field_uniform(x5)};
    z.rr[0] = c * __builtin_amdgcn_logf(u[0]);
    z.rr[1] = c * __builtin_amdgcn_logf(u[2]);
    z.rr[2] = c * __builtin_amdgcn_logf(u[4]);
    z.tr[0] = __builtin_amdgcn_cosf(u[1]);  // cos(2 pi u1)
    z.tr[1] = __builtin_amdgcn_sinf(u[1]);
    z.tr[2] = __builtin_amdgcn_cosf(u[3]);
    z.tr[3] = __builtin_amdgcn_sinf(u[3]);
    z.tr[4] = __builtin_amdgcn_cosf(u[5]);
}

__device__ __forceinline__ float noise_c(float scale)
{
    return -1.38629436111989061883f * scale * scale;
}

// Integer part of x limited to uint32 (below 0 or NaN: 0), as the conversion
// instruction gives it; in C++ the cast of a value out of range has no result.
__device__ __forceinline__ uint32_t cvt_u32_sat(float x)
{
    uint32_t r;
    asm("v_cvt_u32_f32_e32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}

// floor(h + sd(h) s z) limited to [0, avail], with s z = sqrt(rr) tr: the
// standard deviation sqrt(h) (h^(1/4) read literally) and the radius share one
// square root. The conversion to unsigned truncates, which is the floor for
// x >= 0, takes negative x to 0 and x above 2^32 to its largest value, which
// avail then limits: no clamp in float is needed. Rates are non-negative, so
// h >= 0 and the root is finite.
template <int NOISE>
__device__ __forceinline__ int32_t draw_f32(float h, float rr, float tr, int32_t avail)
{
    const float v = NOISE == 1 ? __builtin_amdgcn_sqrtf(h) * rr : h * rr;
    const float x = fmaf(__builtin_amdgcn_sqrtf(v), tr, h);
    return (int32_t)min(cvt_u32_sat(x), (uint32_t)avail);
}

struct RatesF {
    float a0, al, n, be, ga, de, bh;  // bh = beta * eta
};

__device__ __forceinline__ RatesF rates_f32(const Theta& t)
{
    return RatesF{t.a0, t.al, t.n, t.be, t.ga, t.de, t.be * t.et};
}

// The five transitions of a day from the morning's counts (M = A + R + D).
struct Moves {
    int32_t n1, n2, n3, n4, n5;
};

template <int NOISE>
__device__ __forceinline__ Moves moves_f32(int32_t S, int32_t I, int32_t A, int32_t Mi, const RatesF& r,
                                           float invP, const Noise32& z)
{
    const float M = (float)Mi;
    const float pw = __builtin_amdgcn_exp2f(r.n * __builtin_amdgcn_logf(M));
    const float g = fmaf(r.al, __builtin_amdgcn_rcpf(1.0f + pw), r.a0);
    const float If = (float)I;
    const float Af = (float)A;
    const float h1 = (g * invP) * (float)S * If;
    const float h2 = r.ga * If;
    const float h3 = r.be * Af;
    const float h4 = r.de * Af;
    const float h5 = r.bh * If;
    Moves m;
    m.n1 = draw_f32<NOISE>(h1, z.rr[0], z.tr[0], S);
    m.n2 = draw_f32<NOISE>(h2, z.rr[0], z.tr[1], I);
    m.n3 = draw_f32<NOISE>(h3, z.rr[1], z.tr[2], A);
    m.n4 = draw_f32<NOISE>(h4, z.rr[1], z.tr[3], A - m.n3);
    m.n5 = draw_f32<NOISE>(h5, z.rr[2], z.tr[4], I - m.n2);
    return m;
}

template <int NOISE>
__device__ __forceinline__ void day_step_f32(State& s, const RatesF& r, float invP,
                                             const Noise32& z)
{
    const Moves m = moves_f32<NOISE>(s.S, s.I, s.A, s.A + s.R + s.D, r, invP, z);
    s.S -= m.n1;
    s.I += m.n1 - m.n2 - m.n5;
    s.A += m.n2 - m.n3 - m.n4;
    s.R += m.n3;
    s.D += m.n4;
    s.Ru += m.n5;
}

// ---------------------------------------------------------------------------
// One day of the float32 simulate+distance kernels. They are bound by VALU
// issue, so the day keeps what it needs in the form it needs it: R and D as
// R + 1 and D + 1 (the arguments of their logarithms), M = A + R + D as a
// count of its own (recoveries alone raise it), the counter word of the day
// and the address of its row counted up instead of formed from the day. The
// observed days are rows of four words: log2(1 + O) of A, R and D (or, for the
// raw distance, O of A and O + 1 of R and D), and the LDS address of the day's
// row in the future-days bound table, so that a day reads one row and its
// table entries with one address each.
// ---------------------------------------------------------------------------
struct StateD {
    int32_t S, I, A, M, R1, D1;
};

__device__ __forceinline__ StateD state_d(int32_t room, int32_t A0, int32_t R0, int32_t D0, int32_t I0)
{
    return StateD{room - I0, I0, A0, A0 + R0 + D0, R0 + 1, D0 + 1};
}

// the observed words of one day (the fourth: LDS address of the bound row)
template <int DIST>
__device__ __forceinline__ float4 obs_row(int32_t A, int32_t R, int32_t D, uint32_t bound_row)
{
    float4 o;
    if (DIST == 0) {
        o.x = (float)(log1p((double)A) * 1.44269504088896340736);
        o.y = (float)(log1p((double)R) * 1.44269504088896340736);
        o.z = (float)(log1p((double)D) * 1.44269504088896340736);
    } else {
        o.x = __int_as_float(A);
        o.y = __uint_as_float((uint32_t)R + 1u);
        o.z = __uint_as_float((uint32_t)D + 1u);
    }
    o.w = __uint_as_float(bound_row);
    return o;
}

// Simulates the day of counter word w, adds its squared distance to acc (comp:
// the Kahan compensation); lr, ld return log2(1 + R), log2(1 + D) for the
// log1p distance.
template <int NOISE, int DIST, bool KAHAN>
__device__ __forceinline__ void day_distance_f32(StateD& s, const RatesF& r, uint4 words, float invP, float nc,
                                                 const float4& ob, float& acc, float& comp, float& lr, float& ld)
{
    Noise32 z;
    normals_f32(words, nc, z);
    const Moves m = moves_f32<NOISE>(s.S, s.I, s.A, s.M, r, invP, z);
    s.S -= m.n1;
    s.I = (s.I - m.n2) - m.n5 + m.n1;
    s.A = (s.A - m.n3) - m.n4 + m.n2;
    s.M += m.n2;
    s.R1 += m.n3;
    s.D1 += m.n4;
    float d[3];
    if (DIST == 0) {
        lr = __builtin_amdgcn_logf((float)s.R1);
        ld = __builtin_amdgcn_logf((float)s.D1);
        d[0] = __builtin_amdgcn_logf((float)(s.A + 1)) - ob.x;
        d[1] = lr - ob.y;
        d[2] = ld - ob.z;
    } else {
        d[0] = (float)(int32_t)((uint32_t)s.A - __float_as_uint(ob.x));
        d[1] = (float)(int32_t)((uint32_t)s.R1 - __float_as_uint(ob.y));
        d[2] = (float)(int32_t)((uint32_t)s.D1 - __float_as_uint(ob.z));
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        if (KAHAN) {
            const float y = fmaf(d[c], d[c], -comp);
            const float t = acc + y;
            comp = (t - acc) - y;
            acc = t;
        } else {
            acc = fmaf(d[c], d[c], acc);
        }
    }
}

// ---------------------------------------------------------------------------
// float64 path: the same definitions evaluated in the order the oracle writes
// them (no contraction), with the functions of math64.hpp.
// ---------------------------------------------------------------------------

__device__ __forceinline__ void normals_f64(uint4 w, const Math64& tab, double z[5])
{
#pragma clang fp contract(off)
    uint32_t f[6];
    day_fields(w, f);
    double u[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) u[k] = ((double)f[k] + 0.5) * 0x1p-21;
    const double two_pi = 2.0 * 3.14159265358979323846;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const double r = sqrt_mid(-2.0 * log_mid(u[2 * j], tab));
        double sn, cs;
        sincos_turn(two_pi * u[2 * j + 1], sn, cs);
        z[2 * j] = r * cs;
        if (j < 2) z[2 * j + 1] = r * sn;
    }
}

// Quotient and power for parameters outside math64.hpp's ranges (n above
// POW_N_MAX, or a parameter that is not finite): the library's own, out of line.
__device__ __attribute__((noinline)) double force_general(double M, double n, double a0, double al)
{
#pragma clang fp contract(off)
    return a0 + al / (1.0 + pow(M, n));
}

__device__ __attribute__((noinline)) double div_general(double x, double y) { return x / y; }

__device__ __forceinline__ bool theta_mid(const float t[8])
{
    bool ok = t[2] >= 0.0f && t[2] <= POW_N_MAX;
#pragma unroll
    for (int k = 0; k < 8; ++k) ok = ok && fabsf(t[k]) < INFINITY;
    return ok;
}

// g of eq. (4) from p = pow_arg(M, n), M = A + R + D >= A0 >= 1
__device__ __forceinline__ double force_f64(PowArg p, double a0, double al, const Math64& tab)
{
#pragma clang fp contract(off)
    return a0 + div_mid(al, 1.0 + pow_exp(p, tab));
}

template <int NOISE>
__device__ __forceinline__ double sd_f64(double h, double scale)
{
    return NOISE == 0 ? scale * sqrt_mid(h) : scale * sqrt_mid(sqrt_mid(h));
}

// Integer part of x, limited to int32 (NaN: 0), as the conversion instruction
// gives it; in C++ the cast of a value out of range has no result.
__device__ __forceinline__ int32_t cvt_i32_sat(double x)
{
    int32_t r;
    asm("v_cvt_i32_f64_e32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}

// floor(h + sd z) limited to [0, 2^31 - 1] (NaN: 0); the caller limits it to
// what the source holds
template <int NOISE>
__device__ __forceinline__ int32_t draw_f64(double h, double z, double scale)
{
#pragma clang fp contract(off)
    const double x = h + sd_f64<NOISE>(h, scale) * z;
    return max(cvt_i32_sat(x), 0);  // truncation is the floor of x >= 0
}

// What the source gives of a draw d >= 0 if it may hold less than nothing, after a
// negative kappa: then any draw but 0 takes that.
__device__ __forceinline__ int32_t taken(int32_t d, int32_t avail) { return d > 0 ? min(d, avail) : 0; }

template <bool MID>
__device__ __forceinline__ int32_t give(int32_t d, int32_t avail) { return MID ? min(d, avail) : taken(d, avail); }

// NEG: some lane's kappa may be negative (mid is false for those). Their draws are taken
// again behind a branch that a wavefront without them skips: a condition in each of the
// five cost the kernel with given parameters 5 %, the branch costs 1 to 2 (200000 samples
// of 100 days: 300 -> 303 us where 1 in 1000 reaches the last day, 608 -> 621 where half do).
template <int NOISE, bool NEG = false>
__device__ __forceinline__ void day_step_f64(State& s, const Theta& t, bool mid, double P, double rP,
                                             double scale, const double z[5], const Math64& tab)
{
#pragma clang fp contract(off)
    const double M = (double)(s.A + s.R + s.D), n = (double)t.n, a0 = (double)t.a0, al = (double)t.al;
    const double g = mid ? force_f64(pow_arg(M, n, tab), a0, al, tab) : force_general(M, n, a0, al);
    const double If = (double)s.I, Af = (double)s.A;
    const double h0 = g * (double)s.S * If;
    const double h1 = mid ? div_by(h0, P, rP) : div_general(h0, P);
    const int32_t d1 = draw_f64<NOISE>(h1, z[0], scale), d2 = draw_f64<NOISE>((double)t.ga * If, z[1], scale),
                  d3 = draw_f64<NOISE>((double)t.be * Af, z[2], scale), d4 = draw_f64<NOISE>((double)t.de * Af, z[3], scale),
                  d5 = draw_f64<NOISE>((double)t.be * (double)t.et * If, z[4], scale);
    int32_t n1 = min(d1, s.S), n2 = min(d2, s.I), n3 = min(d3, s.A), n4 = min(d4, s.A - n3), n5 = min(d5, s.I - n2);
    if (NEG && !mid) {
        n1 = taken(d1, s.S);
        n2 = taken(d2, s.I);
        n3 = taken(d3, s.A);
        n4 = taken(d4, s.A - n3);
        n5 = taken(d5, s.I - n2);
    }
    s.S -= n1;
    s.I += n1 - n2 - n5;
    s.A += n2 - n3 - n4;
    s.R += n3;
    s.D += n4;
    s.Ru += n5;
}

// ln(1 + X) of a count (X + 1 is exact in float64)
__device__ __forceinline__ double log1p_count_f64(int32_t X, const Math64& tab)
{
    return log_mid((double)X + 1.0, tab);
}

// Observed series for the float64 distance: log1p(O), or O for the raw
// distance. Observed counts below 0 take the library's log1p (NaN or -inf).
template <int DIST>
__device__ __forceinline__ void stage_obs_f64(const int32_t* obs, int T, double* lds, const Math64& tab)
{
    for (int q = threadIdx.x; q < 3 * T; q += blockDim.x) {
        const int32_t O = obs[q];
        lds[q] = DIST == 0 ? (O >= 0 ? log1p_count_f64(O, tab) : log1p((double)O)) : (double)O;
    }
}

// Logarithm of one plus a count below 0, out of line.
__device__ __attribute__((noinline)) double log1p_general(double x) { return log1p(x); }

// A sample with a negative kappa, whose counts can be negative. No prior draws it. It is
// taken as parameters outside the ranges are: not mid.
__device__ __forceinline__ bool negative_start(const float t[8]) { return t[7] < 0.0f; }

// Up to ROWS_PER_WAVE_MAX float64 trajectories run by one wavefront (one
// wavefront per workgroup), in windows of W = ROW_PAIRS / nr
// days (at most ROW_DAYS_MAX): the lanes
// draw the normals of the window's (row, day) pairs in parallel, one pair a
// lane; then four lanes walk each row through the window's days; the lanes form
// the window's squared distance terms in parallel, and lane r adds its row's
// terms in day order (the order of the one-lane-per-sample kernel, so each
// result is the same double).
//
// A walk is a serial chain, so what bounds it is its length in instructions:
// a float64 instruction occupies the SIMD for the same four cycles whatever
// its lane mask. Four of a day's five draws need only the counts of the
// morning, so the four lanes of a row make them as one (each lane its own rate
// and normal, the counts exchanged within the quad by DPP); the fifth waits
// for g. A day's M = A + R + D depends on the previous day's recoveries n2
// alone, so M^n is taken in two halves: its logarithm beside the infections of
// the day before, its exponential beside the four draws of its own day. With
// every row within math64.hpp's ranges a day is one basic block, in which the
// two chains interleave. A day takes 0.46 us with its share of the other
// phases (49 days of 114 rows: 28 us); with one lane per row, all five draws in
// turn and the library's functions it took 1.9 us (94 us).
//
// Rows r < nr: theta rth[8 r .. 8 r + 7] and sample index rix[r], in LDS.
// Scratch in LDS: zs [5 ROW_PAIRS] doubles (normals, then the distance terms),
// xs [4 ROW_PAIRS] int32. Returns row r's distance on lane r < nr (other lanes 0).
constexpr int ROWS_PER_WAVE_MAX = 16;
constexpr int ROW_PAIRS = 64;
constexpr int ROW_DAYS_MAX = 32;

// value of lane L of the calling lane's group of four
template <int L>
__device__ __forceinline__ int32_t quad_lane(int32_t x)
{
    return __builtin_amdgcn_mov_dpp(x, L * 0x55, 0xF, 0xF, true);
}

// One row's walk state and constants, alike on its four lanes.
struct RowWalk {
    State s;
    int32_t M;
    PowArg p;              // of M
    double a0, al, nn, rate;
    double P, rP, scale;
    bool mid, ofA;
    int role;
};

// nd days of a row: normals zr [nd][5], counts A, R, D to xr [nd][4]
template <int NOISE, bool MID>
__device__ __forceinline__ void walk_window(RowWalk& w, int nd, const double* zr, int32_t* xr, const Math64& tab)
{
#pragma clang fp contract(off)
    State& s = w.s;
    double z1 = zr[0], zq = zr[1 + w.role];
#pragma unroll 1
    for (int u = 0; u < nd; ++u) {
        const int v = u + 1 < nd ? u + 1 : u;
        const double z1n = zr[5 * v], zqn = zr[5 * v + 1 + w.role];
        const double g = MID || w.mid ? force_f64(w.p, w.a0, w.al, tab)
                                      : force_general((double)w.M, w.nn, w.a0, w.al);
        const int32_t d4 = draw_f64<NOISE>(w.rate * (double)(w.ofA ? s.A : s.I), zq, w.scale);
        const int32_t n2 = give<MID>(quad_lane<0>(d4), s.I);
        w.M += n2;
        if (MID || w.mid) w.p = pow_arg((double)w.M, w.nn, tab);
        const double h0 = g * (double)s.S * (double)s.I;
        const double h1 = MID || w.mid ? div_by(h0, w.P, w.rP) : div_general(h0, w.P);
        const int32_t n1 = give<MID>(draw_f64<NOISE>(h1, z1, w.scale), s.S);
        const int32_t n3 = give<MID>(quad_lane<1>(d4), s.A);
        const int32_t n4 = give<MID>(quad_lane<2>(d4), s.A - n3);
        const int32_t n5 = give<MID>(quad_lane<3>(d4), s.I - n2);
        s.S -= n1;
        s.I += n1 - n2 - n5;
        s.A += n2 - n3 - n4;
        s.R += n3;
        s.D += n4;
        const int32_t ar = w.role == 0 ? s.A : s.R;
        xr[4 * u + w.role] = w.role < 2 ? ar : s.D;  // the fourth is not read
        z1 = z1n;
        zq = zqn;
    }
}

template <int NOISE, int DIST, bool EXIT = false>
__device__ __forceinline__ double simulate_rows_f64_wave(int nr, const float* rth, const uint64_t* rix,
                                                         Key key, uint32_t series, uint32_t domain,
                                                         int32_t P, int32_t A0, int32_t R0, int32_t D0,
                                                         int T, double scale, const double* lobs,
                                                         const Math64& tab, double* zs, int32_t* xs,
                                                         double exit_at = 0.0)
{
#pragma clang fp contract(off)
    const int lane = threadIdx.x & 63;
    const int W = min(ROW_PAIRS / nr, ROW_DAYS_MAX);
    // the row's walk: lanes 4 r .. 4 r + 3
    const int row = (lane >> 2) < nr ? (lane >> 2) : 0, role = lane & 3;
    const bool walker = (lane >> 2) < nr;
    RowWalk wk;
    {
        float th[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) th[k] = rth[8 * row + k];
        wk.mid = theta_mid(th) && !negative_start(th);
        wk.P = (double)P;
        wk.rP = 1.0 / wk.P;
        wk.scale = scale;
        wk.a0 = (double)th[0];
        wk.al = (double)th[1];
        wk.nn = (double)th[2];
        // this lane's draw: n2 (gamma I), n3 (beta A), n4 (delta A), n5 (beta eta I)
        wk.role = role;
        wk.ofA = role == 1 || role == 2;
        wk.rate = role == 0 ? (double)th[4]
                            : (role == 1 ? (double)th[3]
                                         : (role == 2 ? (double)th[5] : (double)th[3] * (double)th[6]));
        wk.s = init_state(th[7], P, A0, R0, D0);
        wk.M = A0 + R0 + D0;
        wk.p = pow_arg((double)wk.M, wk.nn, tab);  // not used unless mid
    }
    const bool all_mid = __ballot(!wk.mid) == 0ull;
    double acc = 0.0;
    for (int t0 = 1; t0 <= T; t0 += W) {
        const int nd = T - t0 + 1 < W ? T - t0 + 1 : W;
        {
            const int r = lane / nd, u = lane - r * nd;
            if (r < nr) {
                const uint4 w = stream_words(key, rix[r], series, ctr_word3((uint32_t)(t0 + u), domain, 0));
                double z[5];
                normals_f64(w, tab, z);
#pragma unroll
                for (int k = 0; k < 5; ++k) zs[5 * (r * W + u) + k] = z[k];
            }
        }
        wave_lds_sync();
        if (walker) {
            if (all_mid)
                walk_window<NOISE, true>(wk, nd, zs + 5 * row * W, xs + 4 * row * W, tab);
            else
                walk_window<NOISE, false>(wk, nd, zs + 5 * row * W, xs + 4 * row * W, tab);
        }
        wave_lds_sync();
        auto terms = [&](auto logarithm) {
#pragma unroll 1
            for (int p = lane; p < nr * 3 * nd; p += 64) {
                const int r = p / (3 * nd), q = p - r * 3 * nd;
                const int u = q / 3, c = q - 3 * u;
                const int t = t0 - 1 + u;  // 0-based day
                const int32_t X = xs[4 * (r * W + u) + c];
                const double d = (DIST == 0 ? logarithm(X) : (double)X) - lobs[c * T + t];
                zs[5 * r * W + q] = d * d;
            }
        };
        if (DIST == 1 || all_mid)
            terms([&](int32_t X) { return log1p_count_f64(X, tab); });
        else
            terms([&](int32_t X) { return X >= 0 ? log1p_count_f64(X, tab) : log1p_general((double)X); });
        wave_lds_sync();
        if (lane < nr) {
            const double* tr = zs + 5 * lane * W;
            int q = 0;
            for (; q + 6 <= 3 * nd; q += 6) {
                double v[6];
#pragma unroll
                for (int k = 0; k < 6; ++k) v[k] = tr[q + k];
#pragma unroll
                for (int k = 0; k < 6; ++k) acc += v[k];
            }
            for (; q < 3 * nd; ++q) acc += tr[q];
        }
        wave_lds_sync();  // the window's scratch is reused by the next one
        if (EXIT && __ballot(lane < nr && !(acc > exit_at)) == 0ull) break;
    }
    if (EXIT && acc > exit_at) return INFINITY;  // the sum only grows
    return lane < nr ? sqrt_mid(acc) : 0.0;
}

}  // namespace abc
