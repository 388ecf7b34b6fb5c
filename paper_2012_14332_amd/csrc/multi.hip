// Several series in one persistent float32 simulate+distance launch, and its
// C-ABI entry point abc_simulate_distance_multi.
//
// The per-series launches of abc_simulate_distance each end with a tail in
// which the last trajectories of every wavefront's queue run to their last
// day while most lanes of the device are idle. Here the 64-sample chunks of
// all series form one queue: each wavefront owns a fixed stride of chunks
// over it, takes a chunk's 64 samples into its ring (prior draw, rates,
// initial state and the per-sample Philox words, prepared by the whole
// wavefront), and every lane carries the series of the sample it holds --
// its horizon, observed rows and future-days bound table in LDS, tolerance
// and Philox series word. Series are laid out in the queue longest horizon
// first, so a launch ends on its shortest trajectories and pays one tail.
// The day step, the early exit and the distance are those of the one-series
// kernel: every distance is bit-identical to abc_simulate_distance's.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "bound.hpp"
#include "common.hpp"
#include "model.hpp"

namespace abc {

constexpr int MS_MAX = ABC_MULTI_MAX;

struct MSeries {
    int32_t P, A0, R0, D0, T;
    uint32_t series;   // Philox series word
    uint32_t u0, b1;   // its per-series Philox constants
    float invP;
    float exit_f32;    // squared-distance early-exit bound in log2 units (or raw)
    int32_t obs_off;   // float offset of the observed rows [T][4] in LDS
    int32_t tab_off;   // float offset of the bound table [ntb][2][LB_Q] in the tables, -1: none
    int32_t ntb, lb_sh;
    int64_t chunk0;    // first chunk of the series in the launch's queue
    int64_t n;
    uint64_t first;
    const int32_t* obs;
    float* dist;
};

struct MultiArgs {
    MSeries s[MS_MAX];
    int32_t m;
    int32_t refill_min;
    int64_t nchunks;
    float lo[8];
    float width[8];
    Key key;
    uint32_t domain;
    float scale;
    int32_t obs_words;  // floats of all observed rows (a multiple of 4)
    int32_t tab_words;  // floats of all bound tables (a multiple of 4)
    int32_t zero_off;   // float offset of a row of zeros among them for series without one, -1: none
    unsigned long long* days;
};

// What a lane reads from LDS when it starts a sample of series j (three reads).
struct alignas(16) SerLds {
    int32_t A0, M0, R1, D1;    // A0, A0 + R0 + D0, R0 + 1, D0 + 1
    float invP, exitb;
    uint32_t wend, b1;         // wend: fourth counter word of the last day
    uint32_t obs;              // LDS address of the first observed row
    int32_t room;              // P - A0 - R0 - D0 (S0 + I0)
    float* dist;
};

// One prepared sample: rates, I0 and the per-sample Philox words. Its series
// and offset follow from the chunk in the ring, which is wave-uniform, so they
// are not stored (48 bytes a slot).
struct alignas(16) MSlot {
    float a0, al, n, be, ga, de, bh;
    int32_t i0;
    uint32_t c1base, g3, h3, f3;
};

typedef __attribute__((address_space(1))) float global_float;

struct MLane {
    StateD s;
    RatesF r;
    PhiloxDays ph;
    global_float* out;  // the sample's distance
    uint32_t w;         // fourth counter word of the next day; 0: no sample (idle)
    uint32_t p;         // LDS address of the day's observed row
    float acc, comp;
    // the lane's series, cached at the start of each sample
    uint32_t wend;
    float invP, exitb;
    uint32_t b1;
};

// BOUND: some series of the launch has a future-days bound table.
template <int NOISE, int DIST, bool KAHAN, bool BOUND>
__global__ __launch_bounds__(1024) void k_simulate_multi_f32(MultiArgs a)
{
    constexpr int RING = 64;
    extern __shared__ float lds_f[];
    float* tabs = lds_f + a.obs_words;
    SerLds* ser = reinterpret_cast<SerLds*>(tabs + a.tab_words);
    MSlot* ring_all = reinterpret_cast<MSlot*>(ser + MS_MAX);

    // observed rows of every series (obs_row)
    const uint32_t tabs_at = lds_address(tabs);
    for (int j = 0; j < a.m; ++j) {
        const MSeries& sj = a.s[j];
        for (int q = threadIdx.x; q < sj.T; q += blockDim.x) {
            const int row = sj.tab_off >= 0 ? sj.tab_off + 2 * LB_Q * ((q + 1) >> sj.lb_sh) : a.zero_off;
            *reinterpret_cast<float4*>(lds_f + sj.obs_off + 4 * q) =
                obs_row<DIST>(sj.obs[q], sj.obs[sj.T + q], sj.obs[2 * sj.T + q],
                              tabs_at + (uint32_t)sizeof(float) * (uint32_t)row);
        }
    }
    if (a.zero_off >= 0)
        for (int q = threadIdx.x; q < 2 * LB_Q; q += blockDim.x) tabs[a.zero_off + q] = 0.0f;
    const uint32_t wdom = a.domain << 4;
    if (threadIdx.x < (unsigned)a.m) {
        const MSeries& sj = a.s[threadIdx.x];
        SerLds e;
        e.A0 = sj.A0;
        e.M0 = sj.A0 + sj.R0 + sj.D0;
        e.R1 = sj.R0 + 1;
        e.D1 = sj.D0 + 1;
        e.invP = sj.invP;
        e.exitb = sj.exit_f32;
        e.wend = ((uint32_t)sj.T << 8) | wdom;
        e.b1 = sj.b1;
        e.obs = lds_address(lds_f) + (uint32_t)sizeof(float) * (uint32_t)sj.obs_off;
        e.room = sj.P - e.M0;
        e.dist = sj.dist;
        ser[threadIdx.x] = e;
    }
    if (BOUND) {
        // future-days bound tables, one series at a time; b_s of R and D in
        // float64 staged where the ring will live
        double* stage = reinterpret_cast<double*>(ring_all);
        for (int j = 0; j < a.m; ++j) {
            const MSeries& sj = a.s[j];
            if (sj.tab_off < 0) continue;
            __syncthreads();
            for (int q = threadIdx.x; q < 2 * sj.T; q += blockDim.x)
                stage[q] = log1p((double)sj.obs[sj.T + q]) * 1.44269504088896340736;
            __syncthreads();
            build_future_bound(stage, sj.T, sj.lb_sh, sj.ntb, (double)sj.exit_f32, tabs + sj.tab_off);
        }
    }
    __syncthreads();

    __builtin_amdgcn_s_setprio(1);
    const int lane = threadIdx.x & 63;
    // the wavefront index is uniform over the wave: kept scalar, so is
    // everything of the queue derived from it
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    MSlot* ring = ring_all + wv * RING;
    const int64_t wg = (int64_t)blockIdx.x * (blockDim.x >> 6) + wv;
    const int64_t nw = (int64_t)gridDim.x * (blockDim.x >> 6);
    if (wg >= a.nchunks) return;
    // queue positions of this wave (the host keeps them within 32 bits); its
    // j-th chunk is wg + j nw
    const uint32_t Q = __builtin_amdgcn_readfirstlane((uint32_t)(((a.nchunks - 1 - wg) / nw + 1) << 6));
    const float nc = noise_c(a.scale);
    const float dscale = DIST == 0 ? 0.693147180559945309417f : 1.0f;
    // the chunk in the ring (wave-uniform): its series, the offset of its
    // first sample in that series, and how many of its 64 positions hold a
    // sample (fewer only in a series' last chunk)
    int cur_ls = 0;
    int64_t cur_base = 0;
    uint32_t cur_valid = 0;
    // chunk c into the ring: series by the chunk ranges
    auto fill = [&](int64_t c) {
        int ls = 0;
        for (int j = 1; j < a.m; ++j)
            if (c >= a.s[j].chunk0) ls = j;
        ls = __builtin_amdgcn_readfirstlane(ls);
        const MSeries& sj = a.s[ls];
        cur_ls = ls;
        cur_base = (c - sj.chunk0) << 6;
        cur_valid = (uint32_t)min(sj.n - cur_base, (int64_t)64);
        const int64_t k = cur_base + lane;
        MSlot& sl = ring[lane];
        if (k < sj.n) {
            const uint64_t i = sj.first + (uint64_t)k;
            float thv[8];
            prior_draw(a.key, i, sj.series, a.domain, a.lo, a.width, thv);
            const Theta th = theta_from(thv);
            const RatesF r = rates_f32(th);
            const State s0 = init_state(th.ka, sj.P, sj.A0, sj.R0, sj.D0);
            PhiloxDays ph;
            ph.begin(i, sj.u0, a.key);
            sl.a0 = r.a0; sl.al = r.al; sl.n = r.n; sl.be = r.be;
            sl.ga = r.ga; sl.de = r.de; sl.bh = r.bh; sl.i0 = s0.I;
            sl.c1base = ph.c1base; sl.g3 = ph.g3; sl.h3 = ph.h3; sl.f3 = ph.f3;
        }
    };

    uint32_t qb = 0;
    uint32_t filled = 0xFFFFFFFFu;
    const uint32_t row1 = lds_address(lds_f);
    MLane l{};  // idle, with a valid state (no people) and row
    l.s = state_d(0, 0, 0, 0, 0);
    l.p = row1;
    uint64_t days_done = 0;  // of the whole wavefront

    while (true) {
        // refill: the idle lanes take the next queue positions in lane order,
        // once at least refill_min of them are idle; a pass may span the end
        // of one chunk and the start of the next
        uint64_t m = __ballot(l.w == 0u);
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
                const uint32_t pos = off + rank;
                if (in_mask(took) && pos < cur_valid) {
                    const MSlot sl = ring[pos];
                    const SerLds e = ser[cur_ls];
                    l.r = RatesF{sl.a0, sl.al, sl.n, sl.be, sl.ga, sl.de, sl.bh};
                    l.s = StateD{e.room - sl.i0, sl.i0, e.A0, e.M0, e.R1, e.D1};
                    l.ph.c1base = sl.c1base; l.ph.g3 = sl.g3; l.ph.h3 = sl.h3; l.ph.f3 = sl.f3;
                    l.out = (global_float*)e.dist + (cur_base + (int64_t)pos);
                    l.wend = e.wend; l.p = e.obs;
                    l.invP = e.invP; l.exitb = e.exitb; l.b1 = e.b1;
                    l.w = 256u | wdom;
                    l.acc = 0.0f;
                    l.comp = 0.0f;
                }
                qb += (uint32_t)__popcll(took);
                m &= ~took;
            }
            m = __ballot(l.w == 0u);
        }
        if (m == ~0ull && qb >= Q) break;
        days_done += (uint64_t)__popcll(~m);
        // idle lanes take the day too and drop it (as in k_simulate_f32)
        const bool live = l.w != 0u;
        {
            const float4 ob = lds_row(l.p);
            const uint4 words = l.ph.day(l.w, l.b1, a.key);
            float lr, ld;
            day_distance_f32<NOISE, DIST, KAHAN>(l.s, l.r, words, l.invP, nc, ob, l.acc, l.comp, lr, ld);
            float sum = l.acc;
            if (BOUND) sum += future_bound(__float_as_uint(ob.w), lr, ld);
            const bool exited = sum > l.exitb;
            const bool done = exited | (l.w == l.wend);
            if (done & live) *l.out = exited ? INFINITY : finish_distance_f32(l.acc, dscale);
            const bool idle = done | !live;
            l.w = idle ? 0u : l.w + 256u;
            l.p = idle ? row1 : l.p + (uint32_t)sizeof(float4);
        }
    }
    if (a.days && lane == 0) atomicAdd(a.days, (unsigned long long)days_done);
}

static size_t multi_lds_bytes(int obs_words, int tab_words, int block, int stage_doubles)
{
    const size_t ring = sizeof(MSlot) * 64 * (size_t)(block / 64);
    const size_t stage = sizeof(double) * (size_t)stage_doubles;
    return sizeof(float) * ((size_t)obs_words + (size_t)tab_words) + sizeof(SerLds) * MS_MAX +
           (ring > stage ? ring : stage);
}

template <int NOISE, int DIST, bool KAHAN>
static void launch_multi(const MultiArgs& a, unsigned grid, int block, size_t lds, hipStream_t s)
{
    if constexpr (DIST == 0) {
        if (a.tab_words > 0) {
            hipLaunchKernelGGL((k_simulate_multi_f32<NOISE, DIST, KAHAN, true>), dim3(grid), dim3(block), lds, s, a);
            return;
        }
    }
    hipLaunchKernelGGL((k_simulate_multi_f32<NOISE, DIST, KAHAN, false>), dim3(grid), dim3(block), lds, s, a);
}

}  // namespace abc

using namespace abc;

extern "C" abc_status abc_simulate_distance_multi(const abc_sim_job* jobs, int32_t m,
                                                  const abc_model* model, const abc_prior* prior,
                                                  uint64_t seed, uint32_t domain,
                                                  unsigned long long* days, void* stream)
{
    abc_status rc;
    ABC_REQUIRE(jobs != nullptr && m >= 1 && m <= MS_MAX, "need 1 <= m <= %d jobs", MS_MAX);
    if ((rc = check_model(model))) return rc;
    ABC_REQUIRE((model->flags & (ABC_FP64 | ABC_SUPPORT)) == 0,
                "the multi-series launch runs the float32 path with in-kernel prior draws "
                "(ABC_FP64 and ABC_SUPPORT are not options here)");
    ABC_REQUIRE(domain <= 15u, "domain %u > 15", domain);
    MultiArgs a{};
    if ((rc = prior_lo_width(prior, a.lo, a.width))) return rc;
    for (int k = 0; k < 8; ++k)
        ABC_REQUIRE(prior->lo[k] >= 0.0f, "model rates must be non-negative: prior lo[%d] < 0", k);
    int64_t total = 0;
    for (int j = 0; j < m; ++j) {
        const abc_sim_job& jb = jobs[j];
        if ((rc = check_series(jb.ser, true))) return set_error(rc, "job %d: %s", j, abc_last_error());
        ABC_REQUIRE(jb.n >= 0 && jb.n <= ((int64_t)1 << 36), "job %d: n = %lld outside [0, 2^36]",
                    j, (long long)jb.n);
        ABC_REQUIRE(!(jb.eps_exit < 0.0f) && !isnan(jb.eps_exit), "job %d: eps_exit must be >= 0 (or +INF)", j);
        ABC_REQUIRE(jb.n == 0 || jb.dist != nullptr, "job %d: dist is NULL", j);
        total += jb.n;
    }
    ABC_REQUIRE(total <= ((int64_t)1 << 36), "%lld samples in total exceed 2^36", (long long)total);
    if (total == 0) return ABC_OK;

    const int noise = (model->flags & ABC_NOISE_LITERAL) ? 1 : 0;
    const int distm = (model->flags & ABC_DIST_RAW) ? 1 : 0;
    const bool kahan = (model->flags & ABC_KAHAN) != 0;
    const bool bound = distm == 0 && !(model->flags & ABC_NO_BOUND);

    // queue order: longest horizon first (stable), jobs with samples only
    std::vector<int> order;
    for (int j = 0; j < m; ++j)
        if (jobs[j].n > 0) order.push_back(j);
    std::stable_sort(order.begin(), order.end(),
                     [&](int x, int y) { return jobs[x].ser->T > jobs[y].ser->T; });
    a.m = (int32_t)order.size();
    a.key = make_key(seed);
    a.domain = domain;
    a.scale = model->noise_scale;
    a.days = days;
    const LaunchShape shape = launch_shape();
    int block = shape.block, bpc = shape.blocks_per_cu;
    // With early exits a large launch takes two 1024-thread workgroups per CU, a
    // smaller one 512-thread workgroups with at least seven chunks per wavefront:
    // three series of 1e7 samples take 1.49 ms instead of 1.60 ms with two
    // 512-thread workgroups, three of 3e5 samples 0.117 ms instead of 0.127 ms.
    // Where a job has none, its trajectories are most of the work and end together:
    // 512-thread workgroups with one chunk per wavefront, up to four per CU. Three
    // series of T = 100 without exits, one / two / three / four per CU: 1e5 samples each
    // 206 / 176 / 174 / 171 us, 3e5 441 / 386 / 368 / 353, 1e6 1386 / 1205 / 1152 /
    // 1131. So it is with raw distances over short horizons, whose exits come late (T =
    // 100: 1e5 169 / 155 / 158 / 158, T = 400: 359 / 407 / 468 / 466).
    if (!shape.chosen) {
        DeviceInfo di;
        if ((rc = device_info(&di))) return rc;
        bool late = distm == 1 && jobs[order[0]].ser->T <= 150;  // the longest
        for (int j : order) late = late || isinf(jobs[j].eps_exit);
        const int64_t per = (total / 64) / ((int64_t)di.num_cu * 8 * (late ? 1 : 7));
        block = !late && per >= 4 ? 1024 : 512;
        bpc = late ? (per < 1 ? 1 : (per > 4 ? 4 : (int)per)) : (per >= 2 ? 2 : 1);
    }
    a.refill_min = abc_get_refill_min();
    int obs_words = 0, maxT = 0;
    int64_t chunk = 0;
    std::vector<int> sh(a.m, 0), ntb(a.m, 0);
    for (int q = 0; q < a.m; ++q) {
        const abc_sim_job& jb = jobs[order[q]];
        MSeries& s = a.s[q];
        s.P = (int32_t)jb.ser->P;
        s.A0 = jb.ser->A0;
        s.R0 = jb.ser->R0;
        s.D0 = jb.ser->D0;
        s.T = jb.ser->T;
        s.series = jb.series;
        const uint64_t p1 = (uint64_t)PH_M1 * (uint64_t)jb.series;
        s.u0 = (uint32_t)(p1 >> 32) ^ a.key.k0;
        s.b1 = (uint32_t)p1 ^ (a.key.k0 + PH_W0);
        s.invP = 1.0f / (float)jb.ser->P;
        // the same exit bound as abc_simulate_distance, in log2 units for log1p
        const double e2 = (double)jb.eps_exit * (double)jb.eps_exit;
        const double unit = distm ? 1.0 : 2.08136898100560809980;
        s.exit_f32 = isinf(jb.eps_exit) ? INFINITY : (float)(e2 * unit * (1.0 + 0x1p-18));
        s.obs_off = obs_words;
        obs_words += 4 * s.T;
        s.chunk0 = chunk;
        chunk += (jb.n + 63) >> 6;
        s.n = jb.n;
        s.first = jb.first;
        s.obs = jb.ser->obs;
        s.dist = jb.dist;
        if (s.T > maxT) maxT = s.T;
        if (bound && !isinf(jb.eps_exit)) {
            while ((s.T >> sh[q]) + 1 > LB_MAX_BLOCKS) ++sh[q];
            ntb[q] = (s.T >> sh[q]) + 1;
        }
    }
    a.nchunks = chunk;
    a.obs_words = obs_words;
    const int stage_doubles = 2 * maxT + LB_MAX_SEG * 2 * LB_Q;
    DeviceInfo info;
    if ((rc = device_info(&info))) return rc;
    const int num_cu = info.num_cu, max_lds = info.max_lds;
    // where the rows and the rings of a workgroup of this size do not fit, a
    // smaller workgroup needs fewer rings
    while (block > 64 && multi_lds_bytes(a.obs_words, 0, block, stage_doubles) > (size_t)max_lds)
        block = (block / 2 + 63) & ~63;
    // bound tables: coarser time blocks for the series with the most rows until
    // blocks_per_cu workgroups fit a CU's LDS (160 KiB) and one fits the
    // workgroup limit; without room at all, no tables. Series without a table
    // beside others with one look up a row of zeros.
    auto tab_words = [&]() {
        int w = 0;
        bool with = false, without = false;
        for (int q = 0; q < a.m; ++q) {
            w += 2 * LB_Q * ntb[q];
            (ntb[q] > 0 ? with : without) = true;
        }
        return w + (with && without ? 2 * LB_Q : 0);
    };
    const size_t lds_target = std::min((size_t)max_lds, (size_t)(163840 / (bpc > 0 ? bpc : 1)));
    while (multi_lds_bytes(a.obs_words, tab_words(), block, stage_doubles) > lds_target) {
        int qmax = -1;
        for (int q = 0; q < a.m; ++q)
            if (ntb[q] > 1 && (qmax < 0 || ntb[q] > ntb[qmax])) qmax = q;
        if (qmax < 0) break;
        ++sh[qmax];
        ntb[qmax] = (a.s[qmax].T >> sh[qmax]) + 1;
    }
    if (multi_lds_bytes(a.obs_words, tab_words(), block, stage_doubles) > (size_t)max_lds)
        for (int q = 0; q < a.m; ++q) ntb[q] = 0;
    a.tab_words = tab_words();
    a.zero_off = -1;
    int tw = 0;
    for (int q = 0; q < a.m; ++q) {
        a.s[q].ntb = ntb[q];
        a.s[q].lb_sh = sh[q];
        a.s[q].tab_off = ntb[q] > 0 ? tw : -1;
        tw += 2 * LB_Q * ntb[q];
    }
    if (tw < a.tab_words) a.zero_off = tw;
    const size_t lds = multi_lds_bytes(a.obs_words, a.tab_words, block, stage_doubles);
    if (lds > (size_t)max_lds)
        return set_error(ABC_EUNSUPPORTED, "%d series with %d observed days need %zu B of LDS "
                         "per workgroup of %d (> %d)", a.m, obs_words / 4, lds, block, max_lds);
    // resident workgroups: what the LDS allows per CU, at most blocks_per_cu
    int per_cu = (int)(163840 / lds);
    if (per_cu < 1) per_cu = 1;
    if (per_cu > bpc) per_cu = bpc;
    const int64_t need = (a.nchunks + block / 64 - 1) / (block / 64);
    int64_t g = (int64_t)num_cu * per_cu;
    if (g > need) g = need;
    const hipStream_t s = as_stream(stream);
    const unsigned grid = (unsigned)g;
    if (kahan) {
        if (noise == 0 && distm == 0) launch_multi<0, 0, true>(a, grid, block, lds, s);
        else if (noise == 0) launch_multi<0, 1, true>(a, grid, block, lds, s);
        else if (distm == 0) launch_multi<1, 0, true>(a, grid, block, lds, s);
        else launch_multi<1, 1, true>(a, grid, block, lds, s);
    } else {
        if (noise == 0 && distm == 0) launch_multi<0, 0, false>(a, grid, block, lds, s);
        else if (noise == 0) launch_multi<0, 1, false>(a, grid, block, lds, s);
        else if (distm == 0) launch_multi<1, 0, false>(a, grid, block, lds, s);
        else launch_multi<1, 1, false>(a, grid, block, lds, s);
    }
    return check_launch("k_simulate_multi_f32");
}
