// The renderer with a team of T lanes per ray (T a power of two, 1 to 64): the
// form for batches too small to fill the card with one lane per ray.
//
// A lane per ray walks its samples one after another, each a chain of
// dependent loads (occupancy word, eight links, then eight records one by
// one); a batch of a few thousand rays then leaves most of the card without a
// wave and its time is the longest ray's chain.  The samples of a ray depend
// on each other only through the optical depth in front of them, which is a
// prefix sum: a team takes T consecutive sample positions at once, one per
// lane, gathers and interpolates them independently, and composites them with
// a prefix sum over the team (FP64, in registers through data-parallel-primitive
// moves).  Every sample's interpolants, weight and activation are the same
// operations in the same order as in the one-lane form; only FP64 sums are
// grouped differently.  Samples behind the early-termination point that share
// its window are evaluated and discarded.
//
// Pose gradient in ONE march.  Row k of a ray's pose Jacobian is
//   sum_i [delta (c_k,i T_{i+1} + A_k,i - Chat_k) grad sigma_i + dact_k,i w_i grad s_k,i]
// (Eq. 9-14), in which only Chat_k is unknown until the march ends, and it
// enters linearly: the sums without it and S = sum_i delta grad sigma_i are
// accumulated (FP64, because their difference cancels) while the ray is
// composited, and Chat_k S is taken off at the end.  The records of a sample
// are gathered once instead of twice.
//
// Gauss-Newton composites first, each team keeping the positions of its lit windows, then
// gathers those again with their spatial derivatives and sums its Jacobian rows
// in FP32 in sample order, lane after lane, as one lane per ray would: the solve of a
// badly conditioned frame multiplies their rounding.  Prefixes and frame sums are
// FP64 sums that the team's width groups, so the last bits may differ between widths.
//
// Grid gradient: the march keeps (density, three colour pre-activations) of
// its lit samples in LDS, GRID_WINDOWS windows of them, so that the backward
// pass needs only their links again; a ray with more is marched and gathered
// again from the first window that did not fit.  The scatter is the shared
// wave-wide merge.
#include "internal.hpp"
#include "scatter.hpp"

namespace pxm {

enum { TEAM_FORWARD = 0, TEAM_FUSED = 1, TEAM_GN = 2, TEAM_BACKWARD = 3 };

struct TeamIO {
    const float* tgt_rgb;       // fused, Gauss-Newton
    const float* tgt_depth;
    const float* fw;
    const float* g_rgb;         // backward: upstream gradients and the forward's outputs
    const float* g_depth;
    const float* rgb_in;
    const float* depth_in;
    const int32_t* nsamp_in;
    float* rgb;
    float* depth;
    int32_t* nsamp;
    double* loss;
    float* grad;
    double* grad_pose;
    double* gn;
};

// Windows with light that the march keeps for the second pass, in LDS.  Grid
// gradient: per lane a float4 and a position, in the work-mask region of the
// wave's block (this kernel has no masks).  Gauss-Newton: a position per lane.
constexpr int GRID_WINDOWS = 6, GN_WINDOWS = 48;
static_assert(GRID_WINDOWS * 5 <= MARK_WORDS, "the kept samples fit in the work-mask region");

// ---------------------------------------------------------------------------
// team-wide moves (every lane of the wave active)
// ---------------------------------------------------------------------------

// Waves per workgroup.  Four share one atomic per value and frame; eight keep
// a CU's registers until the slowest of them ends (pose gradient of the
// 816,000-ray room frame 843 us with eight, 727 with four, 715 with two), two
// send twice the atomics (2000 rays, Gauss-Newton: 41 us with two, 31 with four).
constexpr int TEAM_WAVES = SUM_WAVES;

struct Team {
    int T;                      // lanes per ray
    int sub;                    // lane's place in its team
    int base;                   // first lane of the team
    unsigned long long mask;    // the team's lanes
};

template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_f64(double v) {
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, ROWS, 0xf, false);
    return __longlong_as_double((long long)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
}

// Inclusive prefix sum over the team.
__device__ __forceinline__ double team_scan(double v, const Team& tm) {
    double o;
    if (tm.T > 1) { o = dpp_f64<0x111, 0xf>(v); v += tm.sub >= 1 ? o : 0.0; }    // row_shr:1
    if (tm.T > 2) { o = dpp_f64<0x112, 0xf>(v); v += tm.sub >= 2 ? o : 0.0; }    // row_shr:2
    if (tm.T > 4) { o = dpp_f64<0x114, 0xf>(v); v += tm.sub >= 4 ? o : 0.0; }    // row_shr:4
    if (tm.T > 8) { o = dpp_f64<0x118, 0xf>(v); v += tm.sub >= 8 ? o : 0.0; }    // row_shr:8
    if (tm.T > 16) v += dpp_f64<0x142, 0xa>(v);                                  // row_bcast:15 -> rows 1, 3
    if (tm.T > 32) v += dpp_f64<0x143, 0xc>(v);                                  // row_bcast:31 -> rows 2, 3
    return v;
}

// The previous lane's value; `first` on the team's first lane.
__device__ __forceinline__ double team_prev(double v, double first, const Team& tm) {
    const double o = dpp_f64<0x138, 0xf>(v);                                     // wave_shr:1
    return tm.sub == 0 ? first : o;
}

// The team's last lane's value, on all of its lanes.
__device__ __forceinline__ double team_last(double v, const Team& tm) {
    return tm.T > 1 ? __shfl(v, tm.base + tm.T - 1, WAVE) : v;
}

__device__ __forceinline__ double team_sum(double v, const Team& tm) {
    return team_last(team_scan(v, tm), tm);
}

// ---------------------------------------------------------------------------
// one window of samples, composited
// ---------------------------------------------------------------------------

// What a lit sample hands on: its weight, the transmittance behind it, its
// colours and the inclusive prefixes A_i, AD_i of Eq. 9 and 10.
struct Lit {
    bool lit;
    float wt, Tn;
    float c[3];
    double A[3], AD;
};

// Prefixes carried from window to window (the same on all lanes of a team).
struct Carry {
    double L;
    double A[3], AD;
    float T;            // transmittance behind L; kept by teams of one only
};

// Optical depth of the window's samples (sr <= 0 or NaN: no light), their
// weights and, with PREFIX, the inclusive sums behind each.  With STOPS a
// sample whose transmittance falls below t_stop ends its ray: `last` is its
// lane (64: none) and later samples of the window are dropped.
template <bool PREFIX, bool STOPS>
__device__ __forceinline__ void composite(const KOpts& op, const Team& tm, bool have, float sr, const float s[3],
                                          float t, Carry& cy, Lit& q, int& last) {
    q.lit = have && sr > 0.f;
    const float x = q.lit ? sr * op.step_vox : 0.f;
    const double Li = cy.L + team_scan((double)x, tm);
    const float Tb = tm.T == 1 ? cy.T : trans_of(team_prev(Li, cy.L, tm));
    q.Tn = cy.T = trans_of(Li);
    last = WAVE;
    if (STOPS) {
        const unsigned long long m = __ballot(q.lit && q.Tn < op.t_stop) & tm.mask;
        if (m) last = __ffsll((long long)m) - 1;
        q.lit = q.lit && lane_id() <= last;
    }
    q.wt = q.lit ? Tb * (-expm1f(-x)) : 0.f;
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) q.c[ch] = q.lit ? act_fwd(op.act, s[ch]) : 0.f;
    const float tt = q.lit ? t : 0.f;
    cy.L = team_last(Li, tm);
    if (PREFIX) {
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) {
            q.A[ch] = cy.A[ch] + team_scan((double)q.wt * (double)q.c[ch], tm);
            cy.A[ch] = team_last(q.A[ch], tm);
        }
        q.AD = cy.AD + team_scan((double)q.wt * (double)tt, tm);
        cy.AD = team_last(q.AD, tm);
    } else {
        // only the totals are wanted: this lane's share, summed over the team at the end
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) cy.A[ch] = fma((double)q.wt, (double)q.c[ch], cy.A[ch]);
        cy.AD = fma((double)q.wt, (double)tt, cy.AD);
    }
}

// Sums of one ray's pose Jacobian rows, without (P, Q) and with (S, St) the
// factor Chat_k; this lane's samples.
template <bool VIEW>
struct PoseSums {
    double P[4][3], Q[4][3], S[3], St[3];
    float V[VIEW ? 3 : 1][3];
};

// Grid-gradient factors of a lit sample (Eq. 8-10).
__device__ __forceinline__ void grid_factors(const KOpts& op, const Lit& q, const float s[3], float t,
                                             const double Chat[3], double Dhat, const float gC[3], float gDr,
                                             float& gsig, float gs[3]) {
    const float delta = op.step_vox;
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) gs[ch] = act_bwd(op.act, s[ch]) * q.wt * gC[ch];
    gsig = delta * (gC[0] * (q.c[0] * q.Tn + (float)(q.A[0] - Chat[0]))
                  + gC[1] * (q.c[1] * q.Tn + (float)(q.A[1] - Chat[1]))
                  + gC[2] * (q.c[2] * q.Tn + (float)(q.A[2] - Chat[2]))
                  + gDr * (t * q.Tn + (float)(q.AD - Dhat)));
}

// ---------------------------------------------------------------------------
// Gauss-Newton: pose Jacobian rows of (R, G, B, z-depth)
// ---------------------------------------------------------------------------

// Sums of a ray's samples, the same on all lanes of its team.
struct JacAcc {
    float go[4][3];
    float gd[4][3];
    float gv[4][3];
};

// Value of lane I of the team (T lanes) on all of its lanes: a broadcast within
// pairs, quads or rows of 16 lanes.
template <int T, int I>
__device__ __forceinline__ float team_get(float v) {
    constexpr int CTRL = T == 2 ? (I ? 0xF5 : 0xA0) : T == 4 ? I * 0x55 : 0x150 + I;   // quad_perm, row_newbcast
    return T == 1 ? v : __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}

// Adds the window's rows in lane order.  gp[k][a]: gradient of output k with
// respect to position (zero for a lane without light), t its distance,
// dact[k] ev[k][a] the view-direction term.
template <bool VIEW, int T, int I>
__device__ __forceinline__ void jacobian_add(unsigned long long lit, float inv_vs, float t, const float gp[4][3], const float dact[3],
                                             const float ev[3][3], JacAcc& ja) {
    constexpr unsigned long long LANE = T == 1 ? ~0ull : T == 2 ? 0x5555555555555555ull << I
                                      : T == 4 ? 0x1111111111111111ull << I : 0x0001000100010001ull << I;
    if (lit & LANE) {                                       // some team has light here (wave-uniform)
        const float tb = team_get<T, I>(t);
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const float p = team_get<T, I>(gp[k][a]);
                ja.go[k][a] = fmaf(p, inv_vs, ja.go[k][a]);
                ja.gd[k][a] = fmaf(tb, p * inv_vs, ja.gd[k][a]);
                if (VIEW && k < 3)
                    ja.gv[k][a] = fmaf(team_get<T, I>(dact[k < 3 ? k : 0]), team_get<T, I>(ev[k < 3 ? k : 0][a]),
                                       ja.gv[k][a]);
            }
    }
    if constexpr (I + 1 < T) jacobian_add<VIEW, T, I + 1>(lit, inv_vs, t, gp, dact, ev, ja);
}

// Row k is the pose gradient of output k alone (unit upstream on it), so a
// sample's factors are those of Eq. 8-10 with gC = e_k (colour rows) or
// dL/d range = 1/s (depth row).
template <bool VIEW>
__device__ __forceinline__ void jacobian_window(const KGrid& g, const KOpts& op, const Team& tm, const Ray& ray,
                                                const Sample& s, const Interp& v, const Lit& q, const double Chat[3],
                                                double Dhat, JacAcc& ja) {
    const float delta = op.step_vox, inv_vs = (float)g.inv_vs;
    float gp[4][3], dact[3], ev[3][3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        dact[a] = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            gp[k][a] = 0.f;
            if (k < 3) ev[k < 3 ? k : 0][a] = 0.f;
        }
    }
    const float t = q.lit ? s.t : 0.f;
    if (q.lit) {
        float gsig[4];
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) {
            dact[ch] = act_bwd(op.act, v.s[ch]) * q.wt;
            gsig[ch] = delta * (q.c[ch] * q.Tn + (float)(q.A[ch] - Chat[ch]));
        }
        gsig[3] = delta * (s.t * q.Tn + (float)(q.AD - Dhat)) / ray.s;
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                float p = gsig[k] * v.dsig[a];
                if (k < 3) p = fmaf(dact[k < 3 ? k : 0], v.ds[k < 3 ? k : 0][a], p);
                gp[k][a] = p;
                if (VIEW && k < 3) ev[k < 3 ? k : 0][a] = v.ev[k < 3 ? k : 0][a];
            }
    }
    const unsigned long long lit = __ballot(q.lit);
    if (tm.T == 16) jacobian_add<VIEW, 16, 0>(lit, inv_vs, t, gp, dact, ev, ja);
    else if (tm.T == 4) jacobian_add<VIEW, 4, 0>(lit, inv_vs, t, gp, dact, ev, ja);
    else if (tm.T == 2) jacobian_add<VIEW, 2, 0>(lit, inv_vs, t, gp, dact, ev, ja);
    else jacobian_add<VIEW, 1, 0>(lit, inv_vs, t, gp, dact, ev, ja);
}

// ---------------------------------------------------------------------------
// the kernel
// ---------------------------------------------------------------------------

// 64 / T rays per wave.  Bound by the latency of each window's chain (occupancy
// words, links, then the records of eight corners one after another) at the
// waves the registers allow: 4 on a SIMD forward, 3 with the grid gradient, 2
// with the pose sums (60 registers of FP64).  With both gradients the limit of 2
// costs 16 spilled registers at SH degree 2 and is worth them: 4096 rays 89 -> 58 us,
// 83,583 rays 832 -> 570 us (a limit of 3 on the pose kernels spills 90 registers and
// takes four times as long).  The view term spills 55 for the pose alone and 61 with
// both (32 and 42 at degree 0): batches above 120,000 to 150,000 rays leave the team
// for it (one_lane_pose).
template <int MODE, bool GRID, bool POSE, bool VIEW, int DEG>
__global__ void __launch_bounds__(WAVE * TEAM_WAVES, POSE && MODE != TEAM_BACKWARD ? 2 : 1) k_team(KGrid g, KRays rs, KOpts op, int log_t, TeamIO io) {
    constexpr bool BACKWARD = MODE == TEAM_BACKWARD;
    constexpr bool GAUSS_NEWTON = MODE == TEAM_GN;
    constexpr bool ONE_MARCH = POSE && MODE == TEAM_FUSED;  // pose sums of the compositing march
    constexpr bool KEEP = (GRID && MODE == TEAM_FUSED) || GAUSS_NEWTON;   // windows kept for the second pass
    extern __shared__ __align__(16) float smem[];
    WaveStage wc{};
    if (GRID) wc = wave_stage(smem, io.grad, (uint64_t)g.n_alloc * (RecL<DEG>::S * sizeof(float)));
    const int lane = lane_id();
    constexpr int KEPT = GAUSS_NEWTON ? GN_WINDOWS : GRID_WINDOWS;
    float4* keep = reinterpret_cast<float4*>(wc.marks) + lane;
    int32_t* keep_at = (GRID ? reinterpret_cast<int32_t*>(wc.marks) + 4 * GRID_WINDOWS * WAVE
                             : reinterpret_cast<int32_t*>(smem) + (threadIdx.x / WAVE) * GN_WINDOWS * WAVE) + lane;
    Team tm;
    tm.T = 1 << log_t;
    tm.sub = lane & (tm.T - 1);
    tm.base = lane - tm.sub;
    tm.mask = (tm.T == WAVE ? ~0ull : (1ull << tm.T) - 1ull) << tm.base;
    const int64_t r = (ray_tile(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x) >> log_t;
    const bool inr = r < rs.n;
    int f = 0;
    Ray ray;
    ray.empty = true;
    float Y[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float GY[9][3];
    float gC[3] = {0.f, 0.f, 0.f};
    float gDr = 0.f;
    double Chat[3] = {0.0, 0.0, 0.0}, Dhat = 0.0;
    int64_t limit = 0;                                      // sample positions to march at most
    bool wanted = inr;
    if (BACKWARD && inr) {
        gC[0] = io.g_rgb[3 * r];
        gC[1] = io.g_rgb[3 * r + 1];
        gC[2] = io.g_rgb[3 * r + 2];
        gDr = io.g_depth[r];
        wanted = gC[0] != 0.f || gC[1] != 0.f || gC[2] != 0.f || gDr != 0.f;
    }
    if (wanted) {
        f = frame_of(rs.off, rs.F, r);
        setup_ray(g, rs, op, r, f, ray);
        sh9(ray.d[0], ray.d[1], ray.d[2], Y);
        if (VIEW) sh9_grad(ray.d[0], ray.d[1], ray.d[2], GY);
        if (!ray.empty) limit = BACKWARD ? io.nsamp_in[r] : op.max_samples;
        if (BACKWARD) {
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) Chat[ch] = io.rgb_in[3 * r + ch];
            Dhat = (double)io.depth_in[r] * (double)ray.s;
            gDr = gDr / ray.s;
        }
    }
    PoseSums<VIEW> ps;
    PoseAcc pa = {{0.f, 0.f, 0.f}, {0.f, 0.f, 0.f}, {0.f, 0.f, 0.f}};
    JacAcc ja;
    if (GAUSS_NEWTON) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int a = 0; a < 3; ++a) ja.go[k][a] = ja.gd[k][a] = ja.gv[k][a] = 0.f;
    }
    if (ONE_MARCH) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
#pragma unroll
            for (int k = 0; k < 4; ++k) ps.P[k][a] = ps.Q[k][a] = 0.0;
            ps.S[a] = ps.St[a] = 0.0;
#pragma unroll
            for (int k = 0; k < (VIEW ? 3 : 1); ++k) ps.V[k][a] = 0.f;
        }
    }
    Carry cy = {0.0, {0.0, 0.0, 0.0}, 0.0, 1.f};
    int64_t kept = 0;                                       // kept sample positions of the ray
    int windows = 0;                                        // kept windows: of the wave (grid), of the team (Gauss-Newton)
    bool spilled = false;
    int64_t resume = 0;                                     // the team's position at the first one not kept
    // The march.  A second one goes over the kept positions again: of a ray whose
    // windows did not all fit, from `resume`, scattering as it goes; or of a
    // Gauss-Newton ray, for its Jacobian.
    auto march = [&](auto second, int64_t o, int64_t lim) {
        constexpr bool SECOND = decltype(second)::value;
        constexpr bool SCATTER = GRID && (SECOND || BACKWARD);
        constexpr bool POSE_HERE = POSE && (GAUSS_NEWTON ? SECOND : !SECOND);
        OccCache oc;
        occ_cache_init(oc);
        bool on = o < lim, dark = true;                     // dark: this lane's last sample had no light (Gauss-Newton)
        while (__ballot(on)) {
            const int64_t oo = o + tm.sub;
            int64_t nxt = oo + 1;
            Sample s;
            bool inside = false, work = false;
            if (on && oo < lim) {
                inside = sample_at(g, ray, ray.k_first + oo, s);
                if (inside) {
                    work = true;
                    if (g.occ0) {
                        int64_t nk;
                        const int cls = occ_classify(g, ray, ray.k_first + oo, s.c, oc, nk);
                        work = cls == OCC_CELL;
                        if (cls == OCC_JUMP) nxt = nk - ray.k_first;
                    }
                }
            }
            const int run = __popcll(__ballot(inside) & tm.mask);   // positions inside come first
            int last = WAVE;
            if (__ballot(work)) {                           // the whole wave composites
                int idx[8];
                Interp v;
                v.sig = v.s[0] = v.s[1] = v.s[2] = 0.f;
                bool have = false;
                if (work) {
                    have = load_links(g, s.base, idx) > 0;
                    if (have && g.probe && (!GAUSS_NEWTON || __ballot(dark))) have = gather_density<DEG>(g, idx, s.f) > 0.f;
                    if (have) gather_interp<POSE_HERE, POSE_HERE && VIEW, DEG>(g, idx, Y, GY, s.f, v);
                    if (GAUSS_NEWTON) dark = !(have && v.sig > 0.f);
                }
                Lit q;
                composite<ONE_MARCH || SECOND || BACKWARD, !BACKWARD && !SECOND>(op, tm, have, v.sig, v.s, s.t, cy, q,
                                                                                 last);
                // the grid gradient keeps the windows of the wave, whose scatters merge; Gauss-Newton
                // each team its own: the rays of a sparse subset are lit at different samples, and
                // the wave's windows are then many more (256^3 room, 12 frames of 25k rays, two lanes
                // per ray: 1018 us, one lane and the wave's windows 1518)
                if (KEEP && !SECOND && (GRID ? __ballot(q.lit) : __ballot(q.lit) & tm.mask)) {
                    if (windows < KEPT) {
                        if (GRID) keep[windows * WAVE] = make_float4(v.sig, v.s[0], v.s[1], v.s[2]);
                        keep_at[windows * WAVE] = q.lit ? (int32_t)oo : -1;
                        ++windows;
                    } else if (!spilled) {
                        spilled = true;
                        resume = o;
                    }
                }
                if (ONE_MARCH && !SECOND && q.lit) {
                    const double delta = (double)op.step_vox, t = (double)s.t;
                    double a[4];
#pragma unroll
                    for (int ch = 0; ch < 3; ++ch) a[ch] = delta * ((double)(q.c[ch] * q.Tn) + q.A[ch]);
                    a[3] = delta * ((double)(s.t * q.Tn) + q.AD);
#pragma unroll
                    for (int x = 0; x < 3; ++x) {
                        const double ds = (double)v.dsig[x];
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            double gk = a[k] * ds;
                            if (k < 3) gk += (double)(act_bwd(op.act, v.s[k < 3 ? k : 0]) * q.wt * v.ds[k < 3 ? k : 0][x]);
                            ps.P[k][x] += gk;
                            ps.Q[k][x] = fma(t, gk, ps.Q[k][x]);
                        }
                        ps.S[x] = fma(delta, ds, ps.S[x]);
                        ps.St[x] = fma(delta * t, ds, ps.St[x]);
                        if (VIEW) {
#pragma unroll
                            for (int k = 0; k < 3; ++k)
                                ps.V[VIEW ? k : 0][x] = fmaf(act_bwd(op.act, v.s[k]) * q.wt, v.ev[k][x], ps.V[VIEW ? k : 0][x]);
                        }
                    }
                }
                if (GAUSS_NEWTON && SECOND) jacobian_window<VIEW>(g, op, tm, ray, s, v, q, Chat, Dhat, ja);
                if (BACKWARD || SCATTER) {
                    float gsig = 0.f, gs[3] = {0.f, 0.f, 0.f}, w[8];
                    if (q.lit) {
                        grid_factors(op, q, v.s, s.t, Chat, Dhat, gC, gDr, gsig, gs);
                        if (POSE_HERE) {
                            const float inv_vs = (float)g.inv_vs;
#pragma unroll
                            for (int a = 0; a < 3; ++a) {
                                const float gp = (gsig * v.dsig[a] + gs[0] * v.ds[0][a] + gs[1] * v.ds[1][a]
                                                  + gs[2] * v.ds[2][a]) * inv_vs;
                                pa.go[a] += gp;
                                pa.gd[a] = fmaf(s.t, gp, pa.gd[a]);
                                if (VIEW) pa.gv[a] += gs[0] * v.ev[0][a] + gs[1] * v.ev[1][a] + gs[2] * v.ev[2][a];
                            }
                        }
                        if (SCATTER) trilinear_weights(s.f, w);
                    }
                    if (SCATTER) scatter_merged<DEG>(q.lit, s.base, idx, w, gsig, gs, Y, wc, io.grad);
                }
            }
            // the ray ends at its last sample, at the box, or at the cap
            if (on) {
                if (last < WAVE) {
                    kept = o + (last - tm.base) + 1;
                    on = false;
                } else if (run < tm.T) {
                    kept = o + run;
                    on = false;
                }
            }
            // past the window, or past the empty block its last position lies in
            const int64_t past = __shfl(nxt, tm.base + tm.T - 1, WAVE);
            o = past > o + tm.T ? past : o + tm.T;
            if (on && o >= lim) {
                kept = lim;
                on = false;
            }
        }
    };
    march(std::integral_constant<bool, false>{}, 0, limit);
    if (!BACKWARD) {
        if (ONE_MARCH) {
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) Chat[ch] = cy.A[ch];
            Dhat = cy.AD;
        } else {
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) Chat[ch] = team_sum(cy.A[ch], tm);
            Dhat = team_sum(cy.AD, tm);
        }
    }
    const float C[3] = {(float)Chat[0], (float)Chat[1], (float)Chat[2]};
    const float z = inr && !BACKWARD ? (float)Dhat / ray.s : 0.f;
    const bool head = inr && tm.sub == 0;
    if (!BACKWARD && head) {
        if (io.rgb) {
            io.rgb[3 * r] = C[0];
            io.rgb[3 * r + 1] = C[1];
            io.rgb[3 * r + 2] = C[2];
        }
        if (io.depth) io.depth[r] = z;
        if (MODE == TEAM_FORWARD) io.nsamp[r] = (int32_t)kept;
    }
    if (MODE == TEAM_FORWARD) return;
    // the loss (Eq. 4, 5, 11); invalid depth drops the ray (Sec. 6.1)
    bool valid = BACKWARD ? wanted : false;
    float e[4] = {0.f, 0.f, 0.f, 0.f}, wf = 0.f;
    if (!BACKWARD && inr) {
        const float Dt = io.tgt_depth[r];
        valid = isfinite(Dt) && Dt > 0.f;
        if (valid) {
            wf = io.fw[f];
            e[0] = C[0] - io.tgt_rgb[3 * r];
            e[1] = C[1] - io.tgt_rgb[3 * r + 1];
            e[2] = C[2] - io.tgt_rgb[3 * r + 2];
            e[3] = z - Dt;
        }
    }
    if (MODE == TEAM_FUSED) {
        double lval = 0.0;
        if (valid) {
            float rho, drho;
            if (op.depth_loss == LOSS_L2) { rho = e[3] * e[3]; drho = 2.f * e[3]; }
            else { rho = fabsf(e[3]); drho = e[3] > 0.f ? 1.f : (e[3] < 0.f ? -1.f : 0.f); }
            lval = (double)wf * ((double)e[0] * e[0] + (double)e[1] * e[1] + (double)e[2] * e[2])
                 + (double)op.lambda_d * wf * rho;
            gC[0] = 2.f * wf * e[0];
            gC[1] = 2.f * wf * e[1];
            gC[2] = 2.f * wf * e[2];
            gDr = op.lambda_d * wf * drho / ray.s;
        }
        if (io.loss) {
            double lv[1] = {lval};
            frame_sum<1>(f, valid && head, lv, io.loss);
        }
    }
    if (KEEP) {
        cy = Carry{0.0, {0.0, 0.0, 0.0}, 0.0, 1.f};
        for (int b = 0; GRID ? b < windows : __ballot(b < windows) != 0; ++b) {
            const int32_t at = GRID || b < windows ? keep_at[b * WAVE] : -1;
            const bool have = valid && at >= 0;
            Sample s;
            s.t = 0.f;
            s.base = 0;
            int idx[8];
            Interp v;
            v.sig = v.s[0] = v.s[1] = v.s[2] = 0.f;
            if (have) {
                sample_at(g, ray, ray.k_first + at, s);
                load_links(g, s.base, idx);
                if (GAUSS_NEWTON) {
                    gather_interp<GAUSS_NEWTON, GAUSS_NEWTON && VIEW, DEG>(g, idx, Y, GY, s.f, v);
                } else {
                    const float4 kv = keep[b * WAVE];
                    v.sig = kv.x;
                    v.s[0] = kv.y;
                    v.s[1] = kv.z;
                    v.s[2] = kv.w;
                }
            }
            Lit q;
            int last;
            composite<true, false>(op, tm, have, v.sig, v.s, s.t, cy, q, last);
            if (GAUSS_NEWTON) {
                jacobian_window<VIEW>(g, op, tm, ray, s, v, q, Chat, Dhat, ja);
            } else {
                float gsig = 0.f, gs[3] = {0.f, 0.f, 0.f}, w[8];
                if (q.lit) {
                    grid_factors(op, q, v.s, s.t, Chat, Dhat, gC, gDr, gsig, gs);
                    trilinear_weights(s.f, w);
                }
                scatter_merged<DEG>(q.lit, s.base, idx, w, gsig, gs, Y, wc, io.grad);
            }
        }
        if (GRID ? spilled : __ballot(spilled) != 0)
            march(std::integral_constant<bool, true>{}, resume, valid && spilled ? kept : 0);
    }
    if (POSE && !GAUSS_NEWTON) {
        if (ONE_MARCH) {
            const double up[4] = {gC[0], gC[1], gC[2], gDr}, hat[4] = {Chat[0], Chat[1], Chat[2], Dhat};
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                double go = 0.0, gd = 0.0;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    go += up[k] * (ps.P[k][a] - hat[k] * ps.S[a]);
                    gd += up[k] * (ps.Q[k][a] - hat[k] * ps.St[a]);
                }
                pa.go[a] = (float)(go * g.inv_vs);
                pa.gd[a] = (float)(gd * g.inv_vs);
                if (VIEW) pa.gv[a] = gC[0] * ps.V[0][a] + gC[1] * ps.V[VIEW ? 1 : 0][a] + gC[2] * ps.V[VIEW ? 2 : 0][a];
            }
        }
        double six[6] = {0, 0, 0, 0, 0, 0};
        if (valid) pose_six<VIEW>(ray, pa, six);
        frame_sum<6>(f, valid, six, io.grad_pose);
    }
    if (GAUSS_NEWTON) {
        double vals[GN_VALUES];
#pragma unroll
        for (int i = 0; i < GN_VALUES; ++i) vals[i] = 0.0;
        if (valid && head) {
            // Jacobian rows J[k] = (g_o, o x g_o + d x g_d (+ d x g_view)), then the ray's
            // terms of the normal equations
            const float* o = ray.o;
            const float* d = ray.d;
            float J[4][6];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float gd[3] = {ja.gd[q][0], ja.gd[q][1], ja.gd[q][2]};
                if (VIEW) { gd[0] += ja.gv[q][0]; gd[1] += ja.gv[q][1]; gd[2] += ja.gv[q][2]; }
                const float* go = ja.go[q];
                J[q][0] = go[0];
                J[q][1] = go[1];
                J[q][2] = go[2];
                J[q][3] = (o[1] * go[2] - o[2] * go[1]) + (d[1] * gd[2] - d[2] * gd[1]);
                J[q][4] = (o[2] * go[0] - o[0] * go[2]) + (d[2] * gd[0] - d[0] * gd[2]);
                J[q][5] = (o[0] * go[1] - o[1] * go[0]) + (d[0] * gd[1] - d[1] * gd[0]);
            }
            const double w1 = (double)wf;
            const double Wk[4] = {w1, w1, w1, w1 * (double)op.lambda_d};
            int q = 0;
#pragma unroll
            for (int i = 0; i < 6; ++i)
#pragma unroll
                for (int j = i; j < 6; ++j) {
                    double acc = 0.0;
#pragma unroll
                    for (int k = 0; k < 4; ++k) acc += Wk[k] * (double)J[k][i] * (double)J[k][j];
                    vals[q++] = acc;
                }
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                double acc = 0.0;
#pragma unroll
                for (int k = 0; k < 4; ++k) acc += Wk[k] * (double)J[k][i] * (double)e[k];
                vals[21 + i] = acc;
            }
            double E = 0.0;
#pragma unroll
            for (int k = 0; k < 4; ++k) E += Wk[k] * (double)e[k] * (double)e[k];
            vals[27] = E;
        }
        frame_sum<GN_VALUES>(f, valid && head, vals, io.gn);
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

template <int MODE, bool GRID, bool POSE, bool VIEW, int DEG>
static void team_go(const KGrid& g, const KRays& rs, const KOpts& op, int log_t, const TeamIO& io, hipStream_t st) {
    const int waves = MODE == TEAM_FORWARD ? 1 : TEAM_WAVES;   // nothing to sum over a workgroup forward
    const unsigned blocks = (unsigned)(((rs.n << log_t) + waves * WAVE - 1) / (waves * WAVE));
    const size_t lds = GRID ? waves * WAVE_LDS_FLOATS * sizeof(float)
                     : MODE == TEAM_GN ? waves * GN_WINDOWS * WAVE * sizeof(int32_t) : 0;
    hipLaunchKernelGGL((k_team<MODE, GRID, POSE, VIEW, DEG>), dim3(blocks), dim3(waves * WAVE), lds, st, g, rs, op, log_t,
                       io);
}

template <int MODE, bool GRID, bool POSE, bool VIEW>
static void team_deg(const KGrid& g, const KRays& rs, const KOpts& op, int log_t, const TeamIO& io, hipStream_t st) {
    if (g.deg == 0) team_go<MODE, GRID, POSE, VIEW, 0>(g, rs, op, log_t, io, st);
    else if (g.deg == 1) team_go<MODE, GRID, POSE, VIEW, 1>(g, rs, op, log_t, io, st);
    else team_go<MODE, GRID, POSE, VIEW, 2>(g, rs, op, log_t, io, st);
}

// Lanes per ray, as a power of two: the widest team whose waves are at most
// about five per SIMD (1024 SIMDs), or, for teams wider than 2^narrow, about
// as many as are resident with the kernel's registers.  A wider team shortens
// a ray's chain of windows; past these limits the waves queue and the windows
// hold more positions without work, so the chain no longer pays for them.
// Measured on the 256^3 room (us; lanes per ray 1, 2, 4, ..., 64; "-" the kernel
// with one lane per ray and the work masks):
//   forward       2,000 rays  -160 | 162  95  64  44  26  19  16
//                19,200 rays  -169 | 171 106  75  59  48  52  63
//               163,200 rays  -175 | 184 166 184
//   pose          2,000 rays  -258 | 239 140  97  63  37  27  22
//                19,200 rays  -273 | 253 152 107  99  85 107 147
//               163,200 rays  -365 | 301 278 359
//               816,000 rays -1154 | 727 926
//   grid          2,000 rays  -828 | 644 333 194 119  58  40  33
//                19,200 rays  -768 | 840 420 278 204 154 163 207
//                83,583 rays  -788 | 802 634 510 531 502
//               362,400 rays  -909 | 1049 971 1099
//   grid + pose   2,000 rays  -855 | 717 380 226 137  66  47  38
//                19,200 rays  -782 | 916 469 301 228 179 194 251
//               163,200 rays  -787 | 1002 781 834
//               816,000 rays -1419 | 1914 2061
// Two lanes for the pose alone stay ahead up to 400,000 rays (PAIRS), with four
// or more lanes' limit as before; fused pose step, us, one lane and two: a frame of
// 360,150 rays of the 256^3 room 964 -> 851, 12 sparse frames of 30k 1111 -> 988; a
// frame of 576,000 989 -> 1071.  (Larger batches leave the teams: launch_backward,
// one_lane_pose.)
// The one-lane kernels stay where they are faster: forward and grid gradients of
// large batches, which this returns 0 for.
int team_lanes_log2(int64_t n_rays, int want) {
    constexpr int64_t PAIRS = 12500, MANY = 5300, RESIDENT = 2700;
    const bool grid = want & 1, pose = want & 2;
    const int narrow = grid ? 4 : pose ? 1 : 6;
    int lt = 0;
    while (lt < 6 && (n_rays << (lt + 1)) <= WAVE * (lt + 1 > narrow ? RESIDENT : grid || !pose ? MANY : PAIRS)) ++lt;
    return lt;
}

hipError_t team_forward(const KGrid& g, const KRays& rs, const KOpts& op, int log_t, float* rgb, float* depth,
                        int32_t* nsamp, hipStream_t st) {
    TeamIO io{};
    io.rgb = rgb;
    io.depth = depth;
    io.nsamp = nsamp;
    team_deg<TEAM_FORWARD, false, false, false>(g, rs, op, log_t, io, st);
    return hipGetLastError();
}

hipError_t team_fused(const KGrid& g, const KRays& rs, const KOpts& op, int log_t, const float* tgt_rgb,
                      const float* tgt_depth, const float* fw, int want, float* rgb, float* depth, double* loss,
                      float* grad, double* grad_pose, hipStream_t st) {
    TeamIO io{};
    io.tgt_rgb = tgt_rgb;
    io.tgt_depth = tgt_depth;
    io.fw = fw;
    io.rgb = rgb;
    io.depth = depth;
    io.loss = loss;
    io.grad = grad;
    io.grad_pose = grad_pose;
    const bool G = want & 1, P = want & 2, V = op.flags & 1;
    if (G && P && V) team_deg<TEAM_FUSED, true, true, true>(g, rs, op, log_t, io, st);
    else if (G && P) team_deg<TEAM_FUSED, true, true, false>(g, rs, op, log_t, io, st);
    else if (G) team_deg<TEAM_FUSED, true, false, false>(g, rs, op, log_t, io, st);
    else if (P && V) team_deg<TEAM_FUSED, false, true, true>(g, rs, op, log_t, io, st);
    else if (P) team_deg<TEAM_FUSED, false, true, false>(g, rs, op, log_t, io, st);
    else team_deg<TEAM_FUSED, false, false, false>(g, rs, op, log_t, io, st);
    return hipGetLastError();
}

hipError_t launch_gn(const KGrid& g, const KRays& rs, const KOpts& op, const float* tgt_rgb, const float* tgt_depth,
                     const float* fw, double* gn, hipStream_t st) {
    // The ordered sums are made for teams of 16, 4, 2 and 1.  Sixteen and four stand while
    // their waves are at most about five per SIMD, two for longer: rays of a sparse
    // subset gain from a shorter chain, those of whole frames little.  256^3 room, us for
    // T = 1, 2, 4, 16 ("-": the kernel before, one lane per ray, both marches through work masks):
    //   whole frames                             sparse frames
    //    172,800 rays      472  387  427          64,000 rays -  801 |  828  488  336  398
    //    307,200 rays      590  570  680         160,000 rays -  830 |  843  554  611  851
    //    600,000 rays      790  854 1151         300,000 rays - 1124 | 1201 1018 1027 1626
    //    816,000 rays -2081 | 975 1114 1509      600,000 rays - 1572 | 1691 1495 1822 3105
    const int log_t = rs.n <= 21200 ? 4 : rs.n <= 84800 ? 2 : rs.n <= 620000 ? 1 : 0;
    TeamIO io{};
    io.tgt_rgb = tgt_rgb;
    io.tgt_depth = tgt_depth;
    io.fw = fw;
    io.gn = gn;
    if (op.flags & 1) team_deg<TEAM_GN, false, true, true>(g, rs, op, log_t, io, st);
    else team_deg<TEAM_GN, false, true, false>(g, rs, op, log_t, io, st);
    return hipGetLastError();
}

hipError_t team_backward(const KGrid& g, const KRays& rs, const KOpts& op, int log_t, const float* rgb,
                         const float* depth, const int32_t* nsamp, const float* g_rgb, const float* g_depth,
                         float* grad, double* grad_pose, hipStream_t st) {
    TeamIO io{};
    io.rgb_in = rgb;
    io.depth_in = depth;
    io.nsamp_in = nsamp;
    io.g_rgb = g_rgb;
    io.g_depth = g_depth;
    io.grad = grad;
    io.grad_pose = grad_pose;
    if (grad) team_deg<TEAM_BACKWARD, true, false, false>(g, rs, op, log_t, io, st);
    else if (op.flags & 1) team_deg<TEAM_BACKWARD, false, true, true>(g, rs, op, log_t, io, st);
    else team_deg<TEAM_BACKWARD, false, true, false>(g, rs, op, log_t, io, st);
    return hipGetLastError();
}

}  // namespace pxm
