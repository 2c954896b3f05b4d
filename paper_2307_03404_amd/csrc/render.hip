// Forward, backward and fused kernels of the sparse-voxel volume renderer with
// one lane per ray: the form for batches that fill the card, and of the
// launch tunings 1 and 2 (team.hip holds the others).
//
// One lane per ray.  A wave holds 64 rays of one pixel tile (the ray packer
// orders full frames in 8x8 tiles), so the lanes gather nearly the same
// vertices at the same sample index and share cache lines.
//
// Forward (Eq. 1-3): march the kept sample positions, skip empty bricks and
// cells (exact: they interpolate to zero density) and composite colour and
// range.  Backward (Eq. 6-14): replay exactly the
// forward's nsamp positions, re-deriving sigma, c, w and T_{i+1} (nothing is
// stored per sample), and scatter or reduce the gradients.
#include <atomic>
#include <type_traits>

#include "internal.hpp"
#include "scatter.hpp"

namespace pxm {

struct FwdResult {
    float C[3];
    float D;            // expected range (world units), Eq. 3
    double Cd[3];       // the same sums in FP64, for the backward of the same kernel
    double Dd;
    int n;              // kept sample positions
    int mark_last;      // last word of the work-position mask written
    bool mark_overflow; // a work position lay beyond the mask
    long long occ;      // samples in cells with an allocated corner
    long long occ_corners;
    long long grad_corners;   // allocated corners of samples with sigma_raw > 0
};

// Forward march of one ray (Eq. 1-3).  With the occupancy bitfield, samples
// in empty bricks are stepped over in one jump and empty cells cost one bit
// test; both are exact (such samples interpolate to zero density) and still
// count as kept positions.
//
// With a non-null `marks` the march also records, for the backward of the
// same kernel, which of its positions carry light (the only ones the backward
// has work at): bit o of the lane's mask is set for
// position k_first + o, in words marks[w * WAVE] (w < MARK_WORDS) written
// in order from a register; out.mark_last is the last word written and
// out.mark_overflow is set if a marked position lay beyond the mask.
template <int DEG>
__device__ __forceinline__ void ray_forward(const KGrid& g, const KOpts& op, const Ray& ray,
                                            const float Y[9], FwdResult& out,
                                            uint32_t* marks = nullptr, int64_t mstride = WAVE) {
    // colour and range are summed in FP64: the backward differences them
    // with its own prefix sums (Eq. 9, 10), and in FP32 that difference
    // would carry rounding that grows with the number of samples
    double C0 = 0.0, C1 = 0.0, C2 = 0.0, D = 0.0;
    float T = 1.f;
    double L = 0.0;
    int n = 0;
    long long occ = 0, occc = 0, gradc = 0;
    int mw = 0;                     // current mark word
    uint32_t mbits = 0;
    bool movf = false;
    if (!ray.empty) {
        const float delta = op.step_vox;
        int64_t k = ray.k_first;
        OccCache oc;
        occ_cache_init(oc);
        int lit_run = 0;                // samples with light since the last one without
        while (n < op.max_samples) {
            Sample s;
            if (!sample_at(g, ray, k, s)) break;
            if (g.occ0) {
                int64_t nxt;
                const int cls = occ_classify(g, ray, k, s.c, oc, nxt);
                if (cls == OCC_JUMP) {
                    if (nxt - k >= (int64_t)(op.max_samples - n)) {
                        n = op.max_samples;
                        break;
                    }
                    n += (int)(nxt - k);
                    k = nxt;
                    continue;
                }
                if (cls == OCC_EMPTY_CELL) {
                    ++n;
                    ++k;
                    continue;
                }
            }
            ++n;
            ++k;
            int idx[8];
            const int na = load_links(g, s.base, idx);
            if (na == 0) continue;
            ++occ;
            occc += na;
            if (g.probe && __ballot(lit_run < LIT_RUN) && !(gather_density<DEG>(g, idx, s.f) > 0.f)) {
                lit_run = 0;
                continue;
            }
            Interp v;
            gather_interp<false, false, DEG>(g, idx, Y, nullptr, s.f, v);
            const float sr = v.sig, s0 = v.s[0], s1 = v.s[1], s2 = v.s[2];
            if (!(sr > 0.f)) {
                lit_run = 0;
                continue;
            }
            ++lit_run;
            gradc += na;
            if (marks) {
                const int64_t o = k - 1 - ray.k_first;
                if (o >= (int64_t)MARK_WORDS * 32) {
                    movf = true;
                } else {
                    const int w = (int)(o >> 5);
                    while (mw < w) {
                        marks[mw * mstride] = mbits;
                        mbits = 0u;
                        ++mw;
                    }
                    mbits |= 1u << (int)(o & 31);
                }
            }
            const float x = sr * delta;
            const float wt = T * (-expm1f(-x));
            C0 = fma((double)wt, (double)act_fwd(op.act, s0), C0);
            C1 = fma((double)wt, (double)act_fwd(op.act, s1), C1);
            C2 = fma((double)wt, (double)act_fwd(op.act, s2), C2);
            D = fma((double)wt, (double)s.t, D);
            L += (double)x;
            T = trans_of(L);
            if (T < op.t_stop) break;
        }
    }
    if (marks) marks[mw * mstride] = mbits;
    out.mark_last = mw;
    out.mark_overflow = movf;
    out.Cd[0] = C0; out.Cd[1] = C1; out.Cd[2] = C2;
    out.Dd = D;
    out.C[0] = (float)C0; out.C[1] = (float)C1; out.C[2] = (float)C2;
    out.D = (float)D;
    out.n = n;
    out.occ = occ;
    out.occ_corners = occc;
    out.grad_corners = gradc;
}

// Running state of a backward march.
struct BwdState {
    double A[3];        // sum_{j<=i} c_j w_j
    double AD;          // sum_{j<=i} t_j w_j
    float T;            // T_i
    double L;           // sum_{j<i} sigma_j delta
    int lit_run;        // samples with light since the last one without
};

// Backward work of one occupied sample (Eq. 6-14): updates the running state
// and the pose accumulators; returns true with the sample's grid-gradient
// factors (gsig = dL/d sigma_raw, gs = dL/ds_c) when it carries light.  PROBE:
// the position is not known to carry light.
template <bool POSE, bool VIEW, int DEG, bool PROBE>
__device__ __forceinline__ bool backward_sample(const KGrid& g, const KOpts& op, const Ray& ray,
                                                const float Y[9], const float GY[9][3],
                                                const Sample& s, const double Chat[3], double Dhat,
                                                const float gC[3], float gDr, BwdState& st,
                                                PoseAcc& pa, int idx[8], float w[8], float& gsig,
                                                float gs[3]) {
    if (load_links(g, s.base, idx) == 0) return false;
    if (PROBE && g.probe && __ballot(st.lit_run < LIT_RUN) && !(gather_density<DEG>(g, idx, s.f) > 0.f)) {
        st.lit_run = 0;
        return false;
    }
    Interp v;
    gather_interp<POSE, POSE && VIEW, DEG>(g, idx, Y, GY, s.f, v);
    trilinear_weights(s.f, w);
    const float sr = v.sig;
    if (PROBE) st.lit_run = sr > 0.f ? st.lit_run + 1 : 0;
    if (!(sr > 0.f)) return false;      // sigma = 0: no light, zero gradient (ReLU)
    const float delta = op.step_vox;
    const float x = sr * delta;
    const float wt = st.T * (-expm1f(-x));
    st.L += (double)x;
    const float Tn = trans_of(st.L);
    float c[3];
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
        c[ch] = act_fwd(op.act, v.s[ch]);
        gs[ch] = act_bwd(op.act, v.s[ch]) * wt * gC[ch];      // Eq. 8 through act
        st.A[ch] = fma((double)wt, (double)c[ch], st.A[ch]);
    }
    st.AD = fma((double)wt, (double)s.t, st.AD);
    // Eq. 9 and Eq. 10 with inclusive prefixes A = sum_{j<=i} c_j w_j; the
    // suffix A - C-hat is formed in FP64
    gsig = delta * (gC[0] * (c[0] * Tn + (float)(st.A[0] - Chat[0]))
                  + gC[1] * (c[1] * Tn + (float)(st.A[1] - Chat[1]))
                  + gC[2] * (c[2] * Tn + (float)(st.A[2] - Chat[2]))
                  + gDr * (s.t * Tn + (float)(st.AD - Dhat)));
    if (POSE) {
        // Appendix A: the spatial gradient of the interpolant, dL/dp =
        // gsig grad(sigma) + sum_c gs_c grad(s_c), in world units
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
    st.T = Tn;
    return true;
}

// Minimum over the 64 lanes (every lane active), returned to all of them.
// Data-parallel-primitive moves within rows of 16 lanes (shift right by 1,
// 2, 4, 8), then the last lane of each row broadcast into the next rows,
// leave the wave's minimum in lane 63; a lane with no source lane reads the
// identity INT64_MAX.  No LDS round trip, unlike a butterfly of shuffles.
__device__ __forceinline__ int64_t wave_min(int64_t v) {
    constexpr int ID_LO = -1, ID_HI = 0x7fffffff;            // INT64_MAX
    auto step = [&](auto ctrl, auto row_mask) {
        const int lo = __builtin_amdgcn_update_dpp(ID_LO, (int)(uint32_t)v, decltype(ctrl)::value,
                                                   decltype(row_mask)::value, 0xf, false);
        const int hi = __builtin_amdgcn_update_dpp(ID_HI, (int)((uint64_t)v >> 32), decltype(ctrl)::value,
                                                   decltype(row_mask)::value, 0xf, false);
        const int64_t o = (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
        v = o < v ? o : v;
    };
    using std::integral_constant;
    step(integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});   // row_shr:1
    step(integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});   // row_shr:2
    step(integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});   // row_shr:4
    step(integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});   // row_shr:8
    step(integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});   // row_bcast:15 -> rows 1, 3
    step(integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});   // row_bcast:31 -> rows 2, 3
    const int lo = __builtin_amdgcn_readlane((int)(uint32_t)v, 63);
    const int hi = __builtin_amdgcn_readlane((int)((uint64_t)v >> 32), 63);
    return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// The smallest marked position offset >= o in a lane's work mask (words
// marks[w * WAVE], w <= last), or -1.
__device__ __forceinline__ int next_mark(const uint32_t* marks, int last, int o) {
    int w = o >> 5;
    if (w > last) return -1;
    uint32_t b = marks[w * WAVE] & (0xffffffffu << (o & 31));
    while (b == 0u) {
        if (++w > last) return -1;
        b = marks[w * WAVE];
    }
    return w * 32 + __ffs(b) - 1;
}

// Which lanes of a wave take part in a step of the grid backward.  The wave
// stands at its lanes' smallest pending sample index, and as a rule the lanes
// at that index work (neighbouring rays then share cells, and a cell's
// gradient is added once for all of them).  Rays of a sparse pixel subset share
// few cells, and their samples lie at so many indices that a step finds a
// handful of lanes: the steps then number the union of the lanes' indices.  So
// each wave counts what its steps have merged, and once that is less than half
// (MERGED_FEW) of what could have been, a step that holds less than half of the
// pending lanes (FIRST_FEW) takes all of them instead, each at its own next
// index.  512^3 room, 16 frames of 30k rays each: fused step 4.58 -> 3.62 ms,
// backward alone 4.98 -> 4.27.  Always taking all is slower where rays do share
// cells (8 frames of 50k rays of the 256^3 room 2.91 ms in step, 3.19 always
// all, 2.81 by this rule; 8 full frames of the 512^3 room 17.4, 18.4, 17.4);
// rules of a quarter and an eighth merged give up part of the gain (4.03, 4.19).
// The fixed-point scatter keeps to the common index: its rounding, and so its
// bits, follow what is merged.
constexpr int MERGED_FEW = 2, FIRST_FEW = 2;
constexpr int MERGE_EVIDENCE = 16;                          // lanes that could have merged before it counts

// The wave's next index after k: nothing pending is below k + 1, where as a rule
// some lane stands; the reduction is for the others (backward of a 1200 x 680
// frame of the 256^3 room 841 -> 822 us, of 8 frames of the 512^3 room 14.7 ->
// 14.3 ms).
__device__ __forceinline__ int64_t next_step(int64_t k, int64_t mine) {
    return __ballot(mine == k + 1) ? k + 1 : wave_min(mine);
}

struct StepRule {
    int could = 0, did = 0;                                 // lanes beyond each step's first; of them merged

    __device__ __forceinline__ bool takes_part(bool pending, bool first) const {
        const bool apart = could >= MERGE_EVIDENCE && did * MERGED_FEW < could;
        if (!apart || (int)__popcll(__ballot(first)) * FIRST_FEW >= (int)__popcll(__ballot(pending))) return first;
        return pending;
    }

    __device__ __forceinline__ void count(bool have, int cells) {
        const int n = (int)__popcll(__ballot(have));
        if (n) {
            could += n - 1;
            did += n - cells;
        }
    }
};

// Backward march of one ray over its first n kept positions (Eq. 6-14).
//   Chat, Dhat: the forward's colour and expected range
//   gC, gDr:    dL/dC-hat and dL/d(range)
// With GRID the lanes of a wave work together in steps (StepRule), so that the
// scatters of rays that share cells merge: every lane must call this (lanes
// without a ray pass n = 0).  Each lane looks up its own next work position; a
// common walk over the indices at which any lane has one took 987 us where this
// takes 822 (backward of a 1200 x 680 frame of the 256^3 room).  Without GRID
// every lane marches on its own.
template <bool GRID, bool POSE, bool VIEW, int DEG, bool FIX = false>
__device__ __forceinline__ void ray_backward(const KGrid& g, const KOpts& op, const Ray& ray,
                                             const float Y[9], int n, const double Chat[3],
                                             double Dhat, const float gC[3], float gDr,
                                             float* __restrict__ grad, const WaveStage& wc,
                                             PoseAcc& pa, const uint32_t* marks = nullptr,
                                             int mark_last = 0, bool mark_overflow = true) {
    float GY[9][3];
    if (VIEW) sh9_grad(ray.d[0], ray.d[1], ray.d[2], GY);
    BwdState st = {{0.0, 0.0, 0.0}, 0.0, 1.f, 0.0, 0};
    const int64_t ks = ray.k_first, ke = ray.k_first + (n > 0 ? n : 0);
    bool has = n > 0;
    StepRule rule;
    if (GRID && marks && __ballot(mark_overflow && n > 0) == 0) {
        // the forward of this kernel marked every work position: visit only those
        int off = has ? next_mark(marks, mark_last, 0) : -1;
        int64_t mine = off >= 0 ? ks + off : INT64_MAX;
        for (int64_t k = wave_min(mine); k != INT64_MAX; k = next_step(k, mine)) {
            const bool pending = off >= 0;
            const bool work = FIX ? mine == k : rule.takes_part(pending, mine == k);
            bool have = false;
            int idx[8];
            float w[8];
            float gsig = 0.f, gs[3] = {0.f, 0.f, 0.f};
            Sample s;
            if (work && sample_at(g, ray, mine, s))
                have = backward_sample<POSE, VIEW, DEG, false>(g, op, ray, Y, GY, s, Chat, Dhat, gC, gDr, st,
                                                   pa, idx, w, gsig, gs);
            rule.count(have, scatter_merged<DEG, FIX>(have, s.base, idx, w, gsig, gs, Y, wc, grad));
            if (work) {
                off = next_mark(marks, mark_last, off + 1);
                mine = off >= 0 ? ks + off : INT64_MAX;
            }
        }
    } else if (GRID) {
        // each lane looks up its own next position in an occupied cell
        int64_t pos = ks;
        Sample s;
        OccCache oc;
        occ_cache_init(oc);
        auto seek = [&]() {
            while (pos < ke) {
                if (!sample_at(g, ray, pos, s)) return false;   // left the box: nothing further on this ray
                if (!g.occ0) return true;
                int64_t nxt;
                const int cls = occ_classify(g, ray, pos, s.c, oc, nxt);
                if (cls == OCC_CELL) return true;
                pos = cls == OCC_JUMP ? (nxt < ke ? nxt : ke) : pos + 1;
            }
            return false;
        };
        int64_t mine = has && seek() ? pos : INT64_MAX;
        for (int64_t k = wave_min(mine); k != INT64_MAX; k = next_step(k, mine)) {
            const bool pending = mine != INT64_MAX;
            const bool first = mine == k;
            const bool work = FIX ? first : rule.takes_part(pending, first);
            bool have = false;
            int idx[8];
            float w[8];
            float gsig = 0.f, gs[3] = {0.f, 0.f, 0.f};
            if (work)
                have = backward_sample<POSE, VIEW, DEG, true>(g, op, ray, Y, GY, s, Chat, Dhat, gC, gDr, st,
                                                   pa, idx, w, gsig, gs);
            rule.count(have, scatter_merged<DEG, FIX>(have, s.base, idx, w, gsig, gs, Y, wc, grad));
            if (work) {
                ++pos;
                mine = seek() ? pos : INT64_MAX;
            }
        }
    } else if (marks && !mark_overflow) {
        // per lane: straight from one marked position to the next
        for (int off = has ? next_mark(marks, mark_last, 0) : -1; off >= 0;
             off = next_mark(marks, mark_last, off + 1)) {
            Sample s;
            if (!sample_at(g, ray, ks + off, s)) break;
            int idx[8];
            float w[8];
            float gsig, gs[3];
            backward_sample<POSE, VIEW, DEG, false>(g, op, ray, Y, GY, s, Chat, Dhat, gC, gDr, st, pa, idx, w,
                                        gsig, gs);
        }
    } else {
        int64_t k = ks;
        OccCache oc;
        occ_cache_init(oc);
        while (k < ke) {
            Sample s;
            if (!sample_at(g, ray, k, s)) break;
            if (g.occ0) {
                int64_t nxt;
                const int cls = occ_classify(g, ray, k, s.c, oc, nxt);
                if (cls == OCC_JUMP) {
                    k = nxt < ke ? nxt : ke;
                    continue;
                }
                if (cls == OCC_EMPTY_CELL) {
                    ++k;
                    continue;
                }
            }
            int idx[8];
            float w[8];
            float gsig, gs[3];
            backward_sample<POSE, VIEW, DEG, true>(g, op, ray, Y, GY, s, Chat, Dhat, gC, gDr, st, pa, idx, w,
                                        gsig, gs);
            ++k;
        }
    }
}

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------

// Rays per workgroup of the forward kernel: one wave, which leaves its registers
// as soon as its own rays end (64 sparse frames of the 512^3 room 7.15 ms with
// four waves, 6.56 with one; the 1200x680 room frame 370 -> 351 us).
constexpr int FORWARD_RAYS = WAVE;

template <int DEG>
__global__ void __launch_bounds__(FORWARD_RAYS) k_forward(KGrid g, KRays rs, KOpts op, float* __restrict__ rgb,
                                                 float* __restrict__ depth, int32_t* __restrict__ nsamp) {
    const int64_t r = ray_tile(blockIdx.x, gridDim.x) * FORWARD_RAYS + threadIdx.x;
    if (r >= rs.n) return;
    const int f = frame_of(rs.off, rs.F, r);
    Ray ray;
    setup_ray(g, rs, op, r, f, ray);
    float Y[9];
    sh9(ray.d[0], ray.d[1], ray.d[2], Y);
    FwdResult fr;
    ray_forward<DEG>(g, op, ray, Y, fr);
    rgb[3 * r] = fr.C[0];
    rgb[3 * r + 1] = fr.C[1];
    rgb[3 * r + 2] = fr.C[2];
    depth[r] = fr.D / ray.s;
    nsamp[r] = fr.n;
}

// What the backward passes know of a ray: its upstream gradients, and the forward's outputs.
struct BackwardRay {
    Ray ray;
    float Y[9], gC[3], gDr;
    double Chat[3], Dhat;
    int f, n;           // frame, positions to replay
    bool active;        // has an upstream gradient
};

__device__ __forceinline__ void backward_ray(const KGrid& g, const KRays& rs, const KOpts& op, int64_t r,
                                             const float* __restrict__ rgb, const float* __restrict__ depth,
                                             const int32_t* __restrict__ nsamp, const float* __restrict__ g_rgb,
                                             const float* __restrict__ g_depth, BackwardRay& b) {
#pragma unroll
    for (int k = 0; k < 9; ++k) b.Y[k] = 0.f;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        b.gC[c] = 0.f;
        b.Chat[c] = 0.0;
    }
    b.gDr = 0.f;
    b.Dhat = 0.0;
    b.f = b.n = 0;
    b.ray.empty = true;
    b.active = r < rs.n;
    if (!b.active) return;
    b.gC[0] = g_rgb[3 * r];
    b.gC[1] = g_rgb[3 * r + 1];
    b.gC[2] = g_rgb[3 * r + 2];
    const float gD = g_depth[r];
    b.active = b.gC[0] != 0.f || b.gC[1] != 0.f || b.gC[2] != 0.f || gD != 0.f;
    if (!b.active) return;
    b.f = frame_of(rs.off, rs.F, r);
    setup_ray(g, rs, op, r, b.f, b.ray);
    sh9(b.ray.d[0], b.ray.d[1], b.ray.d[2], b.Y);
    b.Chat[0] = rgb[3 * r];
    b.Chat[1] = rgb[3 * r + 1];
    b.Chat[2] = rgb[3 * r + 2];
    b.Dhat = (double)depth[r] * (double)b.ray.s;
    b.gDr = gD / b.ray.s;
    b.n = b.ray.empty ? 0 : nsamp[r];
}

// It keeps no work masks, so its LDS (the staging alone) holds 13 waves on a CU,
// and its 137 registers (of 168 there) 3 on a SIMD.  With the mask region allocated, and so 2,
// the backward of a 1200 x 680 frame of the 256^3 room took 827 us and takes 762,
// of 8 frames of the 512^3 room 14.2 and 11.7 ms, of a frame of the 32^3 map 467
// and 372 us.
template <int DEG>
__global__ void __launch_bounds__(WAVE) __attribute__((amdgpu_waves_per_eu(3, 3))) k_backward(KGrid g, KRays rs, KOpts op,
                                                  const float* __restrict__ rgb,
                                                  const float* __restrict__ depth,
                                                  const int32_t* __restrict__ nsamp,
                                                  const float* __restrict__ g_rgb,
                                                  const float* __restrict__ g_depth,
                                                  float* __restrict__ grad) {
    extern __shared__ __align__(16) float smem[];
    const WaveStage wc = wave_stage(smem, grad, (uint64_t)g.n_alloc * (RecL<DEG>::S * sizeof(float)));
    BackwardRay b;
    backward_ray(g, rs, op, ray_tile(blockIdx.x, gridDim.x) * WAVE + threadIdx.x, rgb, depth, nsamp, g_rgb, g_depth, b);
    PoseAcc pa = {{0.f, 0.f, 0.f}, {0.f, 0.f, 0.f}, {0.f, 0.f, 0.f}};
    ray_backward<true, false, false, DEG>(g, op, b.ray, b.Y, b.n, b.Chat, b.Dhat, b.gC, b.gDr, grad, wc, pa);
}

// The pose gradient of batches above POSE_BACKWARD_ONE rays: one lane per ray, one
// wave per workgroup.  Bound by the latency of its gathers at 2 to 3 waves per SIMD.
// us of this kernel and of the better of two and four lanes per ray: 160,000 sparse
// rays of the 256^3 room 602 and 380, 300,000 713 and 660, 600,000 894 and 961 (with
// the view term 1166 and 1270); frames of 307,200 rays 314 and 365, of 816,000 469 and
// 629 (564 with one lane in a team); 300,000 rays of the 32^3 map 253 and 320, of a
// fog in it 783 and 858.
constexpr int64_t POSE_BACKWARD_ONE = 220000;

template <bool VIEW, int DEG>
__global__ void __launch_bounds__(WAVE) k_backward_pose(KGrid g, KRays rs, KOpts op, const float* __restrict__ rgb,
                                                        const float* __restrict__ depth,
                                                        const int32_t* __restrict__ nsamp,
                                                        const float* __restrict__ g_rgb,
                                                        const float* __restrict__ g_depth,
                                                        double* __restrict__ grad_pose) {
    BackwardRay b;
    backward_ray(g, rs, op, ray_tile(blockIdx.x, gridDim.x) * WAVE + threadIdx.x, rgb, depth, nsamp, g_rgb, g_depth, b);
    PoseAcc pa = {{0.f, 0.f, 0.f}, {0.f, 0.f, 0.f}, {0.f, 0.f, 0.f}};
    const WaveStage none{};
    ray_backward<false, true, VIEW, DEG>(g, op, b.ray, b.Y, b.n, b.Chat, b.Dhat, b.gC, b.gDr, nullptr, none, pa);
    double six[6] = {0, 0, 0, 0, 0, 0};
    if (b.active) pose_six<VIEW>(b.ray, pa, six);
    frame_sum<6>(b.f, b.active, six, grad_pose);
}

// Fused step, in one launch (PH 0) or split in two (PH 1: forward and loss,
// PH 2: backward).  The forward launch needs no LDS and few registers, so it
// runs at the occupancy of a forward-only kernel; it leaves each ray's work
// mask and backward inputs in `sp`, from which the backward launch resumes.
template <bool GRID, bool POSE, bool VIEW, int PH, int DEG, bool FIX>
__global__ void __launch_bounds__(256, (PH == 1 ? 4 : 1)) k_fused(KGrid g, KRays rs, KOpts op,
                                               const float* __restrict__ tgt_rgb,
                                               const float* __restrict__ tgt_depth,
                                               const float* __restrict__ fw,
                                               float* __restrict__ rgb_out,
                                               float* __restrict__ depth_out,
                                               double* __restrict__ loss,
                                               float* __restrict__ grad,
                                               double* __restrict__ grad_pose,
                                               int64_t* __restrict__ stats,
                                               unsigned* __restrict__ ws, int persistent,
                                               KSplit sp) {
    __shared__ int64_t s_tile;
    extern __shared__ __align__(16) float smem[];
    WaveStage wc{};
    if (GRID && PH != 1) {
        wc = wave_stage(smem, grad, (uint64_t)g.n_alloc * (RecL<DEG>::S * sizeof(float)));
        wc.gfix = sp.gfix;
    }
    const int64_t n_tiles = (rs.n + blockDim.x - 1) / blockDim.x;
    // Persistent form: workgroups take tiles in order from one queue counter
    // (ws[0]), so the tiles in flight at any time are neighbours in the
    // image and gather from one compact region of the grid.
    for (;;) {
        int64_t tile;
        if (persistent) {
            if (threadIdx.x == 0) s_tile = (int64_t)atomicAdd(ws, 1u);
            __syncthreads();
            tile = s_tile;
            __syncthreads();
            if (tile >= n_tiles) break;
        } else {
            tile = ray_tile(blockIdx.x, gridDim.x);
        }
        const int64_t r = tile * blockDim.x + threadIdx.x;
        const bool inr = r < rs.n;
        int f = 0;
        Ray ray;
        ray.empty = true;
        FwdResult fr;
        bool valid = false;
        double lval = 0.0;
        PoseAcc pa = {{0.f, 0.f, 0.f}, {0.f, 0.f, 0.f}, {0.f, 0.f, 0.f}};
        float Y[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        float gC[3] = {0.f, 0.f, 0.f};
        float gDr = 0.f;
        int nb = 0;
        fr.mark_last = 0;
        fr.mark_overflow = false;
        uint32_t* marks = PH == 1 ? ((GRID || POSE) && inr ? sp.marks + r : nullptr)
                        : GRID ? wc.marks + lane_id()
                        : POSE ? reinterpret_cast<uint32_t*>(smem) + (threadIdx.x / WAVE) * (MARK_WORDS * WAVE)
                                     + lane_id()
                               : nullptr;
        if (PH == 2) {
            // resume from the forward launch: backward inputs and work mask
            if (inr) {
                f = frame_of(rs.off, rs.F, r);
                setup_ray(g, rs, op, r, f, ray);
                sh9(ray.d[0], ray.d[1], ray.d[2], Y);
                const float Dt = tgt_depth[r];
                valid = isfinite(Dt) && Dt > 0.f;
                nb = sp.nb[r];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    fr.Cd[c] = sp.sums[c * sp.n_pad + r];
                    gC[c] = sp.up[c * sp.n_pad + r];
                }
                fr.Dd = sp.sums[3 * sp.n_pad + r];
                gDr = sp.up[3 * sp.n_pad + r];
                const int mi = sp.minfo[r];
                fr.mark_last = mi & 0xff;
                fr.mark_overflow = (mi >> 8) != 0;
                if (marks && !fr.mark_overflow)
                    for (int w = 0; w <= fr.mark_last; ++w) marks[w * WAVE] = sp.marks[w * sp.n_pad + r];
            } else {
                fr.Cd[0] = fr.Cd[1] = fr.Cd[2] = fr.Dd = 0.0;
            }
        } else if (inr) {
            f = frame_of(rs.off, rs.F, r);
            setup_ray(g, rs, op, r, f, ray);
            sh9(ray.d[0], ray.d[1], ray.d[2], Y);
            ray_forward<DEG>(g, op, ray, Y, fr, marks, PH == 1 ? sp.n_pad : (int64_t)WAVE);
            const float z = fr.D / ray.s;
            if (rgb_out) {
                rgb_out[3 * r] = fr.C[0];
                rgb_out[3 * r + 1] = fr.C[1];
                rgb_out[3 * r + 2] = fr.C[2];
            }
            if (depth_out) depth_out[r] = z;
            // Eq. 4, 5, 11; invalid depth drops the ray (Sec. 6.1)
            const float Dt = tgt_depth[r];
            valid = isfinite(Dt) && Dt > 0.f;
            if (valid) {
                const float wf = fw[f];
                const float e0 = fr.C[0] - tgt_rgb[3 * r];
                const float e1 = fr.C[1] - tgt_rgb[3 * r + 1];
                const float e2 = fr.C[2] - tgt_rgb[3 * r + 2];
                const float ed = z - Dt;
                float rho, drho;
                if (op.depth_loss == LOSS_L2) { rho = ed * ed; drho = 2.f * ed; }
                else { rho = fabsf(ed); drho = ed > 0.f ? 1.f : (ed < 0.f ? -1.f : 0.f); }
                lval = (double)wf * ((double)e0 * e0 + (double)e1 * e1 + (double)e2 * e2)
                     + (double)op.lambda_d * wf * rho;
                gC[0] = 2.f * wf * e0;
                gC[1] = 2.f * wf * e1;
                gC[2] = 2.f * wf * e2;
                gDr = op.lambda_d * wf * drho / ray.s;
                nb = fr.n;
            }
            if (PH == 1) {
                // hand the backward inputs to the backward launch
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    sp.sums[c * sp.n_pad + r] = fr.Cd[c];
                    sp.up[c * sp.n_pad + r] = gC[c];
                }
                sp.sums[3 * sp.n_pad + r] = fr.Dd;
                sp.up[3 * sp.n_pad + r] = gDr;
                sp.nb[r] = nb;
                sp.minfo[r] = fr.mark_last | (fr.mark_overflow ? 0x100 : 0);
            }
        } else {
            fr.C[0] = fr.C[1] = fr.C[2] = fr.D = 0.f;
            fr.Cd[0] = fr.Cd[1] = fr.Cd[2] = fr.Dd = 0.0;
        }
        if ((GRID || POSE) && PH != 1)
            ray_backward<GRID, POSE, VIEW, DEG, FIX>(g, op, ray, Y, nb, fr.Cd, fr.Dd, gC, gDr, grad, wc, pa, marks,
                                           fr.mark_last, fr.mark_overflow);
        if (loss && PH != 2) {
            double lv[1] = {lval};
            if (!GRID && POSE && PH == 0 && !persistent) frame_sum<1>(f, valid, lv, loss);
            else seg_sum_atomic<1>(f, valid, lv, loss);
        }
        if (POSE && PH != 1) {
            double six[6] = {0, 0, 0, 0, 0, 0};
            if (valid) pose_six<VIEW>(ray, pa, six);
            if (!GRID && PH == 0 && !persistent) frame_sum<6>(f, valid, six, grad_pose);
            else seg_sum_atomic<6>(f, valid, six, grad_pose);
        }
        if (stats && PH != 2) {
            long long sv[4] = {inr ? fr.occ : 0, inr ? fr.occ_corners : 0,
                               valid ? fr.grad_corners : 0, valid ? 1 : 0};
            add_stats(inr, sv, stats);
        }
        if (!persistent) break;
    }
    if (persistent && threadIdx.x == 0) {
        // the last workgroup to finish re-arms the queue for the next launch
        __threadfence();
        const unsigned prev = atomicAdd(ws + 1, 1u);
        if (prev == gridDim.x - 1) {
            atomicExch(ws, 0u);
            atomicExch(ws + 1, 0u);
        }
    }
}

// Deterministic scatter, last step: grad += fixed-point sum x 2^-FIX_SHIFT
// (one conversion of an exact integer sum), and the buffer is zeroed for the
// next call.  Padding fields of a record are left alone.
__global__ void __launch_bounds__(256) k_fix_finalize(unsigned long long* __restrict__ gfix,
                                                      float* __restrict__ grad, int64_t n, int S,
                                                      int used) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const long long v = (long long)gfix[i];
        if (v != 0 && (int)(i % S) < used) grad[i] += (float)((double)v / FIX_SCALE);
        gfix[i] = 0ull;
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

static inline unsigned blocks_for(int64_t n, int block) {
    return (unsigned)((n + block - 1) / block);
}

// Calls f(std::integral_constant<int, DEG>) for the grid's SH degree.
template <class F>
static void by_degree(int deg, F&& f) {
    if (deg == 0) f(std::integral_constant<int, 0>{});
    else if (deg == 1) f(std::integral_constant<int, 1>{});
    else f(std::integral_constant<int, 2>{});
}

hipError_t launch_forward(const KGrid& g, const KRays& rs, const KOpts& op, float* rgb,
                          float* depth, int32_t* nsamp, hipStream_t st) {
    const int lt = team_lanes_log2(rs.n, 0);
    if (lt > 0) return team_forward(g, rs, op, lt, rgb, depth, nsamp, st);
    by_degree(g.deg, [&](auto D) {
        hipLaunchKernelGGL(k_forward<decltype(D)::value>, dim3(blocks_for(rs.n, FORWARD_RAYS)), dim3(FORWARD_RAYS),
                           0, st, g, rs, op, rgb, depth, nsamp);
    });
    return hipGetLastError();
}

hipError_t launch_backward(const KGrid& g, const KRays& rs, const KOpts& op, const float* rgb,
                           const float* depth, const int32_t* nsamp, const float* g_rgb,
                           const float* g_depth, float* grad_data, double* grad_pose,
                           hipStream_t st) {
    if (!((grad_data != nullptr) ^ (grad_pose != nullptr))) return hipErrorInvalidValue;
    if (grad_pose && rs.n > POSE_BACKWARD_ONE) {
        by_degree(g.deg, [&](auto D) {
            constexpr int DEG = decltype(D)::value;
            auto go = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, dim3(blocks_for(rs.n, WAVE)), dim3(WAVE), 0, st, g, rs, op, rgb, depth, nsamp, g_rgb,
                                   g_depth, grad_pose);
            };
            (op.flags & 1) ? go(k_backward_pose<true, DEG>) : go(k_backward_pose<false, DEG>);
        });
        return hipGetLastError();
    }
    const int lt = team_lanes_log2(rs.n, grad_data ? 1 : 2);
    if (lt > 0 || grad_pose)
        return team_backward(g, rs, op, lt, rgb, depth, nsamp, g_rgb, g_depth, grad_data, grad_pose, st);
    by_degree(g.deg, [&](auto D) {
        // one wave per workgroup: each wave stages its MFMA operands in 11.5 KB of LDS
        hipLaunchKernelGGL((k_backward<decltype(D)::value>), dim3(blocks_for(rs.n, WAVE)), dim3(WAVE),
                           STAGE_LDS_FLOATS * sizeof(float), st, g, rs, op, rgb, depth, nsamp, g_rgb, g_depth, grad_data);
    });
    return hipGetLastError();
}

static size_t device_lds() {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 65536;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess || v <= 0)
        return 65536;
    return (size_t)v;
}

static int device_cus() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 256;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        return 256;
    return cus;
}

// Persistent grid: as many workgroups as the device holds at once (from the
// kernel's register and LDS use), never more than there are tiles.
// The per-CU figure is cached per kernel and block size; concurrent callers
// may both compute it, and they store the same value.
template <bool GRID, bool POSE, bool VIEW, int PH, int DEG, bool FIX>
static unsigned resident_blocks(int block, size_t lds, int64_t tiles) {
    static std::atomic<int> per_cu[4];                    // by block 64/128/256/512, 0 = unknown
    const int slot = block == 64 ? 0 : block == 128 ? 1 : block == 256 ? 2 : 3;
    int n = per_cu[slot].load(std::memory_order_relaxed);
    if (n <= 0) {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_fused<GRID, POSE, VIEW, PH, DEG, FIX>, block,
                                                         lds) != hipSuccess || n <= 0)
            n = 1;
        per_cu[slot].store(n, std::memory_order_relaxed);
    }
    static const int cus = device_cus();
    const int64_t cap = (int64_t)cus * n;
    return (unsigned)(tiles < cap ? tiles : cap);
}

template <bool GRID, bool POSE, bool VIEW, int PH, int DEG, bool FIX>
static void fused_phase(int64_t tiles, dim3 block, hipStream_t st, const KGrid& g, const KRays& rs,
                        const KOpts& op, const float* tgt_rgb, const float* tgt_depth,
                        const float* fw, float* rgb, float* depth, double* loss, float* grad,
                        double* gp, int64_t* stats, unsigned* ws, int persistent, const KSplit& sp) {
    const size_t lds = PH == 1 ? 0
                     : GRID ? (block.x / WAVE) * WAVE_LDS_FLOATS * sizeof(float)
                     : POSE ? (block.x / WAVE) * MARK_WORDS * WAVE * sizeof(uint32_t) : 0;
    const dim3 grid(persistent ? resident_blocks<GRID, POSE, VIEW, PH, DEG, FIX>(block.x, lds, tiles)
                               : (unsigned)tiles);
    hipLaunchKernelGGL((k_fused<GRID, POSE, VIEW, PH, DEG, FIX>), grid, block, lds, st, g, rs, op, tgt_rgb,
                       tgt_depth, fw, rgb, depth, loss, grad, gp, stats, ws, persistent, sp);
}

// variant 0: one workgroup per tile; 1: persistent workgroups on the tile
// queue; 2: a forward launch then a backward launch, both persistent, with
// the per-ray state in the workspace
template <bool GRID, bool POSE, bool VIEW, int DEG, bool FIX>
static void fused_go(int64_t tiles, dim3 block, hipStream_t st, const KGrid& g, const KRays& rs,
                     const KOpts& op, const float* tgt_rgb, const float* tgt_depth,
                     const float* fw, float* rgb, float* depth, double* loss, float* grad,
                     double* gp, int64_t* stats, unsigned* ws, int variant,
                     unsigned long long* gfix) {
    if (variant == 2) {
        KSplit sp = split_state(ws, rs.n);
        sp.gfix = gfix;
        fused_phase<GRID, POSE, VIEW, 1, DEG, false>(tiles, block, st, g, rs, op, tgt_rgb, tgt_depth, fw,
                                                     rgb, depth, loss, grad, gp, stats, ws, 1, sp);
        fused_phase<GRID, POSE, VIEW, 2, DEG, FIX>(tiles, block, st, g, rs, op, tgt_rgb, tgt_depth, fw,
                                                   rgb, depth, loss, grad, gp, stats, ws, 1, sp);
    } else {
        KSplit sp{};
        sp.gfix = gfix;
        fused_phase<GRID, POSE, VIEW, 0, DEG, FIX>(tiles, block, st, g, rs, op, tgt_rgb, tgt_depth, fw,
                                                   rgb, depth, loss, grad, gp, stats, ws, variant, sp);
    }
}

// The pose alone of many rays: one lane per ray in two marches, the second of which
// visits the lit samples only, against a team in one march, whose sums take more
// registers (the view term spills 55).  us, this form and the better team:
//   dense maps: the first march ends at a sample's densities (32^3 map: 160,000 rays 289
//     and 256, 300,000 367 and 440, 816,000 678 and 1044; with the view term 64,000
//     317 and 195, 120,000 331 and 336, 160,000 318 and 367);
//   with the view term (256^3 room: 160,000 sparse rays 852 and 757, 300,000 1172 and
//     1406, 600,000 1572 and 1978; frames of 172,800 527 and 527, of 816,000 917 and 1225;
//     frames in raster order, 120,000 rays 473 and 549, 156,400 566 and 641);
//   SH degrees 0 and 1, whose records are cheap to read twice (degree 0: 160,000
//     sparse rays 595 and 433, 300,000 732 and 797, 600,000 908 and 1117; a frame of
//     816,000 546 and 679);
//   degree 2 on sparse maps stays with the teams (300,000 1074 and 951, 600,000 1474
//     and 1343, a frame of 816,000 859 and 810).
static bool one_lane_pose(const KGrid& g, const KOpts& op, int64_t n_rays, int want) {
    if ((want & 3) != 2) return false;
    if (op.flags & 1) return n_rays > (g.probe ? 120000 : 150000);
    return g.probe ? n_rays > 200000 : g.deg < 2 && n_rays > 250000;
}

hipError_t launch_fused(const KGrid& g, const KRays& rs, const KOpts& op, const float* tgt_rgb,
                        const float* tgt_depth, const float* frame_weight, int want, float* rgb,
                        float* depth, double* loss, float* grad_data, double* grad_pose,
                        int64_t* stats, unsigned* ws, int block, int variant,
                        unsigned long long* gfix, hipStream_t st) {
    // variant 0 takes a team of lanes per ray where that is faster (team_lanes_log2;
    // for the pose alone also of one lane, which needs one march only); the counters and the fixed-point
    // scatter, whose result does not depend on the launch form, stay with one
    const int lt = team_lanes_log2(rs.n, want);
    const bool alone = one_lane_pose(g, op, rs.n, want);
    if (variant == 0 && !alone && !gfix && !(want & 4) && (lt > 0 || (want & 3) == 2))
        return team_fused(g, rs, op, lt, tgt_rgb, tgt_depth, frame_weight, want, rgb, depth, loss, grad_data, grad_pose, st);
    // a wave works alone: workgroups of one wave leave no registers and LDS with
    // waves that wait for the slowest of four (64 uneven frames of the 512^3
    // room 35.0 ms with 256 rays per workgroup, 31.6 with 64)
    if (variant == 0) block = WAVE;
    if (want & 1) {
        // the grid scatter needs WAVE_LDS_FLOATS of LDS per wave: shrink the
        // workgroup if the device cannot give this many waves' worth
        static const size_t max_lds = device_lds();
        while (block > WAVE && (size_t)(block / WAVE) * WAVE_LDS_FLOATS * sizeof(float) > max_lds)
            block /= 2;
    }
    const int64_t tiles = (rs.n + block - 1) / block;
    if (tiles > 0x7fffffffLL) return hipErrorInvalidValue;  // 32-bit grid and queue counters
    const dim3 blk(block);
    const bool G = want & 1, P = want & 2, V = (op.flags & 1) != 0;
    int64_t* sp = (want & 4) ? stats : nullptr;
    by_degree(g.deg, [&](auto D) {
        constexpr int DEG = decltype(D)::value;
        if (G && P) {
            if (V) {
                if (gfix) fused_go<true, true, true, DEG, true>(tiles, blk, st, g, rs, op, tgt_rgb, tgt_depth, frame_weight, rgb, depth, loss, grad_data, grad_pose, sp, ws, variant, gfix);
                else fused_go<true, true, true, DEG, false>(tiles, blk, st, g, rs, op, tgt_rgb, tgt_depth, frame_weight, rgb, depth, loss, grad_data, grad_pose, sp, ws, variant, gfix);
            } else {
                if (gfix) fused_go<true, true, false, DEG, true>(tiles, blk, st, g, rs, op, tgt_rgb, tgt_depth, frame_weight, rgb, depth, loss, grad_data, grad_pose, sp, ws, variant, gfix);
                else fused_go<true, true, false, DEG, false>(tiles, blk, st, g, rs, op, tgt_rgb, tgt_depth, frame_weight, rgb, depth, loss, grad_data, grad_pose, sp, ws, variant, gfix);
            }
        } else if (G) {
            if (gfix) fused_go<true, false, false, DEG, true>(tiles, blk, st, g, rs, op, tgt_rgb, tgt_depth, frame_weight, rgb, depth, loss, grad_data, grad_pose, sp, ws, variant, gfix);
            else fused_go<true, false, false, DEG, false>(tiles, blk, st, g, rs, op, tgt_rgb, tgt_depth, frame_weight, rgb, depth, loss, grad_data, grad_pose, sp, ws, variant, gfix);
        } else if (P) {
            if (V) fused_go<false, true, true, DEG, false>(tiles, blk, st, g, rs, op, tgt_rgb, tgt_depth, frame_weight, rgb, depth, loss, grad_data, grad_pose, sp, ws, variant, nullptr);
            else fused_go<false, true, false, DEG, false>(tiles, blk, st, g, rs, op, tgt_rgb, tgt_depth, frame_weight, rgb, depth, loss, grad_data, grad_pose, sp, ws, variant, nullptr);
        } else {
            fused_go<false, false, false, DEG, false>(tiles, blk, st, g, rs, op, tgt_rgb, tgt_depth, frame_weight, rgb, depth, loss, grad_data, grad_pose, sp, ws, variant, nullptr);
        }
    });
    if (G && gfix) {
        // fold the exact integer sums into the float gradient, once per entry
        const int S = record_floats(g.deg);
        const int64_t n = g.n_alloc * S;
        const int64_t wgs = (n + 255) / 256;
        hipLaunchKernelGGL(k_fix_finalize, dim3((unsigned)(wgs < (1 << 20) ? wgs : (1 << 20))), dim3(256), 0,
                           st, gfix, grad_data, n, S, 1 + 3 * (g.deg + 1) * (g.deg + 1));
    }
    return hipGetLastError();
}

}  // namespace pxm
