// Total-variation gradient in gather form: every allocated vertex's record
// is written by exactly one thread per field, no atomics.
//
//   TV = sum_m lambda_m sum_{u allocated, not on an upper face}
//            sqrt(dx_m(u)^2 + dy_m(u)^2 + dz_m(u)^2 + eps),
//   dx_m(u) = val_m(u + x) - val_m(u)  (empty vertices read as 0).
// dTV/d val_m(v) = lambda_m [ -(dx+dy+dz)(v)/root(v)             if v has a term
//                           + dx(v-x)/root(v-x)                    if v-x has a term
//                           + dy(v-y)/root(v-y) + dz(v-z)/root(v-z)  (likewise) ]
//
// Blocks of 8^3 lattice vertices, one workgroup each.  The workgroup tests the
// block against the occupancy bitfield, loads the links of the block and its
// one-vertex halo (10^3) into LDS in one pass and lists its allocated vertices
// with the terms that touch each.  Then Q lanes per vertex (7 at SH degree 2)
// each take one float4 of its record: they request that float4 of the 13
// records the four terms read at once, and write the result; no barrier follows
// the list, so a vertex costs one round trip and waves do not wait for each
// other.  The 13 records lie in neighbouring rows that the workgroup's other
// waves read too, and come from L1 and L2.
//
// On the 256^3 room (1.68 M records; 376 MB read and written are 73 us at the
// rate of a large copy) and the 512^3 room (4.03 M) this takes 206 and 481 us,
// where staging 6^3 halos of records in LDS, sub-block by sub-block, took 318
// and 1120: a chain of barriers per sub-block and 13 scattered LDS reads per
// field.  The vector ALU is then busy half of the time, and the L2s fetch the
// records three times over (halos, and rows that leave L2 before their turn).
// Cubes of 2^3 blocks (on flat lattices 8 blocks in another shape) dealt to the XCDs in turn: one contiguous eighth each gave
// 266 and 665 us (an XCD with a whole wall of the room works longest), single
// blocks in turn 240 and 527, cubes of 4^3 233 and 538.
//
// SET writes the gradient (grad = dTV) instead of adding to it, which saves
// the read of the gradient: a step that zeroes its gradient can run the TV
// term first and let the rendering backward add onto it.
#include "internal.hpp"

namespace pxm {

constexpr int TB8 = 8;                  // block edge (vertices)
constexpr int TH8 = TB8 + 2;            // with halo
constexpr int TH83 = TH8 * TH8 * TH8;   // 1000 link positions
constexpr int PER_CUBE = 8;             // blocks of a cube
constexpr uint32_t NONE = 0xffffffffu;  // no record
constexpr int TV_THREADS = 256;
constexpr int64_t TV_LAUNCH = 1 << 23;  // blocks per launch: a grid holds fewer than 2^32 threads
// a listed vertex: its position in the halo block and the TV terms that touch
// it (its own, and those of its -x, -y, -z neighbours)
constexpr int TERM_POS = 0x3ff, TERM_OWN = 0x400, TERM_X = 0x800, TERM_Y = 0x1000, TERM_Z = 0x2000;
static_assert(TH83 <= TERM_POS + 1, "halo positions fit in the low bits");

__device__ __forceinline__ int hidx8(int x, int y, int z) { return (x * TH8 + y) * TH8 + z; }

// dTV / d val of one field from the values of the 13 records around vertex v:
// f* ahead of it, b* behind it, and those one step ahead of a step behind.
struct TvHood {
    float v, fx, fy, fz, bx, bxy, bxz, by, byx, byz, bz, bzx, bzy;
};

// NORMAL: eps is a normal number, so the sums of squares are, and need no scaling.
template <bool NORMAL>
__device__ __forceinline__ float tv_rsqrt(float x) {
    return NORMAL ? __builtin_amdgcn_rsqf(x) : rsqrtf(x);
}

template <bool NORMAL>
__device__ __forceinline__ float tv_field(const TvHood& h, int e, float eps) {
    float acc = 0.f;
    {
        const float dx = h.fx - h.v, dy = h.fy - h.v, dz = h.fz - h.v;
        const float t = (dx + dy + dz) * tv_rsqrt<NORMAL>(dx * dx + dy * dy + dz * dz + eps);
        if (e & TERM_OWN) acc -= t;
    }
    {
        const float dx = h.v - h.bx, dy = h.bxy - h.bx, dz = h.bxz - h.bx;
        const float t = dx * tv_rsqrt<NORMAL>(dx * dx + dy * dy + dz * dz + eps);
        if (e & TERM_X) acc += t;
    }
    {
        const float dx = h.byx - h.by, dy = h.v - h.by, dz = h.byz - h.by;
        const float t = dy * tv_rsqrt<NORMAL>(dx * dx + dy * dy + dz * dz + eps);
        if (e & TERM_Y) acc += t;
    }
    {
        const float dx = h.bzx - h.bz, dy = h.bzy - h.bz, dz = h.v - h.bz;
        const float t = dz * tv_rsqrt<NORMAL>(dx * dx + dy * dy + dz * dz + eps);
        if (e & TERM_Z) acc += t;
    }
    return acc;
}

// Cubes along y and z, and the logarithm of a cube's blocks along each axis.
struct TvCubes {
    int ny, nz, lx, ly, lz;
};

// first: the launch's first block (a launch holds at most TV_LAUNCH of them).
// WIDE: the map's records span 4 GiB or more; otherwise s_rec holds byte offsets,
// and an address is one 32-bit add.
template <int DEG, bool SET, bool NORMAL, bool WIDE>
__global__ void __launch_bounds__(TV_THREADS) k_tv(KGrid g, float lam_d, float lam_sh, float eps,
                                                   float* __restrict__ grad, TvCubes cs, int64_t first) {
    constexpr int S = RecL<DEG>::S, Q = RecL<DEG>::Q, USED = RecL<DEG>::USED;
    __shared__ uint32_t s_rec[TH83];        // records of the block and its halo (NONE: empty or outside)
    __shared__ int s_list[TB8 * TB8 * TB8]; // its allocated vertices
    __shared__ int s_n;
    const int t = threadIdx.x;
    // Cubes of blocks go round the XCDs (workgroup b runs on XCD b mod 8), so
    // that blocks sharing halos share an L2 and no XCD gets a whole wall of the
    // map; the turn shifts from round to round, as a row of cubes may hold eight.
    const int64_t b = first + blockIdx.x;
    const int64_t round = b / (8 * PER_CUBE);
    const int64_t cube = round * 8 + ((b + 3 * round + round / 8) & 7);
    const int in = (int)((b / 8) % PER_CUBE);
    const int bz = ((int)(cube % cs.nz) << cs.lz) + (in & ((1 << cs.lz) - 1));
    const int by = ((int)((cube / cs.nz) % cs.ny) << cs.ly) + ((in >> cs.lz) & ((1 << cs.ly) - 1));
    const int bx = ((int)(cube / ((int64_t)cs.nz * cs.ny)) << cs.lx) + (in >> (cs.lz + cs.ly));
    const int x0 = bx * TB8, y0 = by * TB8, z0 = bz * TB8;
    const int X = g.R[0], Y = g.R[1], Z = g.R[2];
    if (x0 >= X || y0 >= Y || z0 >= Z) return;              // workgroup-uniform, as below
    // An allocated vertex v of this block is a corner of cell min(v, R-2) per
    // axis, which lies in cell brick (bx, by, bz) whenever that brick exists.
    if (g.occ1 && bx < g.B[0] && by < g.B[1] && bz < g.B[2]) {
        const int c[3] = {x0, y0, z0};
        if (brick_empty(g, c)) return;
    }
    if (t == 0) s_n = 0;
    {
        // all of a thread's link loads are issued before the first LDS write
        constexpr int LINK_ITERS = (TH83 + TV_THREADS - 1) / TV_THREADS;
        int ids[LINK_ITERS];
#pragma unroll
        for (int k = 0; k < LINK_ITERS; ++k) {
            const int p = t + k * TV_THREADS;
            const int x = x0 + p / (TH8 * TH8) - 1, y = y0 + (p / TH8) % TH8 - 1, z = z0 + p % TH8 - 1;
            ids[k] = -1;
            if (p < TH83 && (uint32_t)x < (uint32_t)X && (uint32_t)y < (uint32_t)Y && (uint32_t)z < (uint32_t)Z)
                ids[k] = g.link[((int64_t)x * Y + y) * Z + z];
        }
#pragma unroll
        for (int k = 0; k < LINK_ITERS; ++k) {
            const int p = t + k * TV_THREADS;
            if (p < TH83)
                s_rec[p] = (uint32_t)ids[k] >= (uint64_t)g.n_alloc ? NONE
                         : WIDE ? (uint32_t)ids[k] : (uint32_t)ids[k] * (uint32_t)(S * sizeof(float));
        }
    }
    __syncthreads();
    // A wave lists the vertices of two 4^3 sub-blocks, so that waves at work
    // together share records.  The order between waves does not matter.
#pragma unroll
    for (int j = 0; j < TB8 * TB8 * TB8 / TV_THREADS; ++j) {
        const int p = j * TV_THREADS + t, sb = p >> 6;
        const int ix = (sb >> 2) * 4 + ((p >> 4) & 3), iy = ((sb >> 1) & 1) * 4 + ((p >> 2) & 3);
        const int iz = (sb & 1) * 4 + (p & 3);
        const int h = hidx8(ix + 1, iy + 1, iz + 1);
        const bool a = s_rec[h] != NONE;
        const unsigned long long m = __ballot(a);
        int base = 0;
        if (lane_id() == 0 && m) base = atomicAdd(&s_n, __popcll(m));
        base = __builtin_amdgcn_readfirstlane(base);
        if (a) {
            const int x = x0 + ix, y = y0 + iy, z = z0 + iz;
            const bool ix_ = x < X - 1, iy_ = y < Y - 1, iz_ = z < Z - 1;
            int e = h;
            if (ix_ && iy_ && iz_) e |= TERM_OWN;
            if (x >= 1 && iy_ && iz_ && s_rec[h - TH8 * TH8] != NONE) e |= TERM_X;
            if (y >= 1 && ix_ && iz_ && s_rec[h - TH8] != NONE) e |= TERM_Y;
            if (z >= 1 && ix_ && iy_ && s_rec[h - 1] != NONE) e |= TERM_Z;
            s_list[base + __popcll(m & ((1ull << lane_id()) - 1))] = e;
        }
    }
    __syncthreads();
    const int items = s_n * Q;
    const char* data = reinterpret_cast<const char*>(g.data);
    char* gout = reinterpret_cast<char*>(grad);
    for (int i = t; i < items; i += TV_THREADS) {
        const int e = s_list[i / Q];
        const uint32_t q = i % Q;
        const int h = e & TERM_POS;
        auto off = [&](uint32_t rec) {                      // bytes from the array's start to the lane's float4
            if constexpr (WIDE) return (size_t)rec * (S * sizeof(float)) + q * 16u;
            else return rec + q * 16u;
        };
        auto at = [&](int p) -> float4 {
            const uint32_t rec = s_rec[p];
            return rec != NONE ? *reinterpret_cast<const float4*>(data + off(rec)) : make_float4(0.f, 0.f, 0.f, 0.f);
        };
        constexpr int DX = TH8 * TH8, DY = TH8, DZ = 1;
        const float4 v = at(h), fx = at(h + DX), fy = at(h + DY), fz = at(h + DZ);
        const float4 px = at(h - DX), pxy = at(h - DX + DY), pxz = at(h - DX + DZ);
        const float4 py = at(h - DY), pyx = at(h - DY + DX), pyz = at(h - DY + DZ);
        const float4 pz = at(h - DZ), pzx = at(h - DZ + DX), pzy = at(h - DZ + DY);
        float* out = reinterpret_cast<float*>(gout + off(s_rec[h]));
        const bool whole = 4 * q + 4 <= USED;               // else one used field and padding
        float4 old = make_float4(0.f, 0.f, 0.f, 0.f);
        if (!SET) {
            if (whole) old = *reinterpret_cast<const float4*>(out);
            else old.x = out[0];
        }
        const float lam = q == 0 ? lam_d : lam_sh;          // field 0 is the density
        float4 r;
        r.x = lam * tv_field<NORMAL>({v.x, fx.x, fy.x, fz.x, px.x, pxy.x, pxz.x, py.x, pyx.x, pyz.x, pz.x, pzx.x, pzy.x}, e, eps);
        r.y = lam_sh * tv_field<NORMAL>({v.y, fx.y, fy.y, fz.y, px.y, pxy.y, pxz.y, py.y, pyx.y, pyz.y, pz.y, pzx.y, pzy.y}, e, eps);
        r.z = lam_sh * tv_field<NORMAL>({v.z, fx.z, fy.z, fz.z, px.z, pxy.z, pxz.z, py.z, pyx.z, pyz.z, pz.z, pzx.z, pzy.z}, e, eps);
        r.w = lam_sh * tv_field<NORMAL>({v.w, fx.w, fy.w, fz.w, px.w, pxy.w, pxz.w, py.w, pyx.w, pyz.w, pz.w, pzx.w, pzy.w}, e, eps);
        if (!SET) {
            r.x += old.x;
            r.y += old.y;
            r.z += old.z;
            r.w += old.w;
        }
        if (whole) *reinterpret_cast<float4*>(out) = r;
        else out[0] = r.x;
    }
}

template <int DEG, bool SET>
static void tv_go(const KGrid& g, float lambda_density, float lambda_sh, float eps, float* grad_data,
                  hipStream_t st) {
    // A cube of 8 blocks is halved along the axes in turn, but not along one that
    // has no second block to share it with: half of the workgroups would be empty.
    int nb[3], l[3] = {0, 0, 0}, nc[3];
    for (int a = 0; a < 3; ++a) nb[a] = (g.R[a] + TB8 - 1) / TB8;
    for (int k = 0; k < 3; ++k) {
        int best = -1;
        for (int a = 2; a >= 0; --a)
            if ((nb[a] >> l[a]) > 1 && (best < 0 || l[a] < l[best])) best = a;
        ++l[best < 0 ? 2 : best];
    }
    for (int a = 0; a < 3; ++a) nc[a] = (nb[a] + (1 << l[a]) - 1) >> l[a];
    const TvCubes cs = {nc[1], nc[2], l[0], l[1], l[2]};
    const int64_t blocks = ((int64_t)nc[0] * nc[1] * nc[2] + 7) / 8 * (8 * PER_CUBE);
    const bool normal = eps >= 1.17549435e-38f;
    const bool wide = (uint64_t)g.n_alloc * (RecL<DEG>::S * sizeof(float)) >= NONE;
    auto go = [&](auto kernel) {
        for (int64_t first = 0; first < blocks; first += TV_LAUNCH)
            hipLaunchKernelGGL(kernel, dim3((unsigned)(blocks - first < TV_LAUNCH ? blocks - first : TV_LAUNCH)), dim3(TV_THREADS), 0, st,
                               g, lambda_density, lambda_sh, eps, grad_data, cs, first);
    };
    if (wide) normal ? go(k_tv<DEG, SET, true, true>) : go(k_tv<DEG, SET, false, true>);
    else normal ? go(k_tv<DEG, SET, true, false>) : go(k_tv<DEG, SET, false, false>);
}

hipError_t launch_tv(const KGrid& g, float lambda_density, float lambda_sh, float eps,
                     float* grad_data, bool set, hipStream_t st) {
    if (tv_staged_wins(g)) return launch_tv_staged(g, lambda_density, lambda_sh, eps, grad_data, set, st);
    auto by_set = [&](auto D) {
        constexpr int DEG = decltype(D)::value;
        if (set) tv_go<DEG, true>(g, lambda_density, lambda_sh, eps, grad_data, st);
        else tv_go<DEG, false>(g, lambda_density, lambda_sh, eps, grad_data, st);
    };
    if (g.deg == 0) by_set(std::integral_constant<int, 0>{});
    else if (g.deg == 1) by_set(std::integral_constant<int, 1>{});
    else by_set(std::integral_constant<int, 2>{});
    return hipGetLastError();
}

}  // namespace pxm
