// Occupancy bitfield used to skip empty space exactly.
//
// Level 0: one 64-bit word per block of 4^3 cells, block (qx, qy, qz) at
//          linear index (qx * Qy + qy) * Qz + qz, Q = ceil((R - 1) / 4); cell
//          (x, y, z) is bit (x & 3) * 16 + (y & 3) * 4 + (z & 3) of its block's
//          word.  A cell is occupied iff one of its 8 corner links is a valid
//          record id; cells beyond R - 2 are empty.
// Level 1: one bit per brick of 8^3 cells, brick (bx, by, bz) at linear index
//          (bx * By + by) * Bz + bz, stored after level 0 (32-bit words).
// Both levels are rebuilt from the link table on the caller's stream; a
// bitfield that does not match the link table gives wrong renders.  The
// 4^3 blocks let a march keep the word of the block it is in and load the
// next only when it crosses into another block.
#include "internal.hpp"

namespace pxm {

void occ_layout(const int R[3], int64_t& w0_words, int Q[3], int B[3], int64_t& w1_words) {
    for (int a = 0; a < 3; ++a) {
        Q[a] = (R[a] - 1 + 3) / 4;
        B[a] = (R[a] - 1 + 7) / 8;
    }
    w0_words = 2 * (int64_t)Q[0] * Q[1] * Q[2];
    w1_words = ((int64_t)B[0] * B[1] * B[2] + 31) / 32;
}

// A group of lanes per 4 x 4 cells of (x, y) and a run of blocks along z: the 5 x 5
// rows of links it needs, one link per lane, are requested at once, each row's
// ballot is its allocation bits, a cell's bit along z is its own or the next, rows of
// cells are ORs of four rows of vertices, and lane l assembles the word of block l.
// A group is a wave (runs of OCC_RUN blocks), or the 4 to 32 lanes that hold a short
// row whole.  Bound by the link reads (511^3: 152 us; a lane per cell that read its
// own 8 corners took 506, reading the table once takes 105; 1024 x 1024 x 8 14 us, 61
// with a wave to every row).
constexpr int OCC_RUN = 15;                                 // 60 cells, 61 of the 64 vertices

__global__ void __launch_bounds__(256) k_occ0(KGrid g, uint64_t* __restrict__ occ0, int64_t n_items, int runs, int log_g) {
    const int group = 1 << log_g, in = lane_id() & (group - 1), first = lane_id() - in;
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x / WAVE);
    const int64_t n_waves = (n_items + (WAVE >> log_g) - 1) >> (6 - log_g);
    for (int64_t w = (int64_t)blockIdx.x * (blockDim.x / WAVE) + threadIdx.x / WAVE; w < n_waves; w += waves) {
        const int64_t it = (w << (6 - log_g)) + (first >> log_g);
        const int64_t q2 = it / runs;
        const int qz = (int)(it - q2 * runs) * OCC_RUN;
        const int qx = (int)(q2 / g.Q[1]), qy = (int)(q2 - (int64_t)qx * g.Q[1]);
        const int x0 = 4 * qx, y0 = 4 * qy, z = 4 * qz + in;   // x0 past the lattice: no cells
        int32_t l[25];
#pragma unroll
        for (int k = 0; k < 25; ++k) {
            const int x = x0 + k / 5, y = y0 + k % 5;
            l[k] = -1;
            if (x < g.R[0] && y < g.R[1] && z < g.R[2]) l[k] = g.link[(int64_t)x * g.sx + (int64_t)y * g.sy + z];
        }
        unsigned long long row[25];
#pragma unroll
        for (int k = 0; k < 25; ++k) row[k] = __ballot((uint32_t)l[k] < (uint64_t)g.n_alloc);
        // cells beyond R - 2 on an axis are empty, and so is what another group's bits
        // shift in: a group holds a vertex more than its cells
        const int cells = g.R[2] - 1 - 4 * qz;
        const unsigned long long in_z = (cells >= 64 ? ~0ull : (1ull << cells) - 1ull) << first;
        uint64_t word = 0ull;
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            const int cx = c >> 2, cy = c & 3, k = 5 * cx + cy;
            unsigned long long m = row[k] | row[k + 1] | row[k + 5] | row[k + 6];
            m = x0 + cx < g.R[0] - 1 && y0 + cy < g.R[1] - 1 ? (m | (m >> 1)) & in_z : 0ull;
            word |= ((m >> ((first + 4 * in) & 63)) & 0xfull) << (4 * c);
        }
        if (in < OCC_RUN && 4 * in < group && qz + in < g.Q[2] && it < n_items) occ0[q2 * g.Q[2] + qz + in] = word;
    }
}

// One lane per brick: the OR of its (up to) 2 x 2 x 2 level-0 words; the
// wave's 64 bricks fill two level-1 words.
__global__ void k_occ1(KGrid g, const uint64_t* __restrict__ occ0, uint32_t* __restrict__ occ1,
                       int64_t nwords1) {
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nb = (int64_t)g.B[0] * g.B[1] * g.B[2];
    bool any = false;
    if (b < nb) {
        const int bx = (int)(b / ((int64_t)g.B[1] * g.B[2])), by = (int)((b / g.B[2]) % g.B[1]);
        const int bz = (int)(b % g.B[2]);
        for (int i = 0; i < 8; ++i) {
            const int qx = 2 * bx + ((i >> 2) & 1), qy = 2 * by + ((i >> 1) & 1), qz = 2 * bz + (i & 1);
            if (qx < g.Q[0] && qy < g.Q[1] && qz < g.Q[2])
                any |= occ0[((int64_t)qx * g.Q[1] + qy) * g.Q[2] + qz] != 0ull;
        }
    }
    const unsigned long long m = __ballot(any);
    const int lane = lane_id();
    const int64_t word = b >> 5;
    if ((lane == 0 || lane == 32) && word < nwords1)
        occ1[word] = lane == 0 ? (uint32_t)m : (uint32_t)(m >> 32);
}

hipError_t launch_occupancy(const KGrid& g, uint32_t* occ, hipStream_t st) {
    int64_t w0, w1;
    int Q[3], B[3];
    occ_layout(g.R, w0, Q, B, w1);
    KGrid k = g;
    for (int a = 0; a < 3; ++a) {
        k.Q[a] = Q[a];
        k.B[a] = B[a];
    }
    const int runs = (Q[2] + OCC_RUN - 1) / OCC_RUN;
    const int64_t n_items = (int64_t)Q[0] * Q[1] * runs;
    int log_g = 2;                                        // lanes that hold a whole row of vertices, or a wave
    while (log_g < 6 && (1 << log_g) < g.R[2]) ++log_g;
    const int64_t per_wg = (int64_t)(256 >> log_g), wgs = (n_items + per_wg - 1) / per_wg;
    hipLaunchKernelGGL(k_occ0, dim3((unsigned)(wgs < (1 << 20) ? wgs : (1 << 20))), dim3(256), 0, st, k,
                       reinterpret_cast<uint64_t*>(occ), n_items, runs, log_g);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t nb = (int64_t)B[0] * B[1] * B[2];
    hipLaunchKernelGGL(k_occ1, dim3((unsigned)((nb + 255) / 256)), dim3(256), 0, st, k,
                       reinterpret_cast<const uint64_t*>(occ), occ + w0, w1);
    return hipGetLastError();
}

}  // namespace pxm
