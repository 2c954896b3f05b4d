// Dynamic-grid edits: coarse-to-fine growth and pruning (Sec. 6.1: the map is
// a dynamic voxel grid that grows to a peak of 512^3).
//
// Both edits are stream compactions: a flag per item, an exclusive prefix
// count that numbers the flagged items in order, and a write pass.  Flags are
// packed 32 to a word; a chunk is EDIT_WORDS words (one workgroup), and the
// count takes three steps:
//   flag kernel   the chunk's words, the exclusive prefix of each word's
//                 popcount inside the chunk, and the chunk's total;
//   k_scan_chunks one workgroup turns the chunk totals into exclusive chunk
//                 offsets and writes the grand total to the caller's n_out;
//   write pass    flagged item i gets id = chunk offset + word prefix +
//                 popcount of the lower bits of its word.
//
// Growth.  R vertices per axis become 2R - 1: fine vertex 2v is coarse vertex
// v, voxel size halves, the origin stays.  A fine vertex is allocated when a
// coarse cell whose closed box holds it has an allocated corner; records are
// numbered in lattice order.  Along an axis, fine coordinate 2v lies in the
// cells of coarse vertices v-1 .. v+1 (clipped to the lattice) and 2v+1 in
// those of v .. v+1, so the flag is an OR over that box of coarse vertices.
// It is evaluated bit-parallel: the coarse allocation bits of each (x, y)
// row, OR-ed over the 1-3 x 1-3 neighbouring rows, then dilated along z by
// shifts.  The compaction runs over fine rows padded to whole words.
// A fine record is the coarse trilinear interpolant at its vertex, density
// halved (density is per voxel, so each world-length step keeps its optical
// depth): 1, 2, 4 or 8 coarse records with exact power-of-two weights,
// summed in FP64 in corner order and rounded once to FP32.
//
// Pruning.  Records with density <= tau are dropped, the others keep their
// order and get new ids, and the link table is rewritten (dropped -> -1).
#include "internal.hpp"

namespace pxm {

namespace {

constexpr int EDIT_THREADS = 256;
constexpr int EDIT_WORDS = EDIT_CHUNK / 32;             // words per chunk, one per thread
constexpr int KEEP_ITERS = EDIT_CHUNK / EDIT_THREADS;   // records per thread in the prune flags
constexpr int SCAN_THREADS = 1024;
constexpr int LINK_PER_THREAD = 8;
constexpr int LINK_ITEMS = LINK_PER_THREAD * EDIT_THREADS;   // link-table items per workgroup pass
static_assert(EDIT_WORDS == EDIT_THREADS, "one thread per flag word of a chunk");

__device__ __forceinline__ bool link_ok(int32_t l, int64_t n) { return (uint32_t)l < (uint64_t)n; }

// Exclusive prefix of `v` over the workgroup's threads; `total` gets the sum.
__device__ __forceinline__ int block_exclusive(int v, int& total) {
    __shared__ int s_wave[EDIT_THREADS / WAVE];
    const int lane = lane_id(), w = threadIdx.x / WAVE;
    int incl = v;
    for (int d = 1; d < WAVE; d <<= 1) {
        const int o = __shfl_up(incl, d, WAVE);
        if (lane >= d) incl += o;
    }
    if (lane == WAVE - 1) s_wave[w] = incl;
    __syncthreads();
    int before = 0;
    total = 0;
#pragma unroll
    for (int i = 0; i < EDIT_THREADS / WAVE; ++i) {
        before += i < w ? s_wave[i] : 0;
        total += s_wave[i];
    }
    return before + incl - v;
}

// Chunk epilogue: thread t owns word t of the chunk.
__device__ __forceinline__ void finish_chunk(uint32_t bits, int64_t gw, int64_t nw, uint32_t* words, int32_t* wpre,
                                             int32_t* chunk_total) {
    const int cnt = __popc(bits);
    int total;
    const int pre = block_exclusive(cnt, total);
    if (gw < nw) {
        words[gw] = bits;
        wpre[gw] = pre;
    }
    if (threadIdx.x == 0) chunk_total[blockIdx.x] = total;
}

// ---------------------------------------------------------------- pruning

// Record r survives iff its density exceeds tau.  Pass `it` of wave w covers
// 64 consecutive records, i.e. words 8 it + 2w and 8 it + 2w + 1 of the chunk.
__global__ __launch_bounds__(EDIT_THREADS) void k_keep_flags(const float* __restrict__ data, int S, float tau, int64_t n,
                                                             uint32_t* __restrict__ words, int32_t* __restrict__ wpre,
                                                             int32_t* __restrict__ chunk_total) {
    __shared__ uint32_t s_words[EDIT_WORDS];
    const int64_t base = (int64_t)blockIdx.x * EDIT_CHUNK;
    const int lane = lane_id(), w = threadIdx.x / WAVE;
    for (int it = 0; it < KEEP_ITERS; ++it) {
        const int64_t r = base + it * EDIT_THREADS + threadIdx.x;
        const bool f = r < n && data[r * S] > tau;
        const unsigned long long m = __ballot(f);
        if (lane == 0) s_words[it * 8 + 2 * w] = (uint32_t)m;
        if (lane == 32) s_words[it * 8 + 2 * w + 1] = (uint32_t)(m >> 32);
    }
    __syncthreads();
    finish_chunk(s_words[threadIdx.x], (int64_t)blockIdx.x * EDIT_WORDS + threadIdx.x, (n + 31) / 32, words, wpre,
                 chunk_total);
}

// One workgroup: exclusive scan of the chunk totals in place; *n_out = sum.
// Thread t owns a contiguous run of ceil(nc / SCAN_THREADS) totals.
__global__ __launch_bounds__(SCAN_THREADS) void k_scan_chunks(int32_t* __restrict__ chunk, int64_t nc,
                                                              int64_t* __restrict__ n_out) {
    __shared__ int64_t s_wave[SCAN_THREADS / WAVE];
    const int64_t per = (nc + SCAN_THREADS - 1) / SCAN_THREADS;
    const int64_t b0 = min((int64_t)threadIdx.x * per, nc), b1 = min(b0 + per, nc);
    int64_t sum = 0;
    for (int64_t b = b0; b < b1; ++b) sum += chunk[b];
    const int lane = lane_id(), w = threadIdx.x / WAVE;
    int64_t incl = sum;
    for (int d = 1; d < WAVE; d <<= 1) {
        const int64_t o = __shfl_up(incl, d, WAVE);
        if (lane >= d) incl += o;
    }
    if (lane == WAVE - 1) s_wave[w] = incl;
    __syncthreads();
    int64_t before = 0;
    for (int i = 0; i < w; ++i) before += s_wave[i];
    int64_t run = before + incl - sum;
    for (int64_t b = b0; b < b1; ++b) {
        const int32_t c = chunk[b];
        chunk[b] = (int32_t)run;
        run += c;
    }
    if (threadIdx.x == SCAN_THREADS - 1) *n_out = before + incl;
}

// id of item i among the flagged ones, or -1.
__device__ __forceinline__ int32_t compact_id(const uint32_t* words, const int32_t* wpre,
                                              const int32_t* chunk_off, int64_t i) {
    const int64_t w = i >> 5;
    const uint32_t bits = words[w];
    const int b = (int)(i & 31);
    if (!((bits >> b) & 1u)) return -1;
    return chunk_off[w / EDIT_WORDS] + wpre[w] + __popc(bits & ((1u << b) - 1u));
}

// 8 lanes per record: lanes p < S/4 copy float4 p of it (at most 7), lane 7
// writes its remap entry.
__global__ __launch_bounds__(EDIT_THREADS) void k_prune_copy(const float* __restrict__ data, int S, int64_t n,
                                                             const uint32_t* __restrict__ words,
                                                             const int32_t* __restrict__ wpre,
                                                             const int32_t* __restrict__ chunk_off,
                                                             int32_t* __restrict__ remap, float* __restrict__ out) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n * 8; t += stride) {
        const int64_t r = t >> 3;
        const int part = (int)(t & 7);
        const int32_t id = compact_id(words, wpre, chunk_off, r);
        if (part == 7) {
            remap[r] = id;
        } else if (id >= 0 && part < S / 4) {
            reinterpret_cast<float4*>(out + (int64_t)id * S)[part] =
                reinterpret_cast<const float4*>(data + r * S)[part];
        }
    }
}

__global__ __launch_bounds__(EDIT_THREADS) void k_relink(const int32_t* link, int64_t nv, int64_t n_alloc,
                                                         const int32_t* __restrict__ remap, int32_t* link_out) {
    const int64_t stride = (int64_t)gridDim.x * LINK_ITEMS;
    for (int64_t v0 = (int64_t)blockIdx.x * LINK_ITEMS; v0 < nv; v0 += stride) {
        int32_t l[LINK_PER_THREAD];
#pragma unroll
        for (int k = 0; k < LINK_PER_THREAD; ++k) {
            const int64_t v = v0 + k * EDIT_THREADS + threadIdx.x;
            l[k] = v < nv ? link[v] : -1;
        }
#pragma unroll
        for (int k = 0; k < LINK_PER_THREAD; ++k) l[k] = link_ok(l[k], n_alloc) ? remap[l[k]] : -1;
#pragma unroll
        for (int k = 0; k < LINK_PER_THREAD; ++k) {
            const int64_t v = v0 + k * EDIT_THREADS + threadIdx.x;
            if (v < nv) link_out[v] = l[k];
        }
    }
}

// ---------------------------------------------------------------- growth

struct Lattice {
    int R[3];     // coarse vertices per axis
    int Rf[3];    // fine vertices per axis, 2R - 1
    int WC;       // coarse allocation words per (x, y) row
    int WF;       // fine flag words per (x, y) row
};

// Coarse allocation bits, rows padded to WC words: one lane per padded item,
// a ballot per 64.  The loop runs over a multiple of 64 items so every wave
// reaches the ballot whole.
__global__ __launch_bounds__(EDIT_THREADS) void k_coarse_bits(KGrid g, Lattice L, int64_t n_items,
                                                              uint32_t* __restrict__ vbits) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t padded = (n_items + WAVE - 1) / WAVE * WAVE;
    const int lane = lane_id();
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < padded; i += stride) {
        bool f = false;
        if (i < n_items) {
            const uint32_t w = (uint32_t)(i >> 5);
            const uint32_t row = w / (uint32_t)L.WC;
            const int z = (int)(w - row * (uint32_t)L.WC) * 32 + (int)(i & 31);
            f = z < L.R[2] && link_ok(g.link[(int64_t)row * L.R[2] + z], g.n_alloc);
        }
        const unsigned long long m = __ballot(f);
        const int64_t w0 = (i - lane) >> 5;
        if (lane == 0 && w0 * 32 < n_items) vbits[w0] = (uint32_t)m;
        if (lane == 32 && (w0 + 1) * 32 < n_items) vbits[w0 + 1] = (uint32_t)(m >> 32);
    }
}

// 64 coarse bits of row `row` starting at coarse z = p (p >= -1; bits outside
// the lattice read 0).
__device__ __forceinline__ uint64_t coarse_window(const uint32_t* vbits, int64_t row, int WC, int p) {
    const uint32_t* r = vbits + row * WC;
    if (p < 0) {
        const uint64_t v = (uint64_t)r[0] | ((WC > 1 ? (uint64_t)r[1] : 0ull) << 32);
        return v << 1;
    }
    const int wi = p >> 5, sh = p & 31;
    const uint64_t lo = wi < WC ? r[wi] : 0u, hi = wi + 1 < WC ? r[wi + 1] : 0u;
    return (lo | (hi << 32)) >> sh;
}

// Bits 0 .. 15 of x at the even positions 0 .. 30.
__device__ __forceinline__ uint32_t spread16(uint32_t x) {
    x &= 0xffffu;
    x = (x | (x << 8)) & 0x00ff00ffu;
    x = (x | (x << 4)) & 0x0f0f0f0fu;
    x = (x | (x << 2)) & 0x33333333u;
    return (x | (x << 1)) & 0x55555555u;
}

// One thread per fine flag word: fine row (fx, fy), fine z in [32 l, 32 l + 32).
// Window bit k is coarse z = 16 l - 1 + k; fine z = 32 l + j sits on or after
// coarse vertex 16 l + (j >> 1), window bit (j >> 1) + 1.
__global__ __launch_bounds__(EDIT_THREADS) void k_grow_flags(const uint32_t* __restrict__ vbits, Lattice L, int64_t nw,
                                                             uint32_t* __restrict__ words, int32_t* __restrict__ wpre,
                                                             int32_t* __restrict__ chunk_total) {
    const int64_t gw = (int64_t)blockIdx.x * EDIT_WORDS + threadIdx.x;
    uint32_t bits = 0;
    if (gw < nw) {
        const uint32_t row = (uint32_t)(gw / L.WF);
        const int l = (int)(gw - (int64_t)row * L.WF);
        const int fx = (int)(row / (uint32_t)L.Rf[1]), fy = (int)(row - (uint32_t)fx * L.Rf[1]);
        const int vx = fx >> 1, vy = fy >> 1;
        const int x0 = (fx & 1) ? vx : max(vx - 1, 0), x1 = (fx & 1) ? vx + 1 : min(vx + 1, L.R[0] - 1);
        const int y0 = (fy & 1) ? vy : max(vy - 1, 0), y1 = (fy & 1) ? vy + 1 : min(vy + 1, L.R[1] - 1);
        uint64_t W = 0;
        for (int x = x0; x <= x1; ++x)
            for (int y = y0; y <= y1; ++y) W |= coarse_window(vbits, (int64_t)x * L.R[1] + y, L.WC, 16 * l - 1);
        const uint64_t D2 = W | (W >> 1);     // bit k: coarse k or k+1   (odd fine z)
        const uint64_t D3 = D2 | (W << 1);    // bit k: coarse k-1 .. k+1 (even fine z)
        // fine z = 32 l + 2 i takes bit i + 1 of D3, 32 l + 2 i + 1 that of D2
        bits = spread16((uint32_t)(D3 >> 1)) | (spread16((uint32_t)(D2 >> 1)) << 1);
        const int in_row = L.Rf[2] - 32 * l;
        if (in_row < 32) bits &= (1u << in_row) - 1u;
    }
    finish_chunk(bits, gw, nw, words, wpre, chunk_total);
}

// A group of lanes per fine row (the power of two that ROW_STEPS steps of 4 links per
// lane fill, a whole wave from 257 links on), whose steps are requested together: a
// link costs a shift, a popcount and a quarter of a store.  Bound by the writes:
// 511^3 links 115 us (537 MB written), 220 where each lane found the row of its link by
// division; 2047 x 2047 x 15 links with their count 225 us, 809 with a wave to every row.
constexpr int ROW_STEPS = 2;

__global__ __launch_bounds__(EDIT_THREADS) void k_fine_link(Lattice L, int log_g, const uint32_t* __restrict__ words,
                                                            const int32_t* __restrict__ wpre,
                                                            const int32_t* __restrict__ chunk_off,
                                                            int32_t* __restrict__ link_fine) {
    const int group = 1 << log_g, lane = threadIdx.x & (group - 1);
    const int64_t rows = (int64_t)L.Rf[0] * L.Rf[1];
    const int64_t groups = (int64_t)gridDim.x * (EDIT_THREADS >> log_g);
    for (int64_t row = (int64_t)blockIdx.x * (EDIT_THREADS >> log_g) + (threadIdx.x >> log_g); row < rows; row += groups) {
        const int64_t w0 = row * L.WF;
        int32_t* out = link_fine + row * L.Rf[2];
        for (int z0 = 0; z0 < L.Rf[2]; z0 += ROW_STEPS * group * 4) {
            uint32_t bits[ROW_STEPS];
            int32_t base[ROW_STEPS];
#pragma unroll
            for (int k = 0; k < ROW_STEPS; ++k) {
                const int z = z0 + (k * group + lane) * 4;
                bits[k] = 0u;
                base[k] = 0;
                if (z < L.Rf[2]) {
                    const int64_t w = w0 + (z >> 5);
                    bits[k] = words[w];
                    base[k] = chunk_off[w / EDIT_WORDS] + wpre[w];
                }
            }
#pragma unroll
            for (int k = 0; k < ROW_STEPS; ++k) {
                const int z = z0 + (k * group + lane) * 4, b = z & 31;
                int32_t id = base[k] + __popc(bits[k] & ((1u << b) - 1u));
                int32_t l[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const bool on = (bits[k] >> (b + j)) & 1u;
                    l[j] = on ? id : -1;
                    id += on;
                }
                if (z + 4 <= L.Rf[2]) {
                    __builtin_memcpy(out + z, l, 16);        // 16 bytes at any multiple of 4
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (z + j < L.Rf[2]) out[z + j] = l[j];
                }
            }
        }
    }
}

// Component c of the eight fine records: sums over corners in (x, y, z) bit order,
// an empty corner 0, in FP64, scaled by their power of two at the end (which
// rounds as scaling each term would) and rounded once to FP32.  Pairs too: an
// FP32 sum of two overflows before its scale brings it back, and rounds twice
// where the scaled value is subnormal.  Sums share their common beginnings.
__device__ __forceinline__ void fine_values(const float v[8][4], int c, float scale, float r[8][4]) {
    const double h = 0.5 * (double)scale, q = 0.25 * (double)scale, e = 0.125 * (double)scale;
    double d[8];
#pragma unroll
    for (int b = 0; b < 8; ++b) d[b] = (double)v[b][c];
    const double s0 = 0.0 + d[0];                           // a sum starts at +0
    const double s01 = s0 + d[1], s3 = s01 + d[2] + d[3];
    r[0][c] = (float)(s0 * (double)scale);
    r[1][c] = (float)(s01 * h);
    r[2][c] = (float)((s0 + d[2]) * h);
    r[3][c] = (float)(s3 * q);
    r[4][c] = (float)((s0 + d[4]) * h);
    r[5][c] = (float)((s01 + d[4] + d[5]) * q);
    r[6][c] = (float)((s0 + d[2] + d[4] + d[6]) * q);
    r[7][c] = (float)((s3 + d[4] + d[5] + d[6] + d[7]) * e);
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// No record: past the end of every buffer, on a 16-byte boundary, and the 16 bytes
// from it end before the offset wraps to the buffer's start.
constexpr uint32_t NOWHERE = 0xfffffff0u;
static_assert(NOWHERE % 16 == 0 && NOWHERE + 12u > NOWHERE, "each word of an access there is out of range");

// Float4s of an array of records, by byte offset.  Not WIDE: a buffer resource of
// the array's size (under 4 GiB), past whose end a load gives 0 and a store does
// nothing, so neither needs a branch.  WIDE: record ids and pointers.
template <bool WIDE>
struct Records {
    float4* base;
    int Q;
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ Records(void* p, int64_t n, int S) : base(static_cast<float4*>(p)), Q(S / 4) {
        rsrc = __builtin_amdgcn_make_buffer_rsrc(p, 0, WIDE ? 0 : (int)(uint32_t)(n * S * 4), 0x00020000);
    }
    // what the list holds for a record id
    __device__ static uint32_t key(int32_t id, int S) {
        return id < 0 ? NOWHERE : WIDE ? (uint32_t)id : (uint32_t)id * (uint32_t)(4 * S);
    }
    __device__ f32x4 load(uint32_t key, uint32_t part) const {
        if constexpr (WIDE) {
            if (key == NOWHERE) return f32x4{0.f, 0.f, 0.f, 0.f};
            return *reinterpret_cast<const f32x4*>(base + (int64_t)key * Q + part);
        } else {
            return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, key == NOWHERE ? key : key + 16 * part, 0, 0));
        }
    }
    __device__ void store(uint32_t key, uint32_t part, f32x4 v) const {
        if constexpr (WIDE) {
            if (key != NOWHERE) *reinterpret_cast<f32x4*>(base + (int64_t)key * Q + part) = v;
        } else {
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rsrc, key == NOWHERE ? key : key + 16 * part, 0, 0);
        }
    }
};

// Records by coarse vertex: coarse vertex v owns the fine vertices
// 2v + o, o in {0,1}^3, and all eight interpolate from the corners v + o' of
// coarse cell v (o' a subset of o's bits; weight 1/2 per odd axis).  A wave
// takes 64 coarse vertices, a lane each (of one row, or of several rows of at most
// 32): it reads their fine links and lists, in LDS, the records around those with an allocated fine vertex (a
// tenth of a sparse map's).  Then a group of 8 lanes takes a listed vertex: lane
// p < S/4 (7 at SH degree 2) fetches float4 p of the 8 corner records and writes
// float4 p of each allocated fine record.
// 256^3 room to 511^3, 20.3 M records of 112 bytes: 1048 us (listing 200), of
// which the writes alone, filled in order, would take 408; 8 lanes for every
// coarse vertex, with branches around each corner and record, took 1446.
// Requesting the next vertex's records early, two z-neighbours' records in one
// store and other orders over the XCDs were no faster.
template <bool WIDE>
__global__ __launch_bounds__(EDIT_THREADS) void k_fine_data(KGrid g, Lattice L, int log_g, const int32_t* __restrict__ link_fine,
                                                            int64_t n_fine, float* __restrict__ out) {
    __shared__ u32x4 s_keys[EDIT_THREADS / WAVE][WAVE][4];   // per listed vertex: 8 corner records, 8 fine records
    const int lane = lane_id(), wave = threadIdx.x / WAVE;
    const int group = 1 << log_g, per_wave = WAVE >> log_g;  // lanes per row segment, segments per wave
    const int segs = (L.R[2] + group - 1) / group;           // segments per row
    const int64_t rows = (int64_t)L.R[0] * L.R[1], items = (rows * segs + per_wave - 1) / per_wave;
    const int64_t waves = (int64_t)gridDim.x * (EDIT_THREADS / WAVE);
    const int S = record_floats(g.deg), Q = S / 4;           // float4 parts per record (at most 7)
    const Records<WIDE> src(const_cast<float*>(g.data), g.n_alloc, S), dst(out, n_fine, S);
    for (int64_t it = ray_tile(blockIdx.x, gridDim.x) * (EDIT_THREADS / WAVE) + wave; it < items; it += waves) {
        const uint32_t seg = (uint32_t)(it * per_wave) + (lane >> log_g), row = seg / (uint32_t)segs;   // fewer than 2^31
        const int vx = (int)(row / (uint32_t)L.R[1]), vy = (int)(row - (uint32_t)vx * L.R[1]);   // vx past the lattice: no vertex
        const int vz = (int)(seg - row * segs) * group + (lane & (group - 1));
        int32_t l[8], f[8];
        bool any = false;
#pragma unroll
        for (int o = 0; o < 8; o += 2) {                     // z pairs, 8 bytes at any multiple of 4
            const int ox = o >> 2, oy = (o >> 1) & 1;
            const int32_t* pair = link_fine + ((int64_t)(2 * vx + ox) * L.Rf[1] + (2 * vy + oy)) * L.Rf[2] + 2 * vz;
            f[o] = f[o + 1] = -1;
            if (vx + ox < L.R[0] && vy + oy < L.R[1]) {
                if (vz + 1 < L.R[2]) __builtin_memcpy(f + o, pair, 8);
                else if (vz < L.R[2]) f[o] = pair[0];
            }
        }
#pragma unroll
        for (int o = 0; o < 8; ++o) {
            if (!link_ok(f[o], n_fine)) f[o] = -1;
            any |= f[o] >= 0;
        }
        const unsigned long long m = __ballot(any);
        if (m == 0ull) continue;
        if (any) {
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const int ox = b >> 2, oy = (b >> 1) & 1, oz = b & 1;
                l[b] = -1;
                if (vx + ox < L.R[0] && vy + oy < L.R[1] && vz + oz < L.R[2])
                    l[b] = g.link[(int64_t)(vx + ox) * g.sx + (int64_t)(vy + oy) * g.sy + (vz + oz)];
            }
#pragma unroll
            for (int b = 0; b < 8; ++b) l[b] = link_ok(l[b], g.n_alloc) ? l[b] : -1;
            u32x4* e = s_keys[wave][__popcll(m & ((1ull << lane) - 1))];
            auto key4 = [&](const int32_t* id) {
                return u32x4{src.key(id[0], S), src.key(id[1], S), src.key(id[2], S), src.key(id[3], S)};
            };
            e[0] = key4(l);
            e[1] = key4(l + 4);
            e[2] = key4(f);
            e[3] = key4(f + 4);
        }
        // the list is this wave's own: order its LDS writes before the reads
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int n = __popcll(m), p = lane & 7;
        for (int base = 0; base < n; base += WAVE / 8) {
            const int i = base + (lane >> 3);
            u32x4 l0 = u32x4(NOWHERE), l1 = u32x4(NOWHERE);
            if (i < n && p < Q) {
                l0 = s_keys[wave][i][0];
                l1 = s_keys[wave][i][1];
            }
            f32x4 cur[8];
#pragma unroll
            for (int b = 0; b < 8; ++b) cur[b] = src.load(b < 4 ? l0[b & 3] : l1[b & 3], p);
            u32x4 f0 = u32x4(NOWHERE), f1 = u32x4(NOWHERE);
            if (i < n && p < Q) {
                f0 = s_keys[wave][i][2];
                f1 = s_keys[wave][i][3];
            }
            float v[8][4], r[8][4];
#pragma unroll
            for (int b = 0; b < 8; ++b)
#pragma unroll
                for (int c = 0; c < 4; ++c) v[b][c] = cur[b][c];
#pragma unroll
            for (int c = 0; c < 4; ++c) fine_values(v, c, c == 0 && p == 0 ? 0.5f : 1.f, r);   // the density is halved
#pragma unroll
            for (int o = 0; o < 8; ++o)
                dst.store(o < 4 ? f0[o & 3] : f1[o & 3], p, f32x4{r[o][0], r[o][1], r[o][2], r[o][3]});
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // the next list overwrites this one
        __builtin_amdgcn_wave_barrier();
    }
}

unsigned stride_blocks(int64_t items, int per_block = EDIT_THREADS) {
    const int64_t b = (items + per_block - 1) / per_block;
    return (unsigned)(b < 1 ? 1 : b > (1 << 20) ? (1 << 20) : b);
}

// Lanes for a row of n items, per_lane to a lane: the logarithm of a power of two, at most a wave.
int group_log2(int n, int per_lane) {
    int lg = 0;
    while (lg < 6 && per_lane << lg < n) ++lg;
    return lg;
}

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

Lattice lattice(const KGrid& g) {
    Lattice L;
    for (int a = 0; a < 3; ++a) {
        L.R[a] = g.R[a];
        L.Rf[a] = 2 * g.R[a] - 1;
    }
    L.WC = (L.R[2] + 31) / 32;
    L.WF = (L.Rf[2] + 31) / 32;
    return L;
}

// Workspace of a compaction over nw flag words: words, word prefixes, chunk
// totals (then offsets), each 256-byte aligned.
struct Compaction {
    uint32_t* words;
    int32_t* wpre;
    int32_t* chunk;
    int64_t n_chunks;
};

size_t compaction_words_bytes(int64_t nw) {
    return 2 * align256(nw * 4) + align256((nw + EDIT_WORDS - 1) / EDIT_WORDS * 4);
}

Compaction carve(void* ws, int64_t nw) {
    char* p = static_cast<char*>(ws);
    Compaction c;
    c.words = reinterpret_cast<uint32_t*>(p);
    c.wpre = reinterpret_cast<int32_t*>(p + align256(nw * 4));
    c.chunk = reinterpret_cast<int32_t*>(p + 2 * align256(nw * 4));
    c.n_chunks = (nw + EDIT_WORDS - 1) / EDIT_WORDS;
    return c;
}

hipError_t scan(const Compaction& c, int64_t* n_out, hipStream_t st) {
    hipLaunchKernelGGL(k_scan_chunks, dim3(1), dim3(SCAN_THREADS), 0, st, c.chunk, c.n_chunks, n_out);
    return hipGetLastError();
}

}  // namespace

size_t prune_workspace_bytes(int64_t n_alloc) { return compaction_words_bytes((n_alloc + 31) / 32) + 4 * n_alloc; }

size_t grow_workspace_bytes(const int R[3]) {
    const int64_t rows_c = (int64_t)R[0] * R[1], rows_f = (int64_t)(2 * R[0] - 1) * (2 * R[1] - 1);
    const int64_t wc = (R[2] + 31) / 32, wf = (2 * R[2] - 1 + 31) / 32;
    return align256(rows_c * wc * 4) + compaction_words_bytes(rows_f * wf);
}

hipError_t launch_upsample_link(const KGrid& g, int32_t* link_fine, int64_t* n_fine, void* ws, hipStream_t st) {
    const Lattice L = lattice(g);
    const int64_t rows_c = (int64_t)L.R[0] * L.R[1], rows_f = (int64_t)L.Rf[0] * L.Rf[1];
    uint32_t* vbits = static_cast<uint32_t*>(ws);
    const int64_t n_coarse_items = rows_c * L.WC * 32, nw = rows_f * L.WF;
    const Compaction c = carve(static_cast<char*>(ws) + align256(rows_c * L.WC * 4), nw);
    hipLaunchKernelGGL(k_coarse_bits, dim3(stride_blocks(n_coarse_items)), dim3(EDIT_THREADS), 0, st, g, L,
                       n_coarse_items, vbits);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_grow_flags, dim3((unsigned)c.n_chunks), dim3(EDIT_THREADS), 0, st, vbits, L, nw, c.words,
                       c.wpre, c.chunk);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = scan(c, n_fine, st)) != hipSuccess) return e;
    const int log_g = group_log2(L.Rf[2], 4 * ROW_STEPS);
    hipLaunchKernelGGL(k_fine_link, dim3(stride_blocks(rows_f, EDIT_THREADS >> log_g)), dim3(EDIT_THREADS), 0, st, L, log_g, c.words,
                       c.wpre, c.chunk, link_fine);
    return hipGetLastError();
}

hipError_t launch_upsample_data(const KGrid& g, const int32_t* link_fine, int64_t n_fine, float* data_fine,
                                hipStream_t st) {
    const Lattice L = lattice(g);
    // a row of at most 32 vertices shares its wave: 1024 x 1024 x 8 vertices, one in
    // a hundred allocated, 393 us, 996 with a wave to every row
    const int log_g = group_log2(L.R[2], 1);
    const int64_t segs = (int64_t)L.R[0] * L.R[1] * ((L.R[2] + (1 << log_g) - 1) >> log_g);
    const uint64_t bytes = (uint64_t)(g.n_alloc > n_fine ? g.n_alloc : n_fine) * (4 * record_floats(g.deg));
    hipLaunchKernelGGL(bytes < NOWHERE ? k_fine_data<false> : k_fine_data<true>, dim3(stride_blocks(segs, EDIT_THREADS >> log_g)), dim3(EDIT_THREADS), 0, st, g, L, log_g, link_fine,
                       n_fine, data_fine);
    return hipGetLastError();
}

hipError_t launch_prune(const KGrid& g, float tau, int32_t* link_out, float* data_out, int64_t* n_out, void* ws,
                        hipStream_t st) {
    const int64_t n = g.n_alloc, nv = (int64_t)g.R[0] * g.R[1] * g.R[2], nw = (n + 31) / 32;
    const Compaction c = carve(ws, nw);
    int32_t* remap = reinterpret_cast<int32_t*>(static_cast<char*>(ws) + compaction_words_bytes(nw));
    hipError_t e;
    if (c.n_chunks > 0) {
        hipLaunchKernelGGL(k_keep_flags, dim3((unsigned)c.n_chunks), dim3(EDIT_THREADS), 0, st, g.data,
                           record_floats(g.deg), tau, n, c.words,
                           c.wpre, c.chunk);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if ((e = scan(c, n_out, st)) != hipSuccess) return e;
    if (n > 0) {
        hipLaunchKernelGGL(k_prune_copy, dim3(stride_blocks(n * 8)), dim3(EDIT_THREADS), 0, st, g.data,
                           record_floats(g.deg), n, c.words,
                           c.wpre, c.chunk, remap, data_out);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_relink, dim3(stride_blocks(nv, LINK_ITEMS)), dim3(EDIT_THREADS), 0, st, g.link, nv, n, remap, link_out);
    return hipGetLastError();
}

}  // namespace pxm
