// merf_ingest.hip -- device-side scene ingest: packing of stored blocks into
// apron bricks, and max-pooling of a binary occupancy mask into the coarser
// levels of the empty-space hierarchy (Sec. 6 builds its occupancy grids by
// max-pooling the full-resolution mask; Sec. 5.3 stores the grid in a
// block-sparse format); and the empty-space distance grid the renderer skips
// with, derived from the occupancy levels.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "merf_device.h"

namespace merf {

namespace {

constexpr int kBrickVoxels = kBrick * kBrick * kBrick;   // 729

// One thread per voxel of a brick: copy the 8 channels of voxel
// (8 b + l) from its stored block, or zeros for an absent block, outside the
// grid, or for the shared zero brick (slot == nbricks).
__global__ void k_pack_bricks(const uint8_t *__restrict__ blocks, const int32_t *__restrict__ block_index,
                              const int32_t *__restrict__ brick_pos, int nbricks, int L, int nbl,
                              uint8_t *__restrict__ bricks) {
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t total = (int64_t)(nbricks + 1) * kBrickVoxels;
    if (gid >= total) return;
    const int slot = (int)(gid / kBrickVoxels), v = (int)(gid % kBrickVoxels);
    uint2 val = make_uint2(0u, 0u);
    if (slot < nbricks) {
        const int pos = brick_pos[slot];
        const int bx = pos & 1023, by = (pos >> 10) & 1023, bz = pos >> 20;
        const int lz = v / (kBrick * kBrick), ly = (v / kBrick) % kBrick, lx = v % kBrick;
        const int x = bx * kBlock + lx, y = by * kBlock + ly, z = bz * kBlock + lz;
        if (x < L && y < L && z < L) {
            const int src = block_index[((size_t)(z / kBlock) * nbl + (y / kBlock)) * nbl + (x / kBlock)];
            if (src >= 0) {
                const size_t off = ((((size_t)src * kBlock + (z % kBlock)) * kBlock + (y % kBlock)) * kBlock +
                                    (x % kBlock)) * kChannels;
                val = *reinterpret_cast<const uint2 *>(blocks + off);
            }
        }
    }
    *reinterpret_cast<uint2 *>(bricks + (size_t)slot * kBrickBytes + (size_t)v * kChannels) = val;
}

// Max-pooling of a mask, several levels in one launch (PoolLevels).  Pooling
// reads the mask once and is bound by that: a workgroup takes `rows`
// consecutive output rows (of one z) of one level, reads the f x f input rows
// of each as whole vectors of V, consecutive lanes on consecutive addresses
// and eight in flight a thread, and ORs what is not zero (most of a mask is)
// into one row image in LDS; an output cell is then the OR of f bytes there.
// A level of few rows with many vectors each is split over workgroups by
// input z (parts); these only store ones, over zeros that k_pool_clear wrote.
// Three levels of a 512^3 mask take 35 us (3.9 TB/s of the mask; a plain copy
// reaches 5.2 TB/s of traffic).  (A thread per output cell reading its f^3
// bytes one by one took 1.26 ms a
// level of a 512^3 mask.)
constexpr int kPoolFlight = 8;
template <typename V>
__global__ __launch_bounds__(256) void k_pool_rows(const PoolLevels lv) {
    extern __shared__ uint32_t image[];                       // [rows][rin rounded up to 4 bytes]
    int l = 0;
    while (l + 1 < lv.n && (int)blockIdx.x >= lv.level[l + 1].first_block) ++l;
    const PoolLevel L = lv.level[l];
    const int f = L.factor, rin = L.rin, rout = rin / f, t = (int)threadIdx.x, nt = (int)blockDim.x;
    const int words = (rin + 3) / 4, nvec = rin / (int)sizeof(V), per_z = (rout + L.rows - 1) / L.rows;
    const int block = (int)blockIdx.x - L.first_block, part = block % L.parts;
    const int oz = block / L.parts / per_z, oy = (block / L.parts - oz * per_z) * L.rows;
    const int rows = min(L.rows, rout - oy), ny = rows * f, z1 = (part + 1) * f / L.parts;
    for (int i = t; i < rows * words; i += nt) image[i] = 0u;
    __syncthreads();
    // a thread keeps its vector v of the row; its group of threads takes every
    // groups-th input row y of each z.  Output row y / f: with more than one,
    // f y < 2^16, so the rounded-up reciprocal is exact.
    const int lanes = min(nvec, nt), groups = nt / lanes, g = t / lanes;
    const uint32_t rf = rows > 1 ? (65536u + (uint32_t)f - 1u) / (uint32_t)f : 0u;
    for (int v = t - g * lanes; g < groups && v < nvec; v += lanes) {
        const V *in = reinterpret_cast<const V *>(L.in + ((size_t)oz * f * rin + (size_t)oy * f) * rin) + v;
        int z = part * f / L.parts, y = g;
        bool seen = false;
        while (z < z1 && !seen) {
            V x[kPoolFlight];
            int at[kPoolFlight];
#pragma unroll
            for (int u = 0; u < kPoolFlight; ++u) {
                const bool in_range = z < z1 && y < ny;
                x[u] = in_range ? in[((size_t)z * rin + y) * nvec] : V{};
                at[u] = (int)(((uint32_t)y * rf) >> 16) * words;
                y += groups;
                if (y >= ny) {
                    y = g;
                    ++z;
                }
            }
#pragma unroll
            for (int u = 0; u < kPoolFlight; ++u) {
                if constexpr (sizeof(V) == 16) {
                    uint32_t *w = image + at[u] + 4 * v;
                    if (x[u].x) atomicOr(w, x[u].x);
                    if (x[u].y) atomicOr(w + 1, x[u].y);
                    if (x[u].z) atomicOr(w + 2, x[u].z);
                    if (x[u].w) atomicOr(w + 3, x[u].w);
                    // one output cell holds the whole vector: its other
                    // vectors at this v add nothing
                    seen = seen || (rows == 1 && f % 16 == 0 && (x[u].x | x[u].y | x[u].z | x[u].w));
                } else {
                    if (x[u])
                        atomicOr(image + at[u] + v * (int)sizeof(V) / 4, (uint32_t)x[u] << (8 * (v * (int)sizeof(V) % 4)));
                }
            }
        }
    }
    __syncthreads();
    for (int i = t; i < rows * rout; i += nt) {
        const int j = i / rout, x = i - j * rout;
        uint32_t any = 0u;
        if (f % 4 == 0) {
            for (int k = 0; k < f / 4; ++k) any |= image[j * words + x * (f / 4) + k];
        } else {
            const uint8_t *c = reinterpret_cast<const uint8_t *>(image + j * words) + x * f;
            for (int k = 0; k < f; ++k) any |= c[k];
        }
        uint8_t *o = L.out + ((size_t)oz * rout + oy) * rout + i;
        if (L.parts == 1) *o = any ? 1 : 0;
        else if (any) *o = 1;
    }
}

__global__ __launch_bounds__(256) void k_pool_clear(uint8_t *__restrict__ out, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) out[i] = 0;
}

// Empty-space distance grid, step 1: the cell of the finest level is
// occupied when every level marks the cell containing it (the levels nest,
// so each finest cell lies in one cell of every level).  Output is the seed
// of the distance transform: 0 for occupied, 255 for empty.
__global__ void k_occ_combine(const OccLevels lv, uint8_t *__restrict__ out) {
    const int rf = lv.res[lv.n - 1];
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= (int64_t)rf * rf * rf) return;
    const int x = (int)(gid % rf), y = (int)((gid / rf) % rf), z = (int)(gid / ((int64_t)rf * rf));
    bool occ = true;
    for (int l = 0; l < lv.n && occ; ++l) {
        const int r = lv.res[l], k = rf / r;
        occ = lv.occ[l][((size_t)(z / k) * r + (y / k)) * r + (x / k)] != 0;
    }
    out[gid] = occ ? 0 : 255;
}

// Step 2, one pass per axis: the Chebyshev (L-infinity) distance to the
// nearest occupied cell is separable,
//   d(c) = min over cells t of the line through c along the axis of
//          max(|c_a - t_a|, d_prev(t)),
// starting from the seed and applied along x, then y, then z; values are
// capped at 255 (a cap only shortens skips).  One workgroup per line, the
// line staged in LDS; each cell scans outwards and stops once the offset
// reaches its best distance.
__global__ void k_dist_axis(const uint8_t *__restrict__ in, uint8_t *__restrict__ out, int r, int axis) {
    __shared__ uint8_t line[kMaxDistRes];
    const int64_t lid = blockIdx.x;
    int64_t base, stride;
    if (axis == 0) { base = lid * r; stride = 1; }
    else if (axis == 1) { base = (lid / r) * r * r + lid % r; stride = r; }
    else { base = lid; stride = (int64_t)r * r; }
    for (int c = (int)threadIdx.x; c < r; c += (int)blockDim.x) line[c] = in[base + c * stride];
    __syncthreads();
    for (int c = (int)threadIdx.x; c < r; c += (int)blockDim.x) {
        int best = line[c];
        for (int dd = 1; dd < best; ++dd) {
            if (c - dd >= 0) best = min(best, max(dd, (int)line[c - dd]));
            if (c + dd < r) best = min(best, max(dd, (int)line[c + dd]));
        }
        out[base + c * stride] = (uint8_t)best;
    }
}

// Forward empty extents.  E(c) of octant (sx, sy, sz) is the edge of the
// largest empty cube with a corner at cell c that extends the octant's way
// (cells outside the grid are empty; at most 255).  A cube of edge m at c is
// its face in c's z plane, its face in c's y plane and the two cubes of edge
// m - 1 one step along (sy, sz) from c, with and without a step along sx:
//   E(c)   = min(Fxy(c), Fxz(c), 1 + E(c + (0, sy, sz)), 1 + E(c + (sx, sy, sz))),
// with Fxy the largest empty square at c in its z plane, which in the same way
// is a row and two squares,
//   Fxy(c) = min(Gx(c), 1 + Fxy(c + (0, sy, 0)), 1 + Fxy(c + (sx, sy, 0))),
// Fxz likewise, and Gx the run of empty cells from c along x (0 at an occupied
// cell).  So three kernels take a cell a constant number of steps each and are
// bound by their traffic, 43 bytes a cell for the eight grids: 167 us for 256^3
// cells (4.3 TB/s; a plain copy reaches 5.2).
// (Growing from the cube on the diagonal needs all three faces and the runs
// along y and z, 63 bytes a cell: 278 us.  A bisection of each extent in a
// table of prefix sums takes 64 lookups per cell and octant: 4.25 ms.)
// Bytes are held as pairs of 16-bit lanes (the even and the odd cells of a
// word), so packed 16-bit instructions do two cells at a time, and a lane
// group holds a whole row of x in registers: a step along the diagonal is then
// a shift by one cell through the row and a step of the row's address.
// Lines of rows are independent; their rows are loaded several steps ahead.
// Rows in scratch are padded to rp = 16 n cells; padding is outside the grid.
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// N cells of one lane: e the even and o the odd cells of each word.
template <int N>
struct Cells {
    static constexpr int W = N / 4;
    u16x2 e[W], o[W];
};
__device__ __forceinline__ u16x2 as_u16x2(uint32_t w) { return __builtin_bit_cast(u16x2, w); }
__device__ __forceinline__ uint32_t as_u32(u16x2 v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ u16x2 splat(int v) { return u16x2{(unsigned short)v, (unsigned short)v}; }

template <int N>
struct Row {
    uint32_t w[N / 4];
};
template <int N>
__device__ __forceinline__ Row<N> load_row(const uint8_t *p) {
    Row<N> x;
    if constexpr (N == 16) {
        const uint4 v = *reinterpret_cast<const uint4 *>(p);
        x.w[0] = v.x; x.w[1] = v.y; x.w[2] = v.z; x.w[3] = v.w;
    } else {
        x.w[0] = *reinterpret_cast<const uint32_t *>(p);
    }
    return x;
}
template <int N>
__device__ __forceinline__ void store_row(uint8_t *p, const Row<N> &x) {
    if constexpr (N == 16) *reinterpret_cast<uint4 *>(p) = make_uint4(x.w[0], x.w[1], x.w[2], x.w[3]);
    else *reinterpret_cast<uint32_t *>(p) = x.w[0];
}
template <int N>
__device__ __forceinline__ Cells<N> unpack(const Row<N> &x) {
    Cells<N> c;
#pragma unroll
    for (int i = 0; i < N / 4; ++i) {
        c.e[i] = as_u16x2(x.w[i] & 0x00ff00ffu);
        c.o[i] = as_u16x2((x.w[i] >> 8) & 0x00ff00ffu);
    }
    return c;
}
template <int N>
__device__ __forceinline__ Row<N> pack(const Cells<N> &c) {
    Row<N> x;
#pragma unroll
    for (int i = 0; i < N / 4; ++i) x.w[i] = as_u32(c.e[i]) | as_u32(c.o[i]) << 8;
    return x;
}
template <int N>
__device__ __forceinline__ Cells<N> fill_cells(int v) {
    Cells<N> c;
#pragma unroll
    for (int i = 0; i < N / 4; ++i) c.e[i] = c.o[i] = splat(v);
    return c;
}
template <int N>
__device__ __forceinline__ Cells<N> min_cells(const Cells<N> &a, const Cells<N> &b) {
    Cells<N> c;
#pragma unroll
    for (int i = 0; i < N / 4; ++i) {
        c.e[i] = __builtin_elementwise_min(a.e[i], b.e[i]);
        c.o[i] = __builtin_elementwise_min(a.o[i], b.o[i]);
    }
    return c;
}
template <int N>
__device__ __forceinline__ Cells<N> plus_one(const Cells<N> &a) {
    Cells<N> c;
#pragma unroll
    for (int i = 0; i < N / 4; ++i) {
        c.e[i] = a.e[i] + splat(1);
        c.o[i] = a.o[i] + splat(1);
    }
    return c;
}
// The cells one further along x (neg: one back); past the row's end 255.
// last: this lane holds the row's end on that side.
template <int N>
__device__ __forceinline__ Cells<N> shift_x(const Cells<N> &a, bool neg, bool last) {
    constexpr int W = N / 4;
    Cells<N> c;
    if (!neg) {
        uint32_t in = (uint32_t)__shfl_down((int)as_u32(a.e[0]), 1, 64);
        in = last ? 255u : in;
#pragma unroll
        for (int i = 0; i < W; ++i) {
            c.e[i] = a.o[i];
            c.o[i] = as_u16x2(as_u32(a.e[i]) >> 16 | (i + 1 < W ? as_u32(a.e[i + 1 < W ? i + 1 : i]) : in) << 16);
        }
    } else {
        uint32_t in = (uint32_t)__shfl_up((int)as_u32(a.o[W - 1]), 1, 64);
        in = last ? 255u << 16 : in;
#pragma unroll
        for (int i = 0; i < W; ++i) {
            c.o[i] = a.e[i];
            c.e[i] = as_u16x2(as_u32(a.o[i]) << 16 | (i > 0 ? as_u32(a.o[i > 0 ? i - 1 : i]) : in) >> 16);
        }
    }
    return c;
}

// What the cubes (or squares) of the row before allow: 1 + the smaller of each
// cell's and of the next one's along x.
template <int N>
__device__ __forceinline__ Cells<N> grow(const Cells<N> &a, bool neg, bool last) {
    return plus_one<N>(min_cells<N>(a, shift_x<N>(a, neg, last)));
}

// Rows of a wave: a row takes rp / N lanes, a wave as many rows as fit.
template <int N>
struct Lanes {
    int per_row, i, row;            // lanes of a row, this lane's place in it, the row (in the wave)
    __device__ __forceinline__ explicit Lanes(int rp) {
        const int lane = (int)threadIdx.x & 63;
        per_row = rp / N;
        row = lane / per_row;
        i = lane - row * per_row;
        if (row >= 64 / per_row) row = 1 << 20;               // a lane left over
    }
};

// Step 1, a lane group per row of x: the cells occupied at every level and the
// runs of empty cells along +x (gx[0]) and -x (gx[1]).  The next occupied cell
// past a lane's own comes from the nearest lane that has one (a ballot and one
// shuffle each way).  Bound by its instructions, most of them once a lane: with
// 16 cells a lane it takes 27 us for 256^3 cells, with 4 it takes 37.
constexpr int kRunWaves = 4;
template <int N>
__global__ __launch_bounds__(64 * kRunWaves) void k_runs_x(const OccLevels lv, const OctantScratch sc) {
    const int r = sc.r, rp = sc.rp;
    const Lanes<N> ln(rp);
    const uint32_t wave = blockIdx.x * (uint32_t)kRunWaves + threadIdx.x / 64u;
    const uint32_t row = wave * (uint32_t)(64 / ln.per_row) + (uint32_t)ln.row;
    const bool live = row < (uint32_t)r * (uint32_t)r;
    const int y = (int)(row % (uint32_t)r), z = (int)(row / (uint32_t)r), x0 = ln.i * N;
    uint32_t occ = 0u;                                        // bit k: cell x0 + k
    if (live) {
        const uint8_t *fine = lv.occ[lv.n - 1] + ((size_t)z * r + y) * r;
        uint8_t b[N];
        if (x0 + N <= r && (reinterpret_cast<uintptr_t>(fine + x0) & 3) == 0) {
#pragma unroll
            for (int w = 0; w < N / 4; ++w) {
                const uint32_t v = reinterpret_cast<const uint32_t *>(fine + x0)[w];
#pragma unroll
                for (int k = 0; k < 4; ++k) b[4 * w + k] = (uint8_t)(v >> (8 * k));
            }
        } else {
#pragma unroll
            for (int k = 0; k < N; ++k) b[k] = x0 + k < r ? fine[x0 + k] : (uint8_t)0;
        }
#pragma unroll
        for (int k = 0; k < N; ++k) occ |= b[k] ? 1u << k : 0u;
        // coarser levels for the cells occupied at the finest
        for (int l = 0; l + 1 < lv.n && occ; ++l) {
            const int rl = lv.res[l], q = r / rl;
            const uint8_t *o = lv.occ[l] + ((size_t)(z / q) * rl + y / q) * rl;
            int cell = x0 / q, left = q - (x0 - cell * q);    // cells of q left in the coarse one
            uint8_t c[N];                                     // (loads in flight together; none past the row)
#pragma unroll
            for (int k = 0; k < N; ++k) {
                c[k] = o[min(cell, rl - 1)];
                if (--left == 0) {
                    ++cell;
                    left = q;
                }
            }
#pragma unroll
            for (int k = 0; k < N; ++k) occ &= c[k] ? ~0u : ~(1u << k);
        }
    }
    const uint64_t have = __builtin_amdgcn_ballot_w64(occ != 0);
    const int lane = (int)threadIdx.x & 63, first = lane - ln.i;   // first lane of the row
    const uint64_t in_row = (ln.per_row == 64 ? ~0ull : (1ull << ln.per_row) - 1) << (first & 63);
    const uint64_t after = lane < 63 ? have & in_row & (~0ull << (lane + 1)) : 0ull;
    const uint64_t before = have & in_row & ((1ull << lane) - 1);
    const int la = after ? __builtin_ctzll(after) : lane, lb = before ? 63 - __builtin_clzll(before) : lane;
    const uint32_t oa = (uint32_t)__shfl((int)occ, la, 64), ob = (uint32_t)__shfl((int)occ, lb, 64);
    // distances from this lane's last / first cell to the next occupied one
    int run = after ? (la - lane - 1) * N + __builtin_ctz(oa | 1u << 31) : 255;
    uint8_t g[N];
#pragma unroll
    for (int k = N - 1; k >= 0; --k) {
        run = (occ >> k & 1u) ? 0 : min(run + 1, 255);
        g[k] = (uint8_t)run;
    }
    auto put = [&](uint8_t *to) {
        Row<N> w;
#pragma unroll
        for (int i = 0; i < N / 4; ++i)
            w.w[i] = (uint32_t)g[4 * i] | (uint32_t)g[4 * i + 1] << 8 | (uint32_t)g[4 * i + 2] << 16 | (uint32_t)g[4 * i + 3] << 24;
        if (live) store_row<N>(to + (size_t)row * rp + x0, w);
    };
    if (sc.gx[0]) put(sc.gx[0]);
    run = before ? (lane - lb - 1) * N + (N - 1 - (31 - __builtin_clz(ob | 1u))) : 255;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        run = (occ >> k & 1u) ? 0 : min(run + 1, 255);
        g[k] = (uint8_t)run;
    }
    if (sc.gx[1]) put(sc.gx[1]);
}

// Step 2: the squares of the planes that x spans with y (blockIdx.z = 0) and
// with z (1), for each sign of x (bit 0 of the combination) and of the other
// axis (bit 1): a lane group per line of rows marches along that axis, from its
// far end.
constexpr int kRowsAhead = 8;
template <int N>
__global__ __launch_bounds__(64) void k_squares_x(const OctantScratch sc, int first_xy, int first_xz) {
    const bool along_z = blockIdx.z != 0;
    const int r = sc.r, rp = sc.rp, combo = (along_z ? first_xz : first_xy) + (int)blockIdx.y, sx = combo & 1;
    const Lanes<N> ln(rp);
    const int line = (int)blockIdx.x * (64 / ln.per_row) + ln.row;
    const bool live = line < r, last = ln.i == (sx ? 0 : ln.per_row - 1), up = combo >> 1;
    const int64_t stride = (int64_t)rp * (along_z ? r : 1), step = up ? stride : -stride;
    int64_t at = (live ? (int64_t)line * rp * (along_z ? 1 : r) : 0) + ln.i % ln.per_row * N + (up ? 0 : (int64_t)(r - 1) * stride);
    const uint8_t *gx = sc.gx[sx];
    uint8_t *f = (along_z ? sc.fxz : sc.fxy)[combo];
    Cells<N> sq = fill_cells<N>(255);
    Row<N> ahead[kRowsAhead];
#pragma unroll
    for (int u = 0; u < kRowsAhead; ++u) ahead[u] = load_row<N>(gx + at + (int64_t)min(u, r - 1) * step);
    for (int s0 = 0; s0 < r; s0 += kRowsAhead) {
        Row<N> cur[kRowsAhead];
#pragma unroll
        for (int u = 0; u < kRowsAhead; ++u) {
            cur[u] = ahead[u];
            ahead[u] = load_row<N>(gx + at + (int64_t)min(kRowsAhead + u, r - 1 - s0) * step);
        }
#pragma unroll
        for (int u = 0; u < kRowsAhead; ++u) {
            if (s0 + u < r) {
                sq = min_cells<N>(unpack<N>(cur[u]), grow<N>(sq, sx != 0, last));
                if (live) store_row<N>(f + at, pack<N>(sq));
                at += step;
            }
        }
    }
}

// Step 3: for each octant, a lane group per diagonal of rows in (y, z).  Line d starts at row y = d of the
// far z; where y leaves the grid the line goes on as another diagonal, from
// the far y.
template <int N>
__global__ __launch_bounds__(64) void k_extents(const OctantScratch sc, int first_octant, bool words, uint8_t *__restrict__ out) {
    constexpr int kAhead = N == 16 ? 4 : 8;
    const int r = sc.r, rp = sc.rp, o = first_octant + (int)blockIdx.y, sx = o & 1, sy = o >> 1 & 1, sz = o >> 2;
    const Lanes<N> ln(rp);
    const int line = (int)blockIdx.x * (64 / ln.per_row) + ln.row;
    const bool live = line < r, last = ln.i == (sx ? 0 : ln.per_row - 1);
    const int x0 = ln.i % ln.per_row * N, d = live ? line : 0;
    const uint8_t *fxy = sc.fxy[sx | sy << 1], *fxz = sc.fxz[sx | sz << 1];
    uint8_t *to = out + (sc.single ? 0 : (size_t)o * r * r * r);
    // rows (y, z) of step s: z from the far end, y from d the same way
    auto y_of = [&](int s) {
        const int y = sy ? d + s : d - s;
        return y >= r ? y - r : y < 0 ? y + r : y;
    };
    auto row_of = [&](int s) { return (uint32_t)((sz ? s : r - 1 - s) * r + y_of(s)); };
    Cells<N> e = fill_cells<N>(255);
    Row<N> a0[kAhead], a1[kAhead];
    auto fetch = [&](int u, int s) {
        const size_t at = (size_t)row_of(min(s, r - 1)) * rp + x0;
        a0[u] = load_row<N>(fxy + at);
        a1[u] = load_row<N>(fxz + at);
    };
#pragma unroll
    for (int u = 0; u < kAhead; ++u) fetch(u, u);
    for (int s0 = 0; s0 < r; s0 += kAhead) {
        Row<N> b0[kAhead], b1[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            b0[u] = a0[u];
            b1[u] = a1[u];
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) fetch(u, s0 + kAhead + u);
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int s = s0 + u;
            if (s < r) {
                if (y_of(s) == (sy ? 0 : r - 1)) e = fill_cells<N>(255);      // the row before it is outside
                e = min_cells<N>(grow<N>(e, sx != 0, last), min_cells<N>(unpack<N>(b0[u]), unpack<N>(b1[u])));
                const Row<N> w = pack<N>(e);
                if (live) {
                    uint8_t *p = to + (size_t)row_of(s) * r + x0;
#pragma unroll
                    for (int i = 0; i < N / 4; ++i) {
                        if (words) {
                            if (x0 + 4 * i < r) reinterpret_cast<uint32_t *>(p)[i] = w.w[i];
                        } else {
#pragma unroll
                            for (int k = 0; k < 4; ++k)
                                if (x0 + 4 * i + k < r) p[4 * i + k] = (uint8_t)(w.w[i] >> (8 * k));
                        }
                    }
                }
            }
        }
    }
}

}  // namespace

namespace {

template <int N>
hipError_t octant_extents(const OccLevels &lv, bool together, uint8_t *scratch, uint8_t *out, hipStream_t stream) {
    OctantScratch sc{};
    sc.r = lv.res[lv.n - 1];
    sc.rp = (sc.r + 15) / 16 * 16;
    sc.single = !together;
    const size_t r = (size_t)sc.r, n = r * r * r, grid = r * r * (size_t)sc.rp;
    const unsigned rows = 64u / (unsigned)(sc.rp / N);        // rows of a wave
    const size_t run_rows = 64u / (unsigned)(sc.rp / 16) * kRunWaves;         // rows of a workgroup of k_runs_x
    const unsigned row_blocks = (unsigned)((r * r + run_rows - 1) / run_rows), line_blocks = (unsigned)((r + rows - 1) / rows);
    const bool words = r % 4 == 0 && reinterpret_cast<uintptr_t>(out) % 4 == 0;
    for (int o = 0; o < (sc.single ? 8 : 1); ++o) {
        const int sx = o & 1, sy = o >> 1 & 1, sz = o >> 2;
        size_t k = 0;
        auto next = [&]() { return scratch + grid * k++; };
        if (sc.single) {
            sc.gx[0] = sc.gx[1] = nullptr;
            sc.gx[sx] = next();
            sc.fxy[sx | sy << 1] = next();
            sc.fxz[sx | sz << 1] = next();
        } else {
            for (int i = 0; i < 2; ++i) sc.gx[i] = next();
            for (int i = 0; i < 4; ++i) {
                sc.fxy[i] = next();
                sc.fxz[i] = next();
            }
        }
        const unsigned combos = sc.single ? 1 : 4, octants = sc.single ? 1 : 8;
        hipLaunchKernelGGL(k_runs_x<16>, dim3(row_blocks), dim3(64 * kRunWaves), 0, stream, lv, sc);
        hipLaunchKernelGGL(k_squares_x<N>, dim3(line_blocks, combos, 2), dim3(64), 0, stream, sc, sx | sy << 1, sx | sz << 1);
        hipLaunchKernelGGL(k_extents<N>, dim3(line_blocks, octants), dim3(64), 0, stream, sc, o, words,
                           out + (sc.single ? (size_t)o * n : 0));
    }
    return hipGetLastError();
}

}  // namespace

// The marching steps: a row of up to 256 cells takes at most 64 lanes of four
// (few lines march, so each takes more lanes); larger ones have 16 cells a lane.
hipError_t launch_octant_extents(const OccLevels &lv, bool together, uint8_t *scratch, uint8_t *out, hipStream_t stream) {
    const int r = lv.res[lv.n - 1];
    if (r <= 0 || r > kMaxDistRes || (together && r > kOctMaxRes)) return hipErrorInvalidValue;
    return r <= 256 ? octant_extents<4>(lv, together, scratch, out, stream)
                    : octant_extents<16>(lv, together, scratch, out, stream);
}

hipError_t launch_pack_bricks(const uint8_t *blocks, const int32_t *block_index, const int32_t *brick_pos,
                              int nbricks, int L, uint8_t *bricks, hipStream_t stream) {
    const int64_t total = (int64_t)(nbricks + 1) * kBrickVoxels;
    const int64_t grid = (total + 255) / 256;
    hipLaunchKernelGGL(k_pack_bricks, dim3((unsigned)grid), dim3(256), 0, stream, blocks, block_index, brick_pos,
                       nbricks, L, L / kBlock, bricks);
    return hipGetLastError();
}

hipError_t launch_distance_grid(const OccLevels &lv, uint8_t *tmp0, uint8_t *tmp1, uint8_t *dist,
                                hipStream_t stream) {
    const int r = lv.res[lv.n - 1];
    const int64_t n = (int64_t)r * r * r;
    if (n <= 0 || r > kMaxDistRes) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_occ_combine, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, lv, tmp0);
    const dim3 lines((unsigned)((int64_t)r * r)), block(256);
    hipLaunchKernelGGL(k_dist_axis, lines, block, 0, stream, tmp0, tmp1, r, 0);
    hipLaunchKernelGGL(k_dist_axis, lines, block, 0, stream, tmp1, tmp0, r, 1);
    hipLaunchKernelGGL(k_dist_axis, lines, block, 0, stream, tmp0, dist, r, 2);
    return hipGetLastError();
}

namespace {

// Whether every row of a level's input starts on a multiple of a bytes.
bool rows_aligned(const PoolLevel &p, uintptr_t a) { return reinterpret_cast<uintptr_t>(p.in) % a == 0 && p.rin % a == 0; }

hipError_t launch_pool_stage(PoolLevels &lv, hipStream_t stream) {
    if (lv.n == 0) return hipSuccess;
    // vectors of 16 bytes where every level's rows are aligned to them, else
    // of 4, else bytes
    bool a16 = true, a4 = true;
    for (int l = 0; l < lv.n; ++l) {
        a16 = a16 && rows_aligned(lv.level[l], 16);
        a4 = a4 && rows_aligned(lv.level[l], 4);
    }
    const int64_t vec = a16 ? 16 : a4 ? 4 : 1;
    // A workgroup's share: output rows of one z that need up to 2048 vectors
    // (eight in flight per thread of 256) and 8 KB of row images, or one row.
    // A row of more than 16384 vectors (64 per thread) is split: the 16^3 level
    // of a 512^3 mask has 256 rows of 32768, one for each of 256 compute units.
    int64_t blocks = 0;
    size_t lds = 0;
    for (int l = 0; l < lv.n; ++l) {
        PoolLevel &p = lv.level[l];
        const int64_t rout = p.rin / p.factor, words = (p.rin + 3) / 4;
        const int64_t per_row = (int64_t)p.factor * p.factor * (p.rin / vec);
        p.rows = (int32_t)std::max<int64_t>(1, std::min<int64_t>(rout, std::min(2048 / per_row, 2048 / words)));
        p.parts = (int32_t)std::min<int64_t>(p.factor, (per_row + 16383) / 16384);
        p.first_block = (int32_t)blocks;
        blocks += rout * ((rout + p.rows - 1) / p.rows) * p.parts;
        lds = std::max(lds, (size_t)(p.rows * words * 4));
        if (p.parts > 1)
            hipLaunchKernelGGL(k_pool_clear, dim3((unsigned)((rout * rout * rout + 255) / 256)), dim3(256), 0, stream, p.out,
                               rout * rout * rout);
    }
    const dim3 grid((unsigned)blocks), block(256);
    if (a16) hipLaunchKernelGGL(k_pool_rows<uint4>, grid, block, lds, stream, lv);
    else if (a4) hipLaunchKernelGGL(k_pool_rows<uint32_t>, grid, block, lds, stream, lv);
    else hipLaunchKernelGGL(k_pool_rows<uint8_t>, grid, block, lds, stream, lv);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_maxpool(const uint8_t *mask, int res, const int32_t *factors, int n, uint8_t *const *out,
                          hipStream_t stream) {
    if (n > kMaxPoolLevels) return hipErrorInvalidValue;
    // Two launches at most: the levels that no other level refines are pooled
    // from the mask, the others from the coarsest of those that does (a
    // maximum of maxima), which is f^3 times smaller.
    PoolLevels direct{}, nested{};
    for (int l = 0; l < n; ++l) {
        int from = -1;
        for (int m = 0; m < n; ++m) {
            if (factors[m] >= factors[l] || factors[l] % factors[m] != 0) continue;
            bool refined = false;                             // is m itself pooled from the mask?
            for (int k = 0; k < n; ++k) refined = refined || (factors[k] < factors[m] && factors[m] % factors[k] == 0);
            if (!refined && (from < 0 || factors[m] > factors[from])) from = m;
        }
        if (from < 0) direct.level[direct.n++] = PoolLevel{mask, out[l], res, factors[l], 0, 0, 0};
        else nested.level[nested.n++] = PoolLevel{out[from], out[l], res / factors[from], factors[l] / factors[from], 0, 0, 0};
    }
    hipError_t e = launch_pool_stage(direct, stream);
    return e == hipSuccess ? launch_pool_stage(nested, stream) : e;
}

}  // namespace merf
