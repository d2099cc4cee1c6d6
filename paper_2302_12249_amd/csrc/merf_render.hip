// merf_render.hip -- gfx950 kernels of the MERF deferred volume renderer.
//
// One wave64 renders an 8x8 tile of pixels, one ray per lane, so the rays of
// a wave are coherent and their plane and grid gathers fall on nearby texels.
// Per lane (MERF, arXiv 2302.12249):
//   1. pinhole ray (o, d);
//   2. the ray is cut at the parameters where the region of the
//      piecewise-projective contraction changes (Sec. 4.2, Eq. 7); each piece
//      maps to a straight contracted segment, handled one at a time;
//   3. each segment is marched on a uniform lattice of contracted step s
//      (sample at each interval midpoint, last interval shortened); a sample
//      is evaluated only if every occupancy level marks its cell occupied
//      (Sec. 6); in empty space the march jumps to the first lattice sample
//      past the exit of an empty box (ray-box slab test in contracted space,
//      exact because the segment is straight): by default the largest empty
//      cube ahead, from a grid derived from the levels at upload, otherwise
//      the empty cell of the first empty level;
//   4. evaluated samples are parked in LDS; the wave shades up to 64 parked
//      samples at once, whoever's they are: gather the 3D grid (trilinear,
//      one brick per sample thanks to the apron) and the three planes
//      (bilinear), dequantise (Eq. 8; the fp32 path applies it to the
//      interpolated codes, the same value up to rounding), sum (Eq. 5),
//      decode (Eq. 6); each lane then composites its own samples in ray
//      order (Eq. 1-2);
//   5. marching stops when the transmittance drops below t_min (Sec. 6);
//   6. the deferred MLP h(C_d, F, d) runs once per pixel (Eq. 3, App. B).
// Before a launch, a prepass (k_tile_cost, k_tile_order) marches a few
// probe rays per tile and orders the tiles by their estimated work, heaviest
// first; the served kernel (k_render_served) runs the same per-tile code on
// requests of several scenes described in device memory.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <hip/hip_bf16.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "merf_device.h"
#include "merf_segments.h"

namespace merf {

namespace {

constexpr float kRcp255 = 1.0f / 255.0f;
constexpr float kNegLog2e = -1.44269504088896340736f;
// Samples are never skipped past a cell exit by more than this (contracted
// units): FP32 error of the exit parameter is below 1e-6.
constexpr float kSkipGuard = 2e-6f;

// ---------------------------------------------------------------------------
// Eq. 8: code b -> 2 m b / 255 - m, correctly rounded to float32.
// k = m (2b - 255) is an exact small integer; q = k * RN(1/255) is then
// corrected by one residual step (Markstein), which gives the correctly
// rounded quotient k / 255 for every code and m in {7, 14} (checked
// exhaustively by the test-suite).
// ---------------------------------------------------------------------------
__device__ __forceinline__ float deq_f32(uint32_t b, float m2, float m255) {
    float k = fmaf((float)b, m2, -m255);
    float q = k * kRcp255;
    float r = fmaf(-q, 255.0f, k);
    return fmaf(r, kRcp255, q);
}


__device__ __forceinline__ uint32_t byte_of(uint32_t w, int i) { return (w >> (8 * i)) & 0xffu; }

// Two codes as the float16 subnormals b * 2^-24, which are exact: mixed-
// precision FMAs (v_fma_mix_f32) then take them as operands directly, so an
// interpolation term costs one instruction instead of a convert and an FMA.
// The sums come out scaled by 2^-24 exactly (a power of two, far from the
// float32 range limits), which the Eq. 8 scale absorbs.
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ f16x2 as_f16x2(uint32_t w) { return __builtin_bit_cast(f16x2, w); }
// bytes 0 and 2 of w
__device__ __forceinline__ f16x2 codes02(uint32_t w) { return as_f16x2(w & 0x00ff00ffu); }
// bytes 1 and 3 of w
__device__ __forceinline__ f16x2 codes13(uint32_t w) { return as_f16x2(__builtin_amdgcn_perm(0u, w, 0x0c030c01u)); }
// byte 0 of a and byte 0 of b
__device__ __forceinline__ f16x2 codes0_0(uint32_t a, uint32_t b) {
    return as_f16x2(__builtin_amdgcn_perm(b, a, 0x0c040c00u));
}

// byte j of a and byte j of b
template <int j>
__device__ __forceinline__ f16x2 codes_jj(uint32_t a, uint32_t b) {
    return as_f16x2(__builtin_amdgcn_perm(b, a, 0x0c000c00u | ((4u + j) << 16) | (uint32_t)j));
}

// Eq. 8 to float16 of a code given as the subnormal b 2^-24, with
// a24 = 2^24 RN32(2m/255) (the scale the upload computes, times 2^24): the
// product is b RN32(2m/255) exactly, so this is RN16(RN32(b a - m)), which
// equals the correctly rounded float16 of the exact 2mb/255 - m for every
// code and m in {7, 14} (checked exhaustively on the host, and bit for bit on
// the device through merf_dequantize, which runs this routine).  Returned
// widened to float; the compiler fuses the FMA and the rounding to float16
// into one mixed-precision instruction.
__device__ __forceinline__ float deq_f16(_Float16 code, float a24, float m) {
    return (float)(_Float16)fmaf((float)code, a24, -m);
}

// Projective map of region reg (Eq. 7): y_j = (2 - 1/|x_j|) s, y_k = x_k/|x_j|.
__device__ __forceinline__ float3 map_region(int reg, float3 x) {
    if (reg == 0) return x;
    int j = (reg - 1) >> 1;
    float s = ((reg - 1) & 1) ? -1.0f : 1.0f;
    float xj = j == 0 ? x.x : (j == 1 ? x.y : x.z);
    float ia = rcp(fabsf(xj));
    float3 y = make_float3(x.x * ia, x.y * ia, x.z * ia);
    float yj = (2.0f - ia) * s;
    if (j == 0) y.x = yj; else if (j == 1) y.y = yj; else y.z = yj;
    return y;
}

// Contracted image of the ray's point at infinity in region reg.
__device__ __forceinline__ float3 limit_point(int reg, float3 d) {
    int j = (reg - 1) >> 1;
    float s = ((reg - 1) & 1) ? -1.0f : 1.0f;
    float dj = j == 0 ? d.x : (j == 1 ? d.y : d.z);
    float ia = rcp(fabsf(dj));
    float3 y = make_float3(d.x * ia, d.y * ia, d.z * ia);
    if (j == 0) y.x = 2.0f * s; else if (j == 1) y.y = 2.0f * s; else y.z = 2.0f * s;
    return y;
}

// Preimage of a contracted point in region reg (world-length deltas).
__device__ __forceinline__ float3 unmap_region(int reg, float3 y) {
    if (reg == 0) return y;
    int j = (reg - 1) >> 1;
    float s = ((reg - 1) & 1) ? -1.0f : 1.0f;
    float yj = j == 0 ? y.x : (j == 1 ? y.y : y.z);
    float a = rcp(2.0f - s * yj);
    float3 x = make_float3(y.x * a, y.y * a, y.z * a);
    if (j == 0) x.x = s * a; else if (j == 1) x.y = s * a; else x.z = s * a;
    return x;
}

// 24-bit multiply (v_mul_u32_u24, full rate; a 32-bit integer multiply is
// quarter rate): both factors below 2^24, the low 32 bits of the product.
__device__ __forceinline__ uint32_t mul24(uint32_t a, uint32_t b) { return __umul24(a, b); }

// Cell of a grid of r cells a side at scaled coordinate v = (p + 2) r / 4,
// clamped to [0, r - 1] on both sides (one median instruction), so that a
// lookup stays inside the grid whatever the point.
__device__ __forceinline__ int cell_index(float v, int r) { return max(min((int)v, r - 1), 0); }

// Byte offset of cell (x, y, z) of an r^3 z-major grid; every factor is
// below 2^24 (r <= 1024).
__device__ __forceinline__ uint32_t cell_offset(int x, int y, int z, int r) {
    return mul24((uint32_t)z, mul24((uint32_t)r, (uint32_t)r)) + mul24((uint32_t)y, (uint32_t)r) + (uint32_t)x;
}

// Number of lanes below this one whose bit is set in the wave mask m.
__device__ __forceinline__ int lanes_below(uint64_t m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Sigmoid of x given as -x log2(e).
__device__ __forceinline__ float sigmoid_l2(float x) {
    return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(x));
}

// XCD-aware tile order.  Consecutive workgroups are dispatched round-robin
// over the 8 XCDs (workgroup b runs on XCD b % 8 as that XCD's (b / 8)-th),
// with no balancing between XCDs.  Each XCD therefore gets runs of
// kXcdChunk consecutive tiles (neighbouring tiles gather neighbouring texels
// and share that XCD's L2), and the runs are dealt to the XCDs in turn over
// the whole launch, so every XCD gets a similar share of the image's work.
// Workgroups past the last whole round of runs keep their own tile.
constexpr int kXcdChunk = 4;
__device__ __forceinline__ int xcd_remap(int bid, int n) {
    constexpr int nx = 8;
    const int full = n / (nx * kXcdChunk) * (nx * kXcdChunk);
    if (bid >= full) return bid;
    const int x = bid % nx, i = bid / nx;
    return ((i / kXcdChunk) * nx + x) * kXcdChunk + i % kXcdChunk;
}

struct Accum {
    float T, cd0, cd1, cd2, f0, f1, f2, f3;
};

struct Counters {
    uint32_t occ_lookups, visited, evaluated, contributing, opens;
};

// Phase profile of the statistics variant (RenderBatch::phases): shader-clock
// timestamps taken at points every lane of the wave passes together, so each
// interval is wave time, added to the phase it belongs to.  Lane i keeps the
// sum of slot i (one register for all slots; a wave's sums stay below 2^32).
template <bool kOn>
struct PhaseClock {
    uint32_t t = 0, v = 0;          // low word of the last timestamp; this lane's sum
    __device__ __forceinline__ void start() {
        if (kOn) t = (uint32_t)__builtin_amdgcn_s_memtime();
    }
    __device__ __forceinline__ void count(int slot, uint32_t x = 1) {
        if (kOn) v += (int)threadIdx.x == slot ? x : 0u;
    }
    __device__ __forceinline__ void lap(int slot) {
        if (kOn) {
            const uint32_t n = (uint32_t)__builtin_amdgcn_s_memtime();
            count(slot, n - t);     // modulo 2^32: intervals are far shorter
            t = n;
        }
    }
};

template <typename T>
__device__ __forceinline__ T load_at(const uint8_t *base, uint32_t off) {
    return *reinterpret_cast<const T *>(base + off);
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// 16-byte load: two adjacent 8-byte texels.
__device__ __forceinline__ u32x4 load_pair(const uint8_t *base, uint32_t off) {
    return *reinterpret_cast<const u32x4 *>(base + off);
}

// Byte offsets of the 20 texels one sample reads.  Planes: the (u, v) and
// (u + 1, v) texels of row v start at op[p] and those of row v + 1 at
// op[p] + prow.  Grid: the 2x2x2 footprint of brick slot brick_index[bi]
// starts at byte ol of that brick.  A coordinate clamped to the last texel has
// that texel as its low one and fraction 0: the high one then lies past the
// row, the plane or (planes) the array, is read with weight 0 and changes
// nothing (any byte is a finite code; the scene's allocation reaches a row
// past the planes).  That leaves a floor and a fraction per axis, two
// instructions fewer than clamping the low texel to the last but one.
struct Footprint {
    uint32_t op[3], prow, bi, ol;
    float ex, ey, ez;   // plane texel fractions
    float fx, fy, fz;   // grid voxel fractions
};

// Scene accessors take the scene as S = const DevScene (a kernel argument)
// or as a constant-address-space DevScene (a slot of a served launch's
// table), so both read it with scalar loads that may be repeated at will.
template <typename S>
__device__ __forceinline__ Footprint footprint(const S &sc, float3 p) {
    Footprint f;
    // ---- three planes, bilinear: P_x(y, z), P_y(x, z), P_z(x, y)
    const float ps = sc.p_scale, ps2 = sc.p_off, pmax = sc.p_max;
    float hx = __builtin_amdgcn_fmed3f(fmaf(p.x, ps, ps2), 0.0f, pmax);
    float hy = __builtin_amdgcn_fmed3f(fmaf(p.y, ps, ps2), 0.0f, pmax);
    float hz = __builtin_amdgcn_fmed3f(fmaf(p.z, ps, ps2), 0.0f, pmax);
    const int jx = (int)hx, jy = (int)hy, jz = (int)hz;
    f.ex = __builtin_amdgcn_fractf(hx); f.ey = __builtin_amdgcn_fractf(hy); f.ez = __builtin_amdgcn_fractf(hz);
    const uint32_t row = (uint32_t)sc.R * kChannels, plane = (uint32_t)sc.R * row;
    f.prow = row;
    // (R <= 8192: texel indices and the row of 8 R bytes are below 2^24, and
    // every offset below 2^31)
    f.op[0] = mul24((uint32_t)jz, row) + (uint32_t)jy * kChannels;
    f.op[1] = plane + mul24((uint32_t)jz, row) + (uint32_t)jx * kChannels;
    f.op[2] = 2u * plane + mul24((uint32_t)jy, row) + (uint32_t)jx * kChannels;
    // ---- sparse 3D grid, trilinear inside one apron brick
    const float gs = sc.g_scale, gs2 = sc.g_off, gmax = sc.g_max;
    float gx = __builtin_amdgcn_fmed3f(fmaf(p.x, gs, gs2), 0.0f, gmax);
    float gy = __builtin_amdgcn_fmed3f(fmaf(p.y, gs, gs2), 0.0f, gmax);
    float gz = __builtin_amdgcn_fmed3f(fmaf(p.z, gs, gs2), 0.0f, gmax);
    const int ix = (int)gx, iy = (int)gy, iz = (int)gz;
    f.fx = __builtin_amdgcn_fractf(gx); f.fy = __builtin_amdgcn_fractf(gy); f.fz = __builtin_amdgcn_fractf(gz);
    f.bi = mul24((uint32_t)(iz >> 3), mul24((uint32_t)sc.nbl, (uint32_t)sc.nbl)) +
           mul24((uint32_t)(iy >> 3), (uint32_t)sc.nbl) + (uint32_t)(ix >> 3);
    f.ol = (uint32_t)((((iz & 7) * kBrick + (iy & 7)) * kBrick + (ix & 7)) * kChannels);
    return f;
}

// The ten 16-byte texel pairs of a sample: 6 plane pairs, 4 grid pairs.
struct Texels {
    u32x4 t[6], g[4];
};

// Issue every load of a sample before waiting on any: the brick index first
// (the brick loads depend on it), then the plane pairs, which overlap its
// round trip, then the brick pairs.  The empty asm takes all ten vectors, so
// the compiler neither splits them into per-word loads nor sinks any to their
// first use, and places one wait before it.  Every array is present on
// the device (a scene without a grid or without planes reads an all-zero
// stand-in), so nothing here branches.
template <typename S>
__device__ __forceinline__ Texels gather(const S &sc, const Footprint &f) {
    Texels x;
    const int brick = load_at<int>(reinterpret_cast<const uint8_t *>(sc.brick_index), f.bi * 4u);
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) {
        x.t[2 * pl] = load_pair(sc.planes, f.op[pl]);
        x.t[2 * pl + 1] = load_pair(sc.planes + f.prow, f.op[pl]);
    }
    constexpr uint32_t sy = kBrick * kChannels, sz = kBrick * kBrick * kChannels;
    // (fewer than 2^31 / kBrickBytes bricks: the upload checks it)
    const uint32_t ob = mul24((uint32_t)brick, kBrickBytes) + f.ol;
    x.g[0] = load_pair(sc.bricks, ob);
    x.g[1] = load_pair(sc.bricks + sy, ob);
    x.g[2] = load_pair(sc.bricks + sz, ob);
    x.g[3] = load_pair(sc.bricks + (sz + sy), ob);
    asm volatile("" : "+v"(x.t[0]), "+v"(x.t[1]), "+v"(x.t[2]), "+v"(x.t[3]), "+v"(x.t[4]), "+v"(x.t[5]),
                 "+v"(x.g[0]), "+v"(x.g[1]), "+v"(x.g[2]), "+v"(x.g[3]));
    return x;
}

// Shaded sample: 1 - alpha and the sigmoids of the diffuse colour and the
// features (Eq. 6).
struct SampleResult {
    float trans;
    float sg[7];
};

// One evaluated sample: gather, dequantise, decode.
// All offsets are 32-bit (the upload keeps every array below 2 GiB) and are
// added to uniform base pointers, so no 64-bit address arithmetic runs per lane.
// kFolded: the sigmoid's -log2(e) lies in the scale of the codes, an operation
// less per channel.  That moves the sums by their last bits, which a float32
// MLP passes on as they are; one with float16 or bfloat16 operands rounds some
// of them to its next value (up to 9e-4 of a pixel), so those modes multiply
// separately, with the roundings of a plain sigmoid(m (2b/255 - 1)).
template <int kFeat, bool kFolded, typename S>
__device__ __forceinline__ SampleResult eval_sample(const S &sc, float3 p, float delta) {
    const Footprint f = footprint(sc, p);
    const Texels x = gather(sc, f);
    // texel words of the 20 texels (lo = channels 0..3, hi = 4..7) and their
    // weights: 8 grid corners, then 4 texels of each plane.  An absent source
    // reads zero codes, so its weights do not matter.
    uint32_t lo[20], hi[20];
    float w[20];
    {
        const float fu[3] = {f.ey, f.ex, f.ex}, fv[3] = {f.ez, f.ez, f.ey};   // (u, v) = (y, z), (x, z), (x, y)
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) {
            const float au = 1.0f - fu[pl], av = 1.0f - fv[pl];
            const u32x4 r0 = x.t[2 * pl], r1 = x.t[2 * pl + 1];
            lo[8 + 4 * pl] = r0.x; hi[8 + 4 * pl] = r0.y; w[8 + 4 * pl] = au * av;
            lo[9 + 4 * pl] = r0.z; hi[9 + 4 * pl] = r0.w; w[9 + 4 * pl] = fu[pl] * av;
            lo[10 + 4 * pl] = r1.x; hi[10 + 4 * pl] = r1.y; w[10 + 4 * pl] = au * fv[pl];
            lo[11 + 4 * pl] = r1.z; hi[11 + 4 * pl] = r1.w; w[11 + 4 * pl] = fu[pl] * fv[pl];
        }
        // corners (x, x + 1) at (y, z), (y + 1, z), (y, z + 1), (y + 1, z + 1)
        const float ax = 1.0f - f.fx, ay = 1.0f - f.fy, az = 1.0f - f.fz;
        const float wyz[4] = {ay * az, f.fy * az, ay * f.fz, f.fy * f.fz};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            lo[2 * i] = x.g[i].x; hi[2 * i] = x.g[i].y; w[2 * i] = ax * wyz[i];
            lo[2 * i + 1] = x.g[i].z; hi[2 * i + 1] = x.g[i].w; w[2 * i + 1] = f.fx * wyz[i];
        }
    }
    // ---- Eq. 8 dequantises each code affinely, q(b) = a b - m with a = 2m/255,
    // and the weights of each present source sum to one, so
    // sum_i w_i q(b_i) = a * sum_i w_i b_i - n m exactly (n sources: 4 for
    // grid + planes).  The FP32 path
    // (kFeat = 0) interpolates the codes and applies the affine map
    // once per channel: the same real number with one convert and one FMA per
    // texel and channel; the two FP32 evaluations differ by rounding only
    // (below 1e-6 relative).  The exact-FP16 path (kFeat = 1) dequantises
    // every code to its correctly rounded float16 value first (deq_f16) and
    // interpolates those values with FP32 weights and FP32 sums.  The
    // FP16-interpolation path (kFeat = 2) computes density as the FP32 path
    // does and interpolates the appearance channels from float16 operands:
    // the weights rounded to float16, the codes exact, each pair of texels
    // summed by one dot product with FP32 accumulation (v_dot2_f32_f16).
    // (a = d_scale or f_scale, n m = -d_off or -f_off, precomputed)
    const float md = sc.m_density, mf = sc.m_feature;
    // ---- density
    float s0 = 0.0f;
    if constexpr (kFeat == 1) {
        // a stand-in source (scene without grid or without planes) reads code
        // 0, whose float16 value is -m: its texels get weight 0 here, so that
        // the sum holds the present sources only (Eq. 5)
#pragma unroll
        for (int i = 0; i < 20; ++i) w[i] *= i < 8 ? sc.grid_w : sc.planes_w;
#pragma unroll
        for (int k = 0; k < 10; ++k) {
            const f16x2 c = codes0_0(lo[2 * k], lo[2 * k + 1]);
            s0 = fmaf(w[2 * k], deq_f16(c.x, sc.d_scale24, md), s0);
            s0 = fmaf(w[2 * k + 1], deq_f16(c.y, sc.d_scale24, md), s0);
        }
    } else {
        // texel pairs: the density codes of texels 2k and 2k + 1 in one word
#pragma unroll
        for (int k = 0; k < 10; ++k) {
            const f16x2 c = codes0_0(lo[2 * k], lo[2 * k + 1]);
            s0 = fmaf(w[2 * k], (float)c.x, s0);
            s0 = fmaf(w[2 * k + 1], (float)c.y, s0);
        }
        s0 = fmaf(s0, sc.d_scale24, sc.d_off);
    }
    SampleResult r;
    float tau = __expf(s0);                       // Eq. 6
    r.trans = __expf(-tau * delta);               // e^{-tau delta} = 1 - alpha (Eq. 1)
    // ---- appearance, of every lane: where alpha is zero its weight is zero,
    // and a wave with no other lane practically never occurs (Sec. 6 reads it
    // only where alpha is not zero)
    {
        // The eight-byte vector instructions that follow (210 of them, 330
        // with float16 features) run faster from 4 modulo 8 bytes than from 0:
        // a four-byte instruction moved across this point made kernels 2.5%
        // faster or slower whatever else it did, so the place is fixed here
        // (float32 features, against 0: sixteen 1080p views 3.06 -> 2.97 ms, a
        // 4K frame with the bf16 MLP 1.176 -> 1.135 ms, a 1080p view 219.7 ->
        // 213.2 us).  With float16 features (kFeat 1) an odd number of
        // four-byte instructions comes first, so they start from 0 (333 -> 322
        // us).  The few of kFeat 2 do not care: 221.7 us wherever they are.
        // Aligning the march or the density as well changes nothing.
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (kFeat == 0) asm volatile(".p2align 3\n s_nop 0");
        else if constexpr (kFeat == 1) asm volatile(".p2align 3");
        __builtin_amdgcn_sched_barrier(0);
        float sa[7];
#pragma unroll
        for (int c = 0; c < 7; ++c) sa[c] = 0.0f;
        // Eq. 8 of the interpolated codes, times -log2(e) for the sigmoid
        auto exponent = [&](float codes) {
            if constexpr (kFolded) return fmaf(codes, sc.f_scale24_l2, sc.f_off_l2);
            else return fmaf(codes, sc.f_scale24, sc.f_off) * kNegLog2e;
        };
        if constexpr (kFeat == 2) {
            // texel pairs (2k, 2k + 1): their weights and the codes of one
            // channel in one register each
#pragma unroll
            for (int k = 0; k < 10; ++k) {
                const f16x2 wk = {(_Float16)w[2 * k], (_Float16)w[2 * k + 1]};
                const uint32_t la = lo[2 * k], lb = lo[2 * k + 1], ha = hi[2 * k], hb = hi[2 * k + 1];
                sa[0] = __builtin_amdgcn_fdot2(wk, codes_jj<1>(la, lb), sa[0], false);
                sa[1] = __builtin_amdgcn_fdot2(wk, codes_jj<2>(la, lb), sa[1], false);
                sa[2] = __builtin_amdgcn_fdot2(wk, codes_jj<3>(la, lb), sa[2], false);
                sa[3] = __builtin_amdgcn_fdot2(wk, codes_jj<0>(ha, hb), sa[3], false);
                sa[4] = __builtin_amdgcn_fdot2(wk, codes_jj<1>(ha, hb), sa[4], false);
                sa[5] = __builtin_amdgcn_fdot2(wk, codes_jj<2>(ha, hb), sa[5], false);
                sa[6] = __builtin_amdgcn_fdot2(wk, codes_jj<3>(ha, hb), sa[6], false);
            }
#pragma unroll
            for (int c = 0; c < 7; ++c) sa[c] = exponent(sa[c]);
        } else if constexpr (kFeat == 1) {
            const float af = sc.f_scale24;
#pragma unroll
            for (int i = 0; i < 20; ++i) {
                const f16x2 l02 = codes02(lo[i]), l13 = codes13(lo[i]);
                const f16x2 h02 = codes02(hi[i]), h13 = codes13(hi[i]);
                sa[0] = fmaf(w[i], deq_f16(l13.x, af, mf), sa[0]);
                sa[1] = fmaf(w[i], deq_f16(l02.y, af, mf), sa[1]);
                sa[2] = fmaf(w[i], deq_f16(l13.y, af, mf), sa[2]);
                sa[3] = fmaf(w[i], deq_f16(h02.x, af, mf), sa[3]);
                sa[4] = fmaf(w[i], deq_f16(h13.x, af, mf), sa[4]);
                sa[5] = fmaf(w[i], deq_f16(h02.y, af, mf), sa[5]);
                sa[6] = fmaf(w[i], deq_f16(h13.y, af, mf), sa[6]);
            }
#pragma unroll
            for (int c = 0; c < 7; ++c) sa[c] *= kNegLog2e;
        } else {
            // per texel pair: channel 2 of both texels from one permute, so
            // 7 permutes or masks extract the 14 codes of the pair
#pragma unroll
            for (int k = 0; k < 10; ++k) {
                const f16x2 c2 = codes_jj<2>(lo[2 * k], lo[2 * k + 1]);
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int i = 2 * k + t;
                    const f16x2 l13 = codes13(lo[i]);
                    const f16x2 h02 = codes02(hi[i]), h13 = codes13(hi[i]);
                    sa[0] = fmaf(w[i], (float)l13.x, sa[0]);
                    sa[1] = fmaf(w[i], (float)(t ? c2.y : c2.x), sa[1]);
                    sa[2] = fmaf(w[i], (float)l13.y, sa[2]);
                    sa[3] = fmaf(w[i], (float)h02.x, sa[3]);
                    sa[4] = fmaf(w[i], (float)h13.x, sa[4]);
                    sa[5] = fmaf(w[i], (float)h02.y, sa[5]);
                    sa[6] = fmaf(w[i], (float)h13.y, sa[6]);
                }
            }
#pragma unroll
            for (int c = 0; c < 7; ++c) sa[c] = exponent(sa[c]);
        }
#pragma unroll
        for (int c = 0; c < 7; ++c) r.sg[c] = sigmoid_l2(sa[c]);
    }
    return r;
}

// Front-to-back compositing of one shaded sample (Eq. 1-2).
template <bool kStats>
__device__ __forceinline__ void composite(Accum &acc, const SampleResult &r, Counters &cnt) {
    const float alpha = 1.0f - r.trans;
    if (kStats) ++cnt.evaluated;
    if (alpha > 0.0f) {
        if (kStats) ++cnt.contributing;
        const float wt = acc.T * alpha;
        acc.cd0 = fmaf(wt, r.sg[0], acc.cd0);
        acc.cd1 = fmaf(wt, r.sg[1], acc.cd1);
        acc.cd2 = fmaf(wt, r.sg[2], acc.cd2);
        acc.f0 = fmaf(wt, r.sg[3], acc.f0);
        acc.f1 = fmaf(wt, r.sg[4], acc.f1);
        acc.f2 = fmaf(wt, r.sg[5], acc.f2);
        acc.f3 = fmaf(wt, r.sg[6], acc.f3);
        acc.T *= r.trans;
    }
}

// March state of one straight contracted segment A -> B (region reg) that
// covers the world parameters [ta, tb] of the ray (B itself is recomputed by
// segment_end where needed).
struct Segment {
    float3 A, e;                    // contracted start, unit direction
    float len, iex, iey, iez;       // length; inverse direction (+-inf where e = +-0)
    float tb;                       // world parameter of the end (kInf: last)
    float n, k;                     // interval count, next interval (integers below 2^24)
    int reg, reg_next;              // regions
    uint32_t doff;                  // byte offset of the empty-space grid of this direction's octant
};

// Contracted end point of the segment of region reg that ends at world
// parameter tb (kInf: the limit point of the ray).
__device__ __forceinline__ float3 segment_end(float3 o, float3 d, float tb, int reg) {
    return tb < kInf ? map_region(reg, make_float3(fmaf(tb, d.x, o.x), fmaf(tb, d.y, o.y), fmaf(tb, d.z, o.z)))
                     : limit_point(reg, d);
}

// Set up the segment of the ray that starts at world parameter ta in region
// reg: find where the ray leaves the region (Eq. 7 breakpoints), map both ends.
__device__ __forceinline__ void open_segment(float3 o, float3 d, float ta, int reg, float istep, uint32_t oct_stride,
                                             Segment &s) {
    const RegionExit x = region_exit(o, d, ta, reg);
    const float tb = x.t;
    s.A = map_region(reg, make_float3(fmaf(ta, d.x, o.x), fmaf(ta, d.y, o.y), fmaf(ta, d.z, o.z)));
    const float3 B = segment_end(o, d, tb, reg);
    s.tb = tb;
    s.reg = reg;
    s.reg_next = x.next;
    float3 e = make_float3(B.x - s.A.x, B.y - s.A.y, B.z - s.A.z);
    float len = sqrtf(e.x * e.x + e.y * e.y + e.z * e.z);
    s.k = 0.0f;
    // contracted segments are at most a few units long; anything else is a
    // degenerate ray (NaN / infinite end point) and contributes nothing
    if (!(len > 0.0f && len < 16.0f)) {
        s.n = 0.0f;
        s.len = 0.0f;
        return;
    }
    float il = rcp(len);
    e.x *= il; e.y *= il; e.z *= il;
    s.e = e;
    s.len = len;
    s.n = ceilf(len * istep);       // (len < 16 and a step of at least 1e-6)
    // rcp(+-0) = +-inf: the slab tests below then give +inf (or NaN, which
    // fminf ignores) for an axis the segment does not move along
    s.iex = rcp(e.x);
    s.iey = rcp(e.y);
    s.iez = rcp(e.z);
    s.doff = oct_stride * (uint32_t)((s.iex < 0.0f ? 1 : 0) | (s.iey < 0.0f ? 2 : 0) | (s.iez < 0.0f ? 4 : 0));
}

// Lattice interval k of a segment: its ends u0, u1 (the last interval is
// shortened) and midpoint um.
__device__ __forceinline__ void interval(const Segment &s, float step, float &u0, float &u1, float &um) {
    u0 = s.k * step;
    u1 = __builtin_amdgcn_fmed3f(u0 + step, 0.0f, s.len);
    um = 0.5f * (u0 + u1);
}

// Empty-space grid of the segment's octant at contracted point p.  Returns
// the byte D of p's cell: D > 0 means the cube of D cells a side with a
// corner at that cell, extending the way the segment travels, is empty; 0
// means the cell is occupied (the cube is the cell itself).  ue is the
// segment parameter at which the cube ends (slab test).
// The march is bound by instruction issue, so the cell is clamped and floored
// as a float, which the row offset and the slab test both use, and the far
// face of the cube is the cell's centre plus |D - 1/2| cells with the sign of
// the direction: 29 vector instructions from the point to ue, where selecting
// the face per axis from integer cells took 42.  With a power-of-two
// resolution the face is exact, so ue has the value that the integer form
// gives.  (Multiplying centre and half edge by 1 / e separately saves three
// more instructions, but an ulp of ue then decided one sample in some ten
// million otherwise; the signs as float16 operands of mixed-precision FMAs
// save the same three and were 1.5% slower over a frame.)  An axis without
// motion (1 / e infinite) gives +inf or NaN, which fminf ignores.
// With the sample's own arithmetic below (floor and fraction of a texel
// coordinate, sigmoid exponents scaled at upload, no branch on alpha) the
// 1080p frame fell from 5020 to 4540 vector instructions per wave, 309 to
// 289 us; 128x128 from 54.5 to 47 us, sixteen 1080p views 3.75 to 3.51 ms.
template <typename S>
__device__ __forceinline__ uint32_t dist_lookup(const S &sc, const Segment &s, float3 p, float &ue) {
    // cell of p: (p + 2) r / 4 clamped to [0, r - 1], rounded down
    const float os = sc.dist_scale, os2 = sc.dist_off, qmax = sc.dist_max;
    const float qx = floorf(__builtin_amdgcn_fmed3f(fmaf(p.x, os, os2), 0.0f, qmax));
    const float qy = floorf(__builtin_amdgcn_fmed3f(fmaf(p.y, os, os2), 0.0f, qmax));
    const float qz = floorf(__builtin_amdgcn_fmed3f(fmaf(p.z, os, os2), 0.0f, qmax));
    // (r <= 1024: y r + x is exact in float32, z r^2 in a 24-bit multiply)
    const uint32_t off = mul24((uint32_t)qz, (uint32_t)sc.dist_slice) + (uint32_t)fmaf(qy, sc.dist_resf, qx) + s.doff;
    const uint32_t D = load_at<uint8_t>(sc.dist, off);
    const float h = sc.dist_cell, c = sc.dist_centre;
    const float half = fabsf(fmaf((float)D, h, -0.5f * h));
    const float tx = (fmaf(qx, h, c) + copysignf(half, s.iex) - s.A.x) * s.iex;
    const float ty = (fmaf(qy, h, c) + copysignf(half, s.iey) - s.A.y) * s.iey;
    const float tz = (fmaf(qz, h, c) + copysignf(half, s.iez) - s.A.z) * s.iez;
    ue = fminf(tx, fminf(ty, tz));
    return D;
}

// Next lattice interval after leaving empty space at segment parameter
// uexit: the first whose midpoint lies past the exit less kSkipGuard, at
// least k + 1 and at most n (k < n; a median, so NaN would give k + 1).
__device__ __forceinline__ float skip_past(const Segment &s, float uexit, float istep) {
    const float kn = floorf(fmaf(uexit, istep, 0.5f - kSkipGuard * istep));
    return __builtin_amdgcn_fmed3f(kn, s.k + 1.0f, s.n);
}

// Pinhole ray through the centre of pixel (px, py) (unit direction).
__device__ __forceinline__ void pixel_ray(const DevCamera &cam, int px, int py, float3 &o, float3 &d) {
    const float vx = ((float)px + 0.5f - cam.cx) * cam.inv_fx;
    const float vy = ((float)py + 0.5f - cam.cy) * cam.inv_fy;
    d = make_float3(fmaf(cam.c2w[0], vx, fmaf(cam.c2w[1], vy, cam.c2w[2])),
                    fmaf(cam.c2w[4], vx, fmaf(cam.c2w[5], vy, cam.c2w[6])),
                    fmaf(cam.c2w[8], vx, fmaf(cam.c2w[9], vy, cam.c2w[10])));
    const float inv = __builtin_amdgcn_rsqf(d.x * d.x + d.y * d.y + d.z * d.z);
    d.x *= inv; d.y *= inv; d.z *= inv;
    o = make_float3(cam.c2w[3], cam.c2w[7], cam.c2w[11]);
}

// Camera of a launch tile: the last camera whose first tile is <= tile.
__device__ __forceinline__ int camera_of(const RenderBatch &rb, int tile) {
    int c = 0;
#pragma unroll
    for (int i = 1; i < kCamsPerLaunch; ++i)
        if (i < rb.n_cams && tile >= rb.cams[i].tile_start) c = i;
    return c;
}

// Deferred MLP (Eq. 3, App. B) for the 64 pixels of a wave on the matrix
// cores.  Each layer is computed transposed, H^T = W^T X^T, over 4 blocks of
// 16 pixels: the output of one layer (lane l holds hidden units 4(l/16) .. +3
// of pixel l % 16) is exactly the B operand the next layer needs, so only the
// input features and the final RGB pass through LDS.  A pixel is a column of
// every product, so inactive lanes cannot affect the others.
//   kPrec 0: fp32 inputs, v_mfma_f32_16x16x4f32 (K = 4 per instruction);
//   kPrec 1: fp16 inputs, v_mfma_f32_16x16x16f16 (K = 16);
//   kPrec 2: bf16 inputs, v_mfma_f32_16x16x16bf16_1k (K = 16).
// Accumulation, biases and ReLU are fp32 in every case.
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef _Float16 halfx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
// LDS staging of the inputs, one row per pixel, sized so that four waves fit
// per SIMD (16 workgroups of one wave in a CU's 160 KB):
//   fp32: 36 floats (the 34 inputs zero-padded to nine K = 4 steps), row
//         stride 37 floats -- odd, so the 16 rows one instruction reads fall in
//         different banks;
//   fp16 / bf16: the inputs already converted, 48 halves (three K = 16
//         steps), row stride 52 halves = 26 banks, so the 16 eight-byte reads
//         of one instruction cover the 32 banks once.
// The outputs reuse the buffer as floats with the row stride kOut.
template <int kPrec>
struct MlpLds {
    static constexpr int kWidth = kPrec == 0 ? 36 : 48;      // inputs per row
    static constexpr int kStride = kPrec == 0 ? 37 : 52;     // elements per row
    static constexpr int kOut = kPrec == 0 ? 37 : 26;        // floats per row of the outputs
    static constexpr int kFloats = 64 * (kPrec == 0 ? 37 : 26);
};

// Scale of the split fp32 MLP's inputs, which are at most 1 (deferred_mlp_split).
constexpr int kInputScaleLog2 = 15;

// Sine and cosine for |x| <= 1, times kScale (a power of two), by their Taylor
// series to x^9 and x^10 (errors below 6e-8): as many issue slots as the
// hardware's, which are exact to 1e-6 only, and the doublings below multiply
// that by 8.  kx is kScale x.
template <int kScale>
__device__ __forceinline__ void sincos_unit(float x, float kx, float &s, float &c) {
    constexpr float K = (float)kScale;
    const float x2 = x * x;
    s = fmaf(kx * x2, fmaf(fmaf(fmaf(2.7557319e-6f, x2, -1.9841270e-4f), x2, 8.3333333e-3f), x2, -0.16666667f), kx);
    c = fmaf(fmaf(fmaf(fmaf(fmaf(K * -2.7557319e-7f, x2, K * 2.4801587e-5f), x2, K * -1.3888889e-3f), x2, K * 4.1666667e-2f),
                  x2, K * -0.5f),
             x2, K);
}

// The MLP's 34 inputs, times kScale (1, or a power of two), zero-padded to 48.
template <bool kSeries, int kScale = 1>
__device__ __forceinline__ void mlp_encode(float *x, const Accum &acc, float3 d) {
    constexpr float K = (float)kScale;
    x[0] = K * acc.cd0; x[1] = K * acc.cd1; x[2] = K * acc.cd2;
    x[3] = K * acc.f0; x[4] = K * acc.f1; x[5] = K * acc.f2; x[6] = K * acc.f3;
    x[7] = K * d.x; x[8] = K * d.y; x[9] = K * d.z;
    // sin and cos of 2^k d, k = 0..3: sine and cosine at k = 0 (the series, or
    // the hardware's in the reduced-precision modes), then the double-angle
    // identities sin 2a = 2 sin a cos a and
    // cos 2a = 1 - 2 sin^2 a (three FP32 operations instead of two quarter-
    // rate transcendentals per term; the error stays near 1e-5 absolute).
    // A scale rides along at no cost: every step is the same operation on
    // scaled values, with the same rounding.
    float sn[3], cs[3];
    if constexpr (kSeries) {
        sincos_unit<kScale>(d.x, x[7], sn[0], cs[0]);
        sincos_unit<kScale>(d.y, x[8], sn[1], cs[1]);
        sincos_unit<kScale>(d.z, x[9], sn[2], cs[2]);
    } else {
        static_assert(kSeries || kScale == 1, "the hardware's sines are not scaled");
        sn[0] = __sinf(d.x); sn[1] = __sinf(d.y); sn[2] = __sinf(d.z);
        cs[0] = __cosf(d.x); cs[1] = __cosf(d.y); cs[2] = __cosf(d.z);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            x[10 + 3 * k + a] = sn[a];
            x[22 + 3 * k + a] = cs[a];
            const float s2 = (2.0f / K) * sn[a];
            cs[a] = fmaf(-s2, sn[a], K);
            sn[a] = s2 * x[22 + 3 * k + a];
        }
    }
#pragma unroll
    for (int k = kMlpIn; k < 48; ++k) x[k] = 0.0f;
}

// Half-precision operand type of kPrec 1 (fp16) and 2 (bf16).
template <int kPrec>
using half4_t = typename std::conditional<kPrec == 1, halfx4, bf16x4>::type;
template <int kPrec>
using half_t = typename std::conditional<kPrec == 1, _Float16, __bf16>::type;

template <int kPrec>
__device__ __forceinline__ half4_t<kPrec> to_half4(const float v[4]) {
    using H = half_t<kPrec>;
    return half4_t<kPrec>{(H)v[0], (H)v[1], (H)v[2], (H)v[3]};
}

// 16x16 block product with K = 16 in half precision: lane l supplies
// A[l % 16][4(l/16) .. +3] and B[4(l/16) .. +3][l % 16].
template <int kPrec>
__device__ __forceinline__ floatx4 mfma16(half4_t<kPrec> a, half4_t<kPrec> b, floatx4 c) {
    if constexpr (kPrec == 1) return __builtin_amdgcn_mfma_f32_16x16x16f16(a, b, c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// The fp32 MLP on the float16 matrix cores.  A float32 matrix instruction
// costs its 32 cycles in full (12 fewer of the 68 made a 1080p frame 2.1%
// faster): the vector units wait for it, as they do not for a float16 one.  So
// every operand v is split into two float16 values, h = RN16(v) and
// l = RN16(v - h), and a product becomes all four of (h + l)(h' + l') in float32
// accumulation.  A K = 32 instruction takes h and l of 16 inputs as its 32 slots
// (a lane's eight: h, then l, of the four inputs that the layout gives it), once
// against the weights' h and once against their l: 36 instructions of 16 cycles
// and no conversions of weights, which the upload splits and lays out by lane
// (k_mlp_fragments).
// h + l is v to 2^-23 relative, until l reaches float16's smallest step of
// 2^-24: below that it is v to an absolute 2^-25.  So every operand is scaled by
// a power of two to the top of float16's range (undone exactly in the multiply
// that adds the bias): the inputs, which are at most 1, by 2^15, a layer's
// weights by the largest of them and its hidden units by their bound, to 2^14
// .. 2^15.  The absolute error is then 2^-39 of what the scale is taken from (an
// input of 1, the layer's largest weight, the bound of its hidden units), and
// an operand down to 2^-16 of that keeps the full 2^-23.  A scene whose
// parameters are not finite, or beyond that scaling, takes the float32
// instructions instead.
// Error against float64 (2-norm, six MLPs of normal weights, colours and
// features near 1e-3, 0.1 and 1): 3.4e-7, 3.4e-7 and 3.5e-7 of the values, where
// the float32 instructions with the hardware's sines had 5.9e-7, 6.0e-7 and
// 5.8e-7: mlp_encode's series takes away more than the split adds.  With all of
// the direction's weights zero the split shows alone: 1.7e-7 in each against
// 1.1e-7, 1.1e-7 and 1.3e-7 (unscaled inputs: 4.1e-5, 3.2e-7 and 2.0e-7).
// 1080p 269 -> 258 us, sixteen 1080p views 3.27 -> 3.07 ms, 512x512 85.6 -> 84.0
// us; the scale of the inputs changes none of them.
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_f16(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{a, b}, f16x2));
}
// minus_one: -1 in a register, so that v - h stays one mixed-precision FMA
__device__ __forceinline__ u32x4 split4(const float *v, float minus_one) {
    u32x4 r;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint32_t h = pack_f16(v[2 * i], v[2 * i + 1]);
        r[i] = h;
        r[2 + i] = pack_f16(fmaf((float)as_f16x2(h).x, minus_one, v[2 * i]), fmaf((float)as_f16x2(h).y, minus_one, v[2 * i + 1]));
    }
    return r;
}
__device__ __forceinline__ floatx4 mfma32(u32x4 a, u32x4 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(halfx8, a), __builtin_bit_cast(halfx8, b), c, 0, 0, 0);
}

// Fragment table of a scene's MLP: kMlpHeader words (whether the split form
// holds, then the scales of the two hidden layers and the output), then one
// 16-byte vector per lane for each of:
enum MlpFragment {
    kFragL1 = 0,         // 4: W0 of inputs 16 m + 4 (l / 16) .. + 3, unit l % 16: m 0 h, m 0 l, m 1 h, m 1 l
    kFragTail = 4,       // W0 of inputs 32, 33 (lanes below 16: h h; below 32: l l)
    kFragL2 = 5,         // 2: W1 of inputs 4 (l / 16) .. + 3: h, l
    kFragL3 = 7,         // 2: W2, outputs 0..2: h, l
    kFragBias = 9,       // 2: scaled biases of hidden units 4 (l / 16) .. + 3 (float32)
    kFragments = 11
};
static_assert(kMlpHeader + 64 * 4 * kFragments == kMlpFragWords, "fragment table");

// Row of one pixel's inputs in LDS: 8 groups of four (h, l), then inputs 32
// and 33 (h h l l); a stride of 9 x 16 bytes keeps the 16-byte reads of a
// group of lanes in different banks.
constexpr int kSplitRow = 144;
static_assert(64 * kSplitRow <= 4 * MlpLds<0>::kFloats, "split rows fit the float32 staging");

__device__ __forceinline__ float3 deferred_mlp_split(const float *__restrict__ W, const uint32_t *__restrict__ frag,
                                                     float *xs, const Accum &acc, float3 d, int lane) {
    const int j = lane & 15, g = lane >> 4;
    const u32x4 *F = reinterpret_cast<const u32x4 *>(frag + kMlpHeader) + lane;
    const float *scale = reinterpret_cast<const float *>(frag);
    const float k0 = scale[1], k1 = scale[2], k2 = scale[3];
    u32x4 w1[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) w1[i] = F[64 * (kFragL1 + i)];
    float minus_one = -1.0f;
    asm volatile("" : "+v"(minus_one));
    uint8_t *rows = reinterpret_cast<uint8_t *>(xs);
    {
        float x[48];
        mlp_encode<true, (1 << kInputScaleLog2)>(x, acc, d);
        uint8_t *row = rows + lane * kSplitRow;
#pragma unroll
        for (int q = 0; q < 8; ++q) *reinterpret_cast<u32x4 *>(row + 16 * q) = split4(x + 4 * q, minus_one);
        const u32x4 t = split4(x + 32, minus_one);
        *reinterpret_cast<uint2 *>(row + 128) = make_uint2(t.x, t.z);
    }
    __syncthreads();
    // the weights' low parts first: the sums then round once at their full
    // size for each of the high parts only
    floatx4 c[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) c[mt] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int low = 1; low >= 0; --low) {
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                const u32x4 b = *reinterpret_cast<const u32x4 *>(rows + (16 * mt + j) * kSplitRow + 16 * (4 * m + g));
                c[mt] = mfma32(w1[2 * m + low], b, c[mt]);
            }
        if (low)
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                const uint2 t = *reinterpret_cast<const uint2 *>(rows + (16 * mt + j) * kSplitRow + 128);
                c[mt] = mfma32(w1[4], u32x4{t.x, t.y, 0u, 0u}, c[mt]);
            }
    }
#pragma unroll
    for (int layer = 0; layer < 2; ++layer) {
        const u32x4 wh = F[64 * (layer ? kFragL3 : kFragL2)], wl = F[64 * ((layer ? kFragL3 : kFragL2) + 1)];
        const floatx4 bias = __builtin_bit_cast(floatx4, F[64 * (kFragBias + layer)]);
        const float k = layer ? k1 : k0;
        u32x4 b[4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            float h[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) h[r] = fmaxf(fmaf(c[mt][r], k, bias[r]), 0.0f);
            b[mt] = split4(h, minus_one);
        }
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) c[mt] = mfma32(wl, b[mt], floatx4{0.0f, 0.0f, 0.0f, 0.0f});
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) c[mt] = mfma32(wh, b[mt], c[mt]);
    }
    __syncthreads();   // every lane has read its inputs; reuse xs for the outputs
    const float *b2 = W + kMlpParams - kMlpOut;
    constexpr int kOut = MlpLds<0>::kOut;
    if (g == 0) {
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int r = 0; r < kMlpOut; ++r) xs[(16 * mt + j) * kOut + r] = fmaf(c[mt][r], k2, b2[r]);
    }
    __syncthreads();
    return make_float3(xs[lane * kOut + 0], xs[lane * kOut + 1], xs[lane * kOut + 2]);
}

// Builds the fragment table (one wave, at upload).
__global__ __launch_bounds__(64) void k_mlp_fragments(const float *__restrict__ W, uint32_t *__restrict__ out) {
    const int lane = (int)threadIdx.x, j = lane & 15, g = lane >> 4;
    const float *W0 = W, *b0 = W0 + kMlpIn * kMlpHidden, *W1 = b0 + kMlpHidden, *b1 = W1 + kMlpHidden * kMlpHidden,
                *W2 = b1 + kMlpHidden;
    auto reduce_max = [](float v) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
        return v;
    };
    auto largest = [&](const float *w, int n) {
        float m = 0.0f;
        for (int i = lane; i < n; i += 64) m = fmaxf(m, fabsf(w[i]));
        return reduce_max(m);
    };
    bool finite = true;
    for (int i = lane; i < kMlpParams; i += 64) finite = finite && fabsf(W[i]) < kInf;
    // bounds of the hidden units: inputs are at most 1 (1.01 for the rounding
    // of sines and weights)
    float bound1 = 0.0f, bound2 = 0.0f;
    if (lane < kMlpHidden) {
        for (int k = 0; k < kMlpIn; ++k) bound1 += 1.01f * fabsf(W0[k * kMlpHidden + lane]);
        bound1 += fabsf(b0[lane]);
    }
    bound1 = reduce_max(bound1);
    if (lane < kMlpHidden) {
        for (int k = 0; k < kMlpHidden; ++k) bound2 += fabsf(W1[k * kMlpHidden + lane]) * bound1;
        bound2 += fabsf(b1[lane]);
    }
    bound2 = reduce_max(bound2);
    // exponents: the largest weight and the bound of the hidden units to
    // 2^14 .. 2^15 as float16
    auto exponent = [](float largest, int want) { return largest > 0.0f && largest < kInf ? want - ilogbf(largest) : 0; };
    const int a0 = exponent(largest(W0, kMlpIn * kMlpHidden), 14), a1 = exponent(largest(W1, kMlpHidden * kMlpHidden), 14),
              a2 = exponent(largest(W2, kMlpHidden * kMlpOut), 14), q1 = exponent(bound1, 14), q2 = exponent(bound2, 14);
    const bool ok = __builtin_amdgcn_ballot_w64(!finite) == 0 && bound1 < kInf && bound2 < kInf &&
                    max(max(abs(a0), abs(a1)), max(max(abs(a2), abs(q1)), abs(q2))) <= 40;
    if (lane == 0) {
        float *head = reinterpret_cast<float *>(out);
        out[0] = ok ? 1u : 0u;
        head[1] = ldexpf(1.0f, ok ? q1 - a0 - kInputScaleLog2 : 0);
        head[2] = ldexpf(1.0f, ok ? q2 - a1 - q1 : 0);
        head[3] = ldexpf(1.0f, ok ? -a2 - q2 : 0);
    }
    u32x4 *F = reinterpret_cast<u32x4 *>(out + kMlpHeader) + lane;
    auto put = [&](int at, float v0, float v1, float v2, float v3) {       // h h and l l of four weights
        const float v[4] = {v0, v1, v2, v3};
        const u32x4 s = split4(v, -1.0f);
        F[64 * at] = u32x4{s.x, s.y, s.x, s.y};
        F[64 * (at + 1)] = u32x4{s.z, s.w, s.z, s.w};
    };
    auto w0 = [&](int k) { return ldexpf(W0[k * kMlpHidden + j], a0); };
    auto w1 = [&](int k) { return ldexpf(W1[k * kMlpHidden + j], a1); };
    auto w2 = [&](int k) { return j < kMlpOut ? ldexpf(W2[k * kMlpOut + min(j, kMlpOut - 1)], a2) : 0.0f; };
    for (int m = 0; m < 2; ++m) put(kFragL1 + 2 * m, w0(16 * m + 4 * g), w0(16 * m + 4 * g + 1), w0(16 * m + 4 * g + 2), w0(16 * m + 4 * g + 3));
    put(kFragL2, w1(4 * g), w1(4 * g + 1), w1(4 * g + 2), w1(4 * g + 3));
    put(kFragL3, w2(4 * g), w2(4 * g + 1), w2(4 * g + 2), w2(4 * g + 3));
    {
        const float v[4] = {w0(32), w0(33), 0.0f, 0.0f};
        const u32x4 s = split4(v, -1.0f);
        const uint32_t t = g == 0 ? s.x : g == 1 ? s.z : 0u;
        F[64 * kFragTail] = u32x4{t, t, 0u, 0u};
    }
    for (int l = 0; l < 2; ++l) {
        const float *b = l ? b1 : b0;
        floatx4 v;
        for (int r = 0; r < 4; ++r) v[r] = ldexpf(b[4 * g + r], l ? q2 : q1);
        F[64 * (kFragBias + l)] = __builtin_bit_cast(u32x4, v);
    }
}

// Returns h(x) for this lane's pixel.  All 64 lanes must call it.
template <int kPrec>
__device__ __forceinline__ float3 deferred_mlp_mfma(const float *__restrict__ W, float *xs, const Accum &acc,
                                                    float3 d, int lane) {
    using Lds = MlpLds<kPrec>;
    const int j = lane & 15, g = lane >> 4;
    const float *W0 = W, *b0 = W0 + kMlpIn * kMlpHidden, *W1 = b0 + kMlpHidden, *b1 = W1 + kMlpHidden * kMlpHidden,
                *W2 = b1 + kMlpHidden, *b2 = W2 + kMlpHidden * kMlpOut;
    // Weights and biases first, so their loads overlap the input encoding.
    // Layer-1 A operand W0^T[hidden j][k]: fp32 steps take k = 9g + q,
    // half-precision steps k = 16 (q / 4) + 4g + q % 4; rows past the 34
    // inputs and output columns past 3 are zero (loaded from a valid address,
    // then replaced, so no load is conditional).
    constexpr int kA0 = kPrec == 0 ? 9 : 12;
    float a0[kA0], a1[4], a2[4], c0[4], c1[4];
#pragma unroll
    for (int q = 0; q < kA0; ++q) {
        const int k = kPrec == 0 ? 9 * g + q : 16 * (q >> 2) + 4 * g + (q & 3);
        const float v = W0[min(k, kMlpIn - 1) * kMlpHidden + j];
        a0[q] = k < kMlpIn ? v : 0.0f;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        a1[q] = W1[(4 * g + q) * kMlpHidden + j];
        const float v = W2[(4 * g + q) * kMlpOut + min(j, kMlpOut - 1)];
        a2[q] = j < kMlpOut ? v : 0.0f;
        c0[q] = b0[4 * g + q];
        c1[q] = b1[4 * g + q];
    }
    {
        float x[48];
        mlp_encode<false>(x, acc, d);
        if constexpr (kPrec == 0) {
#pragma unroll
            for (int i = 0; i < Lds::kWidth; ++i) xs[lane * Lds::kStride + i] = x[i];
        } else {
            half4_t<kPrec> *row = reinterpret_cast<half4_t<kPrec> *>(reinterpret_cast<half_t<kPrec> *>(xs) +
                                                                    lane * Lds::kStride);
#pragma unroll
            for (int i = 0; i < Lds::kWidth / 4; ++i) row[i] = to_half4<kPrec>(x + 4 * i);
        }
    }
    __syncthreads();
    // the four blocks of 16 pixels go through each layer together, so four
    // independent accumulation chains keep the matrix core busy
    floatx4 c[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) c[mt] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (kPrec == 0) {
#pragma unroll
        for (int q = 0; q < 9; ++q)
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
                c[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[q], xs[(16 * mt + j) * Lds::kStride + 9 * g + q], c[mt],
                                                             0, 0, 0);
    } else {
#pragma unroll
        for (int ks = 0; ks < 3; ++ks) {
            const half4_t<kPrec> a = to_half4<kPrec>(a0 + 4 * ks);
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                const half_t<kPrec> *xr = reinterpret_cast<const half_t<kPrec> *>(xs) + (16 * mt + j) * Lds::kStride;
                c[mt] = mfma16<kPrec>(a, *reinterpret_cast<const half4_t<kPrec> *>(xr + 16 * ks + 4 * g), c[mt]);
            }
        }
    }
    float h[4][4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) h[mt][r] = fmaxf(c[mt][r] + c0[r], 0.0f);
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) c[mt] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (kPrec == 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) c[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[q], h[mt][q], c[mt], 0, 0, 0);
    } else {
        const half4_t<kPrec> a = to_half4<kPrec>(a1);
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) c[mt] = mfma16<kPrec>(a, to_half4<kPrec>(h[mt]), c[mt]);
    }
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) h[mt][r] = fmaxf(c[mt][r] + c1[r], 0.0f);
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) c[mt] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (kPrec == 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) c[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a2[q], h[mt][q], c[mt], 0, 0, 0);
    } else {
        const half4_t<kPrec> a = to_half4<kPrec>(a2);
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) c[mt] = mfma16<kPrec>(a, to_half4<kPrec>(h[mt]), c[mt]);
    }
    __syncthreads();   // every lane has read its inputs; reuse xs for the outputs
    // output unit r of pixel 16 mt + j is c[mt][r] of lane j (g = 0)
    if (g == 0) {
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int r = 0; r < kMlpOut; ++r) xs[(16 * mt + j) * Lds::kOut + r] = c[mt][r] + b2[r];
    }
    __syncthreads();
    return make_float3(xs[lane * Lds::kOut + 0], xs[lane * Lds::kOut + 1], xs[lane * Lds::kOut + 2]);
}

// Samples a lane may park ahead of its compositing, and the LDS of a wave:
// during the march the parking area (kDeep x 64 x (p, delta)), the results
// of one shading pass (64 x 8 floats, by shading slot) and the 64-entry
// shading map; the MLP staging afterwards.
// A round shades up to 64 samples at the price of one, so while many rays
// march, three each fill it (parking_depth).  Towards the end of a tile few
// rays are left and a round of three each leaves most of the pass empty: they
// then park as many as still fit 64, up to kDeep, which saves whole rounds for
// some samples parked past a termination.  Measured against three always:
// 1080p 289 -> 275 us, sixteen 1080p views 3.52 -> 3.34 ms, 512x512 93 -> 88 us
// (up to 4: 283, 3.47, 90; up to 7: 280, 3.42, 89, with more marched in vain).
constexpr int kQueue = 3;
constexpr int kDeep = 6;
__device__ __forceinline__ int parking_depth(int marching) {
    return marching > 16 ? kQueue : marching > 12 ? 4 : marching > 8 ? 5 : kDeep;
}
static_assert(16 * 4 <= 64 && 12 * 5 <= 64 && 8 * kDeep <= 64, "a deep round is shaded whole");
constexpr int kParkFloats = 4 * 64 * kDeep + 8 * 65 + 64;
template <int kPrec>
constexpr int kLdsFloats = MlpLds<kPrec>::kFloats > kParkFloats ? MlpLds<kPrec>::kFloats : kParkFloats;

// kLevels: empty space is skipped with the occupancy levels themselves
// (skip_mode 1) instead of the distance grid (skip_mode 0).
// kMode: 0 renders; 1 also adds the statistics counters (and records the
// gathers when rb.rec is set); 2 also takes the phase profile.
// March parameters of one tile's rays.
struct TileParams {
    float step, istep, t_min;
    int32_t delta_mode;
};

// Measurement outputs of the statistics variants (kMode >= 1); see RenderBatch.
struct MeasureArgs {
    unsigned long long *stats;
    uint32_t *rec;
    int32_t *rec_count;
    int32_t rec_cap, total_tiles;
    unsigned long long *phases;
};

// One wave renders local tile lt of camera cam (launch tile `tile`, used by
// the measurement outputs only) of scene sc; lane = threadIdx.x.
// kPart: only the pixels of `part`, the tile's lanes of which lane >> part_shift
// is `part`; the others idle as those outside the image do.
template <int kMode, int kMlpPrec, int kFeat, bool kLevels, bool kPart = false, typename S, typename Cam>
__device__ __forceinline__ void render_tile(const S &sc, const Cam &cam, int lt, int tile,
                                            const TileParams tp, const MeasureArgs ma, float *lds, const int lane,
                                            int part = 0, int part_shift = 6) {
    constexpr bool kStats = kMode >= 1, kPhase = kMode == 2;
    // the tile's corner is uniform: kept in scalar registers
    const int tx0 = __builtin_amdgcn_readfirstlane((lt % cam.tiles_x) * kTile);
    const int ty0 = __builtin_amdgcn_readfirstlane((lt / cam.tiles_x) * kTile);
    const int px = tx0 + (lane & (kTile - 1));
    const int py = ty0 + (lane / kTile);
    const bool active = px < cam.width && py < cam.height && (!kPart || lane >> part_shift == part);
    PhaseClock<kPhase> ph;
    ph.start();

    // ---- pinhole ray
    float vx = ((float)px + 0.5f - cam.cx) * cam.inv_fx;
    float vy = ((float)py + 0.5f - cam.cy) * cam.inv_fy;
    float3 d = make_float3(fmaf(cam.c2w[0], vx, fmaf(cam.c2w[1], vy, cam.c2w[2])),
                           fmaf(cam.c2w[4], vx, fmaf(cam.c2w[5], vy, cam.c2w[6])),
                           fmaf(cam.c2w[8], vx, fmaf(cam.c2w[9], vy, cam.c2w[10])));
    float inv = __builtin_amdgcn_rsqf(d.x * d.x + d.y * d.y + d.z * d.z);
    d.x *= inv; d.y *= inv; d.z *= inv;
    const float3 o = make_float3(cam.c2w[3], cam.c2w[7], cam.c2w[11]);

    Counters cnt = {0u, 0u, 0u, 0u, 0u};
    Accum acc = {1.0f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const float step = tp.step, istep = tp.istep;
    Segment s;
    {
        const Candidates C = make_candidates(o, d);
        const float c1 = first_candidate(C);
        open_segment(o, d, 0.0f, region_at(o, d, c1 < kInf ? 0.5f * c1 : 1.0f), istep, sc.dist_oct_stride, s);
    }
    int nseg = 1;
    // samples this lane may park: kQueue while its ray is marching, 0 once the
    // ray has ended (a comparison with pc gives the wave mask of either state
    // in one instruction, where a flag costs two)
    int room = active ? kQueue : 0;
    float known[kMaxLevels] = {0.0f, 0.0f, 0.0f, 0.0f};   // per level: occupied up to this u
    if (kPhase) ph.lap(kPhSetup);

    // The march runs ahead of the shading: every live lane finds up to `deep`
    // occupied samples (cheap skip iterations) and parks them in LDS; then the
    // wave shades up to 64 parked samples at once -- oldest first, whichever
    // lane's ray they belong to -- so the expensive gather-and-decode code
    // runs with as many lanes busy as possible; then every lane composites
    // its own shaded samples in ray order.  Samples parked past an early
    // termination are dropped, so the image is the one a one-sample-at-a-time
    // march gives.
    float4 *pq = reinterpret_cast<float4 *>(lds);             // [kDeep][64] parked (p, delta)
    float4 *rs = pq + kDeep * 64;                             // [65] x 2: results by shading slot
    int *imap = reinterpret_cast<int *>(rs + 2 * 65);         // [64] shading slot -> parked entry
    // slot 64 is a sample that changes nothing, which the branch-free
    // compositing reads for lanes with no sample of their own
    if (lane < 8) reinterpret_cast<float *>(rs + 2 * 64)[lane] = lane == 0 ? 1.0f : 0.0f;
    int pc = 0;                                               // samples parked by this lane
    do {
        if (kPhase) ph.count(kPhRounds);
        // ---- march: live lanes park up to `deep` samples, one step per
        // pass; the wave stops once 64 samples are parked (a round shades no
        // more), so slow lanes do not hold the others back.  Issue priority
        // by phase: a SIMD's waves that are shading go first, then those
        // compositing, then those marching or in the deferred MLP (the same
        // images; the frames are about 1% faster at 1080p and 2% at 4K)
        __builtin_amdgcn_s_setprio(0);
        int parked = 0;                                       // by the whole wave
#pragma unroll
        for (int j = 0; j < kQueue; ++j) parked += __popcll(__builtin_amdgcn_ballot_w64(pc > j));
        // (samples left over from the last round keep the plain depth, so that
        // a deeper round is always shaded whole)
        const int marching = __popcll(__builtin_amdgcn_ballot_w64(room > 0));
        const int deep = parked > 0 ? kQueue : parking_depth(marching);
        room = room > 0 ? deep : 0;
        for (;;) {
            const bool want = pc < room;
            if (__builtin_amdgcn_ballot_w64(want) == 0 || parked >= 64) break;
            if (kPhase) ph.count(kPhMarchPasses);
            // a lane whose segment is done opens the next region's segment,
            // if any, and marches on in the same pass
            const bool open = want && s.k >= s.n;
            if (kPhase ? __builtin_amdgcn_ballot_w64(open) != 0 : true) {
                if (kPhase) ph.lap(kPhMarch);
                if (open) {
                    if (!(s.tb < kInf) || nseg >= 8) {
                        room = 0;
                    } else {
                        open_segment(o, d, s.tb, s.reg_next, istep, sc.dist_oct_stride, s);
                        ++nseg;
                        if (kStats) ++cnt.opens;
                        known[0] = known[1] = known[2] = known[3] = 0.0f;
                    }
                }
                if (kPhase) {
                    ph.lap(kPhOpen);
                    ph.count(kPhOpenPasses);
                }
            }
            const int pc0 = pc;
            if (want && s.k < s.n) {
                // ---- one march step
                float u0, u1, um;
                interval(s, step, u0, u1, um);
                const float3 p = make_float3(fmaf(um, s.e.x, s.A.x), fmaf(um, s.e.y, s.A.y), fmaf(um, s.e.z, s.A.z));
                if (kStats) ++cnt.visited;
                // a sample in empty space moves the march past the point where
                // the segment leaves it.  A cell seen occupied stays known
                // until the segment leaves it (its exit minus the guard), so
                // later samples inside it need no lookup.
                bool occupied = true;
                if constexpr (!kLevels) {
                    // empty-space grid: leave the whole empty cube ahead, or
                    // remember the occupied cell
                    if (!(um < known[0])) {
                        if (kStats) ++cnt.occ_lookups;
                        float ue;
                        if (dist_lookup(sc, s, p, ue) == 0) {
                            known[0] = ue - kSkipGuard;
                        } else {
                            occupied = false;
                            s.k = skip_past(s, ue, istep);
                        }
                    }
                } else {
                    // the occupancy levels, coarse to fine: stop at the first
                    // empty level and leave its cell
                    float uexit = 0.0f;
#pragma unroll
                    for (int l = 0; l < kMaxLevels; ++l) {
                        if (l < sc.occ_levels && occupied && !(um < known[l])) {
                            const int rl = sc.occ_res[l];
                            const float os = (float)rl * 0.25f, os2 = 2.0f * os;
                            const int qx = cell_index(fmaf(p.x, os, os2), rl);
                            const int qy = cell_index(fmaf(p.y, os, os2), rl);
                            const int qz = cell_index(fmaf(p.z, os, os2), rl);
                            if (kStats) ++cnt.occ_lookups;
                            const bool occ = load_at<uint8_t>(sc.occ[l], cell_offset(qx, qy, qz, rl)) != 0;
                            // exit parameter of this cell along the segment (slab test)
                            const float h = sc.occ_cell[l];
                            const float bx = (float)(s.iex > 0.0f ? qx + 1 : qx) * h - 2.0f;
                            const float by = (float)(s.iey > 0.0f ? qy + 1 : qy) * h - 2.0f;
                            const float bz = (float)(s.iez > 0.0f ? qz + 1 : qz) * h - 2.0f;
                            const float tx = (bx - s.A.x) * s.iex;
                            const float ty = (by - s.A.y) * s.iey;
                            const float tz = (bz - s.A.z) * s.iez;
                            const float ue = fminf(tx, fminf(ty, tz));
                            if (occ) {
                                known[l] = ue - kSkipGuard;
                            } else {
                                occupied = false;
                                uexit = ue;
                            }
                        }
                    }
                    if (!occupied) s.k = skip_past(s, uexit, istep);
                }
                if (occupied) {
                    float delta = u1 - u0;
                    if (tp.delta_mode == 1) {
                        float3 y0 = make_float3(fmaf(u0, s.e.x, s.A.x), fmaf(u0, s.e.y, s.A.y), fmaf(u0, s.e.z, s.A.z));
                        float3 y1 = (s.k == s.n - 1.0f)
                                        ? segment_end(o, d, s.tb, s.reg)
                                        : make_float3(fmaf(u1, s.e.x, s.A.x), fmaf(u1, s.e.y, s.A.y), fmaf(u1, s.e.z, s.A.z));
                        bool at_inf = false;
                        if (s.reg != 0) {
                            const int jj = (s.reg - 1) >> 1;
                            const float sg = ((s.reg - 1) & 1) ? -1.0f : 1.0f;
                            const float y1j = jj == 0 ? y1.x : (jj == 1 ? y1.y : y1.z);
                            at_inf = sg * y1j >= 2.0f;
                        }
                        if (at_inf) {
                            delta = kInf;
                        } else {
                            float3 x0 = unmap_region(s.reg, y0), x1 = unmap_region(s.reg, y1);
                            float dx = x1.x - x0.x, dy = x1.y - x0.y, dz = x1.z - x0.z;
                            delta = sqrtf(dx * dx + dy * dy + dz * dz);
                        }
                    }
                    pq[pc * 64 + lane] = make_float4(p.x, p.y, p.z, delta);
                    ++pc;
                    s.k += 1.0f;
                }
            }
            parked += __popcll(__builtin_amdgcn_ballot_w64(pc != pc0));
        }
        if (kPhase) ph.lap(kPhMarch);
        // ---- shade: parked samples numbered level by level (all first
        // samples, then all second ones ...), lane order within a level;
        // slots past 64 wait for the next round
        int total = 0;
        uint64_t level[kQueue];                               // lanes with more than j parked samples
#pragma unroll
        for (int j = 0; j < kQueue; ++j) {
            level[j] = __builtin_amdgcn_ballot_w64(pc > j);
            const int item = total + lanes_below(level[j]);
            if (pc > j && item < 64) imap[item] = j * 64 + lane;
            total += __popcll(level[j]);
        }
#pragma unroll 1
        for (int j = kQueue; j < deep; ++j) {                 // rolled: few rounds are deep
            const uint64_t m = __builtin_amdgcn_ballot_w64(pc > j);
            if (pc > j) imap[total + lanes_below(m)] = j * 64 + lane;
            total += __popcll(m);
        }
        __syncthreads();
        __builtin_amdgcn_s_setprio(2);
        if (lane < total) {
            const int e = imap[lane];
            const float4 q = pq[e];
            const SampleResult r = eval_sample<kFeat, kMlpPrec == 0>(sc, make_float3(q.x, q.y, q.z), q.w);
            rs[2 * lane] = make_float4(r.trans, r.sg[0], r.sg[1], r.sg[2]);
            rs[2 * lane + 1] = make_float4(r.sg[3], r.sg[4], r.sg[5], r.sg[6]);
        }
        __syncthreads();
        __builtin_amdgcn_s_setprio(1);
        if (kPhase) {
            ph.lap(kPhShade);
            ph.count(kPhShadePasses, total > 0 ? 1 : 0);
            ph.count(kPhShadeLanes, (uint32_t)min(total, 64));
        }
        // ---- composite this lane's shaded samples in ray order
        int before = 0;
        auto composite_slot = [&](int j, int item) {
            const bool use = j < pc && item < 64 && !(acc.T < tp.t_min);      // ends with T below t_min (Sec. 6)
            if constexpr (!kStats) {
                // branch-free: an unused slot composites slot 64, whose alpha
                // is 0 and transmittance 1, which leaves every accumulator
                // bit for bit unchanged (a branch around the update made the
                // compiler copy the accumulators, a weight selected to 0 cost
                // two instructions a slot; with the flags of termination and
                // of shaded samples derived only where they are used, a round
                // costs 19 of 106 instructions less: 1080p 275 -> 269 us, the
                // served kernel, which spilled, 5.7% faster)
                const int it = use ? item : 64;
                const float4 ra = rs[2 * it], rbv = rs[2 * it + 1];
                const float wt = acc.T * (1.0f - ra.x);
                acc.cd0 = fmaf(wt, ra.y, acc.cd0);
                acc.cd1 = fmaf(wt, ra.z, acc.cd1);
                acc.cd2 = fmaf(wt, ra.w, acc.cd2);
                acc.f0 = fmaf(wt, rbv.x, acc.f0);
                acc.f1 = fmaf(wt, rbv.y, acc.f1);
                acc.f2 = fmaf(wt, rbv.z, acc.f2);
                acc.f3 = fmaf(wt, rbv.w, acc.f3);
                acc.T *= ra.x;
            } else if (use) {
                const int e = j * 64 + lane;
                if (kStats && ma.rec) {
                    // measurement: record the texel offsets of this sample
                    const uint32_t k = cnt.evaluated;
                    if (k < (uint32_t)ma.rec_cap) {
                        const float4 q = pq[e];
                        const Footprint f = footprint(sc, make_float3(q.x, q.y, q.z));
                        const uint32_t qs = (uint32_t)tile * 64u + (uint32_t)lane;
                        *reinterpret_cast<u32x4 *>(ma.rec + 4 * ((size_t)k * (size_t)ma.total_tiles * 64u + qs)) =
                            u32x4{f.op[0], f.op[1], f.op[2], (f.bi << 13) | f.ol};
                    }
                }
                const float4 ra = rs[2 * item], rbv = rs[2 * item + 1];
                const SampleResult r = {ra.x, {ra.y, ra.z, ra.w, rbv.x, rbv.y, rbv.z, rbv.w}};
                composite<kStats>(acc, r, cnt);
            }
        };
#pragma unroll
        for (int j = 0; j < kQueue; ++j) {
            composite_slot(j, before + lanes_below(level[j]));
            before += __popcll(level[j]);
        }
#pragma unroll 1
        for (int j = kQueue; j < deep; ++j) {
            const uint64_t m = __builtin_amdgcn_ballot_w64(pc > j);
            composite_slot(j, before + lanes_below(m));
            before += __popcll(m);
        }
        // ---- a ray that has terminated parks nothing more and drops what it
        // has; of the others, keep the samples not shaded yet, in order
        const bool terminated = acc.T < tp.t_min;
        room = terminated ? 0 : room;
        if (total <= 64 || terminated) {
            pc = 0;
        } else {
            int done = 0, first = 0;
#pragma unroll
            for (int j = 0; j < kQueue; ++j) {
                done += j < pc && first + lanes_below(level[j]) < 64 ? 1 : 0;
                first += __popcll(level[j]);
            }
            if (done > 0) {
#pragma unroll
                for (int j = 0; j + 1 < kQueue; ++j)
                    if (j + done < pc) pq[j * 64 + lane] = pq[(j + done) * 64 + lane];
                pc -= done;
            }
        }
        __syncthreads();
        if (kPhase) ph.lap(kPhComposite);
    } while (__builtin_amdgcn_ballot_w64((room | pc) > 0) != 0);

    __builtin_amdgcn_s_setprio(0);      // the MLP at the marching waves' priority
    float3 h;
    if (kMlpPrec == 0 && __builtin_amdgcn_readfirstlane((int)*sc.mlp_frag))
        h = deferred_mlp_split(sc.mlp, sc.mlp_frag, lds, acc, d, lane);
    else
        h = deferred_mlp_mfma<kMlpPrec>(sc.mlp, lds, acc, d, lane);
    if (active) {
        // the pixel again from the lane id (an opaque copy, so the compiler
        // recomputes it instead of holding px and py through the march)
        int l2 = lane;
        asm volatile("" : "+v"(l2));
        const int ox = tx0 + (l2 & (kTile - 1));
        const int oy = ty0 + (l2 / kTile);
        float4 rgba = make_float4(acc.cd0 + h.x, acc.cd1 + h.y, acc.cd2 + h.z, 1.0f - acc.T);
        *reinterpret_cast<float4 *>(cam.out + ((int64_t)oy * cam.width + ox) * 4) = rgba;
    }
    if (kPhase) ph.lap(kPhMlp);
    if (kStats && ma.rec_count) ma.rec_count[tile * 64 + lane] = (int32_t)cnt.evaluated;
    if (kStats) {
        unsigned long long v[6] = {active ? 1ull : 0ull, cnt.occ_lookups, cnt.visited, cnt.evaluated, cnt.contributing,
                                   acc.T < tp.t_min ? 1ull : 0ull};
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            unsigned long long x = v[i];
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
            if (lane == 0 && x) atomicAdd(ma.stats + i, x);
        }
        if (kPhase) {
            ph.count(kPhWaves);
            uint32_t x = cnt.opens;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
            ph.count(kPhOpenLanes, x);
            if (lane < kPhSlots && ph.v) atomicAdd(ma.phases + lane, (unsigned long long)ph.v);
        }
    }
}

template <int kMode, int kMlpPrec, int kFeat, bool kLevels>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_render(const DevScene sc, const RenderBatch rb) {
    __shared__ float lds[kLdsFloats<kMlpPrec>];
    const int slot = xcd_remap((int)blockIdx.x, rb.total_tiles);
    int tile = rb.order ? rb.order[slot] : slot;
    if ((unsigned)tile >= (unsigned)rb.total_tiles) tile = slot;   // never leave the launch
    int c = 0;
#pragma unroll
    for (int i = 1; i < kCamsPerLaunch; ++i)
        if (i < rb.n_cams && tile >= rb.cams[i].tile_start) c = i;
    const DevCamera &cam = rb.cams[c];
    const TileParams tp = {rb.step, rb.inv_step, rb.t_min, rb.delta_mode};
    const MeasureArgs ma = {rb.stats, rb.rec, rb.rec_count, rb.rec_cap, rb.total_tiles, rb.phases};
    render_tile<kMode, kMlpPrec, kFeat, kLevels>(sc, cam, tile - cam.tile_start, tile, tp, ma, lds,
                                                    (int)threadIdx.x);
}

// A launch of so few tiles that their waves leave slots of the device idle: each
// tile is rendered by 1 << parts_log2 waves, a part of its pixels each.  A small
// frame lasts as long as its longest wave, and a wave's rounds follow its
// rays' samples: with 16 rays instead of 64 there are fewer of them
// (parking_depth), and its march waits for fewer rays.  Full scene, back to
// back: 128x128 52.6 -> 37.8 us, 200x150 58.6 -> 49; 8x8 pixels 29.7 -> 23.6.
template <int kMlpPrec, int kFeat, bool kLevels>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_render_parts(const DevScene sc, const RenderBatch rb,
                                                                                              const int parts_log2) {
    __shared__ float lds[kLdsFloats<kMlpPrec>];
    const int slot = xcd_remap((int)blockIdx.x, rb.total_tiles << parts_log2);
    const int tile = slot >> parts_log2, part = slot & ((1 << parts_log2) - 1);
    int c = 0;
#pragma unroll
    for (int i = 1; i < kCamsPerLaunch; ++i)
        if (i < rb.n_cams && tile >= rb.cams[i].tile_start) c = i;
    const DevCamera &cam = rb.cams[c];
    const TileParams tp = {rb.step, rb.inv_step, rb.t_min, rb.delta_mode};
    const MeasureArgs ma = {};
    render_tile<0, kMlpPrec, kFeat, kLevels, true>(sc, cam, tile - cam.tile_start, tile, tp, ma, lds,
                                                      (int)threadIdx.x, part, 6 - parts_log2);
}

// Served launch: workgroup b renders position b / 8 of its XCD's share of
// the launch (XCD x = blockIdx % 8 holds the runs of kXcdChunk consecutive
// tiles that xcd_remap deals to x), so neighbouring tiles still share an L2.
// The grid is a fixed class (the server captures one graph per class), the
// smallest that gives every tile a workgroup of its own; workgroups past the
// launch's tiles exit at once.  A launch larger than the largest such class
// is persistent (a grid of the device's wave slots): its workgroups go on
// taking positions from the XCD's counter, asking for the next one as they
// start each tile so that the atomic's round trip overlaps the render, until
// the share is exhausted; the counters are zeroed before such a launch
// (k_zero_ctl).  (A 4096-workgroup persistent grid rendered a 1080p request
// 13% slower than one workgroup per tile, and 5% slower once its workgroups
// no longer counted themselves out on one shared counter at the end.)  Each
// tile belongs to one request, which names its camera, march parameters and
// scene (a slot of the server's scene table).
typedef const __attribute__((address_space(4))) DevScene ConstScene;
typedef const __attribute__((address_space(4))) ServeLaunch ConstLaunch;
typedef const __attribute__((address_space(4))) ServeWork ConstWork;

__device__ __forceinline__ int xcd_share_tile(int x, uint32_t i) {
    return (int)((((i / kXcdChunk) * kXcds + (uint32_t)x) * kXcdChunk) + i % kXcdChunk);
}

// The scene table and the launch descriptors are read through the constant
// address space: they do not change during the launch, so the compiler reads
// them with scalar loads and may repeat a load instead of holding its value.
template <int kMlpPrec, int kFeat, bool kLevels>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_render_served(
    ConstScene *__restrict__ table, ConstLaunch *__restrict__ launch, ServeCtl *__restrict__ ctl) {
    __shared__ float lds[kLdsFloats<kMlpPrec>];
    const int x = (int)(blockIdx.x % kXcds);
    const uint32_t base = gridDim.x / kXcds;      // positions handed out by workgroup index
    uint32_t *counter = ctl->next + x * kCtlStride;
    uint32_t i = blockIdx.x / kXcds;
    // a launch with more positions per XCD than the grid gives it loops
    const bool loops = base < (uint32_t)((launch->total_tiles + kXcds - 1) / kXcds);
    for (;;) {
        // nothing is carried from one tile to the next: opaque copies of the
        // lane id and the launch pointer keep the compiler from hoisting
        // lane-only address arithmetic and descriptor loads out of this loop
        // and holding them in registers through every tile
        // (the lane id is recomputed from the exec mask: a workgroup is one wave)
        int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        ConstLaunch *L = launch;
        asm volatile("" : "+v"(lane), "+s"(L));
        const int n = L->total_tiles, nw = L->n_work;
        const int tile = xcd_share_tile(x, i);
        if (i >= (uint32_t)n || tile >= n) break;
        uint32_t nx = 0;                           // the next position, in flight during the render
        if (loops && lane == 0) nx = base + atomicAdd(counter, 1u);
        int c = 0;
#pragma unroll
        for (int k = 1; k < kCamsPerLaunch; ++k)
            if (k < nw && tile >= L->work[k].cam.tile_start) c = k;
        ConstWork &w = L->work[c];
        const TileParams tp = {w.step, w.inv_step, w.t_min, w.delta_mode};
        const MeasureArgs ma = {nullptr, nullptr, nullptr, 0, 0, nullptr};
        render_tile<0, kMlpPrec, kFeat, kLevels>(table[w.scene], w.cam, tile - w.cam.tile_start, tile, tp, ma, lds,
                                                    lane);
        if (!loops) break;
        __syncthreads();
        i = (uint32_t)__builtin_amdgcn_readfirstlane((int)__shfl(nx, 0, 64));
    }
}

// Zero a served launch's counters (a node of its own before the launch, so
// that no workgroup of the launch has to find out that it is the last one).
__global__ __launch_bounds__(64) void k_zero_ctl(ServeCtl *__restrict__ ctl) {
    if ((int)threadIdx.x < kXcds) ctl->next[threadIdx.x * kCtlStride] = 0u;
}

// Tile cost for the launch order.  kCostRays rays of every 8x8 tile (pixels
// (2,2), (5,2), (2,5) and (5,5) of the tile, clamped to the image) march as
// the renderer does, through empty space to their first occupied sample.
// With kEffort they go on through occupied space, where the opacity of each
// evaluated sample (its density; the rest of the shading is not needed) is
// composited, until the ray terminates (T < t_min), ends, or has evaluated
// kCostEval samples.  The effort E of a tile is the sum of its rays'
// evaluated samples (a march still running after kCostSteps steps counts
// one); its key is 0 for E = 0 and 1 + [E >= 2 kCostRays] +
// [E >= 3 kCostRays] + [E >= 4 kCostRays] otherwise: rays that reach no
// occupied space only march, rays that terminate within a sample or two
// shade little, and rays that keep shading cost the most.  Without kEffort
// the key is the number of rays that reach occupied space (the cheaper
// prepass, for launches so large that the end of the launch is a small part
// of it).
constexpr int kCostSteps = 64;
constexpr int kCostEval = 4;
constexpr int kEffortMaxTiles = 1 << 16;
constexpr int kGroupTiles = 64 / kCostRays;                   // tiles of one k_tile_cost wave
constexpr int kCountBits = kGroupTiles < 32 ? 5 : 7;           // a group's count of one key
constexpr int kScanBits = 64 / kCostKeys;                      // a workgroup's count of one key
static_assert(kCostKeys * kCountBits <= 32 && (uint64_t)64 * kGroupTiles < (1ull << kScanBits), "count fields");
template <bool kEffort>
__global__ __launch_bounds__(64) void k_tile_cost(const DevScene sc, const RenderBatch rb, uint8_t *__restrict__ keys,
                                                  uint32_t *__restrict__ group_counts) {
    const int g = (int)blockIdx.x * 64 + (int)threadIdx.x;
    const int tile = g / kCostRays, sub = g % kCostRays;
    int ev = 0;                                               // samples this ray evaluated
    if (tile < rb.total_tiles) {
        const DevCamera &cam = rb.cams[camera_of(rb, tile)];
        const int lt = tile - cam.tile_start;
        const int px = min((lt % cam.tiles_x) * kTile + (kCostRays == 1 ? 4 : (sub & 1) ? 5 : 2), cam.width - 1);
        const int py = min((lt / cam.tiles_x) * kTile + (kCostRays == 1 ? 4 : (sub & 2) ? 5 : 2), cam.height - 1);
        float3 o, d;
        pixel_ray(cam, px, py, o, d);
        const float step = rb.step, istep = rb.inv_step;
        Segment s;
        const Candidates C = make_candidates(o, d);
        const float c1 = first_candidate(C);
        open_segment(o, d, 0.0f, region_at(o, d, c1 < kInf ? 0.5f * c1 : 1.0f), istep, sc.dist_oct_stride, s);
        int nseg = 1, it = 0;
        float T = 1.0f;
        for (; it < kCostSteps; ++it) {
            if (s.k >= s.n) {
                if (!(s.tb < kInf) || nseg >= 8) break;
                open_segment(o, d, s.tb, s.reg_next, istep, sc.dist_oct_stride, s);
                ++nseg;
                continue;
            }
            float u0, u1, um;
            interval(s, step, u0, u1, um);
            const float3 p = make_float3(fmaf(um, s.e.x, s.A.x), fmaf(um, s.e.y, s.A.y), fmaf(um, s.e.z, s.A.z));
            float ue;
            if (dist_lookup(sc, s, p, ue) == 0) {
                // an occupied sample: the renderer evaluates it
                if (!kEffort) {
                    ev = 1;
                    break;
                }
                T *= eval_sample<0, true>(sc, p, u1 - u0).trans;
                if (++ev >= kCostEval || T < rb.t_min) break;
                s.k += 1.0f;
            } else {
                s.k = skip_past(s, ue, istep);
            }
        }
        if (it == kCostSteps && ev == 0) ev = 1;
    }
    // the kCostRays rays of a tile are consecutive lanes: their effort from
    // the bits of ev (at most kCostEval < 8)
    static_assert(kCostEval < 8 && kCostRays * kCostEval < 256, "effort bits");
    const uint64_t tm = ((1ull << kCostRays) - 1) << ((int)threadIdx.x & ~(kCostRays - 1));
    int key;
    if (kEffort) {
        int effort = 0;
#pragma unroll
        for (int bit = 0; bit < 3; ++bit) effort += __popcll(__ballot((ev >> bit) & 1) & tm) << bit;
        key = effort == 0 ? 0 : 1 + (effort >= 2 * kCostRays) + (effort >= 3 * kCostRays) + (effort >= 4 * kCostRays);
    } else {
        key = __popcll(__ballot(ev > 0) & tm);
    }
    const bool head = tile < rb.total_tiles && sub == 0;
    if (head) keys[tile] = (uint8_t)key;
    // the keys of the wave's kGroupTiles tiles (a group), counted per key in
    // kCountBits-bit fields
    uint32_t packed = 0u;
#pragma unroll
    for (int k = 0; k < kCostKeys; ++k) packed |= (uint32_t)__popcll(__ballot(head && key == k)) << (kCountBits * k);
    if (threadIdx.x == 0) group_counts[blockIdx.x] = packed;
}

// Stable counting sort of a launch's tiles by cost key, highest key first.
// A wave of k_tile_cost covers a group of kGroupTiles consecutive tiles and
// counts their keys.  Here a 64-lane workgroup places 64 groups, a lane per
// group: the lanes sum the counts of all groups (the totals) and of the
// groups before the workgroup's first, a scan over the lanes adds the counts
// of the lower lanes' groups, and each lane then writes its tiles' positions
// in ascending tile order.  Small workgroups find free wave slots while a
// render kernel occupies the device.
constexpr int kOrderLoads = 16;                               // group counts in flight per lane
__global__ __launch_bounds__(64) void k_tile_order(const uint8_t *__restrict__ keys,
                                                   const uint32_t *__restrict__ group_counts, int n,
                                                   int32_t *__restrict__ order) {
    const int lane = (int)threadIdx.x;
    const int ngroups = (n + kGroupTiles - 1) / kGroupTiles;
    const int g0 = (int)blockIdx.x * 64;                      // first group of this workgroup
    int total[kCostKeys], before[kCostKeys];
#pragma unroll
    for (int k = 0; k < kCostKeys; ++k) total[k] = before[k] = 0;
    for (int base = 0; base < ngroups; base += 64 * kOrderLoads) {
        uint32_t w[kOrderLoads];
#pragma unroll
        for (int u = 0; u < kOrderLoads; ++u) {
            const int g = base + 64 * u + lane;
            w[u] = g < ngroups ? group_counts[g] : 0u;
        }
#pragma unroll
        for (int u = 0; u < kOrderLoads; ++u) {
            const bool earlier = base + 64 * u + lane < g0;
#pragma unroll
            for (int k = 0; k < kCostKeys; ++k) {
                const int c = (int)((w[u] >> (kCountBits * k)) & ((1u << kCountBits) - 1u));
                total[k] += c;
                before[k] += earlier ? c : 0;
            }
        }
    }
#pragma unroll
    for (int k = 0; k < kCostKeys; ++k) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            total[k] += __shfl_xor(total[k], off, 64);
            before[k] += __shfl_xor(before[k], off, 64);
        }
    }
    // this lane's group: its counts widened to kScanBits-bit fields and
    // scanned over the lanes
    const int g = g0 + lane;
    const uint32_t mine = g < ngroups ? group_counts[g] : 0u;
    uint64_t x = 0;
#pragma unroll
    for (int k = 0; k < kCostKeys; ++k)
        x |= (uint64_t)((mine >> (kCountBits * k)) & ((1u << kCountBits) - 1u)) << (kScanBits * k);
    uint64_t incl = x;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint64_t y = __shfl_up(incl, off, 64);
        if (lane >= off) incl += y;
    }
    const uint64_t excl = incl - x;
    // first position of each key for this lane's tiles: all tiles of heavier
    // keys, then those of the same key in earlier groups
    int pos[kCostKeys];
    int run = 0;
#pragma unroll
    for (int k = kCostKeys - 1; k >= 0; --k) {
        pos[k] = run + before[k] + (int)((excl >> (kScanBits * k)) & ((1ull << kScanBits) - 1ull));
        run += total[k];
    }
    if (g < ngroups) {
        u32x4 kv[kGroupTiles / 16];
#pragma unroll
        for (int v = 0; v < kGroupTiles / 16; ++v)
            kv[v] = *reinterpret_cast<const u32x4 *>(keys + kGroupTiles * g + 16 * v);
#pragma unroll
        for (int j = 0; j < kGroupTiles; ++j) {
            const int i = kGroupTiles * g + j;
            const int key = (int)byte_of(kv[j >> 4][(j >> 2) & 3], j & 3);
            int at = pos[0];
#pragma unroll
            for (int k = 1; k < kCostKeys; ++k) at = key == k ? pos[k] : at;
            if (i < n) order[at] = i;
#pragma unroll
            for (int k = 0; k < kCostKeys; ++k) pos[k] += key == k ? 1 : 0;
        }
    }
}

__global__ void k_identity_order(int32_t *__restrict__ order, int n) {
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < n) order[i] = i;
}

// Gather replay (measurement only): each lane re-issues, round by round, the
// texel loads the renderer made for its pixel -- the brick slot, then the six
// plane pairs and the four brick pairs -- with the same tile order and wave
// shape, and no arithmetic beyond the addresses.  Its time bounds what the
// renderer's gathers alone can reach on this working set.
__global__ __launch_bounds__(64) void k_gather_replay(const DevScene sc, const uint32_t *__restrict__ rec,
                                                      const int32_t *__restrict__ rec_count, int cap,
                                                      const int32_t *__restrict__ order, int total_tiles,
                                                      float *__restrict__ out) {
    const int slot = xcd_remap((int)blockIdx.x, total_tiles);
    int tile = order ? order[slot] : slot;
    if ((unsigned)tile >= (unsigned)total_tiles) tile = slot;   // an order of another launch
    const uint32_t q = (uint32_t)tile * 64u + threadIdx.x;
    const size_t slots = (size_t)total_tiles * 64u;
    const int n = min(rec_count[q], cap);
    const uint32_t prow = (uint32_t)sc.R * kChannels;
    uint32_t sink = 0u;
    for (int k = 0; __any(k < n); ++k) {
        if (k < n) {
            const u32x4 r = *reinterpret_cast<const u32x4 *>(rec + 4 * ((size_t)k * slots + q));
            const int brick = load_at<int>(reinterpret_cast<const uint8_t *>(sc.brick_index), (r.w >> 13) * 4u);
            Texels x;
#pragma unroll
            for (int pl = 0; pl < 3; ++pl) {
                const uint32_t o = pl == 0 ? r.x : (pl == 1 ? r.y : r.z);
                x.t[2 * pl] = load_pair(sc.planes, o);
                x.t[2 * pl + 1] = load_pair(sc.planes, o + prow);
            }
            constexpr uint32_t sy = kBrick * kChannels, sz = kBrick * kBrick * kChannels;
            const uint32_t ob = (uint32_t)brick * kBrickBytes + (r.w & 8191u);
            x.g[0] = load_pair(sc.bricks, ob);
            x.g[1] = load_pair(sc.bricks, ob + sy);
            x.g[2] = load_pair(sc.bricks, ob + sz);
            x.g[3] = load_pair(sc.bricks, ob + sz + sy);
            asm volatile("" : "+v"(x.t[0]), "+v"(x.t[1]), "+v"(x.t[2]), "+v"(x.t[3]), "+v"(x.t[4]), "+v"(x.t[5]),
                         "+v"(x.g[0]), "+v"(x.g[1]), "+v"(x.g[2]), "+v"(x.g[3]));
            sink ^= x.t[0].x ^ x.g[0].x;
        }
    }
    reinterpret_cast<float4 *>(out)[q] = make_float4((float)n, (float)(sink & 1u), 0.0f, 0.0f);
}

// Eq. 8 dequantisation of a buffer of codes.  prec 1 runs deq_f16, the
// routine the fp16-feature render path applies to every code it reads, with
// the scale a the upload computes for that path.  prec 0 gives the correctly
// rounded float32 value (deq_f32) and prec 2 that value rounded again to
// bfloat16, which is the correctly rounded bfloat16 value, because k/255
// never lies within half a float32 ulp of a bfloat16 rounding boundary (its
// binary expansion repeats with period 8); the test-suite checks all codes.
// Bound by its traffic (one byte read, two or four written a code): a thread
// takes 16 codes as one vector and stores 16-byte vectors.  Buffers that are
// not aligned to that take the codes one by one (kVec false), as do the last
// n % 16.  Float16, 100.7 M codes: 55 us (5.5 TB/s, as a large copy), 142 us
// with a code per thread.
template <int prec>
__device__ __forceinline__ auto dequant_one(uint32_t code, float m2, float m255, float m, float a24) {
    if constexpr (prec == 1) return __float2half_rn(deq_f16(as_f16x2(code).x, a24, m));   // the subnormal b 2^-24
    else if constexpr (prec == 0) return deq_f32(code, m2, m255);
    else return __float2bfloat16(deq_f32(code, m2, m255));
}

template <int prec, bool kVec>
__global__ __launch_bounds__(256) void k_dequant(const uint8_t *__restrict__ codes, int64_t n, float m, float a,
                                                 void *__restrict__ out) {
    using T = decltype(dequant_one<prec>(0u, 0.0f, 0.0f, 0.0f, 0.0f));
    const float m2 = 2.0f * m, m255 = 255.0f * m, a24 = a * 16777216.0f;
    T *o = reinterpret_cast<T *>(out);
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, nt = (int64_t)gridDim.x * blockDim.x;
    int64_t first = 0;
    if constexpr (kVec) {
        for (int64_t i = t; i < n / 16; i += nt) {
            const u32x4 v = reinterpret_cast<const u32x4 *>(codes)[i];
            T x[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) x[k] = dequant_one<prec>(byte_of(v[k >> 2], k & 3), m2, m255, m, a24);
#pragma unroll
            for (int k = 0; k < (int)sizeof(T); ++k) {
                u32x4 w;
                __builtin_memcpy(&w, x + k * (16 / (int)sizeof(T)), 16);
                reinterpret_cast<u32x4 *>(o + 16 * i)[k] = w;
            }
        }
        first = n / 16 * 16;
    }
    for (int64_t i = first + t; i < n; i += nt) o[i] = dequant_one<prec>(codes[i], m2, m255, m, a24);
}

}  // namespace

template <int kMode, int kFeat, bool kLevels>
const void *render_kernel_mlp(int mlp_prec) {
    return mlp_prec == 0 ? (const void *)k_render<kMode, 0, kFeat, kLevels>
         : mlp_prec == 1 ? (const void *)k_render<kMode, 1, kFeat, kLevels>
                         : (const void *)k_render<kMode, 2, kFeat, kLevels>;
}

template <int kMode, bool kLevels>
const void *render_kernel_feat(const RenderBatch &rb) {
    return rb.feat_prec == 2 ? render_kernel_mlp<kMode, 2, kLevels>(rb.mlp_prec)
         : rb.feat_prec == 1 ? render_kernel_mlp<kMode, 1, kLevels>(rb.mlp_prec)
                             : render_kernel_mlp<kMode, 0, kLevels>(rb.mlp_prec);
}

template <int kMode>
const void *render_kernel_mode(const RenderBatch &rb) {
    return rb.skip_mode ? render_kernel_feat<kMode, true>(rb) : render_kernel_feat<kMode, false>(rb);
}

const void *render_kernel(const RenderBatch &rb) {
    if (rb.phases) return render_kernel_mode<2>(rb);
    if (rb.stats) return render_kernel_mode<1>(rb);
    return render_kernel_mode<0>(rb);
}

dim3 render_grid(const RenderBatch &rb) { return dim3((unsigned)rb.total_tiles); }

template <int kFeat, bool kLevels>
const void *parts_kernel_mlp(int mlp_prec) {
    return mlp_prec == 0 ? (const void *)k_render_parts<0, kFeat, kLevels>
         : mlp_prec == 1 ? (const void *)k_render_parts<1, kFeat, kLevels>
                         : (const void *)k_render_parts<2, kFeat, kLevels>;
}

template <bool kLevels>
const void *parts_kernel(const RenderBatch &rb) {
    return rb.feat_prec == 2 ? parts_kernel_mlp<2, kLevels>(rb.mlp_prec)
         : rb.feat_prec == 1 ? parts_kernel_mlp<1, kLevels>(rb.mlp_prec)
                             : parts_kernel_mlp<0, kLevels>(rb.mlp_prec);
}

// Waves a tile of a launch is divided over (log2): up to eight, as long as they
// take at most three quarters of the device's 4096 slots.  With all of them, frames of
// 256x256 or 352x368 pixels gain a little more alone but lose 11% where four
// streams render them side by side (17.8 -> 19.8 and 20.3 -> 22.6 us each); with
// half of them, 304x320 gains nothing (68.7 us alone and 20.3 on four streams,
// against 58.5 and 19.1).  Beyond 4096, waves queue (256x256 52 -> 63 us).
// Sixteen waves a tile gain only below 64 tiles.
int render_parts_log2(const RenderBatch &rb) {
    int k = 0;
    if (rb.stats || rb.phases || rb.order) return k;
    while (k < kPartsMaxLog2 && (int64_t)rb.total_tiles << (k + 1) <= kPartsMaxWaves) ++k;
    return k;
}

template <int kFeat, bool kLevels>
const void *served_kernel_mlp(int mlp_prec) {
    return mlp_prec == 0 ? (const void *)k_render_served<0, kFeat, kLevels>
         : mlp_prec == 1 ? (const void *)k_render_served<1, kFeat, kLevels>
                         : (const void *)k_render_served<2, kFeat, kLevels>;
}

const void *served_kernel(int mlp_prec, int feat_prec, int skip_mode) {
    if (feat_prec == 2) return skip_mode ? served_kernel_mlp<2, true>(mlp_prec) : served_kernel_mlp<2, false>(mlp_prec);
    if (feat_prec == 1) return skip_mode ? served_kernel_mlp<1, true>(mlp_prec) : served_kernel_mlp<1, false>(mlp_prec);
    return skip_mode ? served_kernel_mlp<0, true>(mlp_prec) : served_kernel_mlp<0, false>(mlp_prec);
}

hipError_t launch_zero_ctl(ServeCtl *ctl, hipStream_t stream) {
    hipLaunchKernelGGL(k_zero_ctl, dim3(1), dim3(64), 0, stream, ctl);
    return hipGetLastError();
}

hipError_t launch_render_served(const DevScene *table, const ServeLaunch *launch, ServeCtl *ctl, int mlp_prec,
                                int feat_prec, int skip_mode, int grid, hipStream_t stream) {
    if (grid < kXcds || grid % kXcds != 0) return hipErrorInvalidValue;
    ConstScene *t = (ConstScene *)table;
    ConstLaunch *l = (ConstLaunch *)launch;
    void *args[] = {&t, &l, &ctl};
    return hipLaunchKernel(served_kernel(mlp_prec, feat_prec, skip_mode), dim3((unsigned)grid), dim3(kRenderBlock),
                           args, 0, stream);
}

hipError_t launch_render(const DevScene &sc, const RenderBatch &rb, hipStream_t stream) {
    if (rb.total_tiles <= 0) return hipSuccess;
    if (int parts_log2 = render_parts_log2(rb)) {
        void *args[] = {const_cast<DevScene *>(&sc), const_cast<RenderBatch *>(&rb), &parts_log2};
        return hipLaunchKernel(rb.skip_mode ? parts_kernel<true>(rb) : parts_kernel<false>(rb),
                               dim3((unsigned)rb.total_tiles << parts_log2), dim3(kRenderBlock), args, 0, stream);
    }
    void *args[] = {const_cast<DevScene *>(&sc), const_cast<RenderBatch *>(&rb)};
    return hipLaunchKernel(render_kernel(rb), render_grid(rb), dim3(kRenderBlock), args, 0, stream);
}

hipError_t launch_tile_order(const DevScene &sc, const RenderBatch &rb, uint8_t *keys, uint32_t *group_counts,
                             int32_t *order, hipStream_t stream) {
    if (rb.total_tiles <= 0 || rb.total_tiles > kOrderMaxTiles) return hipErrorInvalidValue;
    const int groups = (rb.total_tiles + kGroupTiles - 1) / kGroupTiles;
    if (rb.total_tiles <= kEffortMaxTiles)
        hipLaunchKernelGGL(k_tile_cost<true>, dim3((unsigned)groups), dim3(64), 0, stream, sc, rb, keys, group_counts);
    else
        hipLaunchKernelGGL(k_tile_cost<false>, dim3((unsigned)groups), dim3(64), 0, stream, sc, rb, keys, group_counts);
    hipLaunchKernelGGL(k_tile_order, dim3((unsigned)((groups + 63) / 64)), dim3(64), 0, stream, keys, group_counts,
                       rb.total_tiles, order);
    return hipGetLastError();
}

hipError_t launch_identity_order(int32_t *order, int n, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_identity_order, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, order, n);
    return hipGetLastError();
}

hipError_t launch_gather_replay(const DevScene &sc, const uint32_t *rec, const int32_t *rec_count, int cap,
                                const int32_t *order, int total_tiles, float *out, hipStream_t stream) {
    if (total_tiles <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather_replay, dim3((unsigned)total_tiles), dim3(64), 0, stream, sc, rec, rec_count, cap,
                       order, total_tiles, out);
    return hipGetLastError();
}

hipError_t launch_mlp_fragments(const float *mlp, uint32_t *frag, hipStream_t stream) {
    hipLaunchKernelGGL(k_mlp_fragments, dim3(1), dim3(64), 0, stream, mlp, frag);
    return hipGetLastError();
}

hipError_t launch_dequant(const uint8_t *codes, int64_t n, float m, float a, int prec, void *out,
                          hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    const bool vec = reinterpret_cast<uintptr_t>(codes) % 16 == 0 && reinterpret_cast<uintptr_t>(out) % 16 == 0;
    // a vector per thread up to 2^17 workgroups, which 2^29 codes fill
    const int64_t items = vec ? std::max<int64_t>(n / 16, std::min<int64_t>(n, 256)) : n;
    const dim3 grid((unsigned)std::min<int64_t>((items + 255) / 256, vec ? 1 << 17 : 4096)), block(256);
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, stream, codes, n, m, a, out); };
    if (prec == 0) vec ? launch(k_dequant<0, true>) : launch(k_dequant<0, false>);
    else if (prec == 1) vec ? launch(k_dequant<1, true>) : launch(k_dequant<1, false>);
    else vec ? launch(k_dequant<2, true>) : launch(k_dequant<2, false>);
    return hipGetLastError();
}

}  // namespace merf
