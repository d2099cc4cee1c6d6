// Where a ray changes region of the contraction (Eq. 7): the breakpoints along
// it and the search for the next one.  Float32 throughout, as the kernels march.
#pragma once

#include <stdint.h>

namespace merf {

namespace {

constexpr float kInf = __builtin_huge_valf();

// Hardware reciprocal (v_rcp_f32, 1 ulp); rcp(+-0) = +-inf.
__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// ---------------------------------------------------------------------------
// Eq. 7 regions: 0 = unit cube, 1 + 2j + (x_j < 0) = outer region of axis j.
// Ties pick the first axis.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int region_of(float x, float y, float z) {
    float ax = fabsf(x), ay = fabsf(y), az = fabsf(z);
    int j = 0;
    float r = ax, v = x;
    if (ay > r) { r = ay; j = 1; v = y; }
    if (az > r) { r = az; j = 2; v = z; }
    if (r <= 1.0f) return 0;
    return 1 + 2 * j + (v < 0.0f ? 1 : 0);
}

struct Candidates {
    float c[12];
};

__device__ __forceinline__ float valid_t(float t) { return t > 0.0f ? t : kInf; }    // (NaN: kInf)

// Parameters t > 0 where the ray can change region: x_j = +-1, x_j = +-x_k.
// Hardware reciprocals (1 ulp) replace divisions: a breakpoint is only needed
// to FP32 accuracy, and a zero denominator still gives +-inf (no candidate).
__device__ __forceinline__ Candidates make_candidates(float3 o, float3 d) {
    Candidates C;
    const float ix = rcp(d.x), iy = rcp(d.y), iz = rcp(d.z);
    C.c[0] = valid_t((1.0f - o.x) * ix);
    C.c[1] = valid_t((-1.0f - o.x) * ix);
    C.c[2] = valid_t((1.0f - o.y) * iy);
    C.c[3] = valid_t((-1.0f - o.y) * iy);
    C.c[4] = valid_t((1.0f - o.z) * iz);
    C.c[5] = valid_t((-1.0f - o.z) * iz);
    C.c[6] = valid_t((o.y - o.x) * rcp(d.x - d.y));
    C.c[7] = valid_t((-o.y - o.x) * rcp(d.x + d.y));
    C.c[8] = valid_t((o.z - o.x) * rcp(d.x - d.z));
    C.c[9] = valid_t((-o.z - o.x) * rcp(d.x + d.z));
    C.c[10] = valid_t((o.z - o.y) * rcp(d.y - d.z));
    C.c[11] = valid_t((-o.z - o.y) * rcp(d.y + d.z));
    return C;
}

// Smallest candidate (kInf if none).
__device__ __forceinline__ float first_candidate(const Candidates &C) {
    float m = C.c[0];
#pragma unroll
    for (int i = 1; i < 12; ++i) m = fminf(m, C.c[i]);
    return m;
}

// Smallest candidate strictly greater than t (kInf if none), for 0 < t < kInf.
// Positive floats order as their bits do, so a candidate's distance above t is
// one subtraction (half the instructions of comparing and selecting each), and
// wraps to more than kInf's own distance when the candidate is not above.  The
// minimum starts at kInf's: a ray that looks across the cube from outside all
// three of its slabs has twelve finite candidates, none above its last exit.
__device__ __forceinline__ float next_candidate(const Candidates &C, float t) {
    const uint32_t base = __float_as_uint(t) + 1u;
    uint32_t m = __float_as_uint(kInf) - base;
#pragma unroll
    for (int i = 0; i < 12; ++i) m = min(m, __float_as_uint(C.c[i]) - base);
    return __uint_as_float(m + base);
}

__device__ __forceinline__ int region_at(float3 o, float3 d, float t) {
    return region_of(o.x + t * d.x, o.y + t * d.y, o.z + t * d.z);
}

struct RegionExit {
    float t;                        // world parameter (kInf: the ray stays in the region)
    int next;                       // the region entered
};

// Where the ray leaves region reg, in which it is just after world parameter
// ta, and the region it enters there.
// Every region is convex, so the ray leaves reg at the first breakpoint after
// ta on one of reg's own boundary planes that it crosses outward: inside the
// cube any face x_j = +-1; in the outer region of axis a (sign s) its face
// x_a = s when |x_a| shrinks, and a plane x_a = +-x_k when |x_k| grows past
// |x_a| there.  The direction of a crossing follows from the signs of the
// direction's components, so it is exact even where several planes meet
// (a ray through a cube edge crosses the seam between two outer regions into
// the region it enters, not out of it).  The region entered is read at the
// midpoint to the next breakpoint of the full set; where that midpoint is
// within rounding of the exit and still reads reg, it is the region across
// the exit plane (the outer region of face x_j = +-1, the cube across a face
// x_a = s, axis k with the sign x_k takes across x_a = +-x_k).
__device__ __forceinline__ RegionExit region_exit(float3 o, float3 d, float ta, int reg) {
    const Candidates C = make_candidates(o, d);
    // the six boundary planes of reg: cube {0..5}; axis 0 {0, 1, 6, 7, 8, 9};
    // axis 1 {2, 3, 6, 7, 10, 11}; axis 2 {4, 5, 8, 9, 10, 11}
    const int ax = (reg - 1) >> 1, neg = (reg - 1) & 1;
    const bool in_cube = reg == 0, a0 = !in_cube && ax == 0, a1 = !in_cube && ax == 1;
    float cr[6];
    cr[0] = in_cube || a0 ? C.c[0] : (a1 ? C.c[2] : C.c[4]);
    cr[1] = in_cube || a0 ? C.c[1] : (a1 ? C.c[3] : C.c[5]);
    cr[2] = in_cube ? C.c[2] : (a0 || a1 ? C.c[6] : C.c[8]);
    cr[3] = in_cube ? C.c[3] : (a0 || a1 ? C.c[7] : C.c[9]);
    cr[4] = in_cube ? C.c[4] : (a0 ? C.c[8] : C.c[10]);
    cr[5] = in_cube ? C.c[5] : (a0 ? C.c[9] : C.c[11]);
    // outer regions: the other axes k1 < k2, and for each plane whether
    // crossing it leaves the region (|x_a| shrinks below 1, or |x_k| grows
    // past |x_a|)
    const int k1 = a0 ? 1 : 0, k2 = ax == 2 ? 1 : 2;
    const float da = ax == 0 ? d.x : (ax == 1 ? d.y : d.z);
    const float dk1 = k1 == 0 ? d.x : d.y, dk2 = k2 == 1 ? d.y : d.z;
    const bool sneg = neg != 0;
    bool out[6];
    out[0] = in_cube || (!sneg && da < 0.0f);
    out[1] = in_cube || (sneg && da > 0.0f);
    out[2] = in_cube || ((dk1 > da) != sneg);
    out[3] = in_cube || ((da + dk1 < 0.0f) != sneg);
    out[4] = in_cube || ((dk2 > da) != sneg);
    out[5] = in_cube || ((da + dk2 < 0.0f) != sneg);
    float tb = kInf;
    int hit = 0;
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const bool nearer = out[i] && cr[i] > ta && cr[i] < tb;    // ties: the first plane
        tb = nearer ? cr[i] : tb;
        hit = nearer ? i : hit;
    }
    // the region across the exit plane (regions are 1 + 2k + (x_k < 0)): from
    // the cube, that of face hit; from axis a, the cube across its faces
    // (planes 0, 1), axis k across x_a = x_k with the sign of x_a (planes 2, 4)
    // and across x_a = -x_k with the other sign (planes 3, 5)
    const int kk = hit < 4 ? k1 : k2;
    const int across = in_cube ? 1 + hit : (hit < 2 ? 0 : 1 + 2 * kk + (neg ^ (hit & 1)));
    RegionExit x = {tb, reg};
    if (tb < kInf) {
        const float n2 = next_candidate(C, tb);
        const int r2 = region_at(o, d, n2 < kInf ? 0.5f * (tb + n2) : 2.0f * tb + 1.0f);
        x.next = r2 != reg ? r2 : across;
    }
    return x;
}

}  // namespace

}  // namespace merf
