// Marching (Sec. 3.4): parameters of a call, Eq. 6 without its divisions, ray clipping and the skip field, shared by the
// wave loop (kn_render.hip) and the fused render (kn_fused.hip).  Included inside each unit's own compile flags; internal
// linkage.
#pragma once

#include "kn_common.h"

#include <math.h>

namespace {

struct MarchParams {
    KnGrid net, occ;
    KnGrid content; // box around everything occupied (res 0: nothing is); rays are clipped against it
    const uint4 *bricks;      // per block of 4^3 voxels: occupancy bits, network, skip value (the fused render)
    const uint32_t *occ_bits; // a bit per voxel (the wave loop: a 32-bit test costs it less than the block's 64 bits)
    int32_t brick_nets;
    const uint8_t *skip_dist;
    int32_t skip_res[3];
    float skip_inv[3];   // 1 / (edge of a skip block) per axis
    float skip_edge_min; // shortest edge of a skip block
    float skip_margin;   // safety margin on the jump radius (position rounding)
    int32_t has_occ;
    // >= 0 on every axis: the occupancy grid refines the network grid by 2^net_shift[a] (same box), so that the
    // network cell of a point is its voxel coordinate shifted right, exactly (scaling the cell edge by a power of two
    // scales the fp32 quotient of Eq. 6 by the same power of two without a rounding difference)
    int32_t net_shift[3];
    float t_near, step;
    int32_t K;
    const int32_t *cell_net; // sparse network grid: cell -> network or -1 (kernels built with OPT_SPARSE read it)
    uint32_t seed_key;       // stratified sampling: kn_mix32(seed) (kernels built with OPT_STRAT use it)
};

// Variants of the marching kernels, chosen at compile time so that the plain path carries none of their cost:
// a sparse network grid (a table look-up per kept point; points in cells without a network are dropped) and
// stratified sampling (lattice points at their drawn offsets instead of the middle of their intervals).
constexpr int OPT_SPARSE = 1, OPT_STRAT = 2;

// One axis of Eq. 6 without the division when the result cannot depend on it: u' = rel * (1/cell)
// differs from the correctly rounded quotient by a few ulp (less than 4.8e-7 |u'|); only when u' sits that close
// to an integer is the division itself evaluated.  `guard` is that bound for the largest |u'| that matters,
// res + 1: beyond it both u' and the quotient are outside [0, res) whatever their last bits are, and callers only
// ask whether the result is inside that range, and which integer it is if so.  Returns floor(quotient) as a float
// (for values inside the range; some value outside the range otherwise; NaN and inf stay what they are).
__device__ __forceinline__ float axis_floor(float rel, float cell, float inv_cell, float guard, float one_minus_guard)
{
    const float u = rel * inv_cell;
    const float f = floorf(u);
    const float frac = u - f;
    if (frac <= guard || frac >= one_minus_guard) return floorf(rel / cell); // (both false for NaN / inf)
    return f;
}

struct GridFast {
    float bmin[3], cell[3], inv[3], resf[3], guard[3], one_minus_guard[3];
    int32_t res1, res2;
};

__host__ __device__ __forceinline__ GridFast make_fast(const KnGrid &g)
{
    GridFast f;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        f.bmin[a] = g.bmin[a];
        f.cell[a] = g.cell[a];
        f.inv[a] = 1.0f / g.cell[a];
        f.resf[a] = (float)g.res[a];
        f.guard[a] = ((float)g.res[a] + 1.0f) * 4.8e-7f + 1e-30f;
        f.one_minus_guard[a] = 1.0f - f.guard[a];
    }
    f.res1 = g.res[1];
    f.res2 = g.res[2];
    return f;
}

// Eq. 6 per axis: integer cell coordinates of a point, false when it is outside the grid
__device__ __forceinline__ bool grid_coords_fast(const GridFast &g, float x, float y, float z, int32_t &ix, int32_t &iy,
                                                 int32_t &iz)
{
    const float fx = axis_floor(x - g.bmin[0], g.cell[0], g.inv[0], g.guard[0], g.one_minus_guard[0]);
    const float fy = axis_floor(y - g.bmin[1], g.cell[1], g.inv[1], g.guard[1], g.one_minus_guard[1]);
    const float fz = axis_floor(z - g.bmin[2], g.cell[2], g.inv[2], g.guard[2], g.one_minus_guard[2]);
    const bool in = (fx >= 0.0f) && (fx < g.resf[0]) && (fy >= 0.0f) && (fy < g.resf[1]) && (fz >= 0.0f) &&
                    (fz < g.resf[2]);
    ix = (int32_t)fx;
    iy = (int32_t)fy;
    iz = (int32_t)fz;
    return in;
}

__device__ __forceinline__ int32_t grid_index_fast(const GridFast &g, float x, float y, float z)
{
    const float fx = axis_floor(x - g.bmin[0], g.cell[0], g.inv[0], g.guard[0], g.one_minus_guard[0]);
    const float fy = axis_floor(y - g.bmin[1], g.cell[1], g.inv[1], g.guard[1], g.one_minus_guard[1]);
    const float fz = axis_floor(z - g.bmin[2], g.cell[2], g.inv[2], g.guard[2], g.one_minus_guard[2]);
    const bool in = (fx >= 0.0f) && (fx < g.resf[0]) && (fy >= 0.0f) && (fy < g.resf[1]) && (fz >= 0.0f) &&
                    (fz < g.resf[2]);
    if (!in) return -1;
    return ((int32_t)fx * g.res1 + (int32_t)fy) * g.res2 + (int32_t)fz;
}

// Conservative range [k_lo, k_hi) of lattice indices whose point can lie inside the AABB (slab
// test widened by the rounding error of x_k = fma(t_k, d, o) and two steps).  Every index
// outside the range is provably outside the box; indices inside it are still tested exactly.
struct PlainDivide {
    __device__ __forceinline__ float operator()(float a, float b) const { return a / b; }
};
template <typename Divide = PlainDivide>
__device__ __forceinline__ void clip_ray(const KnGrid &g, const float o[3], const float d[3], float t_near, float step,
                                         int32_t K, int32_t &k_lo, int32_t &k_hi, Divide divide = Divide{})
{
    if (g.res[0] == 0) { // empty box
        k_lo = k_hi = 0;
        return;
    }
    float tmin = -INFINITY, tmax = INFINITY;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (d[a] != 0.0f) {
            const float lo = g.bmin[a], hi = g.bmin[a] + g.cell[a] * (float)g.res[a];
            const float inv = divide(1.0f, d[a]);
            float t0 = (lo - o[a]) * inv, t1 = (hi - o[a]) * inv;
            if (t0 > t1) { float s = t0; t0 = t1; t1 = s; }
            const float mag = fabsf(lo) + fabsf(hi) + fabsf(o[a]) + g.cell[a];
            const float margin = mag * 2.4e-7f * fabsf(inv) + 1e-6f * (fabsf(t0) + fabsf(t1));
            tmin = fmaxf(tmin, t0 - margin);
            tmax = fminf(tmax, t1 + margin);
        }
    }
    // k such that t_near + (k + 1/2) step lies in [tmin, tmax], widened by two steps
    float a = floorf(divide(tmin - t_near, step) - 0.5f) - 2.0f;
    float b = ceilf(divide(tmax - t_near, step) - 0.5f) + 3.0f;
    a = fminf(fmaxf(a, 0.0f), (float)K); // NaN -> 0
    b = fminf(fmaxf(b, 0.0f), (float)K);
    if (!(tmin <= tmax)) { // empty -> nothing; NaN -> stay conservative (full range)
        if (tmin > tmax) { a = 0.0f; b = 0.0f; } else { a = 0.0f; b = (float)K; }
    }
    k_lo = (int32_t)a;
    k_hi = (int32_t)b;
}

// Jump length bookkeeping shared by the two users of the skip field.  A point whose block has
// Chebyshev distance dist >= 2 to the nearest occupied block lies in an empty block, and so does
// every point within Euclidean distance (dist-1) * (shortest block edge) of it, minus a rounding
// margin: jump(dist) is how many further lattice indices that covers.
struct SkipJump {
    float a, b;
    bool use;
    // strat: with stratified sampling point k + j lies up to j + 1 steps from point k, one more than on the
    // midpoint lattice
    __device__ __forceinline__ SkipJump(const MarchParams &p, const float o[3], const float d[3], bool strat)
    {
        const float dlen = sqrtf(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
        const float inv_step_len = 1.0f / (p.step * dlen); // 1 / distance covered by one lattice step
        a = p.skip_edge_min * inv_step_len;
        b = (p.skip_margin + 1e-6f * (fabsf(o[0]) + fabsf(o[1]) + fabsf(o[2]))) * inv_step_len + (strat ? 2.0f : 1.0f);
        use = p.skip_dist != nullptr && isfinite(inv_step_len);
    }
    // (up to the largest integer)
    __device__ __forceinline__ int32_t jump(int32_t dist) const { return (int32_t)fmaxf(floorf((float)(dist - 1) * a - b), 0.0f); }
};

// skip-field value at a point; -1 = the point is (up to rounding) outside the field
__device__ __forceinline__ int32_t skip_lookup(const MarchParams &p, float x, float y, float z)
{
    const float cx = floorf((x - p.occ.bmin[0]) * p.skip_inv[0]);
    const float cy = floorf((y - p.occ.bmin[1]) * p.skip_inv[1]);
    const float cz = floorf((z - p.occ.bmin[2]) * p.skip_inv[2]);
    if (cx >= 0.0f && cx < (float)p.skip_res[0] && cy >= 0.0f && cy < (float)p.skip_res[1] && cz >= 0.0f &&
        cz < (float)p.skip_res[2])
        return p.skip_dist[((int32_t)cx * p.skip_res[1] + (int32_t)cy) * p.skip_res[2] + (int32_t)cz];
    return -1;
}

// One thread walks a ray through provably empty space: returns the first index in [k, k_hi) whose
// point is not known to be empty (or k_hi).  No index it passes over can be a kept sample.
template <int OPT>
__device__ __forceinline__ int32_t skip_to_content(const MarchParams &p, const GridFast &go, const float o[3],
                                                   const float d[3], int32_t k, int32_t k_hi, uint32_t ray_key)
{
    constexpr bool STRAT = (OPT & OPT_STRAT) != 0;
    if (k >= k_hi) return k_hi; // the ray misses the content box: nothing to walk through
    const SkipJump sj(p, o, d, STRAT);
    if (!sj.use) return k;
    while (k < k_hi) {
        float x, y, z;
        kn_lattice_point<STRAT>(o[0], o[1], o[2], d[0], d[1], d[2], p.t_near, p.step, k, x, y, z, ray_key);
        const int32_t dist = skip_lookup(p, x, y, z);
        if (dist >= 2) {
            const int32_t further = sj.jump(dist); // (saturated where a step is far shorter than a block: the sum would wrap)
            k = further >= k_hi - k ? k_hi : k + 1 + further;
        } else if (dist < 0 && grid_index_fast(go, x, y, z) < 0) {
            k += 1; // exactly outside the AABB (the clip range starts a little before the box)
        } else {
            break;
        }
    }
    return min(k, k_hi);
}

// a grid, for voxel_coords
struct VoxelFast {
    float inv[3], shift[3], guard, one_minus_guard, bmin[3], cell[3];
    int32_t res[3];
};

// float -> floor as an integer, as the instruction defines it for every input: saturated, NaN -> 0
__device__ __forceinline__ int32_t floor_int(float f)
{
    int32_t i;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(i) : "v"(f));
    return i;
}

// Eq. 6 per axis on the grid that is marched through: integer cell coordinates (any value outside [0, res) for points
// outside).  u = x / cell - bmin / cell in one multiply-add differs from the quotient of Eq. 6 by less than `guard` (host:
// voxel_fast); true where some u is that close to an integer: the caller then evaluates the divisions themselves.
__device__ __forceinline__ bool voxel_coords(const VoxelFast &g, float x, float y, float z, int32_t &ix, int32_t &iy, int32_t &iz, float *u = nullptr)
{
    const float ux = fmaf(x, g.inv[0], g.shift[0]), uy = fmaf(y, g.inv[1], g.shift[1]), uz = fmaf(z, g.inv[2], g.shift[2]);
    const float fx = __builtin_amdgcn_fractf(ux), fy = __builtin_amdgcn_fractf(uy), fz = __builtin_amdgcn_fractf(uz);
    ix = floor_int(ux);
    iy = floor_int(uy);
    iz = floor_int(uz);
    if (u) { // (known at compile time)
        u[0] = ux;
        u[1] = uy;
        u[2] = uz;
    }
    return (fminf(fminf(fx, fy), fz) <= g.guard) | (fmaxf(fmaxf(fx, fy), fz) >= g.one_minus_guard);
}

__device__ __forceinline__ bool inside(const VoxelFast &g, int32_t ix, int32_t iy, int32_t iz)
{
    return ((uint32_t)ix < (uint32_t)g.res[0]) & ((uint32_t)iy < (uint32_t)g.res[1]) & ((uint32_t)iz < (uint32_t)g.res[2]);
}

// u = fma(x, fl(1/cell), fl(-bmin * fl(1/cell))) against fl(fl(x - bmin) / cell): with A = max(|bmin|, |bmax|) / cell, the
// roundings of 1/cell, of the product and of u amount to 2^-24 (3 A + res), those of Eq. 6 to 2^-23 res, for every x
// inside the box; 2e-7 (A + res + 1) is above their sum.
inline VoxelFast voxel_fast(const KnGrid &g)
{
    VoxelFast v;
    v.guard = 0.0f;
    for (int a = 0; a < 3; ++a) {
        v.bmin[a] = g.bmin[a];
        v.cell[a] = g.cell[a];
        v.res[a] = g.res[a];
        v.inv[a] = 1.0f / g.cell[a];
        v.shift[a] = -g.bmin[a] * v.inv[a];
        const float reach = fmaxf(fabsf(g.bmin[a]), fabsf(g.bmin[a] + g.cell[a] * (float)g.res[a]));
        v.guard = fmaxf(v.guard, 2e-7f * (reach * v.inv[a] + (float)g.res[a] + 1.0f) + 1e-30f);
    }
    v.one_minus_guard = 1.0f - v.guard;
    return v;
}

// The fused render's walk to content: the first index in [k, k_hi) whose point is in a block that is occupied or next to one (or
// k_hi); no index in front of it can be a kept sample.  From a point whose block has distance D to the nearest occupied block the
// ray jumps out of the empty cube of blocks around it ((2 D - 1)^3 of them, wherever in its block the point is), where skip_to_content
// jumps by the radius of the ball that is empty around every point of the block: half as many dependent look-ups.
// The place f in the block is counted from the block that was looked up.  Next to a block's face Eq. 6 and the approximate u may put
// the point on different sides; the fraction of u would then be a whole block off, and the jump with it.  Counted like this (the
// difference is exact, and the clamp moves it towards the face that Eq. 6 saw the point at) f is as wrong as u is, less than guard / 4 =
// 5e-8 (A + res + 1) of a block (voxel_fast), and that, with the rounding of both points, is inside the margin: a thousandth of the
// shortest block's edge plus 4e-6 of the box plus 1e-6 of the origin, of which the rounding takes 2^-23 (box + |o|) twice.
// exact(x, y, z, ix, iy, iz): Eq. 6 with its divisions, for points within rounding of a voxel's face.
template <bool STRAT, typename Exact>
__device__ __forceinline__ int32_t walk_to_content(const MarchParams &p, const VoxelFast &g, const float o[3], const float d[3], int32_t k,
                                                   int32_t k_hi, uint32_t ray_key, Exact exact)
{
    if (k >= k_hi || !p.skip_dist) return min(k, k_hi);
    float per_block[3]; // lattice steps per block (infinite: the ray does not move along the axis)
#pragma unroll
    for (int a = 0; a < 3; ++a) per_block[a] = __builtin_amdgcn_rcpf(fabsf(d[a] * (p.step * p.skip_inv[a])));
    const float margin = (p.skip_margin + 1e-6f * (fabsf(o[0]) + fabsf(o[1]) + fabsf(o[2]))) * (1.000001f * __builtin_amdgcn_rcpf(p.skip_edge_min));
    while (k < k_hi) {
        float x, y, z, u[3];
        int32_t ix, iy, iz;
        kn_lattice_point<STRAT>(o[0], o[1], o[2], d[0], d[1], d[2], p.t_near, p.step, k, x, y, z, ray_key);
        if (voxel_coords(g, x, y, z, ix, iy, iz, u)) exact(x, y, z, ix, iy, iz);
        if (!inside(g, ix, iy, iz)) { // (the clipped range starts a little in front of the box)
            ++k;
            continue;
        }
        const int32_t dist = p.skip_dist[kn_mad24(kn_mad24(ix >> 2, p.skip_res[1], iy >> 2), p.skip_res[2], iz >> 2)];
        if (dist < 2) break;
        const float block[3] = {(float)(ix >> 2), (float)(iy >> 2), (float)(iz >> 2)};
        float steps = INFINITY;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float f = __builtin_amdgcn_fmed3f(fmaf(u[a], 1.0f / KN_SKIP_BLOCK, -block[a]), 0.0f, 1.0f);
            steps = fminf(steps, ((float)dist - margin - (d[a] > 0.0f ? f : 1.0f - f)) * per_block[a]);
        }
        // (stratified: point k + j lies up to j + 1 steps from point k; saturated, the sum below would wrap)
        const int32_t further = (int32_t)fminf(fmaxf(floorf(steps * 0.999996f) - (STRAT ? 2.0f : 1.0f), 0.0f), 2147483520.0f);
        k = further >= k_hi - k ? k_hi : k + 1 + further;
    }
    return min(k, k_hi);
}

} // namespace
