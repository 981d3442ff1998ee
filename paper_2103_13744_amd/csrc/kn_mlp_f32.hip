// Grouped tiny-MLP evaluation in fp32 (scenes with KN_F32 weights) on the matrix cores' fp32 path.
//
// Same decomposition as the 16-bit kernel: a wavefront takes a contiguous range of tiles (<= 64 consecutive
// entries of the grouped sample list, all of one network) and keeps the network's weights in registers until
// the network changes.  Every layer of Sec. 3.2 / Eq. 7 is computed transposed, out^T = W^T * act^T, with
// v_mfma_f32_16x16x4_f32: the A operand is a 16(out) x 4(in) block of W^T (lane (m, g) = (lane%16, lane/16)
// supplies W[in slot g][out m]), the B operand a 4(in) x 16(samples) block of activations (lane (n, g)
// supplies input slot g of sample n), the accumulator a 16(out) x 16(samples) tile of which lane (n, g)
// holds outputs 4g + 0..3 of sample n.  An accumulator register is therefore already the B operand of one
// MFMA of the next layer: MFMA (t, j) of a layer consumes, from lane group g, hidden unit 16t + 4g + j.
// Which input sits in which slot is free as long as the A operand follows; weights are gathered from the
// canonical layout into that order once per scene (k_pack_weights_f32), as an image of the register file.
//
// Input slots.
//   gamma(x), 16 MFMAs q: group g < 3: axis g, frequency q/2, sin for even q, cos for odd q;
//                         group 3:    q < 12: axis q/4, frequency 8 + (q/2)%2, sin / cos; q = 12..14: x, y, z;
//                                     q = 15: the constant 1 that multiplies b1.
//   gamma(d), 8 MFMAs q:  group g < 3: axis g, frequency q/2, sin / cos; group 3: dx, dy, dz, 1 (b4), 0 x 4.
// b2 initialises accumulators.
//
// Feature layer: layer 3's feature vector has no activation (Sec. 3.2), so feature layer and layer 4 are one affine map of
// the second hidden vector.  The weights' image holds the product of the two (64-bit sums, rounded once), and layer 4 is
// evaluated on the second hidden vector: H/16 * H/4 MFMAs of a sample tile fewer, and a rounding fewer in the results.
// Weights so large or so small that the product, or a sum over it, could leave fp32 where the two layers by themselves
// do not (fold_leaves_range) are kept apart: a scene with such a network is evaluated by the FOLD = false variants.
//
// Density and colour (1 + 3 outputs) would be 4 of 16 rows of their MFMAs.  They are dot products on the vector ALU
// instead, over the hidden units a lane holds, summed over the four lane groups with lane swaps; lane group u keeps the
// (r, g, b, sigma) of sample tile u, so that lane l holds those of sample l of the 64.
//
// What bounds it: the matrix cores (fp32 MFMAs take 32 cycles each; 80 per sample tile at width 32, 224 at width 64), with
// the vector ALU's some 300 instructions per tile beside them, which two wavefronts per SIMD hide in part (cores busy 70 % of
// the kernel at 4 M points; three wavefronts spill and are slower).  Against five separate layers with the heads on the
// matrix cores (112 and 320 MFMAs): 4 M points, 16^3 networks, width 32, 751 -> 633 us, 2 M at width 64 841 -> 675; 800x800
// frame, width 32, 759 -> 619.  Relative error against 64 bits (65,537 points): density 2.4e-7 -> 2.3e-7, colour 1.16e-7 ->
// 1.08e-7; width 64 2.4e-7 -> 2.3e-7, 1.42e-7 -> 1.23e-7.
//
// Encoding: accurate sincosf at frequencies 0, 4 (positions), 0 (directions) and 8 (group 3), up to three steps
// of the double-angle recurrence in between; all in fp32.
#include "kn_common.h"
#include "kn_direct.h"
#include "kn_mlp_f32_core.h"
#include "kn_mlp_shared.h"
#include <hip/hip_ext.h>
#include "kn_probe.h"

namespace {

constexpr int F32_WAVES = 4;
constexpr int F32_TILE_LEN = 64;

// canonical index of the value in register r of lane `lane`; -1 = zero (or, with FOLD, an element of the product of feature
// layer and layer 4 or of its bias, which the packing kernel forms)
template <int H, bool FOLD> __device__ int reg_source(int r, int lane)
{
    using R = Regs<H>;
    constexpr int HQ = R::HQ;
    const int m = lane & 15, g = lane >> 4;
    auto unit = [&](int k) { return 16 * (k >> 2) + 4 * g + (k & 3); }; // hidden unit behind MFMA k for this lane group
    if (r < R::W2) {
        const int t = (r - R::W1) >> 4, q = (r - R::W1) & 15, col = 16 * t + m;
        if (g < 3) return R::oW1 + (3 + 6 * (q >> 1) + 3 * (q & 1) + g) * H + col;
        if (q < 12) return R::oW1 + (3 + 6 * (8 + ((q >> 1) & 1)) + 3 * (q & 1) + (q >> 2)) * H + col;
        return q < 15 ? R::oW1 + (q - 12) * H + col : R::ob1 + col;
    }
    if (r < R::W4) {
        const int t = (r - R::W2) / HQ, k = (r - R::W2) % HQ;
        return R::oW2 + unit(k) * H + 16 * t + m;
    }
    if (r < R::WO) {
        const int t = (r - R::W4) / (HQ + 8), k = (r - R::W4) % (HQ + 8), col = 16 * t + m;
        if (k < HQ) return FOLD ? -1 : R::oW4 + unit(k) * H + col;
        const int q = k - HQ;
        if (g < 3) return R::oW4 + (H + 3 + 6 * (q >> 1) + 3 * (q & 1) + g) * H + col;
        if (q < 3) return R::oW4 + (H + q) * H + col;
        return q == 3 && !FOLD ? R::ob4 + col : -1;
    }
    if (r < R::B2) {
        const int c = (r - R::WO) / HQ, k = (r - R::WO) % HQ;
        return c < 3 ? R::oW5 + unit(k) * 3 + c : R::oW3 + unit(k) * (H + 1);
    }
    if (r < R::BO) return R::ob2 + 16 * ((r - R::B2) >> 2) + 4 * g + ((r - R::B2) & 3);
    if (r < R::W3) return r - R::BO < 3 ? R::ob5 + (r - R::BO) : R::ob3;
    if (r < R::B3) {
        const int t = (r - R::W3) / HQ, k = (r - R::W3) % HQ;
        return R::oW3 + unit(k) * (H + 1) + 1 + 16 * t + m;
    }
    return R::ob3 + 1 + 16 * ((r - R::B3) >> 2) + 4 * g + ((r - R::B3) & 3);
}

// the wavefront's LDS writes before, its reads after
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Whether the product of feature layer and layer 4 may not stand for the two.  Lane j < H of a wavefront bounds output j of each
// layer for every point of the scene's box (|coordinate| <= reach; sines and cosines are at most 1): if the sum of all
// magnitudes in layer 4, with each feature bounded the same way, is far inside fp32, then so are the features, the elements of
// the product and every partial sum over either.  And an element that underflows is off by 2^-150 at most: what that can move a
// colour's pre-activation by has to be below 2^-30.  (NaN and infinity fail the comparisons.)
template <int H>
__device__ bool fold_leaves_range(const float *__restrict__ src, const float *w3, const float *w4, float reach, int j, float *s_h, float *s_moved)
{
    using R = Regs<H>;
    constexpr float LIMIT = 1e38f;
    j = min(j, H - 1); // (the lanes behind repeat the last output)
    float b = fabsf(src[R::ob1 + j]);
#pragma unroll
    for (int i = 0; i < 63; ++i) b += fabsf(src[R::oW1 + i * H + j]) * (i < 3 ? reach : 1.0f);
    s_h[j] = b;
    wave_sync();
    b = fabsf(src[R::ob2 + j]);
#pragma unroll
    for (int i = 0; i < H; ++i) b += fabsf(src[R::oW2 + i * H + j]) * s_h[i];
    wave_sync();
    s_h[j] = b < 1.0f ? 1.0f : b; // (at least 1: the elements of the product are bounded as well)
    wave_sync();
    b = fabsf(src[R::ob3 + 1 + j]);
    float sum = 1.0f;
#pragma unroll 8
    for (int i = 0; i < H; ++i) {
        b += fabsf(w3[i * (H + 1) + 1 + j]) * s_h[i];
        sum += s_h[i];
    }
    float out = 0.0f;
    for (int c = 0; c < 3; ++c) out += fabsf(src[R::oW5 + 3 * j + c]);
    s_moved[j] = out * sum * 7.0064923216240854e-46f; // 2^-150
    wave_sync();
    s_h[j] = b;
    wave_sync();
    b = fabsf(src[R::ob4 + j]);
    float moved = 0.0f;
#pragma unroll 8
    for (int i = 0; i < H; ++i) {
        b += fabsf(w4[i * H + j]) * s_h[i];
        moved += s_moved[i];
    }
#pragma unroll
    for (int i = H; i < H + 27; ++i) b += fabsf(src[R::oW4 + i * H + j]); // (unit directions)
    return !(b <= LIMIT) || !(moved <= 9.3132257e-10f);
}

// One workgroup per network.  Four (H = 64: eight) wavefronts gather the image register by register (which value a register
// holds is uniform but for the lane) and, with FOLD, form the product of the two layers from LDS; one more forms its bias and
// sets `apart` where the product may not be used.
// Bound by the latency of its few trips to memory on small scenes, by memory traffic on large ones.
// Against a thread per element that sums its own product over global memory (which made no bound), creating a scene of 16^3
// networks: width 32 105 -> 66 us (this kernel 45, 232 MB), width 64 469 -> 195 (174, 628 MB); 32^3 931 -> 442 and 3,572 ->
// 1,447; 2^3 24 -> 29 and 25 -> 36 (the bound's chain of layers, and the wait for it).
template <int H> constexpr int PACK_WAVES = H == 32 ? 4 : 8;
template <int H, bool FOLD>
__global__ void __launch_bounds__((PACK_WAVES<H> + FOLD) * KN_WAVE)
    k_pack_weights_f32(const float *__restrict__ w, int64_t P, float reach, float *__restrict__ packed, int32_t *__restrict__ apart)
{
    using R = Regs<H>;
    constexpr int HQ = R::HQ, WAVES = PACK_WAVES<H>;
    __shared__ float s_w3[FOLD ? H * (H + 1) : 1], s_w4[FOLD ? H * H : 1], s_h[H], s_moved[H];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / KN_WAVE), lane = threadIdx.x & (KN_WAVE - 1);
    const float *__restrict__ src = w + blockIdx.x * P;
    float *__restrict__ image = packed + (int64_t)blockIdx.x * R::IMAGE;
    if constexpr (FOLD) {
        constexpr int T = (WAVES + 1) * KN_WAVE, STEPS = (H * (H + 1) + T - 1) / T;
        float v[2][STEPS]; // (all loads in flight together)
#pragma unroll
        for (int q = 0; q < STEPS; ++q) {
            const int i = threadIdx.x + q * T;
            v[0][q] = src[R::oW3 + min(i, H * (H + 1) - 1)];
            v[1][q] = src[R::oW4 + min(i, H * H - 1)];
        }
#pragma unroll
        for (int q = 0; q < STEPS; ++q) {
            const int i = threadIdx.x + q * T;
            if (i < H * (H + 1)) s_w3[i] = v[0][q];
            if (i < H * H) s_w4[i] = v[1][q];
        }
        __syncthreads();
        if (wave == WAVES) {
            if (lane < H) {
                double acc = (double)src[R::ob4 + lane];
#pragma unroll 16
                for (int f = 0; f < H; ++f) acc = fma((double)src[R::ob3 + 1 + f], (double)s_w4[f * H + lane], acc);
                image[image_at<H>(R::W4 + (HQ + 8) * (lane >> 4) + HQ + 3, 48 + (lane & 15))] = (float)acc;
            }
            const bool out_of_range = fold_leaves_range<H>(src, s_w3, s_w4, reach, lane, s_h, s_moved);
            if (__ballot(out_of_range) != 0ull && lane == 0) __hip_atomic_store(apart, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            return;
        }
    }
    constexpr int LAST = (FOLD ? R::W3 : R::N) / 4, BATCH = 3; // groups of four registers, and how many groups' loads are in flight together
    for (int g0 = wave; g0 < LAST; g0 += WAVES * BATCH) {
        int at[BATCH][4];
        f4 v[BATCH];
#pragma unroll
        for (int q = 0; q < BATCH; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j) at[q][j] = reg_source<H, FOLD>(4 * min(g0 + WAVES * q, LAST - 1) + j, lane);
#pragma unroll
        for (int q = 0; q < BATCH; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j) v[q][j] = src[max(at[q][j], 0)];
#pragma unroll
        for (int q = 0; q < BATCH; ++q) {
            const int r = 4 * (g0 + WAVES * q), k = r >= R::W4 && r < R::WO ? (r - R::W4) % (HQ + 8) : -1;
            if (r >= 4 * LAST || (FOLD && k >= 0 && k < HQ)) continue; // (FOLD: elements of the product and its bias are written elsewhere)
#pragma unroll
            for (int j = 0; j < 4; ++j) v[q][j] = at[q][j] < 0 ? 0.0f : v[q][j];
            if (H == 64 || (FOLD && k == HQ && lane >= 48)) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (!(FOLD && k == HQ && j == 3 && lane >= 48)) image[image_at<H>(r + j, lane)] = v[q][j];
            } else {
                *(f4 *)&image[image_at<H>(r, lane)] = v[q];
            }
        }
    }
    if constexpr (FOLD) { // thread: rows 4 kt .. + 3 of the product, columns ct + COLS c
        constexpr int CT = H * H / (4 * WAVES * KN_WAVE), COLS = H / CT;
        static_assert(CT >= 1 && COLS % 16 == 0, "a thread's columns lie in different output tiles at the same lane");
        const int kt = threadIdx.x / COLS, ct = threadIdx.x % COLS;
        double acc[4][CT] = {};
#pragma unroll 4
        for (int f = 0; f < H; ++f) {
            double b[CT];
#pragma unroll
            for (int c = 0; c < CT; ++c) b[c] = (double)s_w4[f * H + ct + COLS * c];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const double a = (double)s_w3[(4 * kt + q) * (H + 1) + 1 + f];
#pragma unroll
                for (int c = 0; c < CT; ++c) acc[q][c] = fma(a, b[c], acc[q][c]);
            }
        }
#pragma unroll
        for (int c = 0; c < CT; ++c) { // hidden unit 4 kt + q is MFMA 4 (kt / 4) + q of lane group kt % 4
            const int col = ct + COLS * c;
            const int r = R::W4 + (HQ + 8) * (col >> 4) + 4 * (kt >> 2), lane = 16 * (kt & 3) + (col & 15);
            if constexpr (H == 32) {
                *(f4 *)&image[image_at<H>(r, lane)] = (f4){(float)acc[0][c], (float)acc[1][c], (float)acc[2][c], (float)acc[3][c]};
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) image[image_at<H>(r + q, lane)] = (float)acc[q][c];
            }
        }
    }
}
// what a wavefront has staged of a chunk: x, y, z, dx, dy, dz per sample
struct Staged {
    const float (*stage)[8];
    __device__ __forceinline__ void operator()(int j, float (&p)[3], float (&d)[3]) const
    {
        const f4 s0 = *(const f4 *)&stage[j][0], s1 = *(const f4 *)&stage[j][4];
        p[0] = s0[0];
        p[1] = s0[1];
        p[2] = s0[2];
        d[0] = s0[3];
        d[1] = s1[0];
        d[2] = s1[1];
    }
};

template <int H, bool FOLD>
__global__ void __launch_bounds__(F32_WAVES *KN_WAVE) __attribute__((amdgpu_waves_per_eu(H == 32 ? 2 : 1, H == 32 ? 2 : 1)))
    k_mlp_f32(const float *__restrict__ packed, KnSampleSrc src, const int32_t *__restrict__ perm,
              const KnTile *__restrict__ tiles, const int32_t *__restrict__ n_tiles, float *__restrict__ sigma,
              float *__restrict__ rgb)
{
    __shared__ float stage[F32_WAVES][KN_WAVE][8]; // x, y, z, dx, dy, dz of the chunk's samples

    const int wave = threadIdx.x / KN_WAVE, lane = threadIdx.x & (KN_WAVE - 1);

    const int total_tiles = *n_tiles;
    const int total_waves = gridDim.x * F32_WAVES;
    // workgroup b runs on XCD b % 8: renumbered so that an XCD (one L2) works on a contiguous eighth of the tile list
    const int xcd_share = gridDim.x >> 3;
    const int block_no = (gridDim.x & 7) == 0 ? (int)(blockIdx.x & 7) * xcd_share + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
    const int wid = __builtin_amdgcn_readfirstlane(block_no * F32_WAVES + wave);
    const int t_lo = __builtin_amdgcn_readfirstlane((int)((int64_t)wid * total_tiles / total_waves));
    const int t_hi = __builtin_amdgcn_readfirstlane((int)((int64_t)(wid + 1) * total_tiles / total_waves));
    if (t_lo >= t_hi) return;

    NetF32<H, FOLD> w;
    auto descriptor = [&](int t) -> KnTile { return tiles[min(t, t_hi - 1)]; };
    auto sample_index = [&](const KnTile &d) {
        const int32_t pos = d.start + min(lane, d.len - 1);
        return perm ? perm[pos] : pos; // (without an index list the sorted list holds the samples themselves)
    };
    KnTile dsc_next = descriptor(t_lo);
    int32_t idx_next = sample_index(dsc_next);
    int32_t net_cur = -1;

    for (int t = t_lo; t < t_hi; ++t) {
        const KnTile tl = dsc_next;
        const int32_t idx = idx_next;
        float x, y, z, dx, dy, dz, dscale;
        int32_t out_idx;
        kn_load_sample(src, idx, x, y, z, dx, dy, dz, dscale, out_idx);
        dsc_next = descriptor(t + 1);
        idx_next = sample_index(dsc_next);
        if (tl.net != net_cur) { // uniform
            w.load(packed, tl.net, lane);
            net_cur = tl.net;
        }
        *(f4 *)&stage[wave][lane][0] = (f4){x, y, z, dx};
        *(f4 *)&stage[wave][lane][4] = (f4){dy, dz, 0.0f, 0.0f};
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

        const f4 out = eval_chunk<H, FOLD>(w, lane, (tl.len + 15) >> 4, Staged{stage[wave]}); // (a small group needs no empty sample tiles)
        __builtin_amdgcn_wave_barrier(); // the staging buffer is rewritten by the next iteration

        if (lane < tl.len) {
            const float sg = fmaxf(out[3], 0.0f) * dscale;
            float col[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) col[c] = 1.0f / (1.0f + expf(-out[c]));
            if (src.out4) {
                *(f4 *)(src.out4 + 4 * (int64_t)out_idx) = (f4){col[0], col[1], col[2], sg};
            } else {
                sigma[out_idx] = sg;
#pragma unroll
                for (int c = 0; c < 3; ++c) rgb[3 * (int64_t)out_idx + c] = col[c];
            }
        }
    }
}

// A small batch in the caller's order: a wavefront takes a few consecutive points and evaluates them network by network
// (kn_direct.hip says when and why).
template <int H, bool FOLD>
__global__ void __launch_bounds__(F32_WAVES *KN_WAVE) __attribute__((amdgpu_waves_per_eu(H == 32 ? 2 : 1, H == 32 ? 2 : 1)))
    k_eval_direct_f32(const float *__restrict__ packed, KnDirectJob job)
{
    __shared__ float stage[F32_WAVES][KN_WAVE][8]; // x, y, z, dx, dy, dz, lane of the sample: the samples of one network
    const int wave = threadIdx.x / KN_WAVE, lane = threadIdx.x & (KN_WAVE - 1);
    const int64_t first = (int64_t)(blockIdx.x * F32_WAVES + wave) << job.lg_points;
    KnDirectPoint pt;
    unsigned long long pending = kn_direct_point(job, first, lane, pt);
    while (pending != 0ull) {
        const int32_t sel = __builtin_amdgcn_readlane(pt.net, (int)__builtin_ctzll(pending));
        NetF32<H, FOLD> w;
        w.load(packed, sel, lane);
        const bool hit = pt.net == sel;
        const unsigned long long hits = __ballot(hit);
        const int c = __popcll(hits), from = (int)__builtin_ctzll(hits);
        // the samples move to the front; the places behind them repeat the first one
        const int hits_below = __popcll(hits & ((1ull << lane) - 1ull)), place = hit ? hits_below : c + lane - hits_below;
        float v[6];
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            const float own = q < 3 ? pt.p[q < 3 ? q : 0] : pt.d[q < 3 ? 0 : q - 3];
            const float first_one = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(own), from));
            v[q] = hit ? own : first_one;
        }
        *(f4 *)&stage[wave][place][0] = (f4){v[0], v[1], v[2], v[3]};
        *(f4 *)&stage[wave][place][4] = (f4){v[4], v[5], __int_as_float(lane), 0.0f};
        pending &= ~hits;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const f4 out = eval_chunk<H, FOLD>(w, lane, (c + 15) / 16, Staged{stage[wave]});
        if (lane < c) {
            const int64_t to = first + __float_as_int(stage[wave][lane][6]);
            job.sigma[to] = fmaxf(out[3], 0.0f);
#pragma unroll
            for (int q = 0; q < 3; ++q) job.rgb[3 * to + q] = 1.0f / (1.0f + expf(-out[q]));
        }
        __builtin_amdgcn_wave_barrier(); // the staging buffer is rewritten by the next pass
    }
}


// Density only, for occupancy extraction (Sec. 3.4): layers 1 and 2 and the density row of layer 3 at the probes of one
// network cell (KnProbeBox).
//
// The probes are a lattice and gamma(x) is a concatenation of what belongs to x, to y and to z, so layer 1 is a sum of three
// vectors that depend on one coordinate each.  A workgroup takes a part of the cell's box of up to job.sub probes per axis,
// forms the vectors of its rows of x (with the bias), y and z once and keeps them in LDS; layer 1 of a probe is then two
// additions per output instead of an encoding and 16 matrix products per 16 outputs, and the probes of the part, numbered z fastest
// and dealt out in chunks of 64, need no order of their own (a lane looks up the rows of its probe wherever they are, so short ranges in z
// leave no lanes empty).  Layer 2 runs on the matrix cores as in k_mlp_f32; the density's partial sums of four tiles are summed over
// the lane groups together, so that lane l ends with probe l of the chunk, and marks its voxel.
//
// Bound: the matrix cores (16 products of 32 cycles per tile at width 32, 64 at width 64; 530 us for 120x100x80 voxels at width 32, where
// they take 400 at the 2.0 GHz of such a load, 1,750 to 1,810 of 1,620 at width 64).  Against an encoding and all of layer 1 per probe, with a
// voxel's probes together (a second pass over every tile with the neighbour's weights where grids do not nest):
// 64^3 voxels on 8^3 networks 519 -> 156 us, on 20^3 1,938 -> 192, 120x100x80 on 16^3 2,986 -> 529; width 64 1,089 -> 500,
// 4,149 -> 631, 6,260 -> 1,748.  The marks: no voxel of twelve 64^3 grids differs from 64 bits, before or after.  Three and
// two wavefronts per SIMD: 1 % faster and 3 % slower.
template <int H>
__global__ void __launch_bounds__(F32_WAVES *KN_WAVE) __attribute__((amdgpu_waves_per_eu(H == 32 ? 4 : 3, H == 32 ? 4 : 3)))
    k_probe_f32(const float *__restrict__ packed, KnProbeJob job)
{
    using R = Regs<H>;
    constexpr int HT = H / 16, HQ = H / 4, ENC = 24;
    extern __shared__ f4 s_probe[];
    const int threads = job.waves * KN_WAVE;
    const int pitch = (job.sub[0] + job.sub[1] + job.sub[2]) | 1; // (odd: the rows' stores below fall on different banks)
    f4 *const tab = s_probe;                                      // [output / 4][row]: the row's part of layer 1; rows of z, y, x
    float *const enc = (float *)(s_probe + HQ * pitch);           // [row][ENC]: sines and cosines of the ten frequencies, coordinate
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / KN_WAVE), lane = tid & (KN_WAVE - 1);
    const int n = lane & 15, g = lane >> 4;

    const int32_t cell = blockIdx.x / job.parts, part = blockIdx.x - cell * job.parts;
    const int32_t net = __builtin_amdgcn_readfirstlane(kn_net_of_cell(job.cell_net, cell));
    if (net < 0) return; // no network: nothing to mark
    KnProbeBox box;
    if (!kn_probe_box(job, cell, box)) return;
    int32_t len[3], cuts[3]; // probes of the cell, parts they are cut into (of equal size or one more)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        len[a] = box.p1[a] - box.p0[a];
        cuts[a] = (len[a] + job.sub[a] - 1) / job.sub[a];
    }
    const int32_t all = cuts[0] * cuts[1] * cuts[2];
    if (part >= all) return;

    const float *__restrict__ image = packed + (int64_t)net * R::IMAGE;
    for (int32_t s = part; s < all; s += job.parts) {
        const int32_t sq = s / cuts[2], at[3] = {sq / cuts[1], sq % cuts[1], s % cuts[2]};
        int32_t lo[3], num[3]; // first probe (counted like box.p0) and probes of the part
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int32_t each = len[a] / cuts[a], more = len[a] % cuts[a];
            lo[a] = box.p0[a] + at[a] * each + min(at[a], more);
            num[a] = each + (at[a] < more ? 1 : 0);
        }
        const int32_t row_y = num[2], row_x = num[2] + num[1], rows = row_x + num[0];

        // ---- encodings of the rows: three accurate evaluations each, at frequencies 0, 4 and 8
        for (int i = tid; i < 3 * rows; i += threads) {
            const int restart = i < rows ? 0 : (i < 2 * rows ? 1 : 2), row = i - restart * rows;
            const bool is_z = row < row_y, is_y = !is_z && row < row_x;
            auto axis = [&](auto x, auto y, auto z) { return is_z ? z : (is_y ? y : x); };
            const float p = kn_probe_coord(axis(job.occ.cell[0], job.occ.cell[1], job.occ.cell[2]), axis(job.occ.bmin[0], job.occ.bmin[1], job.occ.bmin[2]),
                                           axis(box.v0[0], box.v0[1], box.v0[2]), axis(lo[0], lo[1], lo[2]) + row - axis(row_x, row_y, 0));
            float sn[4], cs[4];
            sincosf(p * (restart == 0 ? 1.0f : (restart == 1 ? 16.0f : 256.0f)), &sn[0], &cs[0]);
#pragma unroll
            for (int k = 1; k < 4; ++k) double_angle(sn[k - 1], cs[k - 1], sn[k], cs[k]);
            float *const to = enc + row * ENC + 8 * restart;
            *(f4 *)to = (f4){sn[0], cs[0], sn[1], cs[1]};
            *(f4 *)(to + 4) = restart == 2 ? (f4){p, 0.0f, 0.0f, 0.0f} : (f4){sn[2], cs[2], sn[3], cs[3]};
        }
        __syncthreads();
        // ---- the rows' parts of layer 1: thread = (output, every threads / H-th row)
        {
            const int col = tid & (H - 1);
            const float *const w1 = image;
            float *const out = (float *)(tab + (col >> 2) * pitch) + (col & 3);
            auto weight = [&](int q, int from) { return w1[image_at<H>(R::W1 + 16 * (col >> 4) + q, from + (col & 15))]; };
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                float w[21];
#pragma unroll
                for (int q = 0; q < 16; ++q) w[q] = weight(q, 16 * a);
#pragma unroll
                for (int q = 0; q < 4; ++q) w[16 + q] = weight(4 * a + q, 48);
                w[20] = weight(12 + a, 48);
                const float b1 = a == 0 ? weight(15, 48) : 0.0f;
                const int first = a == 0 ? row_x : (a == 1 ? row_y : 0);
                for (int row = first + tid / H; row < first + num[a]; row += threads / H) {
                    const f4 *const e = (const f4 *)(enc + row * ENC);
                    float acc = b1;
#pragma unroll
                    for (int q = 0; q < 6; ++q) {
                        const f4 v = e[q];
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (4 * q + j < 21) acc = fmaf(w[4 * q + j < 21 ? 4 * q + j : 0], v[j], acc);
                    }
                    out[4 * row] = acc;
                }
            }
        }
        __syncthreads();

        // ---- the probes, 64 at a time
        float w2[HT][HQ], wo[HQ];
        f4 bias2[HT];
#pragma unroll
        for (int t = 0; t < HT; ++t) {
            fetch_registers<H>(image, lane, R::W2 + HQ * t, w2[t], HQ);
            bias2[t] = fetch_registers<H>(image, lane, R::B2 + 4 * t);
        }
        fetch_registers<H>(image, lane, R::WO + 3 * HQ, wo, HQ);
        const float bias_sig = image[image_at<H>(R::BO + 3, 0)];
        const int32_t points = num[0] * num[1] * num[2]; // (at most 48^3: quotients by multiplication are exact)
        const uint32_t by_z = (0x80000000u + (uint32_t)num[2] - 1u) / (uint32_t)num[2], by_y = (0x80000000u + (uint32_t)num[1] - 1u) / (uint32_t)num[1];
        for (int32_t first = wave * KN_WAVE; first < points; first += threads) {
            const int32_t p = min(first + lane, points - 1);
            const int32_t pq = (int32_t)__umulhi(2u * (uint32_t)p, by_z), iz = p - pq * num[2];
            const int32_t ix = (int32_t)__umulhi(2u * (uint32_t)pq, by_y), iy = pq - ix * num[1];
            const int32_t where = iz | (row_y + iy) << 8 | (row_x + ix) << 16;
            float d[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int32_t r = __builtin_amdgcn_ds_bpermute(4 * (16 * u + n), where);
                const f4 *const pz = tab + g * pitch + (r & 255), *const py = tab + g * pitch + ((r >> 8) & 255), *const px = tab + g * pitch + (r >> 16);
                f4 acc[HT], h[HT];
#pragma unroll
                for (int t = 0; t < HT; ++t) {
                    const f4 a = px[4 * t * pitch], b = py[4 * t * pitch], c = pz[4 * t * pitch];
#pragma unroll
                    for (int j = 0; j < 4; ++j) h[t][j] = fmaxf((a[j] + b[j]) + c[j], 0.0f);
                }
#pragma unroll
                for (int t = 0; t < HT; ++t) {
                    acc[t] = bias2[t];
#pragma unroll
                    for (int k = 0; k < HQ; ++k) acc[t] = mfma4(w2[t][k], h[k >> 2][k & 3], acc[t]);
                }
                d[u] = 0.0f;
#pragma unroll
                for (int k = 0; k < HQ; ++k) d[u] = fmaf(wo[k], fmaxf(acc[k >> 2][k & 3], 0.0f), d[u]);
            }
            // sums over the lane groups, tile u's in lane group u
            float half[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const auto v = __builtin_amdgcn_permlane32_swap(__float_as_uint(d[q]), __float_as_uint(d[2 + q]), false, false);
                half[q] = __uint_as_float(v[0]) + __uint_as_float(v[1]);
            }
            const auto v = __builtin_amdgcn_permlane16_swap(__float_as_uint(half[0]), __float_as_uint(half[1]), false, false);
            const float sg = fmaxf((__uint_as_float(v[0]) + __uint_as_float(v[1])) + bias_sig, 0.0f);
            if (sg > job.tau && first + lane < points) {
                const int64_t vx = box.v0[0] + (lo[0] + ix) / 3, vy = box.v0[1] + (lo[1] + iy) / 3, vz = box.v0[2] + (lo[2] + iz) / 3;
                job.occupancy[(vx * job.occ.res[1] + vy) * job.occ.res[2] + vz] = 1;
            }
        }
        __syncthreads(); // the tables are rewritten by the next part
    }
}

} // namespace

int kn_mlp_f32_tile_len(const kn_scene *) { return F32_TILE_LEN; }

// bytes of the packed weights of N networks of width H (0: no kernel for that width)
int64_t kn_mlp_f32_packed_bytes(int32_t H, int64_t N)
{
    if (H != 32 && H != 64) return 0;
    return (int64_t)(H == 32 ? Regs<32>::IMAGE : Regs<64>::IMAGE) * 4 * N;
}

// fills sc->packed_w (kn_mlp_f32_packed_bytes bytes, assigned by the caller) and sets sc->f32_apart; waits for the stream
int kn_mlp_f32_pack_weights(kn_scene *sc, hipStream_t st, const KnHostWord &word)
{
    const int H = sc->desc.hidden;
    if (H != 32 && H != 64) return KN_E_UNSUPPORTED;
    if (!sc->packed_w) return KN_E_INVALID_ARG;
    const float *w = (const float *)sc->desc.weights;
    float *image = (float *)sc->packed_w;
    float reach = 1.0f;
    for (int a = 0; a < 3; ++a) reach = fmaxf(reach, fmaxf(fabsf(sc->desc.aabb_min[a]), fabsf(sc->desc.aabb_max[a])));
    const dim3 grid((unsigned)sc->N), without((H == 32 ? PACK_WAVES<32> : PACK_WAVES<64>) * KN_WAVE), with_fold(without.x + KN_WAVE);
    sc->f32_apart = true;
    if (word.host) {
        *word.host = 0;
        auto pack = H == 32 ? k_pack_weights_f32<32, true> : k_pack_weights_f32<64, true>;
        hipLaunchKernelGGL(pack, grid, with_fold, 0, st, w, sc->P, reach, image, word.dev);
        KN_CHECK_LAUNCH();
        KN_HIP(hipStreamSynchronize(st));
        sc->f32_apart = *word.host != 0;
    }
    if (sc->f32_apart) {
        auto pack = H == 32 ? k_pack_weights_f32<32, false> : k_pack_weights_f32<64, false>;
        hipLaunchKernelGGL(pack, grid, without, 0, st, w, sc->P, reach, image, (int32_t *)nullptr);
        KN_CHECK_LAUNCH();
    }
    return KN_OK;
}

int kn_mlp_f32_launch(const kn_scene *sc, hipStream_t st, const KnSampleSrc &src, const KnBucketOut &b, int64_t max_tiles,
                      float *sigma, float *rgb, hipEvent_t ev_start, hipEvent_t ev_stop)
{
    if (max_tiles <= 0) return KN_OK;
    const float *w = (const float *)sc->packed_w;
    const int H = sc->desc.hidden;
    if (H != 32 && H != 64) return KN_E_UNSUPPORTED;
    // one workgroup of 4 wavefronts per compute unit and resident wavefront (H = 32: two per SIMD, H = 64: one)
    int64_t blocks = kn_div_up(max_tiles, F32_WAVES);
    const int64_t fill = H == 32 ? 512 : 256;
    if (blocks > fill) blocks = fill;
    dim3 grid((unsigned)blocks), block(F32_WAVES * KN_WAVE);
    auto kernel = H == 32 ? (sc->f32_apart ? k_mlp_f32<32, false> : k_mlp_f32<32, true>)
                          : (sc->f32_apart ? k_mlp_f32<64, false> : k_mlp_f32<64, true>);
    if (ev_start && ev_stop)
        hipExtLaunchKernelGGL(kernel, grid, block, 0, st, ev_start, ev_stop, 0, w, src, b.perm, b.tiles, b.n_tiles, sigma, rgb);
    else
        hipLaunchKernelGGL(kernel, grid, block, 0, st, w, src, b.perm, b.tiles, b.n_tiles, sigma, rgb);
    KN_CHECK_LAUNCH();
    return KN_OK;
}

int kn_direct_f32_launch(const kn_scene *sc, hipStream_t st, const KnDirectJob &job, unsigned blocks, hipEvent_t ev_start,
                         hipEvent_t ev_stop)
{
    const int H = sc->desc.hidden;
    if (H != 32 && H != 64) return KN_E_UNSUPPORTED;
    auto kernel = H == 32 ? (sc->f32_apart ? k_eval_direct_f32<32, false> : k_eval_direct_f32<32, true>)
                          : (sc->f32_apart ? k_eval_direct_f32<64, false> : k_eval_direct_f32<64, true>);
    const dim3 grid(blocks), block(F32_WAVES * KN_WAVE);
    if (ev_start && ev_stop) hipExtLaunchKernelGGL(kernel, grid, block, 0, st, ev_start, ev_stop, 0, (const float *)sc->packed_w, job);
    else hipLaunchKernelGGL(kernel, grid, block, 0, st, (const float *)sc->packed_w, job);
    KN_CHECK_LAUNCH();
    return KN_OK;
}

int kn_probe_f32_launch(const kn_scene *sc, hipStream_t st, KnProbeJob job)
{
    const int H = sc->desc.hidden;
    if (H != 32 && H != 64) return KN_E_UNSUPPORTED;
    // up to 48 probes per axis together; fewer in x where that leaves too few workgroups to fill the chip twice
    int64_t parts = 1, probes[3];
    for (int a = 0; a < 3; ++a) {
        probes[a] = 3 * kn_div_up(job.occ.res[a], job.net_res[a]);
        const int64_t cuts = kn_div_up(probes[a], 48);
        job.sub[a] = (int32_t)kn_div_up(probes[a], cuts);
        parts *= cuts;
    }
    while (sc->cells * parts < 2048 && job.sub[0] > 6) {
        parts *= 2;
        job.sub[0] = (job.sub[0] + 1) / 2;
    }
    if (parts > 65536) parts = 65536; // (a workgroup goes on to the cell's next part)
    while (sc->cells * parts > 0x7fffffffLL) parts = kn_div_up(parts, 2);
    job.parts = (int32_t)parts;
    // A wavefront for 64 probes of a part, in the mean.  Four / so, where a cell has one voxel, 27 probes: 32^3 networks 400 -> 143 us, width 64
    // 1,147 -> 451 (three of four wavefronts held places on the compute units, and the one that worked was on the same SIMD in all workgroups);
    // 48^3 voxels on 32^3 networks, 91 probes, 416 -> 247, width 64 1,227 -> 735.
    const int64_t points = KN_PROBES * (int64_t)job.occ.res[0] * job.occ.res[1] * job.occ.res[2] / (sc->cells * parts);
    job.waves = (int32_t)(points >= F32_WAVES * KN_WAVE ? F32_WAVES : points < KN_WAVE ? 1 : kn_div_up(points, KN_WAVE));
    const int pitch = (job.sub[0] + job.sub[1] + job.sub[2]) | 1;
    const size_t lds = (size_t)pitch * (H * 4 + 24 * 4);
    const dim3 grid((unsigned)(sc->cells * parts)), block(job.waves * KN_WAVE);
    const float *w = (const float *)sc->packed_w;
    if (H == 32)
        hipLaunchKernelGGL(k_probe_f32<32>, grid, block, lds, st, w, job);
    else
        hipLaunchKernelGGL(k_probe_f32<64>, grid, block, lds, st, w, job);
    KN_CHECK_LAUNCH();
    return KN_OK;
}
