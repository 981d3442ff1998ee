// The fp32 network on the matrix cores' fp32 path: a network's weights as an image of the register file, and the evaluation of a
// chunk of samples (kn_mlp_f32.hip says how operands and slots are laid out, and packs the images), for every kernel that evaluates
// fp32 scenes.  Included inside units compiled for denormals, NaNs and signed zeros; internal linkage.
#pragma once

#include "kn_common.h"

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4 mfma4(float a, float b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

__device__ __forceinline__ void double_angle(float s, float c, float &s2, float &c2)
{
    s2 = 2.0f * (s * c);
    c2 = fmaf(-2.0f * s, s, 1.0f);
}

template <int H> struct Regs {
    static constexpr int HT = H / 16, HQ = H / 4;
    static constexpr int W1 = 0;                     // (t, q)  -> W1 + 16 t + q
    static constexpr int W2 = W1 + 16 * HT;          // (t, k)  -> W2 + HQ t + k
    static constexpr int W4 = W2 + HQ * HT;          // (t, k)  -> W4 + (HQ + 8) t + k; k < HQ: folded with the feature layer; k >= HQ: gamma(d)
    static constexpr int WO = W4 + (HQ + 8) * HT;    // (c, k)  -> WO + HQ c + k: colour c (c < 3) / density, hidden unit k of the lane group
    static constexpr int B2 = WO + 4 * HQ;           // (t, j): accumulator initial values of this lane
    static constexpr int BO = B2 + 4 * HT;
    static constexpr int W3 = BO + 4;                // (t, k)  -> W3 + HQ t + k: feature rows, (t, j) -> B3 + 4 t + j: their biases;
    static constexpr int B3 = W3 + HQ * HT;          // both only where the feature layer is kept apart
    static constexpr int N = B3 + 4 * HT;
    // Registers WO .. W3 - 1 are the same in the sixteen lanes of a lane group: the image holds them once per group, behind the others.
    static constexpr int GROUPED = W3 - WO, LANED = N - GROUPED, GROUPED_AT = LANED * KN_WAVE;
    static constexpr int IMAGE = GROUPED_AT + ((4 * GROUPED + 31) & ~31); // floats (lines of 128 bytes)
    static_assert(((W2 | W4 | WO | B2 | BO | W3 | B3 | N | HQ) & 3) == 0, "registers are fetched in fours");
    // canonical offsets (Sec. 3.2: five layers, weights before biases)
    static constexpr int oW1 = 0, ob1 = 63 * H, oW2 = ob1 + H, ob2 = oW2 + H * H, oW3 = ob2 + H, ob3 = oW3 + H * (H + 1),
                         oW4 = ob3 + H + 1, ob4 = oW4 + (H + 27) * H, oW5 = ob4 + H, ob5 = oW5 + 3 * H;
};

// Register file image of one network: register r of lane l sits at packed[net * IMAGE + image_at(r, l)].  Width 32: four registers of a
// lane side by side, so that a wavefront fetches them with one 16-byte load per lane (31 loads instead of 124, more than the 63 that can
// be in flight): 300 points 18.2 -> 16 us, 5,000 33 -> 30, 65,537 34 -> 32.5, 4 M 530 -> 520.  Width 64, where weights live in both halves of the
// register file and a load fills either, one by one: in fours 5,000 points 56 -> 59 us, 4 M the same.
// GROUPED registers by lane, half as much again to be fetched / so: 5,003 points on 16^3 networks 29.5 -> 23.1 us, 65,537 32.8 -> 30.6, 100,003 41.5 -> 37.9; width 64 (a
// third) 52.1 -> 47.9, 100,003 89.8 -> 79.9, 1 M 342 -> 337; 64x64 rays 28.4 -> 27.8, 400x300 sparse, width 64, 325 -> 316.
template <int H> __host__ __device__ __forceinline__ constexpr int image_at(int r, int lane)
{
    using R = Regs<H>;
    const bool grouped = r >= R::WO && r < R::W3;
    const int at = grouped ? r - R::WO : (r < R::WO ? r : r - R::GROUPED), stride = grouped ? 4 : KN_WAVE, l = grouped ? lane >> 4 : lane;
    return (grouped ? R::GROUPED_AT : 0) + (H == 32 ? ((at >> 2) * stride + l) * 4 + (at & 3) : at * stride + l);
}
// registers first .. first + n - 1 (multiples of four) of an image
template <int H> __device__ __forceinline__ void fetch_registers(const float *__restrict__ image, int lane, int first, float *to, int n)
{
    if constexpr (H == 32) {
#pragma unroll
        for (int i = 0; i < n; i += 4) {
            const f4 v = *(const f4 *)(image + image_at<H>(first + i, lane));
#pragma unroll
            for (int j = 0; j < 4; ++j) to[i + j] = v[j];
        }
    } else {
#pragma unroll
        for (int i = 0; i < n; ++i) to[i] = image[image_at<H>(first + i, lane)];
    }
}
template <int H> __device__ __forceinline__ f4 fetch_registers(const float *__restrict__ image, int lane, int first)
{
    float v[4];
    fetch_registers<H>(image, lane, first, v, 4);
    return (f4){v[0], v[1], v[2], v[3]};
}
// one network's weights in registers
template <int H, bool FOLD> struct NetF32 {
    using R = Regs<H>;
    static constexpr int HT = H / 16, HQ = H / 4; // output tiles per layer, MFMAs per hidden input vector
    float w1[HT][16], w2[HT][HQ], w4[HT][HQ + 8], wo[4][HQ];
    float w3[FOLD ? 1 : HT][HQ]; // (FOLD: not there)
    f4 bias2[HT], bias3[FOLD ? 1 : HT], bias_out;
    __device__ __forceinline__ void load(const float *__restrict__ packed, int32_t net, int lane)
    {
        const float *__restrict__ image = packed + (int64_t)net * R::IMAGE;
#pragma unroll
        for (int t = 0; t < HT; ++t) {
            fetch_registers<H>(image, lane, R::W1 + 16 * t, w1[t], 16);
            fetch_registers<H>(image, lane, R::W2 + HQ * t, w2[t], HQ);
            fetch_registers<H>(image, lane, R::W4 + (HQ + 8) * t, w4[t], HQ + 8);
            bias2[t] = fetch_registers<H>(image, lane, R::B2 + 4 * t);
            if constexpr (!FOLD) {
                fetch_registers<H>(image, lane, R::W3 + HQ * t, w3[t], HQ);
                bias3[t] = fetch_registers<H>(image, lane, R::B3 + 4 * t);
            }
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) fetch_registers<H>(image, lane, R::WO + HQ * c, wo[c], HQ);
        bias_out = fetch_registers<H>(image, lane, R::BO);
    }
};

// sum over the four lane groups, in all of them
__device__ __forceinline__ float sum_groups(float v)
{
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    const float h = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(h), __float_as_uint(h), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// n_tiles sample tiles (16 u .. 16 u + 15, u < n_tiles <= 4) of a chunk of 64 samples; lane l returns the pre-activations
// (r, g, b, sigma) of sample l.  fetch(j, p, d): position and direction of sample j of the chunk.
template <int H, bool FOLD, typename Fetch> __device__ __forceinline__ f4 eval_chunk(const NetF32<H, FOLD> &w, int lane, int n_tiles, Fetch fetch)
{
    constexpr int HT = H / 16, HQ = H / 4;
    const int n = lane & 15, g = lane >> 4;
    const bool g3 = g == 3;
    const f4 zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
    f4 out = zero4;
#pragma unroll 1
    for (int u = 0; u < n_tiles; ++u) {
        __builtin_amdgcn_s_setprio(0);
        float p[3], d[3];
        fetch(16 * u + n, p, d);
        const float pg = g == 0 ? p[0] : (g == 1 ? p[1] : p[2]);
        const float dg = g == 0 ? d[0] : (g == 1 ? d[1] : d[2]);
        // three accurate evaluations per lane; groups 0..2: axis g at frequencies 0 and 4 and the direction at 0,
        // group 3: the three axes at frequency 8
        const float ang[3] = {g3 ? 256.0f * p[0] : pg, g3 ? 256.0f * p[1] : 16.0f * pg, g3 ? 256.0f * p[2] : dg};
        float cs[3][4], cc[3][4];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            sincosf(ang[c], &cs[c][0], &cc[c][0]);
#pragma unroll
            for (int k = 1; k < 4; ++k) double_angle(cs[c][k - 1], cc[c][k - 1], cs[c][k], cc[c][k]);
        }
        float enc[16], dirv[8];
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int f = q >> 1;
            const float axis_v = (q & 1) ? cc[f >> 2][f & 3] : cs[f >> 2][f & 3];
            const float g3_v = q < 12 ? ((q & 1) ? cc[q >> 2][(q >> 1) & 1] : cs[q >> 2][(q >> 1) & 1])
                                      : (q < 15 ? p[q >= 12 && q < 15 ? q - 12 : 0] : 1.0f);
            enc[q] = g3 ? g3_v : axis_v;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const float axis_v = (q & 1) ? cc[2][q >> 1] : cs[2][q >> 1];
            const float g3_v = q < 3 ? d[q < 3 ? q : 0] : (q == 3 ? 1.0f : 0.0f);
            dirv[q] = g3 ? g3_v : axis_v;
        }
        __builtin_amdgcn_s_setprio(1); // the other wavefront of the SIMD encodes under these: 650 -> 630 us for 4 M points
        f4 acc[HT], h[HT];
        // layer 1: gamma(x) -> H, ReLU
#pragma unroll
        for (int t2 = 0; t2 < HT; ++t2) {
            acc[t2] = zero4;
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[t2] = mfma4(w.w1[t2][q], enc[q], acc[t2]);
        }
#pragma unroll
        for (int t2 = 0; t2 < HT; ++t2)
#pragma unroll
            for (int j = 0; j < 4; ++j) h[t2][j] = fmaxf(acc[t2][j], 0.0f);
        // layer 2: H -> H, ReLU
#pragma unroll
        for (int t2 = 0; t2 < HT; ++t2) {
            acc[t2] = w.bias2[t2];
#pragma unroll
            for (int k = 0; k < HQ; ++k) acc[t2] = mfma4(w.w2[t2][k], h[k >> 2][k & 3], acc[t2]);
        }
#pragma unroll
        for (int t2 = 0; t2 < HT; ++t2)
#pragma unroll
            for (int j = 0; j < 4; ++j) h[t2][j] = fmaxf(acc[t2][j], 0.0f);
        // layer 3: the density; its feature vector is folded into layer 4, or takes the second hidden vector's place
        f4 o = zero4;
#pragma unroll
        for (int k = 0; k < HQ; ++k) o[3] = fmaf(w.wo[3][k], h[k >> 2][k & 3], o[3]);
        if constexpr (!FOLD) {
#pragma unroll
            for (int t2 = 0; t2 < HT; ++t2) {
                acc[t2] = w.bias3[t2];
#pragma unroll
                for (int k = 0; k < HQ; ++k) acc[t2] = mfma4(w.w3[t2][k], h[k >> 2][k & 3], acc[t2]);
            }
#pragma unroll
            for (int t2 = 0; t2 < HT; ++t2) h[t2] = acc[t2];
        }
        // layer 4: [second hidden vector through the folded feature layer (or the features), gamma(d)] -> H, ReLU
#pragma unroll
        for (int t2 = 0; t2 < HT; ++t2) {
            acc[t2] = zero4;
#pragma unroll
            for (int q = 0; q < 8; ++q) acc[t2] = mfma4(w.w4[t2][HQ + q], dirv[q], acc[t2]);
#pragma unroll
            for (int k = 0; k < HQ; ++k) acc[t2] = mfma4(w.w4[t2][k], h[k >> 2][k & 3], acc[t2]);
        }
#pragma unroll
        for (int t2 = 0; t2 < HT; ++t2)
#pragma unroll
            for (int j = 0; j < 4; ++j) h[t2][j] = fmaxf(acc[t2][j], 0.0f);
        // layer 5: H -> colour
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int k = 0; k < HQ; ++k) o[c] = fmaf(w.wo[c][k], h[k >> 2][k & 3], o[c]);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float v = sum_groups(o[c]) + w.bias_out[c];
            out[c] = g == u ? v : out[c];
        }
    }
    return out;
}

} // namespace
