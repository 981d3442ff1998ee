// Pieces of the 16-bit grouped-MLP kernels that more than one translation unit uses: operand types, the layout of a
// network's slot-order weights, the matrix-core step, activation packing and the encodings.  Included inside each
// unit's own compile flags (see build.py); everything has internal linkage.
#pragma once

#include "kn_common.h"
#include "kn_dir_encode.h"

namespace {

using kn_enc::double_angle;
using kn_enc::INV_2PI;
using kn_enc::pk;
using kn_enc::sincos_rev;

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef __bf16 b2 __attribute__((ext_vector_type(2)));
typedef short s2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned u4 __attribute__((ext_vector_type(4)));

template <int H> struct Lay {
    static constexpr int HT = H / 16, HK = H / 32;
    static constexpr int L1 = 0;                          // (t, kb) -> L1 + 2t + kb
    static constexpr int L2 = L1 + 2 * HT;                // (t, kb) -> L2 + t*HK + kb
    static constexpr int L4 = L2 + HT * HK;                   // (t, kb) -> L4 + t*(HK+1) + kb; kb < HK: h2 through the folded
                                                          // feature layer, kb = HK: gamma(d)
    static constexpr int NBLK = L4 + HT * (HK + 1);
    // Behind the blocks, density row of layer 3 and colour rows of layer 5: one block (kb) for both heads, whose rows have period four.  Width 64: stored
    // for four rows, 256 bytes instead of 1,024, and images start on lines (a block is eight of them then, not parts of nine): 160x120 sparse 69.8 -> 66.6 us,
    // 1080p 978 -> 966, 5,003 points 24.3 -> 23.3.  Width 32, by row: 20,011 points 31.2 -> 29.5, but 800x800 143.5 -> 145.5, 400x300 76.5 -> 79 (three
    // more spilled registers in the fused render); on lines 31.2 -> 32.0.
    static constexpr int HEADS = H == 32 ? 64 : 16;       // in 16 bytes
    static constexpr int LO = NBLK * 64;
    static constexpr int TAIL = LO + HEADS * HK;
    static constexpr int TAIL_FLOATS = H + 4;             // b2[H], b5[3], b3 density
    static constexpr int HALFS = H == 32 ? TAIL * 8 + TAIL_FLOATS * 2 : (TAIL * 8 + TAIL_FLOATS * 2 + 63) & ~63;
    static_assert(HALFS % 8 == 0, "blocks are fetched 16 bytes at a time");
    __device__ static constexpr int heads_at(int kb, int lane) { return LO + HEADS * kb + (H == 32 ? lane : 4 * (lane >> 4) + (lane & 3)); }
    // canonical offsets
    static constexpr int oW1 = 0, ob1 = 63 * H, oW2 = ob1 + H, ob2 = oW2 + H * H, oW3 = ob2 + H,
                         ob3 = oW3 + H * (H + 1), oW4 = ob3 + H + 1, ob4 = oW4 + (H + 27) * H, oW5 = ob4 + H,
                         ob5 = oW5 + 3 * H;
};

template <bool BF> __device__ __forceinline__ f4 mfma(u4 a, u4 b, f4 c)
{
    if constexpr (BF)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8, a), __builtin_bit_cast(b8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h8, b), c, 0, 0, 0);
}

// ReLU on two packed 16-bit floats: as signed 16-bit integers every negative float is negative
__device__ __forceinline__ unsigned relu2(unsigned v)
{
    return __builtin_bit_cast(unsigned, __builtin_elementwise_max(__builtin_bit_cast(s2, v), (s2){0, 0}));
}

// accumulators of one layer (HT tiles) -> B operands of the next (HK blocks)
template <int H, bool BF, bool RELU> __device__ __forceinline__ void pack_acts(const f4 *acc, u4 *B)
{
#pragma unroll
    for (int kb = 0; kb < H / 32; ++kb) {
        unsigned r0 = pk<BF>(acc[2 * kb][0], acc[2 * kb][1]);
        unsigned r1 = pk<BF>(acc[2 * kb][2], acc[2 * kb][3]);
        unsigned r2 = pk<BF>(acc[2 * kb + 1][0], acc[2 * kb + 1][1]);
        unsigned r3 = pk<BF>(acc[2 * kb + 1][2], acc[2 * kb + 1][3]);
        if (RELU) { r0 = relu2(r0); r1 = relu2(r1); r2 = relu2(r2); r3 = relu2(r3); }
        B[kb] = (u4){r0, r1, r2, r3};
    }
}

// B operands of layer 1 for one lane: gamma(x) slots of lane group g (see "Slot order").  ang[0..2]: the lane's three
// restart angles in revolutions; ident[0..1]: the packed pairs (x, y), (z, 1) that sit in group 3's last slots.
template <bool BF, bool WRAP> __device__ __forceinline__ void encode_position(f4 ang, u4 ident, unsigned m3, u4 (&Bx)[2])
{
    // s[q] = sin, m[q] = cos of the q-th angle of this lane
    float s[8], m[8];
    sincos_rev<WRAP>(ang[0], s[0], m[0]);
    double_angle(s[0], m[0], s[1], m[1]);
    sincos_rev<WRAP>(ang[1], s[2], m[2]);
    double_angle(s[2], m[2], s[3], m[3]);
    sincos_rev<WRAP>(ang[2], s[4], m[4]);
    double_angle(s[4], m[4], s[5], m[5]);
    double_angle(s[5], m[5], s[6], m[6]);
    double_angle(s[6], m[6], s[7], m[7]);
    unsigned p[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) p[q] = pk<BF>(s[q], m[q]);
    p[6] = (ident[0] & m3) | (p[6] & ~m3);
    p[7] = (ident[1] & m3) | (p[7] & ~m3);
    Bx[0] = (u4){p[0], p[1], p[2], p[3]};
    Bx[1] = (u4){p[4], p[5], p[6], p[7]};
}
// The gamma(d) block of layer 4.  rev: the lane's direction component in revolutions; ident[2..3]: (dx, dy), (dz, 1).
template <bool BF> __device__ __forceinline__ u4 encode_direction(float rev, u4 ident, unsigned m3)
{
    float s[4], m[4];
    sincos_rev<false>(rev, s[0], m[0]); // directions: |d| far below 256 revolutions
    double_angle(s[0], m[0], s[1], m[1]);
    double_angle(s[1], m[1], s[2], m[2]);
    double_angle(s[2], m[2], s[3], m[3]);
    // group 3: slots 0..3 hold dx, dy, dz, 1; its slots 4..7 meet zero weights, any finite value does
    return (u4){(ident[2] & m3) | (pk<BF>(s[0], m[0]) & ~m3), (ident[3] & m3) | (pk<BF>(s[1], m[1]) & ~m3),
                pk<BF>(s[2], m[2]), pk<BF>(s[3], m[3])};
}

} // namespace
