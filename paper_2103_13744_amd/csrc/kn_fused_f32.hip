// The fused render (kn_fused_core.h) of scenes with fp32 weights of width 32 whose feature layer is folded into layer 4.  (Width 64: one
// wavefront per SIMD has nothing to hide its look-ups and weights behind; 0.69 to 1.16 of the wave loop's speed.)
#include "kn_fused_core.h"
#include "kn_mlp_f32_core.h"

namespace {

template <int H> struct Net32 {
    static constexpr bool FLUSHED = false;
    static constexpr int DIR = 0; // (encoded per sample)
    // A sample tile takes 2,560 cycles of the matrix cores: what counts is that no sample is evaluated in vain, that tiles are full and
    // that the wavefronts end together; the march is small beside it.  Rays x slots, at most S samples per ray, frames of 26 kinds against
    // the wave loop: 32 x 512, 32 1.16; 16 x 256, 32 1.20; 16 x 256, 16 1.14 to 1.16; 16 x 128, 16 1.15.  First pools of a quarter of the
    // rays instead of all, 250x200 to 640x480: 0.88 to 0.96 -> 1.01 to 1.24 (an eighth: the same).
    static constexpr int SLOTS = 256, MIN_LG = 2, MAX_LG = 4, MAX_S = 32;
    static constexpr int WAVES_PER_SIMD = 2, MAX_WAVES = 4 * WAVES_PER_SIMD;
    static constexpr int LARGE_POOLS_BELOW = 0x7fffffff, SHARE_LATER = 4;
    static constexpr bool LARGE_POOLS_LATE = false, CHUNKS = false;
    static constexpr int64_t LONG_ROUNDS_BELOW = 0;
    static constexpr int NEED_QUARTERS = 4;
    // Issue priorities (eval_chunk itself sets 0 and 1 for encoding and matrix products): what is not matrix products first, so that they are always in
    // flight.  42 frames of 280x280 to 1842x1378, geometric mean against no priorities outside the evaluation: so 0.997, the 16-bit networks' order
    // (2 and 3 for the evaluation, 1, 0) 1.004, with the evaluation's 0 and 1 in it 1.001; 885x661 on 2^3 networks 504 / 502 / 511 / 506 us.
    static constexpr int PRIO_EVALUATE = 0, PRIO_BETWEEN = 2, PRIO_MARCH = 2;

    static __device__ __forceinline__ void place_direction(const float (&)[3], u4 *) {}

    struct Weights : NetF32<H, true> {
        __device__ __forceinline__ void load(const void *packed, int32_t net, int lane) { NetF32<H, true>::load((const float *)packed, net, lane); }
    };

    __device__ __forceinline__ explicit Net32(int) {}

    template <typename Slot>
    __device__ __forceinline__ f4 evaluate(const Weights &w, int lane, int len, Slot slot, const f4 *slots, const u4 *, const f4 *rays, int P) const
    {
        return eval_chunk<H, true>(w, lane, (len + 15) / 16, [&](int j, float (&p)[3], float (&d)[3]) {
            const int i = slot(j);
            const f4 x = slots[i], v = rays[2 * (i & (P - 1)) + 1];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                p[c] = x[c];
                d[c] = v[c];
            }
        });
    }
    static __device__ __forceinline__ float sigmoid(float v) { return 1.0f / (1.0f + expf(-v)); }
};

} // namespace

int kn_fused_f32_configure()
{
    return fused_configure<Net32<32>>();
}

int kn_fused_f32_launch(const kn_scene *sc, hipStream_t st, const KnFusedJob &job, hipEvent_t ev_start, hipEvent_t ev_stop)
{
    if (sc->desc.hidden != 32) return KN_E_UNSUPPORTED;
    return fused_launch<Net32<32>>(sc, st, job, ev_start, ev_stop);
}
