// The fused render (kn_fused_core.h) of scenes with 16-bit weights.
#include "kn_fused_core.h"
#include "kn_mlp_core.h"

namespace {

template <int H, bool BF, bool WRAP> struct Net16 {
    using L = Lay<H>;
    static constexpr int HT = L::HT, HK = L::HK, NBLK = L::NBLK;
    static constexpr bool FLUSHED = true;
    static constexpr int DIR = 4;

    // (Shapes, pools and rounds were chosen, and the figures of this block measured, when the march's look-ups went out one by one.)
    // Rays and slots per wavefront.  Large pools keep few lanes per ray and cut a ray into many rounds, small ones evaluate more samples
    // behind the termination point; many slots mean many samples per visit of a network, few fit a step of the march (256 points).
    // Rays x slots, 800x800 and 767x577 / 1080p at width 64, us: 32 x 384 183, 167 / 64 x 768 1,211; 16 x 384 173, 163 / 32 x 768 1,100;
    // 16 x 256 169, 156 / 32 x 896 1,100; 32 x 256 182, 164 / 32 x 512 1,225; 16 x 768 at width 64 1,191.
    static constexpr int SLOTS = H == 32 ? 256 : 768, MIN_LG = 2, MAX_LG = H == 32 ? 5 : 6, MAX_S = 32;
    static constexpr int WAVES_PER_SIMD = H == 32 ? 4 : 2, MAX_WAVES = 4 * WAVES_PER_SIMD;
    // Full pools of many rays with few samples each where rays end after few samples, of half as many rays otherwise.  How many a ray
    // takes depends on the scene; coarse lattices need fewer than fine ones.  Half / all, one frame each: 1424x1070, width 32, K = 32 (2^3
    // networks) 294 / 268 us, K = 128 (16^3) 176 / 168, 800x800, K = 512, 169 / 182; width 64, 1424x1070, K = 64 (2^3) 580 / 390, K = 256 (8^3)
    // 340 / 310, K = 512 (16^3) 460 / 457, 1080p, K = 1024, 1,051 / 1,110.  At width 32 they have to be filled more than once.
    static constexpr int LARGE_POOLS_BELOW = H == 32 ? 256 : 512;
    static constexpr bool LARGE_POOLS_LATE = H == 32;
    static constexpr int SHARE_LATER = 1;
    static constexpr int64_t LONG_ROUNDS_BELOW = H == 32 ? 400000 : KN_FUSED_OWN_RAYS + 1; // rays (fused_launch)
    static constexpr bool CHUNKS = H == 32; // how rays beyond the first pools are handed out (CHUNK_SHARE)
    // A round's march ends when fewer than half of the pool's rays have this little of their slots filled: at width 32 a second step
    // for the rest of a ray's slots is mostly thrown away; at width 64, where a visit of a network costs more, it pays.
    static constexpr int NEED_QUARTERS = H == 32 ? 2 : 4;
    // Issue priorities of a wavefront's phases.  At equal ones the four wavefronts of a SIMD drift into the same phase, and all wait for
    // their look-ups or all want the vector ALU; like this one that evaluates gets through, and the others' look-ups are under way meanwhile.
    // Equal / 2, 1, 0 for evaluation, blend and hand-out, march, us per frame: 800x800 161.7 / 153.0, 767x577 stratified 154.9 / 147.9, 695x518
    // 164.7 / 154.9, sparse 800x800 189.2 / 186.4, 146x106 42.8 / 40.6; width 64 (two wavefronts) no change.  1, 0, 0 and 3, 0, 0
    // are within 0.3 % of it, a higher priority outside the evaluation (0, 1, 1) changes nothing.
    static constexpr int PRIO_EVALUATE = 2, PRIO_BETWEEN = 1, PRIO_MARCH = 0;

    static __device__ __forceinline__ void place_direction(const float (&d)[3], u4 *to) // gamma(d) in operand order
    {
        kn_enc::u4 q[4];
        kn_enc::dir_slots<BF>(d[0], d[1], d[2], q);
#pragma unroll
        for (int i = 0; i < 4; ++i) to[i] = q[i];
    }

    struct Weights {
        u4 areg[NBLK], heads[HK];
        f4 bias2[HT], bias_out;
        __device__ __forceinline__ void load(const void *packed, int32_t net, int lane)
        {
            const u4 *__restrict__ wp = (const u4 *)((const uint16_t *)packed + (int64_t)net * L::HALFS);
            const float *__restrict__ tail = (const float *)(wp + L::TAIL);
            // in the order of their use, nothing to be done to them in front of the first layer: that runs while the others' are under way (with the heads
            // in blocks of their own, joined here, 800x800 144.9 -> 143.5 us, sparse 145.5 -> 137.1, 1080p, width 64, 990 -> 970)
#pragma unroll
            for (int b = 0; b < L::L2; ++b) areg[b] = wp[b * KN_WAVE + lane];
#pragma unroll
            for (int t = 0; t < HT; ++t) bias2[t] = *(const f4 *)(tail + 16 * t + 4 * (lane >> 4));
            bias_out = *(const f4 *)(tail + H);
#pragma unroll
            for (int kb = 0; kb < HK; ++kb) heads[kb] = wp[L::heads_at(kb, lane)];
#pragma unroll
            for (int b = L::L2; b < NBLK; ++b) areg[b] = wp[b * KN_WAVE + lane];
        }
    };

    // which word of a sample's slot each of a lane's three restart angles comes from, and its scale (see k_mlp_mfma)
    int n, g, wo0, wo1, wo2;
    unsigned m3;
    float f0, f1, f2_;
    __device__ __forceinline__ explicit Net16(int lane) : n(lane & 15), g(lane >> 4)
    {
        m3 = (g == 3) ? 0xffffffffu : 0u;
        wo0 = g < 3 ? g : 0;
        wo1 = g < 3 ? g : 1;
        wo2 = g < 3 ? g : 2;
        f0 = g < 3 ? INV_2PI : 256.0f * INV_2PI;
        f1 = g < 3 ? 4.0f * INV_2PI : 256.0f * INV_2PI;
        f2_ = g < 3 ? 16.0f * INV_2PI : 256.0f * INV_2PI;
    }

    // pre-activations (r, g, b, sigma) of sample `lane` of a tile of len samples; slot(j): the slot of the tile's sample j
    template <typename Slot>
    __device__ __forceinline__ f4 evaluate(const Weights &w, int, int len, Slot slot, const f4 *slots, const u4 *dirs, const f4 *, int P) const
    {
        const f4 zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
        f4 out = zero4;
        auto sample_tile = [&](int u) {
            f4 o_sig = w.bias_out, o_col = w.bias_out;
            const int i = slot(16 * u + n);
            const float *sp = (const float *)(slots + i);
            const float v0 = sp[wo0], v1 = sp[wo1], v2 = sp[wo2];
            const f4 ang = {v0 * f0, v1 * f1, v2 * f2_, 0.0f};
            const u4 ident = {pk<BF>(v0, v1), pk<BF>(v2, 1.0f), 0u, 0u}; // (group 3: v0..v2 are x, y, z)
            u4 Bx[2];
            encode_position<BF, WRAP>(ang, ident, m3, Bx);
            const u4 Bd = dirs[4 * (i & (P - 1)) + g];
            f4 acc[HT];
            u4 Bh[HK];
#pragma unroll
            for (int t = 0; t < HT; ++t) {
                acc[t] = mfma<BF>(w.areg[L::L1 + 2 * t], Bx[0], zero4);
                acc[t] = mfma<BF>(w.areg[L::L1 + 2 * t + 1], Bx[1], acc[t]);
            }
            pack_acts<H, BF, true>(acc, Bh);
#pragma unroll
            for (int t = 0; t < HT; ++t) {
                acc[t] = w.bias2[t];
#pragma unroll
                for (int kb = 0; kb < HK; ++kb) acc[t] = mfma<BF>(w.areg[L::L2 + t * HK + kb], Bh[kb], acc[t]);
            }
            pack_acts<H, BF, true>(acc, Bh);
#pragma unroll
            for (int kb = 0; kb < HK; ++kb) o_sig = mfma<BF>(w.heads[kb], Bh[kb], o_sig);
#pragma unroll
            for (int t = 0; t < HT; ++t) {
                acc[t] = mfma<BF>(w.areg[L::L4 + t * (HK + 1) + HK], Bd, zero4);
#pragma unroll
                for (int kb = 0; kb < HK; ++kb) acc[t] = mfma<BF>(w.areg[L::L4 + t * (HK + 1) + kb], Bh[kb], acc[t]);
            }
            pack_acts<H, BF, true>(acc, Bh);
#pragma unroll
            for (int kb = 0; kb < HK; ++kb) o_col = mfma<BF>(w.heads[kb], Bh[kb], o_col);
            out = g == u ? (f4){o_col[0], o_col[1], o_col[2], o_sig[3]} : out;
        };
        // (two sample tiles side by side wherever two are there; uniform branches)
        if (len > 16) { sample_tile(0); sample_tile(1); }
        else sample_tile(0);
        if (len > 48) { sample_tile(2); sample_tile(3); }
        else if (len > 32) sample_tile(2);
        return out;
    }
    static __device__ __forceinline__ float sigmoid(float v) { return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * v)); }
};

} // namespace

// The kernel's voxel, block and cell numbers are formed with 24-bit multiplications, and it keeps a sample's network in
// 16 bits.  fp32 networks of width 64, and those whose layers are kept apart, are the wave loop's.
bool kn_fused_supports(const kn_scene *sc)
{
    if (sc->N > 65536 || (sc->desc.wdtype == KN_F32 && (sc->f32_apart || sc->desc.hidden != 32))) return false;
    auto fits = [](const int32_t r[3]) {
        constexpr int64_t lim = 1ll << 24;
        return (int64_t)r[0] * r[1] <= lim && r[0] < lim && r[1] < lim && r[2] < lim;
    };
    return fits(sc->net_grid.res) && (!sc->has_occ || fits(sc->skip_res));
}

int kn_fused_configure()
{
    KN_TRY((fused_configure<Net16<32, false, false>>()));
    KN_TRY((fused_configure<Net16<32, false, true>>()));
    KN_TRY((fused_configure<Net16<32, true, false>>()));
    KN_TRY((fused_configure<Net16<32, true, true>>()));
    KN_TRY((fused_configure<Net16<64, false, false>>()));
    KN_TRY((fused_configure<Net16<64, false, true>>()));
    KN_TRY((fused_configure<Net16<64, true, false>>()));
    KN_TRY((fused_configure<Net16<64, true, true>>()));
    return kn_fused_f32_configure();
}

int kn_fused_launch(const kn_scene *sc, hipStream_t st, const KnFusedJob &job, hipEvent_t ev_start, hipEvent_t ev_stop)
{
    if (sc->desc.wdtype == KN_F32) return kn_fused_f32_launch(sc, st, job, ev_start, ev_stop);
    float reach = 0.0f; // (see the launch of k_mlp_mfma)
    for (int c = 0; c < 3; ++c) reach = fmaxf(reach, fmaxf(fabsf(sc->desc.aabb_min[c]), fabsf(sc->desc.aabb_max[c])));
    const bool wrap = !(reach * (256.0f * INV_2PI) < 250.0f);
    using Launch = decltype(&fused_launch<Net16<32, false, false>>);
    static const Launch table[2][2][2] = {
        {{fused_launch<Net16<32, false, false>>, fused_launch<Net16<32, false, true>>}, {fused_launch<Net16<32, true, false>>, fused_launch<Net16<32, true, true>>}},
        {{fused_launch<Net16<64, false, false>>, fused_launch<Net16<64, false, true>>}, {fused_launch<Net16<64, true, false>>, fused_launch<Net16<64, true, true>>}}};
    if (sc->desc.hidden != 32 && sc->desc.hidden != 64) return KN_E_UNSUPPORTED;
    return table[sc->desc.hidden == 64][sc->desc.wdtype == KN_BF16][wrap](sc, st, job, ev_start, ev_stop);
}
