// Evaluation of small batches without any ordering (scenes with 16-bit weights; kn_mlp_f32.hip holds the fp32 kernel).
//
// kn_eval_grouped orders the whole batch by network first, which is nine launches and four trips through memory.  A
// small batch cannot fill the chip with those, and each costs its latency.  Here a wavefront takes P consecutive points
// (P a power of two up to 64), finds their networks and evaluates them network by network: one launch.  What it gives
// up is that the points of one network meet in full tiles and share one fetch of the weights, so it is for batches whose
// weights, fetched once per wavefront and network, are still little traffic (see kn_direct_lg_points).
//
// What bounds it: the latency of a pass over one network (weights 11.4 / 29 KB per wavefront from the caches, then five
// dependent layers), P times in a row at worst; so P is as small as leaves every resident wavefront one share.
// Measured, 1,000 points on 16^3 networks, width 32, fp16: 45 us -> 15 (the host's share of a call); fp32: 56 -> 15.
#include "kn_direct.h"
#include "kn_mlp_core.h"

namespace {

constexpr int DIRECT_WAVES = 4;

// Same operands and order of operations per sample as k_mlp_mfma: the results are the same bits.
template <int H, bool BF, bool WRAP>
__global__ void __launch_bounds__(DIRECT_WAVES *KN_WAVE) __attribute__((amdgpu_waves_per_eu(H == 32 ? 4 : 2, H == 32 ? 4 : 2)))
    k_eval_direct(const uint16_t *__restrict__ packed, KnDirectJob job)
{
    using L = Lay<H>;
    constexpr int HT = L::HT, HK = L::HK, NBLK = L::NBLK;
    __shared__ f4 stage[DIRECT_WAVES][KN_WAVE][2]; // x, y, z, dx | dy, dz, lane of the sample, - : the samples of one network
    const int wave = threadIdx.x / KN_WAVE, lane = threadIdx.x & (KN_WAVE - 1), n = lane & 15, g = lane >> 4;
    const unsigned m3 = g == 3 ? 0xffffffffu : 0u;
    const f4 zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
    const int64_t first = (int64_t)(blockIdx.x * DIRECT_WAVES + wave) << job.lg_points;
    KnDirectPoint pt;
    unsigned long long pending = kn_direct_point(job, first, lane, pt);
    while (pending != 0ull) {
        const int32_t sel = __builtin_amdgcn_readlane(pt.net, (int)__builtin_ctzll(pending));
        u4 areg[NBLK], heads[HK];
        f4 bias2[HT], bias_out;
        const u4 *__restrict__ wp = (const u4 *)(packed + (int64_t)sel * L::HALFS);
        const float *__restrict__ tail = (const float *)(wp + L::TAIL);
#pragma unroll
        for (int b = 0; b < L::L2; ++b) areg[b] = wp[b * KN_WAVE + lane]; // (in the order of their use)
#pragma unroll
        for (int t = 0; t < HT; ++t) bias2[t] = *(const f4 *)(tail + 16 * t + 4 * g);
        bias_out = *(const f4 *)(tail + H);
#pragma unroll
        for (int kb = 0; kb < HK; ++kb) heads[kb] = wp[L::heads_at(kb, lane)];
#pragma unroll
        for (int b = L::L2; b < NBLK; ++b) areg[b] = wp[b * KN_WAVE + lane];
        const bool hit = pt.net == sel;
        const unsigned long long hits = __ballot(hit);
        if (hit) {
            const int rank = __popcll(hits & ((1ull << lane) - 1ull));
            stage[wave][rank][0] = (f4){pt.p[0], pt.p[1], pt.p[2], pt.d[0]};
            stage[wave][rank][1] = (f4){pt.d[1], pt.d[2], __int_as_float(lane), 0.0f};
        }
        pending &= ~hits;
        const int c = __popcll(hits);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // (density row and colour rows are repeated with period four: every lane group computes the four values of a sample, and
        // group u keeps those of sample tile u)
        f4 out = zero4;
        for (int u = 0; 16 * u < c; ++u) {
            const int i = min(16 * u + n, c - 1);
            const f4 q0 = stage[wave][i][0], q1 = stage[wave][i][1];
            const float pg = g == 0 ? q0[0] : (g == 1 ? q0[1] : q0[2]), dg = g == 0 ? q0[3] : (g == 1 ? q1[0] : q1[1]);
            const bool g3 = g == 3;
            const f4 ang = {g3 ? q0[0] * (256.0f * INV_2PI) : pg * INV_2PI, g3 ? q0[1] * (256.0f * INV_2PI) : pg * (4.0f * INV_2PI),
                            g3 ? q0[2] * (256.0f * INV_2PI) : pg * (16.0f * INV_2PI), g3 ? 0.0f : dg * INV_2PI};
            const u4 ident = {pk<BF>(q0[0], q0[1]), pk<BF>(q0[2], 1.0f), pk<BF>(q0[3], q1[0]), pk<BF>(q1[1], 1.0f)};
            u4 Bx[2];
            encode_position<BF, WRAP>(ang, ident, m3, Bx);
            const u4 Bd = encode_direction<BF>(ang[3], ident, m3);
            f4 o_sig = bias_out, o_col = bias_out, acc[HT];
            u4 Bh[HK];
#pragma unroll
            for (int t = 0; t < HT; ++t) {
                acc[t] = mfma<BF>(areg[L::L1 + 2 * t], Bx[0], zero4);
                acc[t] = mfma<BF>(areg[L::L1 + 2 * t + 1], Bx[1], acc[t]);
            }
            pack_acts<H, BF, true>(acc, Bh);
#pragma unroll
            for (int t = 0; t < HT; ++t) {
                acc[t] = bias2[t];
#pragma unroll
                for (int kb = 0; kb < HK; ++kb) acc[t] = mfma<BF>(areg[L::L2 + t * HK + kb], Bh[kb], acc[t]);
            }
            pack_acts<H, BF, true>(acc, Bh);
#pragma unroll
            for (int kb = 0; kb < HK; ++kb) o_sig = mfma<BF>(heads[kb], Bh[kb], o_sig);
#pragma unroll
            for (int t = 0; t < HT; ++t) {
                acc[t] = mfma<BF>(areg[L::L4 + t * (HK + 1) + HK], Bd, zero4);
#pragma unroll
                for (int kb = 0; kb < HK; ++kb) acc[t] = mfma<BF>(areg[L::L4 + t * (HK + 1) + kb], Bh[kb], acc[t]);
            }
            pack_acts<H, BF, true>(acc, Bh);
#pragma unroll
            for (int kb = 0; kb < HK; ++kb) o_col = mfma<BF>(heads[kb], Bh[kb], o_col);
            out = g == u ? (f4){o_col[0], o_col[1], o_col[2], o_sig[3]} : out;
        }
        if (lane < c) {
            const int64_t to = first + __float_as_int(stage[wave][lane][1][2]);
            job.sigma[to] = fmaxf(out[3], 0.0f);
#pragma unroll
            for (int q = 0; q < 3; ++q)
                job.rgb[3 * to + q] = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * out[q]));
        }
        __builtin_amdgcn_wave_barrier(); // the staging buffer is rewritten by the next pass
    }
}

} // namespace

// A batch goes unordered when its weight traffic takes less time than ordering does.  The traffic is at most one fetch per
// point, or per wavefront and network where there are few networks; what a fetch takes when all wavefronts fetch is in `ns` (40,000 points all over 16^3
// networks: 1.53 in 16 bits, 4.3 at width 64, fp32 3.8 and 11.9), and less than half of it where the weights of all networks fit the 4 MB of an XCD's L2.
// What ordering takes grows with the networks, whose counts every one of its workgroups looks at, and few points of a batch that is all over the grid
// meet.  Near the lines, direct / ordered, points all over the grid (in brackets: nine in ten in a twentieth of the cells), us: 5x8x5
// networks, fp32, 3,000 points 11 / 19, 6,000 (not taken) 20 / 19; 16^3, fp16, 12,000 20 / 22, 16,000 25 / 22 (12 / 19), 24,000 37 / 22 (16 / 19), 28,000
// (not) 43 / 22 (19 / 19); 10x16x10, bf16, width 64, 6,000 24 / 21 (13 / 19), 8,000 (not) 32 / 21 (13 / 19), fp32 6,000 (not) 23 / 19 (20 / 25); 24x20x28, fp16,
// 24,000 40 / 40 (26 / 24), 34,000 (not) 61 / 42 (40 / 27), fp32 8,000 30 / 40 (25 / 26); 32^3, fp16, 28,000 48 / 60 (42 / 38), 40,000 (not) 67 / 70 (56 / 39),
// bf16, width 64, 16,000 68 / 94 (62 / 43), fp32 16,000 54 / 70 (50 / 41).
int kn_direct_lg_points(const kn_scene *sc, int64_t M)
{
    const int H = sc->desc.hidden;
    const bool f32 = sc->desc.wdtype == KN_F32;
    const int64_t resident = 1024 * (f32 ? (H == 32 ? 2 : 1) : (H == 32 ? 4 : 2)); // wavefronts
    int lg = 0;
    while (lg < 6 && (resident << lg) < M) ++lg;
    const double shares = (double)kn_div_up(M, 1ll << lg), networks = (double)(sc->N < (1 << lg) ? sc->N : 1 << lg);
    const double fetches = fmin((double)M, shares * networks);
    const int near = f32 ? (H == 32 ? 109 : 37) : (H == 32 ? 241 : 101); // networks whose images, 2.7 to 3.0 MB, stay in the L2
    const double ns = f32 ? (H == 32 ? 4.74 : 12.4) : (H == 32 ? 1.55 : 4.13), us = 1e-3 * fetches * (sc->N <= near ? ns / 2.25 : ns);
    const bool heavy = f32 || H == 64;
    const double limit = sc->N <= 255 ? 24.0 : sc->N <= 8191 ? (heavy ? 26.0 : 40.0) : sc->N <= 16383 ? 45.0 : (heavy ? 80.0 : 50.0);
    return us <= limit ? lg : -1;
}

int kn_direct_launch(const kn_scene *sc, hipStream_t st, const KnDirectJob &job, hipEvent_t ev_start, hipEvent_t ev_stop)
{
    const int64_t blocks = kn_div_up(kn_div_up(job.M, 1ll << job.lg_points), DIRECT_WAVES);
    if (blocks > 0x7fffffffLL) return KN_E_UNSUPPORTED;
    if (sc->desc.wdtype == KN_F32) return kn_direct_f32_launch(sc, st, job, (unsigned)blocks, ev_start, ev_stop);
    const bool bf = sc->desc.wdtype == KN_BF16;
    float reach = 0.0f; // (see the launch of k_mlp_mfma)
    for (int a = 0; a < 3; ++a) reach = fmaxf(reach, fmaxf(fabsf(sc->desc.aabb_min[a]), fabsf(sc->desc.aabb_max[a])));
    const bool wrap = !(reach * (256.0f * INV_2PI) < 250.0f);
    if (sc->desc.hidden != 32 && sc->desc.hidden != 64) return KN_E_UNSUPPORTED;
    auto kernel = sc->desc.hidden == 32
                      ? (bf ? (wrap ? k_eval_direct<32, true, true> : k_eval_direct<32, true, false>)
                            : (wrap ? k_eval_direct<32, false, true> : k_eval_direct<32, false, false>))
                      : (bf ? (wrap ? k_eval_direct<64, true, true> : k_eval_direct<64, true, false>)
                            : (wrap ? k_eval_direct<64, false, true> : k_eval_direct<64, false, false>));
    const dim3 grid((unsigned)blocks), block(DIRECT_WAVES * KN_WAVE);
    if (ev_start && ev_stop) hipExtLaunchKernelGGL(kernel, grid, block, 0, st, ev_start, ev_stop, 0, (const uint16_t *)sc->packed_w, job);
    else hipLaunchKernelGGL(kernel, grid, block, 0, st, (const uint16_t *)sc->packed_w, job);
    KN_CHECK_LAUNCH();
    return KN_OK;
}
