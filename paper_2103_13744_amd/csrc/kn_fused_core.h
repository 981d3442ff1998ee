// The whole path behind one kernel (Sec. 3.4, Eq. 1-4, Eq. 7): marching with empty-space skipping, grouping by network,
// the fused tiny MLP and blending with early ray termination, in one of the number formats that the networks (Net) come in.
//
// A wavefront owns a pool of P rays (P a power of two, G = 64 / P lanes per ray) and works through them alone, without
// workgroup barriers.  One round: every ray of the pool collects up to S kept samples (P * S slots of LDS per
// wavefront); the samples are evaluated network by network; every ray blends its samples in order and ends, or stays
// for the next round; free places are filled with the next rays of the live list.  Samples, results and encoded
// directions never leave the LDS, a frame needs no slot buffers, no histogram and no host decision in the middle, and a
// ray stops within S samples of its termination point.  Against the wave loop (march, group, evaluate and blend kernels
// per wave, the host waiting for a count), two views each: 30,000 rays, width 32 (200x151) 115, 133 -> 41, 46 us; 800x800 215, 225 -> 135, 158; 1080p,
// width 64, 1623, 1583 -> 1040, 920.  Frames of up to 32,767 rays are this kernel alone: a workgroup also clips its rays and walks them to their
// first lattice point near content (200x151: 67 us with two launches in front of it).
//
// What bounds it: vector-ALU issue while there is work (a march step of 256 points takes about 300 instructions, a tile of 16
// samples about 65, a round about 350 besides), and the end of a frame, when the rays that are left are few.  The rays' costs differ
// (most end within two rounds, some take ten) and neighbours cost alike, so behind a list a workgroup is all of a compute unit's wavefronts, whose
// first pools lie in as many parts of the list, and who share their last rays through the LDS: workgroups of four
// wavefronts, all places in a list filled by an atomic per wavefront and round, 203 us at 800x800 (call, with the set-up's 31), 181
// at 767x577 stratified, 1,093 at 1080p, width 64; like this 164, 148 and 1,038 (145, 136 and 920 since the march's look-ups are under way together).
// Tried and slower, before that: contiguous pieces of the list
// larger than what a wavefront has places for (800x800 +3, 1080p +60: the last pieces decide), hand-out counters per XCD (+3, +20),
// half of the list handed out beforehand (+6, +190), 12 wavefronts per compute unit (+3).
//
// The wavefronts of a SIMD are in different phases at different times, so the latency of the march runs under the
// evaluation of the others.  Results are the bits of the wave loop (kn_render.hip): same lattice points, same operand
// order in the networks (a sample's outputs do not depend on which samples share its tile), same recurrence per ray.
#pragma once

#include "kn_common.h"
#include "kn_fused.h"
#include "kn_march.h"
#include <hip/hip_ext.h>

#include <algorithm>

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned u4 __attribute__((ext_vector_type(4)));

enum { BUSY = 0, IDLE, CLAIMED, GIVEN }; // states of a wavefront while the last rays of a workgroup are shared out

// Rays beyond the first pools.  Width 32: they are handed to a workgroup in chunks, its wavefronts take from those what they have places
// for: an eighth of a workgroup's even share of what is left, so that the chunks become small towards the end.  (An atomic per
// wavefront and round, all on one word, kept the wavefronts waiting: 11 ns each, 45 us for the 4,096 that ask after their first round.  At
// least 8 rays and a sixteenth / 16 and an eighth / 32 and an eighth / 32 and a half, us: 899x900 163 / 124.5 / 115.5 / 116, 800x800 175 / 151.6 / 150.8 /
// 152.6, sparse 197 / 186.9 / 186.3 / 192, 1071x1070 sparse - / 327 / 326 / 343.)
// Width 64: half as many wavefronts, whose rounds take three times as long, take them for themselves (1080p 1,051 us, 1,084 in chunks:
// rays that are under way at the same time lie closer together).
constexpr int CHUNK_SHARE = 8, CHUNK_MIN = 32, CHUNK_MAX = 512;
// Rays in a row that a workgroup which sets up its own rays takes together: some eight groups per workgroup (six in those of a whole
// compute unit), so that those rays that meet content are spread evenly, of rays that meet the same networks.  Six or four groups per workgroup
// and longer ones, the mean of twelve views: 200x151 55.1 us, eight 51.7; at width 64 94 and 74; 128 drawn frames of 4,000 to 32,767 rays: the
// same in the mean at width 32, six 0.98 of eight at width 64.  Shorter groups meet more networks: of two rays, 140x105 63 us instead of 52.
constexpr int OWN_GROUPS = 8, OWN_GROUPS_WHOLE = 6;
constexpr int OWN_GROUP_MIN = 4, OWN_GROUP_MAX = 16;
constexpr int OWN_RAYS_MAX = OWN_GROUP_MAX * (int)((KN_FUSED_OWN_RAYS + 256 * OWN_GROUP_MAX - 1) / (256 * OWN_GROUP_MAX));

// a wavefront's part of the LDS
template <class Net> struct WaveLds {
    static constexpr int RAYS = 1 << Net::MAX_LG;
    f4 slot[Net::SLOTS];      // sample j of pool ray s at j * P + s: (x, y, z, density scale), then (r, g, b, alpha)
    u4 dir[RAYS * Net::DIR];  // the direction of pool ray s as the networks take it
    f4 ray[RAYS * 2];         // (origin, jump scale), (direction, jump offset) of pool ray s
    uint16_t idx[Net::SLOTS]; // the samples' networks, then the slots of the network at hand
};

// lattice points a lane tests per step of the march: enough look-ups in flight, and the work per step that does not
// depend on the number of points (ranks, frontier, skip field) is shared by four
constexpr int STEPS = 4;
constexpr int BLEND = 4; // samples that the blend requests together

struct FusedArgs {
    MarchParams p;
    VoxelFast vox, net; // the grid that is marched through, the network grid
    const void *packed;
    const float *rays_o, *rays_d;
    int32_t n_waves, n_blocks; // wavefronts of a workgroup, workgroups
    int32_t max_lg;    // log2 of the rays of a full pool
    int32_t late_lg, late_s; // when there is no ray left to be taken: log2 of the places that a pool keeps, samples per ray and round
    int32_t few_rays;  // a workgroup starts with fewer wavefronts where its wavefronts would get fewer rays than this
    int32_t R, own_rays, own_group; // own_rays > 0: a workgroup sets up that many rays by itself, groups of own_group, and there is no list
    const int4 *list;  // live rays: (ray, first lattice index, end of the clipped range, -)
    int32_t *ctl;      // [0] = live rays, [1] = rays handed out beyond the wavefronts' first pools
    float eps, bg[3];
    float *rgb_out;
    unsigned long long *counters; // nullable: [0] += samples evaluated, [1] += samples blended
};

// The arguments are read from the kernel's own argument segment where they are used: `opaque` hides where the pointer and
// the lane number come from, so that neither arguments nor values derived from the lane number stay in registers across
// the phases of a round (the evaluation has none to spare).
typedef const __attribute__((address_space(4))) FusedArgs *ArgsPtr;
__device__ __forceinline__ ArgsPtr opaque(ArgsPtr p)
{
    asm volatile("" : "+s"(p));
    return p;
}
__device__ __forceinline__ int opaque(int lane)
{
    asm volatile("" : "+v"(lane));
    return lane;
}

// With 16-bit networks the file is compiled for flushed fp32 denormals (the evaluation's encoding needs that, see build.py).  Where
// lattice points are placed and tested, and in the blend, denormals count: a point at -1e-40 lies outside a box that starts at 0.  There
// the mode register says so; the compiler's own divisions would set it back, so none is left to it in those parts, and neither is a
// multiplication by two (the output modifier does nothing there).
template <class Net> __device__ __forceinline__ void keep_denormals(bool keep)
{
    if constexpr (!Net::FLUSHED) return;
    constexpr int FP32_DENORM = 1 | (4 << 6) | (1 << 11); // MODE, bits 4 and 5
    if (keep) __builtin_amdgcn_s_setreg(FP32_DENORM, 3);
    else __builtin_amdgcn_s_setreg(FP32_DENORM, 0);
}
// a / b rounded to nearest, with denormals kept: the instruction set's scaled division
__device__ __forceinline__ float divide(float a, float b)
{
    bool scaled, unused;
    const float d = __builtin_amdgcn_div_scalef(a, b, false, &unused), n = __builtin_amdgcn_div_scalef(a, b, true, &scaled);
    float r = __builtin_amdgcn_rcpf(d);
    r = fmaf(fmaf(-d, r, 1.0f), r, r);
    float q = n * r;
    q = fmaf(fmaf(-d, q, n), r, q);
    return __builtin_amdgcn_div_fixupf(__builtin_amdgcn_div_fmasf(fmaf(-d, q, n), r, q, scaled), b, a);
}

// Eq. 6 itself
__device__ __forceinline__ void voxel_coords_exact(const VoxelFast &g, float x, float y, float z, int32_t &ix, int32_t &iy, int32_t &iz)
{
    ix = floor_int(divide(x - g.bmin[0], g.cell[0]));
    iy = floor_int(divide(y - g.bmin[1], g.cell[1]));
    iz = floor_int(divide(z - g.bmin[2], g.cell[2]));
    __builtin_amdgcn_sched_barrier(0); // (the divisions of several points side by side would cost more registers than there are)
}
struct ExactDivide {
    __device__ __forceinline__ float operator()(float a, float b) const { return divide(a, b); }
};
__device__ __forceinline__ bool is_finite(float v) { return (__float_as_uint(v) & 0x7f800000u) != 0x7f800000u; } // (the file is compiled without NaNs)

// the first n lanes, 1 <= n <= 64
__device__ __forceinline__ unsigned long long lanes_below(int n) { return ~0ull >> (KN_WAVE - n); }

// LDS writes of the wavefront's lanes before, reads after
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <class Net, bool STRAT>
__global__ void __launch_bounds__(Net::MAX_WAVES *KN_WAVE)
    __attribute__((amdgpu_waves_per_eu(Net::WAVES_PER_SIMD, Net::WAVES_PER_SIMD))) k_render_fused(FusedArgs args_by_value)
{
    constexpr int NQ = Net::SLOTS / KN_WAVE;
    extern __shared__ f4 s_dynamic[];
    WaveLds<Net> *const s_wave = (WaveLds<Net> *)s_dynamic; // one per wavefront of the workgroup
    // sharing of the last rays inside the workgroup: what each wavefront is doing, the number of rays it
    // was given, and how many wavefronts are out of work
    __shared__ int32_t s_state[Net::MAX_WAVES], s_given[Net::MAX_WAVES], s_idle;
    __shared__ int32_t s_lock, s_at, s_end; // what is left of the workgroup's chunk of the list
    __shared__ int32_t s_own;               // live rays of a workgroup that sets up its own

    const ArgsPtr args = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr(); // = &args_by_value
    const int wave = __builtin_amdgcn_readfirstlane(kn_thread() / KN_WAVE), lane = kn_thread() & (KN_WAVE - 1);
    const int n_waves = args->n_waves, n_blocks = args->n_blocks;
    f4 *slots = s_wave[wave].slot;
    u4 *dirs = s_wave[wave].dir;
    f4 *rays = s_wave[wave].ray;
    uint16_t *idx = s_wave[wave].idx;

    // this workgroup's place among all: those of one XCD (b mod 8) side by side
    const int place_of_block = (kn_block() & 7) * (n_blocks >> 3) + (kn_block() >> 3);
    int4 *const own_list = (int4 *)(s_wave + n_waves);
    const int own_rays = args->own_rays;
    if (own_rays > 0) {
        // ---- Small frames: the set-up is part of the kernel.  A workgroup takes groups of rays that lie as far apart as there are
        // workgroups, eight lanes walk a ray, each through an eighth of its range.
        if (kn_thread() == 0) s_own = 0;
        __syncthreads();
        keep_denormals<Net>(true);
        const ArgsPtr a = opaque(args);
        const MarchParams &p = *(const MarchParams *)&a->p;
        const VoxelFast vf = *(const VoxelFast *)&a->vox;
        constexpr int LANES = 8, RAYS = KN_WAVE / LANES;
        const int sub = lane & (LANES - 1);
        for (int j0 = wave * RAYS; j0 < own_rays; j0 += n_waves * RAYS) {
            const int j = j0 + lane / LANES;
            const int group = a->own_group; // (a power of two)
            const int r = (place_of_block + n_blocks * (j / group)) * group + (j & (group - 1));
            int32_t k_lo = 0, k_hi = 0, first = 0x7fffffff;
            if (r < a->R) {
                const float o[3] = {a->rays_o[3 * (int64_t)r], a->rays_o[3 * (int64_t)r + 1], a->rays_o[3 * (int64_t)r + 2]};
                const float d[3] = {a->rays_d[3 * (int64_t)r], a->rays_d[3 * (int64_t)r + 1], a->rays_d[3 * (int64_t)r + 2]};
                clip_ray(*(const KnGrid *)&a->p.content, o, d, a->p.t_near, a->p.step, a->p.K, k_lo, k_hi, ExactDivide{});
                // (a ray with a component that is no finite number has no lattice point inside the box)
                if (!(is_finite(o[0]) & is_finite(o[1]) & is_finite(o[2]) & is_finite(d[0]) & is_finite(d[1]) & is_finite(d[2]))) k_hi = k_lo;
                const int32_t part = (int32_t)(((uint32_t)(k_hi - k_lo) + (LANES - 1)) / LANES);
                const int32_t from = k_lo + sub * part, to = min(from + part, k_hi);
                const int32_t at = walk_to_content<STRAT>(p, vf, o, d, from, to, kn_mix32(a->p.seed_key + (uint32_t)r),
                                                          [&](float x, float y, float z, int32_t &ix, int32_t &iy, int32_t &iz) { voxel_coords_exact(vf, x, y, z, ix, iy, iz); });
                if (at < to) first = at;
            }
#pragma unroll
            for (int w = 1; w < LANES; w <<= 1) first = min(first, __shfl_xor(first, w, KN_WAVE));
            const bool lives = first < k_hi;
            const unsigned long long m = __ballot(lives && sub == 0);
            int base = 0;
            if (lane == 0) base = atomicAdd(&s_own, __popcll(m));
            base = __builtin_amdgcn_readfirstlane(base);
            if (sub == 0 && r < a->R) {
                if (lives) {
                    own_list[base + __popcll(m & ((1ull << lane) - 1ull))] = make_int4(r, first, k_hi, 0);
                } else {
#pragma unroll
                    for (int c = 0; c < 3; ++c) a->rgb_out[3 * (int64_t)r + c] = a->bg[c];
                }
            }
        }
        keep_denormals<Net>(false);
        __syncthreads();
    }
    const int n_live = own_rays > 0 ? s_own : args->ctl[0];
    const int peers = own_rays > 0 ? 1 : n_blocks; // workgroups that share the list
    const int few_rays = args->few_rays;
    // as many wavefronts as get few_rays rays each; the others take what is shared out
    const int users = min(n_waves, max(1, (n_live + peers * few_rays - 1) / (peers * few_rays)));
    const int total_waves = peers * users;
    // rays per pool: as many as take the list (a part of it, 1 / SHARE_LATER, where the rest is better handed out later), up to the pool's size
    int lgP = Net::MIN_LG;
    // (LARGE_POOLS_LATE: the largest only where they are filled a second time)
    const int max_lg = Net::LARGE_POOLS_LATE && n_live < 3 * (total_waves << (Net::MAX_LG - 1)) ? Net::MAX_LG - 1 : args->max_lg;
    while (lgP < max_lg && (own_rays > 0 ? 1 : Net::SHARE_LATER) * ((int64_t)total_waves << lgP) < n_live) ++lgP;

    // First pools: equal contiguous shares of the list's head.  A workgroup takes four that lie side by side (rays that meet the
    // same networks) from each of up to four parts of the list (rays that cost differently); inside a part, shares that lie side by
    // side go to the workgroups of one XCD (b mod 8), which find each other's networks in its L2.  A workgroup's shares
    // scattered one by one: the same for large frames, 164x94 rays with a network per sample 79 -> 96 us instead of 72.
    const int part = wave >> 2, width = min(4, users - 4 * part);
    const int wid = own_rays > 0 ? wave : 4 * part * n_blocks + place_of_block * width + (wave & 3);
    const int n_first = own_rays > 0 ? n_live : (int)min((int64_t)n_live, (int64_t)total_waves << lgP); // (its own rays are all there are)
    int at = __builtin_amdgcn_readfirstlane(wave < users ? (int)((int64_t)wid * n_first / total_waves) : 0);
    int end = __builtin_amdgcn_readfirstlane(wave < users ? (int)((int64_t)(wid + 1) * n_first / total_waves) : 0);
    bool more = n_live > n_first;
    if (kn_thread() < n_waves) s_state[kn_thread()] = BUSY;
    if (kn_thread() == 0) s_idle = s_lock = s_at = s_end = 0;
    __syncthreads();

    int ray = -1, k = 0, k_hi = 0; // (the same in all lanes of a ray's group, like everything per ray below)
    float T = 1.0f, c0 = 0.0f, c1 = 0.0f, c2 = 0.0f;
    long long evaluated = 0, blended = 0; // (uniform)

    for (;;) {
        bool moved = false;
        if (at >= end && !more) {
            // ---- The list is exhausted.  The rays that are left differ in cost (most end within two rounds, some take ten),
            // and a wavefront with many long ones would run on alone: one that has run out of rays waits for a part of
            // another wavefront's of its workgroup.  (LDS only; a waiting wavefront ends when all are out of work.)
            unsigned long long live = __ballot(ray >= 0) & lanes_below(1 << lgP);
            int n = __popcll(live);
            const int ln = opaque(lane);
            if (n == 0) {
                if (ln == 0) {
                    __hip_atomic_store(&s_state[wave], IDLE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    __hip_atomic_fetch_add(&s_idle, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
                int st;
                for (;;) {
                    st = __hip_atomic_load(&s_state[wave], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
                    if (__builtin_amdgcn_readfirstlane(st) == GIVEN) break;
                    if (__builtin_amdgcn_readfirstlane(__hip_atomic_load(&s_idle, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP)) == n_waves) break;
                    __builtin_amdgcn_s_sleep(4);
                }
                if (__builtin_amdgcn_readfirstlane(st) != GIVEN) break; // everybody is out of work
                n = __builtin_amdgcn_readfirstlane(s_given[wave]);
                if (ln == 0) __hip_atomic_store(&s_state[wave], BUSY, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                lgP = Net::MAX_LG;
                const int place = ln & ((1 << lgP) - 1);
                if (place < n) {
                    const f4 q0 = slots[2 * place], q1 = slots[2 * place + 1];
                    ray = __float_as_int(q0[0]);
                    k = __float_as_int(q0[1]);
                    k_hi = __float_as_int(q0[2]);
                    T = q0[3];
                    c0 = q1[0];
                    c1 = q1[1];
                    c2 = q1[2];
                }
                live = (1ull << n) - 1ull; // (at most half a pool was given)
                wave_sync();
            } else if (n >= 2 && __builtin_amdgcn_readfirstlane(__hip_atomic_load(&s_idle, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) > 0) {
                int to = -1;
                if (ln == 0)
                    for (int w = 1; w < n_waves && to < 0; ++w) {
                        int expect = IDLE;
                        const int other = wave + w < n_waves ? wave + w : wave + w - n_waves;
                        if (__hip_atomic_compare_exchange_strong(&s_state[other], &expect, CLAIMED, __ATOMIC_ACQUIRE, __ATOMIC_RELAXED,
                                                                 __HIP_MEMORY_SCOPE_WORKGROUP)) {
                            to = other;
                            __hip_atomic_fetch_sub(&s_idle, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        }
                    }
                to = __builtin_amdgcn_readfirstlane(to);
                if (to >= 0) { // the upper half of the live rays moves to wavefront `to`'s part of the LDS
                    const int P = 1 << lgP, place = ln & (P - 1), keep = n - n / 2;
                    const int rank = __popcll(live & ((1ull << place) - 1ull)) - keep;
                    const bool gives = ray >= 0 && rank >= 0;
                    if (gives && ln < P) {
                        s_wave[to].slot[2 * rank] = (f4){__int_as_float(ray), __int_as_float(k), __int_as_float(k_hi), T};
                        s_wave[to].slot[2 * rank + 1] = (f4){c0, c1, c2, 0.0f};
                    }
                    if (gives) ray = -1;
                    if (ln == 0) {
                        s_given[to] = n / 2;
                        // (the LDS is written in order: the rays are there before the state says so)
                        __hip_atomic_store(&s_state[to], GIVEN, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                    n = keep;
                    live = __ballot(ray >= 0) & lanes_below(P);
                }
            }
            // ---- the rays that are left move together, so that each gets more lanes and more slots
            int lg = lgP;
            const int late_lg = Net::LONG_ROUNDS_BELOW > 0 ? args->late_lg : Net::MIN_LG;
            while (lg > late_lg && n <= (1 << (lg - 1))) --lg;
            if (lg < lgP) {
                if ((live >> ln) & 1ull) idx[__popcll(live & ((1ull << ln) - 1ull))] = (uint16_t)ln; // (a leading lane is its place's number)
                wave_sync();
                const int place = ln & ((1 << lg) - 1);
                const int from = place < n ? (int)idx[place] : 0;
                ray = __shfl(ray, from, KN_WAVE);
                k = __shfl(k, from, KN_WAVE);
                k_hi = __shfl(k_hi, from, KN_WAVE);
                T = __shfl(T, from, KN_WAVE);
                c0 = __shfl(c0, from, KN_WAVE);
                c1 = __shfl(c1, from, KN_WAVE);
                c2 = __shfl(c2, from, KN_WAVE);
                if (place >= n) ray = -1;
                moved = true;
                lgP = lg;
                wave_sync();
            }
        }
        const int P = 1 << lgP, G = KN_WAVE >> lgP;
        const int S_max = min(Net::SLOTS >> lgP, Net::LONG_ROUNDS_BELOW > 0 && at >= end && !more ? args->late_s : Net::MAX_S);
        const unsigned long long firsts = lanes_below(P); // lanes that lead a ray's group
        int cnt = 0;
        {
            const ArgsPtr a = opaque(args);
            const int ln = opaque(lane), slot = ln & (P - 1), gl = ln >> lgP;
            // ---- fill the free places of the pool
            const unsigned long long free_places = __ballot(ray < 0) & firsts;
            const int n_free = __popcll(free_places);
            bool fresh = moved;
            if (n_free > 0) {
                if (at >= end && more) {
                    int got = 0, last = 0;
                    if (ln == 0) {
                        if constexpr (Net::CHUNKS) { // (the lock's holder is a resident wavefront and waits for nothing but memory)
                            int expect = 0;
                            while (!__hip_atomic_compare_exchange_strong(&s_lock, &expect, 1, __ATOMIC_ACQUIRE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) {
                                expect = 0;
                                __builtin_amdgcn_s_sleep(1);
                            }
                            got = __hip_atomic_load(&s_at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                            last = __hip_atomic_load(&s_end, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                            const int chunk = min(max((n_live - max(last, n_first)) / (n_blocks * CHUNK_SHARE), CHUNK_MIN), CHUNK_MAX);
                            if (got >= last && last < n_live) {
                                got = min(n_first + atomicAdd(&a->ctl[1], chunk), n_live);
                                last = min(got + chunk, n_live);
                                __hip_atomic_store(&s_end, last, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                            }
                            __hip_atomic_store(&s_at, min(got + n_free, last), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                            __hip_atomic_store(&s_lock, 0, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
                        } else {
                            got = min(n_first + atomicAdd(&a->ctl[1], n_free), n_live);
                            last = min(got + n_free, n_live);
                        }
                    }
                    at = __builtin_amdgcn_readfirstlane(got);
                    last = __builtin_amdgcn_readfirstlane(last);
                    end = min(at + n_free, last);
                    more = end < n_live;
                }
                const int avail = end - at;
                if (avail > 0) {
                    const int rank = __popcll(free_places & ((1ull << slot) - 1ull));
                    if (ray < 0 && rank < avail) {
                        const int4 e = a->own_rays > 0 ? own_list[at + rank] : a->list[at + rank];
                        ray = e.x;
                        k = e.y;
                        k_hi = e.z;
                        T = 1.0f;
                        c0 = c1 = c2 = 0.0f;
                        fresh = true;
                    }
                    at += min(n_free, avail);
                }
            }
            if (__ballot(ray >= 0) == 0ull) continue; // (only where the hand-out counter gave nothing any more)
            if (ray >= 0 && fresh && gl == 0) { // a ray takes its place: what the rounds need of it goes to the LDS
                float o[3], d[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    o[c] = a->rays_o[3 * (int64_t)ray + c];
                    d[c] = a->rays_d[3 * (int64_t)ray + c];
                }
                const SkipJump sj(*(const MarchParams *)&a->p, o, d, STRAT);
                rays[2 * slot] = (f4){o[0], o[1], o[2], sj.use ? sj.a : 0.0f};
                rays[2 * slot + 1] = (f4){d[0], d[1], d[2], sj.use ? sj.b : 1e30f}; // (no jumps)
                Net::place_direction(d, dirs + Net::DIR * slot);
            }
            wave_sync();

            keep_denormals<Net>(true);
            __builtin_amdgcn_s_setprio(Net::PRIO_MARCH);
            // ---- march: up to S kept samples per ray.  A step tests G * STEPS consecutive lattice points, STEPS per lane,
            // with all look-ups of the step in flight together; the skip field is asked at each lane's last point only.
            // What the loop reads of the arguments is copied out in front of it (scalar registers): a scalar load inside costs
            // its latency per step, and there were twenty of them (7,200 cycles per step, 1,300 without).
            if (ray >= 0) {
                const VoxelFast vf = *(const VoxelFast *)&a->vox;
                const float t_near = a->p.t_near, step = a->p.step;
                const uint4 *__restrict__ const bricks = a->p.bricks;
                const int32_t *__restrict__ const cell_net = a->p.cell_net;
                const uint32_t last_block = (uint32_t)(a->p.skip_res[0] * a->p.skip_res[1] * a->p.skip_res[2] - 1); // (points outside look up any block)
                const int32_t skip1 = a->p.skip_res[1], skip2 = a->p.skip_res[2];
                const int32_t has_occ = a->p.has_occ, brick_nets = a->p.brick_nets;
                const int n_lanes = __popcll(__ballot(true));
                const f4 ro = rays[2 * slot], rd = rays[2 * slot + 1];
                const int S = S_max;
                const uint32_t ray_key = kn_mix32(a->p.seed_key + (uint32_t)ray);
                // The march of a round ends when fewer than half of the pool's rays still collect: the others would only wait.
                while (2 * __popcll(__ballot(k < k_hi && 4 * cnt < Net::NEED_QUARTERS * S)) >= n_lanes) {
                  if (k < k_hi && cnt < S) {
                    const int k0 = k + gl * STEPS;
                    float x[STEPS], y[STEPS], z[STEPS];
                    int32_t ix[STEPS], iy[STEPS], iz[STEPS], net[STEPS];
                    bool in[STEPS], close = false;
#pragma unroll
                    for (int c = 0; c < STEPS; ++c) {
                        kn_lattice_point<STRAT>(ro[0], ro[1], ro[2], rd[0], rd[1], rd[2], t_near, step, k0 + c, x[c], y[c], z[c], ray_key);
                        close |= voxel_coords(vf, x[c], y[c], z[c], ix[c], iy[c], iz[c]);
                    }
                    if (close) { // some point within rounding of a voxel's face: the divisions themselves
#pragma unroll
                        for (int c = 0; c < STEPS; ++c) voxel_coords_exact(vf, x[c], y[c], z[c], ix[c], iy[c], iz[c]);
                    }
#pragma unroll
                    for (int c = 0; c < STEPS; ++c) // (saturated integers: whatever the coordinates are, the look-ups stay inside)
                        in[c] = inside(vf, ix[c], iy[c], iz[c]) & (k0 + c < k_hi);
                    int32_t dist = 0;
                    if (has_occ) { // (uniform)
                        // occupancy bits, network and skip-field value of each point's block: one load per point, all in flight together
                        uint4 brick[STEPS];
#pragma unroll
                        for (int c = 0; c < STEPS; ++c)
                            brick[c] = bricks[min((uint32_t)kn_mad24(kn_mad24(ix[c] >> 2, skip1, iy[c] >> 2), skip2, iz[c] >> 2), last_block)];
                        dist = in[STEPS - 1] ? (int32_t)brick[STEPS - 1].w : 0;
#pragma unroll
                        for (int c = 0; c < STEPS; ++c) {
                            const uint64_t bits = (uint64_t)brick[c].y << 32 | brick[c].x;
                            in[c] = in[c] & (((bits >> (((ix[c] & 3) << 4) | ((iy[c] & 3) << 2) | (iz[c] & 3))) & 1ull) != 0ull);
                            net[c] = (int32_t)brick[c].z;
                        }
                    }
                    if (!brick_nets) { // (uniform) a block may lie in several cells, or there is no occupancy grid
                        const VoxelFast vn = *(const VoxelFast *)&a->net;
                        bool close_net = false;
#pragma unroll
                        for (int c = 0; c < STEPS; ++c) {
                            int32_t nx, ny, nz;
                            close_net |= voxel_coords(vn, x[c], y[c], z[c], nx, ny, nz);
                            in[c] = in[c] & inside(vn, nx, ny, nz);
                            net[c] = kn_mad24(kn_mad24(nx, vn.res[1], ny), vn.res[2], nz);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        if (close_net) {
#pragma unroll
                            for (int c = 0; c < STEPS; ++c) {
                                int32_t nx, ny, nz;
                                voxel_coords_exact(vn, x[c], y[c], z[c], nx, ny, nz);
                                in[c] = in[c] & inside(vn, nx, ny, nz);
                                net[c] = kn_mad24(kn_mad24(nx, vn.res[1], ny), vn.res[2], nz);
                            }
                        }
                        if (cell_net) { // (uniform) a sparse grid: the cell's network, or none
                            const uint32_t last_cell = (uint32_t)(vn.res[0] * vn.res[1] * vn.res[2] - 1);
#pragma unroll
                            for (int c = 0; c < STEPS; ++c) net[c] = cell_net[min((uint32_t)net[c], last_cell)];
#pragma unroll
                            for (int c = 0; c < STEPS; ++c) in[c] = in[c] & (net[c] >= 0);
                        }
                    }
                    // ranks in order along the ray: kept points of the lanes in front of this one in the group, then this lane's
                    int own = 0;
#pragma unroll
                    for (int c = 0; c < STEPS; ++c) own += in[c] ? 1 : 0;
                    int incl = own;
                    for (int w = P; w < KN_WAVE; w <<= 1) {
                        const int v = __shfl_up(incl, w, KN_WAVE);
                        if (ln >= w + slot) incl += v; // (lane ln - w belongs to the group as well)
                    }
                    const int total = __shfl(incl, slot + KN_WAVE - P, KN_WAVE);
                    int rank = cnt + incl - own;
                    int stop = 0x7fffffff; // first kept point that does not fit: where the next round resumes
#pragma unroll
                    for (int c = 0; c < STEPS; ++c) {
                        if (in[c] & (rank < S)) {
                            const int at_slot = (rank << lgP) + slot;
                            float dscale = 1.0f;
                            if constexpr (STRAT)
                                dscale = divide(kn_lattice_t<true>(t_near, step, k0 + c + 1, ray_key) - kn_lattice_t<true>(t_near, step, k0 + c, ray_key), step);
                            slots[at_slot] = (f4){x[c], y[c], z[c], dscale};
                            idx[at_slot] = (uint16_t)net[c];
                        }
                        stop = (in[c] & (rank == S)) ? k0 + c : stop;
                        rank += in[c] ? 1 : 0;
                    }
                    // the frontier: every index of this step was tested; the farthest jump extends the known-empty range
                    const bool over = cnt + total > S; // (uniform in the group)
                    int32_t v = over ? -stop : (dist >= 2 ? k0 + STEPS + (int32_t)fmaxf(floorf((float)(dist - 1) * ro[3] - rd[3]), 0.0f) : 0); // (SkipJump::jump)
                    for (int w = P; w < KN_WAVE; w <<= 1) v = max(v, __shfl_xor(v, w, KN_WAVE));
                    k = over ? -v : max(k + G * STEPS, v);
                    cnt = min(cnt + total, S);
                  }
                }
            }
        }
        wave_sync();

        __builtin_amdgcn_s_setprio(Net::PRIO_EVALUATE);
        // ---- evaluate: one network after the other
        keep_denormals<Net>(false);
        {
            const ArgsPtr a = opaque(args);
            const int ln = opaque(lane);
            const Net net(ln);
            const float step = a->p.step;
            // the networks of the slots a lane looks after, ln + 64 q (they are its own ray's)
            uint32_t nq[NQ];
#pragma unroll
            for (int q = 0; q < NQ; ++q) nq[q] = (ln >> lgP) + q * G < cnt ? (uint32_t)idx[ln + KN_WAVE * q] : 0xffffffffu;
            __builtin_amdgcn_wave_barrier();
            for (;;) {
                uint32_t mine = 0xffffffffu;
#pragma unroll
                for (int q = NQ - 1; q >= 0; --q) mine = nq[q] != 0xffffffffu ? nq[q] : mine;
                const unsigned long long pending = __ballot(mine != 0xffffffffu);
                if (pending == 0ull) break;
                const int32_t sel = __builtin_amdgcn_readlane((int)mine, (int)__builtin_ctzll(pending));
                typename Net::Weights w; // (not kept across rounds: the march needs the registers)
                w.load(a->packed, sel, ln);
                int c = 0;
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    const bool hit = nq[q] == (uint32_t)sel;
                    const unsigned long long b = __ballot(hit);
                    if (hit) {
                        idx[c + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(b >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)b, 0u))] = (uint16_t)(ln + KN_WAVE * q);
                        nq[q] = 0xffffffffu;
                    }
                    c += __popcll(b);
                }
                wave_sync();
                for (int t0 = 0; t0 < c; t0 += KN_WAVE) {
                    const int len = min(KN_WAVE, c - t0);
                    // pre-activations (r, g, b, sigma) of sample ln of the tile
                    const f4 out = net.evaluate(w, ln, len, [&](int j) { return (int)idx[min(t0 + j, c - 1)]; }, slots, dirs, rays, P);
                    if (ln < len) { // lane l holds sample l of the tile; its result takes the place of its position
                        const int i = idx[t0 + ln];
                        float sg = fmaxf(out[3], 0.0f);
                        if constexpr (STRAT) sg *= slots[i][3];
                        f4 res;
#pragma unroll
                        for (int q = 0; q < 3; ++q) res[q] = Net::sigmoid(out[q]);
                        res[3] = 1.0f - expf(-sg * step); // alpha (Eq. 4)
                        slots[i] = res;
                    }
                }
                __builtin_amdgcn_wave_barrier();
            }
        }
        wave_sync();

        __builtin_amdgcn_s_setprio(Net::PRIO_BETWEEN);
        // ---- blend (Eq. 2-4): the sequential recurrence, the same in all lanes of a ray's group
        keep_denormals<Net>(true);
        {
            const ArgsPtr a = opaque(args);
            const int ln = opaque(lane), slot = ln & (P - 1), gl = ln >> lgP;
            const float stop_below = a->eps > 0.0f ? a->eps : -INFINITY;
            int used = 0;
            if (ray >= 0) {
                // Four samples per step, requested together: one at a time the recurrence waits for the LDS at each of them (82x49 rays
                // 60.8 -> 54.9 us, 200x151 45.8 -> 44.6, 800x800 163.4 -> 162.0).
                // What is requested beyond a ray's samples lies among its slots: a round has S_max of them, a multiple of BLEND.
                static_assert((Net::SLOTS >> Net::MAX_LG) % BLEND == 0 && Net::MAX_S % BLEND == 0, "S_max is a multiple of BLEND");
                bool goes = cnt > 0;
                for (int j = 0; goes; j += BLEND) {
                    f4 q[BLEND];
#pragma unroll
                    for (int c = 0; c < BLEND; ++c) q[c] = slots[((j + c) << lgP) + slot];
                    asm volatile("" : "+v"(q[0]), "+v"(q[1]), "+v"(q[2]), "+v"(q[3])); // (one wait for the four)
#pragma unroll
                    for (int c = 0; c < BLEND; ++c) {
                        if (goes) {
                            const float wgt = T * q[c][3];
                            c0 = fmaf(wgt, q[c][0], c0);
                            c1 = fmaf(wgt, q[c][1], c1);
                            c2 = fmaf(wgt, q[c][2], c2);
                            T *= (1.0f - q[c][3]);
                            used = j + c + 1;
                            goes = (used < cnt) & !(T < stop_below);
                        }
                    }
                }
                if ((cnt > 0 && T < stop_below) || k >= k_hi) {
                    if (gl == 0) {
                        float *px = a->rgb_out + 3 * (int64_t)ray;
                        px[0] = fmaf(T, a->bg[0], c0);
                        px[1] = fmaf(T, a->bg[1], c1);
                        px[2] = fmaf(T, a->bg[2], c2);
                    }
                    ray = -1;
                }
            }
            if (a->counters) { // (uniform)
                evaluated += __builtin_amdgcn_readlane(kn_wave_inclusive_scan(gl == 0 ? cnt : 0), KN_WAVE - 1);
                blended += __builtin_amdgcn_readlane(kn_wave_inclusive_scan(gl == 0 ? used : 0), KN_WAVE - 1);
            }
        }
        keep_denormals<Net>(false);
        __builtin_amdgcn_wave_barrier(); // the slots are rewritten by the next round
    }
    if (args->counters && lane == 0) {
        atomicAdd(&args->counters[0], (unsigned long long)evaluated);
        atomicAdd(&args->counters[1], (unsigned long long)blended);
    }
}

template <class Net> using FusedFn = decltype(&k_render_fused<Net, false>);

// a workgroup's LDS is above the default limit of dynamic LDS (once per device, from kn_create)
template <class Net> int fused_configure()
{
    constexpr int bytes = Net::MAX_WAVES * (int)sizeof(WaveLds<Net>) + OWN_RAYS_MAX * (int)sizeof(int4);
    KN_HIP(hipFuncSetAttribute((const void *)k_render_fused<Net, false>, hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
    KN_HIP(hipFuncSetAttribute((const void *)k_render_fused<Net, true>, hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
    return KN_OK;
}

template <class Net> int fused_launch(const kn_scene *sc, hipStream_t st, const KnFusedJob &job, hipEvent_t ev_start, hipEvent_t ev_stop)
{
    FusedArgs a;
    a.p = *(const MarchParams *)job.march;
    a.net = voxel_fast(a.p.net);
    a.vox = voxel_fast(a.p.occ);
    a.packed = sc->packed_w;
    a.rays_o = job.rays_o;
    a.rays_d = job.rays_d;
    a.list = job.list;
    a.R = (int32_t)job.R;
    a.ctl = job.ctl;
    a.eps = job.eps;
    for (int c = 0; c < 3; ++c) a.bg[c] = job.bg[c];
    a.rgb_out = job.rgb_out;
    a.counters = job.counters;
    // As many wavefronts as get four rays each, up to what the compute units hold; a multiple of eight workgroups, for the shares of the
    // XCDs.  Behind a list a workgroup is a compute unit's wavefronts.  A frame that sets up its own rays has workgroups of four to seven
    // wavefronts, as many as load the compute units evenly: its rays are spread by then, none waits for the walks of fifteen others, and a
    // compute unit is free for a frame on another stream as soon as the four are done.  One workgroup per compute unit / so, the mean of
    // twelve views, one frame at a time and per frame with three in flight: 200x151 55.9, 39.1 / 51.7, 31.1 us; 170x170 60.3, 33.8 / 53.3, 27.4;
    // 100x100 42.2, 26.7 / 43.0, 23.0; 140x105 49.0, 32.8 / 52.5, 32.0; 200x151 at width 64 80, 54 / 74, 48; 104 drawn frames of 4,000 to 32,767
    // rays 1.03 to 1.05 and 1.03 to 1.11 times as fast in the mean, single ones 0.76 to 1.45: where a workgroup's groups of rays fall into one
    // column of the image the rays' costs are spread worst (an offset from group to group moved that to other frames, the mean stayed).
    // At width 32 without an occupancy grid, where nothing is walked, a workgroup stays a compute unit's wavefronts: with smaller ones 36
    // drawn frames are 0.97 times as fast one at a time and 1.02 in flight.  Behind a list eight wavefronts are 1.06 times as fast in
    // flight, but 0.98 one at a time (74 drawn frames of up to 400,000 rays; 577x433 115 -> 121 us): not taken.
    const int64_t want = kn_div_up(job.R, 1 << Net::MIN_LG);
    const int per_cu = (int)std::min<int64_t>(std::max<int64_t>(kn_div_up(want, 256), 4), Net::MAX_WAVES);
    const bool whole = job.list || (Net::MAX_WAVES == 16 && !a.p.has_occ);
    const int groups = whole ? 1 : per_cu / 4; // workgroups per compute unit
    const int waves = (int)kn_div_up(per_cu, groups);
    const int64_t blocks = std::min<int64_t>(8 * kn_div_up(want, 8 * waves), 256 * groups);
    a.max_lg = Net::MAX_LG - (a.p.K < Net::LARGE_POOLS_BELOW ? 0 : 1);
    a.own_group = OWN_GROUP_MIN;
    while (a.own_group < OWN_GROUP_MAX && job.R > (whole ? OWN_GROUPS_WHOLE : OWN_GROUPS) * blocks * (int64_t)a.own_group) a.own_group *= 2;
    // With hardly two samples of a ray per network the weights' way to the wavefronts is what bounds a frame: there, and with enough
    // rays for all compute units, four rays or more share what a wavefront loads (164x94, 1.2 samples per network, width 32 / 64: 93 -> 80 /
    // 224 -> 172 us); elsewhere every wavefront gets a ray if there is one (100x100, 1.5 samples per network: 47 us, 62 with four).
    const float points = fminf(a.p.net.cell[0], fminf(a.p.net.cell[1], a.p.net.cell[2])) / a.p.step;
    a.few_rays = points < 2.0f && job.R > 12288 ? 4 : 1;
    a.own_rays = job.list ? 0 : (int32_t)(a.own_group * kn_div_up(job.R, a.own_group * blocks));
    // Small frames, where every wavefront has its few rays from the start and the chip is not full: longer rounds, where a round's samples are in few
    // networks or none is evaluated in vain.  32 / 64 samples of a ray in pools of four / 128 of two, us: 16^3 networks, 18.5 points in a
    // cell, 140x77 56 / 51 / 49, 27.7 points 70 / 61 / 54, 37 points 97 / 84 / 80, width 64, 37 points 98 / 92 / 85; 9.2 points 91 / 96 / 103, sparse 4.6
    // points 57 / 61 / 64; fp32 (not taken), 18.5 points 82 / 81 / 92; without termination 89x87, 37 points 101 / 84 / 72, 6.2 points 51 / 48.5 / 48.
    // Behind a list (the last rays of each wavefront; 32 samples / so): width 32, 228x225, 37 points 108 / 95, 260x192 without termination 113 / 101,
    // 425x316, 27.7 points 127 / 117, 800x800 no change; width 64, 288x290, 59 points 190 / 181, but 409x230, 24.6 points 190 / 200.
    a.late_lg = Net::MIN_LG;
    a.late_s = Net::MAX_S;
    if (job.R < Net::LONG_ROUNDS_BELOW) {
        if (a.eps == 0.0f || points >= 24.0f) {
            a.late_lg = Net::MIN_LG - 1;
            a.late_s = 4 * Net::MAX_S;
        } else if (points >= 12.0f)
            a.late_s = 2 * Net::MAX_S;
    }
    a.n_waves = waves;
    a.n_blocks = (int32_t)blocks;
    const size_t lds = waves * sizeof(WaveLds<Net>) + a.own_rays * sizeof(int4);
    const FusedFn<Net> kernel = job.strat ? k_render_fused<Net, true> : k_render_fused<Net, false>;
    const dim3 grid((unsigned)blocks), block(waves * KN_WAVE);
    if (ev_start && ev_stop) hipExtLaunchKernelGGL(kernel, grid, block, lds, st, ev_start, ev_stop, 0, a);
    else hipLaunchKernelGGL(kernel, grid, block, lds, st, a);
    KN_CHECK_LAUNCH();
    return KN_OK;
}

} // namespace
