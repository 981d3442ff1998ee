// Stable ordering of a batch by network (Sec. 3.5: the inputs are ordered so that the inputs of one network are
// consecutive in memory): a least-significant-digit radix sort of at most two passes (keys are below 2^16), in two forms.
//
// kn_reorder_run (kn_eval_grouped) moves the samples themselves.  The points arrive in the caller's order; sorting
// indices alone leaves the grouped-MLP kernel with one random 12-byte gather per position and per direction and
// one scattered write per result.  Here two 16-byte halves per sample, (x, y, z, key) and (dx, dy, dz, caller index),
// each in an array of its own, travel through the passes, after which the kernel reads its samples with two
// contiguous 16-byte loads per lane.
// kn_bucket_run (the stage call kn_bucket, the layer-at-a-time and the static-scratch evaluation) sorts (key, index)
// pairs and leaves the permutation.
//
// kn_order_run and kn_count_run (kn_eval_grouped where nobody asks for the permutation) order by counting, without passes:
// the first indices (batches of up to some 10^5 points), the second the samples.
//
// One pass = (digit, block) count table -> per-digit exclusive scan over the blocks -> stable scatter.  Inside a
// block, stability comes from ranking each 64-element row of a wavefront with ballot-built peer masks and
// wave-private counters: no atomics in the ordering path, so the order is the unique stable one.
// A scatter does not store an element where its rank says: 64 lanes would write to some 40 different runs, one
// memory transaction each, and the pass would run at the rate of a random scatter.  The block first brings its
// elements into sorted order in LDS; then consecutive lanes write consecutive addresses, a few runs per store
// instruction.
// The table of the first pass of kn_reorder_run is counted by the kernel that computes the cell ids (Eq. 6); every
// scatter also leaves the keys alone in their new order (4 bytes each), from which the table of the next pass is
// counted.  (Counting it with one atomic per record from inside the first scatter was tried: 4 M device atomics on
// a 130 KB table take longer than both scatters together.)
// Bucket offsets, counts and the kernel's tile list are then found by a 16-way search over the sorted keys, one
// 16-lane group per network.
//
// Results of kn_eval_grouped: a random 16-byte store costs one memory transaction, an unaligned 12-byte one several,
// so the MLP kernel writes (r, g, b, sigma) as one 16-byte store at the sample's caller index into a staging array,
// and a streaming kernel splits that array into the caller's sigma and rgb arrays.
#include "kn_common.h"

namespace {

constexpr int RO_THREADS = 256;
constexpr int RO_WAVES = RO_THREADS / KN_WAVE; // 4
constexpr int RO_ROWS = 16;                    // 64-record rows per wavefront
constexpr int RO_TILE = RO_THREADS * RO_ROWS;  // 4096 records per block

typedef uint32_t u4 __attribute__((ext_vector_type(4)));

// Eq. 6 for RO_TILE points per block: ids (optional), sort keys (network id, N = outside), and the block's count of
// each value of the keys' lowest digit.  Also clears `zero` (the counter that a later kernel of the call adds to) and
// writes the (zero) results of the points that have no network into the staging array of the results.
__global__ void __launch_bounds__(RO_THREADS)
    k_keys_hist(const float *__restrict__ pts, int64_t M, KnGrid g, const int32_t *__restrict__ cell_net, int32_t *__restrict__ ids,
                int32_t *__restrict__ keys, int32_t N, uint32_t digit_mask, int32_t nblk, int32_t *__restrict__ table,
                int32_t *__restrict__ zero, int64_t n_zero, float *__restrict__ out4)
{
    __shared__ int32_t hist[256];
    for (int64_t i = (int64_t)blockIdx.x * RO_THREADS + threadIdx.x; i < n_zero; i += (int64_t)gridDim.x * RO_THREADS) zero[i] = 0;
    hist[threadIdx.x] = 0;
    __syncthreads();
    // one point: id, key, the zero result of a point without a network, the digit count
    auto point = [&](int64_t i, float x, float y, float z) -> int32_t {
        const int32_t id = kn_net_of_cell(cell_net, kn_grid_index(g, x, y, z));
        const int32_t key = id < 0 ? N : id;
        if (ids) ids[i] = id;
        if (id < 0) *(float4 *)(out4 + 4 * i) = make_float4(0.0f, 0.0f, 0.0f, 0.0f); // no network: the result is zero
        atomicAdd(&hist[(uint32_t)key & digit_mask], 1);
        return key;
    };
    const int64_t tile0 = (int64_t)blockIdx.x * RO_TILE;
    if (tile0 + RO_TILE <= M && ((uintptr_t)pts & 15) == 0) { // (uniform) a whole tile of a 16-byte aligned array
        // four consecutive points per thread and step: three 16-byte loads, one 16-byte store of the keys
#pragma unroll
        for (int r = 0; r < RO_ROWS / 4; ++r) {
            const int64_t i = tile0 + 4 * ((int64_t)r * RO_THREADS + threadIdx.x);
            const float4 a = *(const float4 *)(pts + 3 * i), b = *(const float4 *)(pts + 3 * i + 4), c = *(const float4 *)(pts + 3 * i + 8);
            int4 k;
            k.x = point(i, a.x, a.y, a.z);
            k.y = point(i + 1, a.w, b.x, b.y);
            k.z = point(i + 2, b.z, b.w, c.x);
            k.w = point(i + 3, c.y, c.z, c.w);
            *(int4 *)(keys + i) = k;
        }
    } else {
        const int64_t base = tile0 + threadIdx.x;
        float p[RO_ROWS][3];
#pragma unroll
        for (int r = 0; r < RO_ROWS; ++r) {
            const int64_t i = min(base + r * RO_THREADS, M - 1);
#pragma unroll
            for (int c = 0; c < 3; ++c) p[r][c] = pts[3 * i + c];
        }
#pragma unroll
        for (int r = 0; r < RO_ROWS; ++r) {
            const int64_t i = base + r * RO_THREADS;
            if (i < M) keys[i] = point(i, p[r][0], p[r][1], p[r][2]);
        }
    }
    __syncthreads();
    if (threadIdx.x <= digit_mask) table[(int64_t)threadIdx.x * nblk + blockIdx.x] = hist[threadIdx.x];
}

// Row d of the (digit, block) table -> exclusive prefix along the blocks (in place), totals[d] = the row's sum.
// One workgroup per digit.
__global__ void __launch_bounds__(RO_THREADS) k_digit_scan(int32_t *__restrict__ table, int32_t nblk, int32_t *__restrict__ totals)
{
    __shared__ int32_t lds[16];
    int32_t *row = table + (int64_t)blockIdx.x * nblk;
    int32_t carry = 0;
    for (int32_t base = 0; base < nblk; base += RO_THREADS * 4) {
        const int32_t i0 = base + threadIdx.x * 4;
        int32_t v[4], s = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k] = i0 + k < nblk ? row[i0 + k] : 0;
            s += v[k];
        }
        int32_t tot;
        int32_t run = carry + kn_block_exclusive_scan(s, lds, tot);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (i0 + k < nblk) row[i0 + k] = run;
            run += v[k];
        }
        carry += tot;
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

// (digit, block) counts of a pass from the keys alone, in the order the pass reads them.  Also clears `zero`.
__global__ void __launch_bounds__(RO_THREADS)
    k_key_hist(const int32_t *__restrict__ keys, int64_t M, int shift, uint32_t mask, int32_t nblk, int32_t *__restrict__ table,
               int32_t *__restrict__ zero, int64_t n_zero)
{
    __shared__ int32_t hist[256];
    for (int64_t i = (int64_t)blockIdx.x * RO_THREADS + threadIdx.x; i < n_zero; i += (int64_t)gridDim.x * RO_THREADS) zero[i] = 0;
    hist[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * RO_TILE + 4 * (int64_t)threadIdx.x;
#pragma unroll
    for (int r = 0; r < RO_ROWS / 4; ++r) {
        const int64_t i = base + r * (4 * RO_THREADS);
        if (i + 3 < M) {
            const int4 k = *(const int4 *)(keys + i);
            atomicAdd(&hist[((uint32_t)k.x >> shift) & mask], 1);
            atomicAdd(&hist[((uint32_t)k.y >> shift) & mask], 1);
            atomicAdd(&hist[((uint32_t)k.z >> shift) & mask], 1);
            atomicAdd(&hist[((uint32_t)k.w >> shift) & mask], 1);
        } else {
            for (int64_t j = i; j < M && j < i + 4; ++j) atomicAdd(&hist[((uint32_t)keys[j] >> shift) & mask], 1);
        }
    }
    __syncthreads();
    if (threadIdx.x <= mask) table[(int64_t)threadIdx.x * nblk + blockIdx.x] = hist[threadIdx.x];
}

// Ranking step shared by the scatter kernels.  Wavefront w of block b owns elements [b*RO_TILE + w*RO_ROWS*64,
// +RO_ROWS*64) as rows of 64; order of elements = (block, wave, row, lane).  In: key[r] of the lane's element of row r
// (clamped loads beyond M).  Out: lpos[r], the element's position in the block's sorted order (digit, then input
// order), and delta[d] = (global position) - (position in the block's sorted order) for the elements of digit d.
// cnt and delta are LDS arrays of the caller; contains block barriers: every thread of the block calls it.
__device__ __forceinline__ void rank_block(const uint32_t (&key)[RO_ROWS], int32_t (&lpos)[RO_ROWS], int64_t M, int shift, int bits,
                                           int32_t nblk, const int32_t *__restrict__ table_s, const int32_t *__restrict__ totals,
                                           int32_t (*cnt)[256], int32_t *delta, int32_t *scan_lds)
{
    const int lane = threadIdx.x & (KN_WAVE - 1), w = threadIdx.x / KN_WAVE;
    const uint32_t mask = (1u << bits) - 1u;
#pragma unroll
    for (int i = 0; i < RO_WAVES; ++i) cnt[i][threadIdx.x] = 0;
    // thread d: position of this block's first element with digit d = elements with smaller digits + elements with
    // this digit in earlier blocks
    int32_t digit_base;
    {
        const bool has = threadIdx.x <= mask;
        const int32_t total = has ? totals[threadIdx.x] : 0;
        const int32_t mine = has ? table_s[(int64_t)threadIdx.x * nblk + blockIdx.x] : 0;
        int32_t all;
        digit_base = kn_block_exclusive_scan(total, scan_lds, all) + mine; // (contains the barrier that orders the clearing above)
    }
    const int64_t wbase = (int64_t)blockIdx.x * RO_TILE + (int64_t)w * (RO_ROWS * KN_WAVE);
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
    for (int r = 0; r < RO_ROWS; ++r) {
        const bool valid = wbase + r * KN_WAVE + lane < M;
        const uint32_t d = (key[r] >> shift) & mask;
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            if (b < bits) { // uniform
                const bool bit = (d >> b) & 1u;
                const uint64_t m = __ballot(bit);
                peers &= bit ? m : ~m;
            }
        }
        int32_t prior = 0;
        if (valid) prior = cnt[w][d];
        __builtin_amdgcn_wave_barrier();
        const int n_peers = __popcll(peers);
        const bool leader = valid && (lane == 63 - __clzll(peers));
        if (leader) cnt[w][d] = prior + n_peers;
        __builtin_amdgcn_wave_barrier();
        lpos[r] = prior + __popcll(peers & lt_mask); // rank among the wavefront's elements of the same digit
    }
    __syncthreads();
    {
        // thread d: where the digit's elements start in the block's sorted order, and each wavefront's share of them
        const int d = threadIdx.x;
        int32_t c[RO_WAVES], sum = 0;
#pragma unroll
        for (int i = 0; i < RO_WAVES; ++i) {
            c[i] = cnt[i][d];
            sum += c[i];
        }
        int32_t all;
        int32_t run = kn_block_exclusive_scan(sum, scan_lds, all);
        delta[d] = digit_base - run;
#pragma unroll
        for (int i = 0; i < RO_WAVES; ++i) {
            cnt[i][d] = run;
            run += c[i];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RO_ROWS; ++r) lpos[r] += cnt[w][(key[r] >> shift) & mask];
}

// Stable scatter of one radix pass over (key, value) pairs.  vals == nullptr: the values are the positions (first pass).
__global__ void __launch_bounds__(RO_THREADS)
    k_index_scatter(const int32_t *__restrict__ keys, const int32_t *__restrict__ vals, int32_t *__restrict__ keys_out,
                    int32_t *__restrict__ vals_out, int64_t M, int shift, int bits, int32_t nblk, const int32_t *__restrict__ table_s,
                    const int32_t *__restrict__ totals)
{
    __shared__ uint2 stage[RO_TILE]; // (key, value) in the block's sorted order
    __shared__ int32_t cnt[RO_WAVES][256];
    __shared__ int32_t delta[256];
    __shared__ int32_t scan_lds[16];
    const int lane = threadIdx.x & (KN_WAVE - 1), w = threadIdx.x / KN_WAVE;
    const uint32_t mask = (1u << bits) - 1u;
    const int64_t bbase = (int64_t)blockIdx.x * RO_TILE;
    const int64_t wbase = bbase + (int64_t)w * (RO_ROWS * KN_WAVE);
    const int32_t n_here = (int32_t)min((int64_t)RO_TILE, M - bbase); // elements of this block (>= 1)
    uint32_t key[RO_ROWS];
    int32_t val[RO_ROWS], lpos[RO_ROWS];
#pragma unroll
    for (int r = 0; r < RO_ROWS; ++r) {
        const int64_t i = min(wbase + r * KN_WAVE + lane, M - 1);
        key[r] = (uint32_t)keys[i];
        val[r] = vals ? vals[i] : (int32_t)i;
    }
    rank_block(key, lpos, M, shift, bits, nblk, table_s, totals, cnt, delta, scan_lds);
#pragma unroll
    for (int r = 0; r < RO_ROWS; ++r)
        if (wbase + r * KN_WAVE + lane < M) stage[lpos[r]] = make_uint2(key[r], (uint32_t)val[r]);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < RO_ROWS; ++k) {
        const int32_t sp = k * RO_THREADS + threadIdx.x; // position in the block's sorted order
        if (sp < n_here) {
            const uint2 v = stage[sp];
            const int32_t dst = sp + delta[(v.x >> shift) & mask];
            keys_out[dst] = (int32_t)v.x;
            vals_out[dst] = (int32_t)v.y;
        }
    }
}

// Stable scatter of one radix pass over the samples themselves.  `keys`: the keys in the order of the input.
//   FROM_REC false: the halves are formed here from the caller's arrays (points, dirs), caller index = position.
//   keys_out (nullable): the keys alone in the new order; perm_out (nullable): the caller indices in the new order.
// Dynamic LDS: RO_TILE * 16 bytes (the staging buffer of one half).
template <bool FROM_REC>
__global__ void __launch_bounds__(RO_THREADS)
    k_reorder_scatter(const int32_t *__restrict__ keys, const float *__restrict__ pts, const float *__restrict__ dirs,
                      const u4 *__restrict__ pin, const u4 *__restrict__ din, u4 *__restrict__ pout, u4 *__restrict__ dout,
                      int32_t *__restrict__ keys_out, int32_t *__restrict__ perm_out, int64_t M, int shift, int bits, int32_t nblk,
                      const int32_t *__restrict__ table_s, const int32_t *__restrict__ totals)
{
    constexpr int ROWS = RO_ROWS;
    extern __shared__ u4 stage[]; // RO_TILE halves in the block's sorted order
    __shared__ int32_t cnt[RO_WAVES][256];
    __shared__ int32_t delta[256];
    __shared__ int32_t scan_lds[16];
    const int lane = threadIdx.x & (KN_WAVE - 1), w = threadIdx.x / KN_WAVE;
    const uint32_t mask = (1u << bits) - 1u;
    const int64_t bbase = (int64_t)blockIdx.x * RO_TILE;
    const int64_t wbase = bbase + (int64_t)w * (ROWS * KN_WAVE);
    const int32_t n_here = (int32_t)min((int64_t)RO_TILE, M - bbase); // records of this block (>= 1)
    uint32_t key[ROWS];
    int32_t lpos[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) key[r] = (uint32_t)keys[min(wbase + r * KN_WAVE + lane, M - 1)];
    rank_block(key, lpos, M, shift, bits, nblk, table_s, totals, cnt, delta, scan_lds);

    // first halves: (x, y, z, key)
    {
        u4 h[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const int64_t i = min(wbase + r * KN_WAVE + lane, M - 1);
            if constexpr (FROM_REC) {
                h[r] = pin[i];
            } else {
                const float *p = pts + 3 * i;
                h[r] = (u4){__float_as_uint(p[0]), __float_as_uint(p[1]), __float_as_uint(p[2]), key[r]};
            }
        }
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
            if (wbase + r * KN_WAVE + lane < M) stage[lpos[r]] = h[r];
    }
    __syncthreads();
    int32_t dst[ROWS];
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
        const int32_t sp = k * RO_THREADS + threadIdx.x; // position in the block's sorted order
        if (sp < n_here) {
            const u4 v = stage[sp];
            dst[k] = sp + delta[(v[3] >> shift) & mask];
            pout[dst[k]] = v;
            if (keys_out) keys_out[dst[k]] = (int32_t)v[3];
        }
    }
    __syncthreads();
    // second halves: (dx, dy, dz, caller index)
    {
        u4 h[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const int64_t i = min(wbase + r * KN_WAVE + lane, M - 1);
            if constexpr (FROM_REC) {
                h[r] = din[i];
            } else {
                const float *q = dirs + 3 * i;
                h[r] = (u4){__float_as_uint(q[0]), __float_as_uint(q[1]), __float_as_uint(q[2]), (uint32_t)i};
            }
        }
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
            if (wbase + r * KN_WAVE + lane < M) stage[lpos[r]] = h[r];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
        const int32_t sp = k * RO_THREADS + threadIdx.x;
        if (sp < n_here) {
            const u4 v = stage[sp];
            dout[dst[k]] = v;
            if (perm_out) perm_out[dst[k]] = (int32_t)v[3];
        }
    }
}

// Bucket offsets, counts and the tile list of the grouped MLP from the sorted keys (key j at key_of[key_stride * j]:
// word 3 of each first half of the re-ordered samples, or a plain array).
// A wavefront takes three networks n0, n0+1, n0+2 (n = 0 .. N; N: the points without a network): its four 16-lane
// groups find the number of keys below n0 .. n0+3 by a 16-way search (one load per lane and round, five or six rounds
// for 2^22 keys), so that groups 0..2 know both ends of their bucket; each writes offsets[n] and counts[n], and its
// network's tiles (chunks of at most tile_len records) into slots that the workgroup takes from the zeroed counter
// n_tiles with one atomic (the order of tiles is free: nothing observable depends on it).  offsets has N + 2 entries;
// the group of n = N writes the last two.
constexpr int OT_NETS_PER_WAVE = 3, OT_THREADS = 1024, OT_WAVES = OT_THREADS / KN_WAVE;
__global__ void __launch_bounds__(OT_THREADS)
    k_offsets_tiles(const uint32_t *__restrict__ key_of, int key_stride, int64_t M, int32_t N, int32_t tile_len,
                    int32_t *__restrict__ offsets, int32_t *__restrict__ user_offsets, int32_t *__restrict__ counts,
                    int32_t *__restrict__ user_counts, KnTile *__restrict__ tiles, int32_t *__restrict__ n_tiles)
{
    const int lane = threadIdx.x & (KN_WAVE - 1), t = lane & 15, sub = lane >> 4;
    const int32_t wave_id = (blockIdx.x * blockDim.x + threadIdx.x) / KN_WAVE;
    const int32_t n = wave_id * OT_NETS_PER_WAVE + sub; // the bound this group searches; groups 0..2 own network n
    const bool searches = n <= N + 1;
    const uint32_t bound = (uint32_t)n;
    int64_t lo = 0, hi = searches ? M : 0; // the number of keys below `bound` lies in [lo, hi]
    while (__any(hi > lo)) { // each round cuts the interval to a seventeenth; uniform trip count in the wavefront
        const int64_t len = hi - lo;
        const bool last = len <= 16;
        // probes: strictly inside, increasing in t, distinct (len > 16); the last round tests every position left
        const int64_t pos = last ? lo + t : lo + (int64_t)(t + 1) * len / 17;
        bool below = false;
        if (pos < hi) below = key_of[(int64_t)key_stride * pos] < bound;
        const int c = __popcll((__ballot(below) >> (16 * sub)) & 0xffffull); // keys are sorted: lanes 0 .. c-1
        if (last) {
            lo = hi = lo + c;
        } else {
            const int64_t p_below = lo + (int64_t)c * len / 17;       // probe c-1 (if c > 0): the last one below
            const int64_t p_above = lo + (int64_t)(c + 1) * len / 17; // probe c (if c < 16): the first one not below
            if (c < 16) hi = p_above;
            if (c > 0) lo = p_below + 1;
        }
    }
    const int32_t first = (int32_t)lo;
    const int32_t next = __shfl(first, (lane + 16) & (KN_WAVE - 1), KN_WAVE); // the following group's bound
    const bool mine = sub < OT_NETS_PER_WAVE && n <= N;
    const int32_t count = mine ? next - first : 0;
    if (mine && t == 0) {
        offsets[n] = first;
        if (user_offsets) user_offsets[n] = first;
        if (n == N) {
            offsets[N + 1] = next; // = M
            if (user_offsets) user_offsets[N + 1] = next;
        }
        counts[n] = count;
        if (user_counts) user_counts[n] = count;
    }
    // tiles: bucket N (no network) gets none
    const int32_t n_mine = (mine && n < N) ? (count + tile_len - 1) / tile_len : 0;
    int32_t before = 0, wave_total = 0; // tiles of the groups in front of mine in the wavefront
#pragma unroll
    for (int g = 0; g < OT_NETS_PER_WAVE; ++g) {
        const int32_t v = __shfl(n_mine, 16 * g, KN_WAVE);
        if (g < sub) before += v;
        wave_total += v;
    }
    // one atomic per workgroup: atomics on one address execute one after the other (11 ns each)
    __shared__ int32_t wave_tiles[OT_WAVES], block_base;
    const int wv = threadIdx.x / KN_WAVE;
    if (lane == 0) wave_tiles[wv] = wave_total;
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t all = 0;
        for (int i = 0; i < OT_WAVES; ++i) all += wave_tiles[i];
        block_base = all > 0 ? atomicAdd(n_tiles, all) : 0;
    }
    __syncthreads();
    int32_t base = block_base + before;
    for (int i = 0; i < wv; ++i) base += wave_tiles[i];
    for (int32_t k = t; k < n_mine; k += 16) {
        KnTile tl;
        tl.net = n;
        tl.start = first + k * tile_len;
        tl.len = min(tile_len, count - k * tile_len);
        tl.pad = 0;
        tiles[base + k] = tl;
    }
}

// Ordering of a batch whose order inside a network nobody asks for: the rank of a point in its network comes from an
// atomic, so there are no passes.  Latency bound (kn_order_pays says where it is used).  k_rank counts (counts: zeroed N + 1), k_place turns the counts into starts, every
// workgroup for itself, and writes the list of points and the tiles.
//   A workgroup counts its points per network in LDS and takes its share of each network with one atomic: atomics on one
//   address execute one after the other, 11 ns each, and one per run of lanes with the same network took 398 us of a call for
//   131,072 points in random order over two cells of 16^3 (26 like this, 26 over eight, 39 -> 34 all over the grid).  The lanes
//   go through the networks side by side, so that an atomic instruction meets few lines (one atomic per network by the first
//   point that counted it: 65,537 points, 10x16x10, this kernel 12 us; 5 like this), which 1,024 threads with a point each do
//   faster than 256 with four (131,072 points fp32, 16^3 networks 53 -> 51 us a call, 24x20x16 72 -> 70).
//   STABLE (the permutation is asked for): ranks in the order of the points.  The lanes of a wavefront with the same network are found by ballots, a bit of
//   the network at a time, and the wavefronts of a workgroup take their turns at the counts in LDS; the counts of the workgroups go to a (workgroup,
//   network) table, k_table_scan sums them up (and is no launch more: there is nothing to be cleared), and k_place adds what is in front.
constexpr int RANK_THREADS = 1024, RANK_BINS = 4; // networks per thread whose atomics are in flight together
// tiles of c samples (tile_len: a power of two)
__device__ __forceinline__ int32_t tiles_of(int32_t c, int32_t tile_len) { return (c + tile_len - 1) >> __builtin_ctz((uint32_t)tile_len); }
// rows of a (workgroup, network) table start on lines
__host__ __device__ inline int64_t table_stride(int32_t bins) { return (bins + 31) & ~31; }
template <bool STABLE>
__global__ void __launch_bounds__(RANK_THREADS)
    k_rank(const float *__restrict__ pts, int64_t M, KnGrid g, const int32_t *__restrict__ cell_net, int32_t *__restrict__ ids, int32_t N,
           int32_t *__restrict__ counts, int32_t *__restrict__ table, uint2 *__restrict__ ranks, float *__restrict__ sigma, float *__restrict__ rgb)
{
    extern __shared__ int32_t hist[]; // N + 1
    const int64_t i = (int64_t)blockIdx.x * RANK_THREADS + threadIdx.x;
    float p[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) p[c] = pts[3 * min(i, M - 1) + c];
    for (int n = threadIdx.x; n <= N; n += RANK_THREADS) hist[n] = 0;
    const int32_t id = kn_net_of_cell(cell_net, kn_grid_index(g, p[0], p[1], p[2])), key = id < 0 ? N : id;
    const bool active = i < M;
    if (active) {
        if (ids) ids[i] = id;
        if (id < 0) { // no network: the result is zero
            sigma[i] = 0.0f;
            rgb[3 * i] = rgb[3 * i + 1] = rgb[3 * i + 2] = 0.0f;
        }
    }
    if constexpr (STABLE) {
        const int lane = threadIdx.x & (KN_WAVE - 1), wv = __builtin_amdgcn_readfirstlane(threadIdx.x / KN_WAVE);
        unsigned long long same = __ballot(active); // (active lanes) with this lane's network
        for (int b = 0; N >> b; ++b) {
            const bool bit = (key >> b) & 1;
            const unsigned long long with = __ballot(bit);
            same &= bit ? with : ~with;
        }
        const int before = __popcll(same & ((1ull << lane) - 1ull));
        int32_t base = 0;
        for (int w = 0; w < RANK_THREADS / KN_WAVE; ++w) {
            __syncthreads();
            if (w == wv && active && before == 0) { // the first of each network (distinct addresses)
                base = hist[key];
                hist[key] = base + __popcll(same);
            }
        }
        __syncthreads();
        for (int n = threadIdx.x; n <= N; n += RANK_THREADS) table[blockIdx.x * table_stride(N + 1) + n] = hist[n];
        base = __shfl(base, active ? (int)__builtin_ctzll(same) : 0, KN_WAVE);
        if (active) ranks[i] = make_uint2((uint32_t)key, (uint32_t)(base + before));
        return;
    }
    __syncthreads();
    const int32_t rank = active ? atomicAdd(&hist[key], 1) : 0;
    __syncthreads();
    for (int n = threadIdx.x; n <= N; n += RANK_THREADS * RANK_BINS) {
        int32_t c[RANK_BINS];
#pragma unroll
        for (int q = 0; q < RANK_BINS; ++q) c[q] = n + q * RANK_THREADS <= N ? hist[n + q * RANK_THREADS] : 0;
#pragma unroll
        for (int q = 0; q < RANK_BINS; ++q)
            if (c[q] > 0) c[q] = atomicAdd(&counts[n + q * RANK_THREADS], c[q]);
#pragma unroll
        for (int q = 0; q < RANK_BINS; ++q)
            if (n + q * RANK_THREADS <= N) hist[n + q * RANK_THREADS] = c[q];
    }
    __syncthreads();
    if (active) ranks[i] = make_uint2((uint32_t)key, (uint32_t)(rank + hist[key]));
}

// Dynamic LDS: place_lds(per), the networks' starts and per step the tiles in front; per: steps of 64 networks per wavefront.
// PLACE_AHEAD: steps whose counts are under way together (65,000 points, one after the other / so: 16^3 networks, fp16, 28 / 26 us a call, 24x20x28 55 / 49,
// 32^3 111 / 96).
// PLACE_PART: networks whose tiles a wavefront writes where all of them are one step.  Sixty-four / so, the call: 4^3 networks, 98,305 points 25.6 / 18.8 us, 5x8x5, 112,001
// 26.8 / 19.7, width 64 29.0 / 22.2 (more than PLACE_OWN_TILES tiles each, written one network after the other, 6 us of k_place's 11).
constexpr int PLACE_OWN_TILES = 8, PLACE_AHEAD = 8, PLACE_PART = 8;
constexpr int PLACE_THREADS = 1024, PLACE_WAVES = PLACE_THREADS / KN_WAVE, PLACE_POINTS = 2; // points per thread
constexpr int place_lds(int per) { return (PLACE_THREADS + PLACE_WAVES) * per * 4; }
__global__ void __launch_bounds__(PLACE_THREADS)
    k_place(const uint2 *__restrict__ ranks, int64_t M, int32_t N, int32_t per, int32_t tile_len, const int32_t *__restrict__ counts,
            const int32_t *__restrict__ table, int32_t *__restrict__ perm, int32_t *__restrict__ user_counts, KnTile *__restrict__ tiles,
            int32_t *__restrict__ n_tiles)
{
    extern __shared__ int32_t start[];
    __shared__ int32_t s_sum[2][PLACE_WAVES];
    const int lane = threadIdx.x & (KN_WAVE - 1), wv = threadIdx.x / KN_WAVE, b0 = wv * KN_WAVE * per + lane;
    int32_t *step_tiles = start + PLACE_THREADS * per; // tiles of the wavefront's networks in front of each step
    const int64_t i0 = (int64_t)blockIdx.x * (PLACE_THREADS * PLACE_POINTS) + threadIdx.x;
    uint2 kr[PLACE_POINTS];
#pragma unroll
    for (int r = 0; r < PLACE_POINTS; ++r) kr[r] = ranks[min(i0 + r * PLACE_THREADS, M - 1)];
    if (table) { // (uniform) stable ranks: what the workgroups of k_rank in front counted
#pragma unroll
        for (int r = 0; r < PLACE_POINTS; ++r)
            kr[r].y += (uint32_t)table[min(i0 + r * PLACE_THREADS, M - 1) / RANK_THREADS * table_stride(N + 1) + (int32_t)kr[r].x];
    }
    // exclusive starts of the networks inside the wavefront's share, then across wavefronts (tiles: the same sums, kept for
    // the networks this workgroup writes the tiles of)
    int32_t sum = 0, tile_sum = 0;
    for (int s0 = 0; s0 < per; s0 += PLACE_AHEAD) {
        int32_t c_ahead[PLACE_AHEAD];
#pragma unroll
        for (int q = 0; q < PLACE_AHEAD; ++q) c_ahead[q] = counts[min(b0 + (s0 + q) * KN_WAVE, N)];
#pragma unroll
        for (int q = 0; q < PLACE_AHEAD; ++q) {
            const int s = s0 + q;
            if (s >= per) break; // (uniform)
            const int32_t n = b0 + s * KN_WAVE, c = n <= N ? c_ahead[q] : 0;
            const int32_t inc = kn_wave_inclusive_scan(c);
            start[n] = sum + inc - c;
            sum += __builtin_amdgcn_readlane(inc, KN_WAVE - 1);
            const int32_t t = n < N ? tiles_of(c, tile_len) : 0;
            if (lane == 0) step_tiles[wv * per + s] = tile_sum;
            tile_sum += __builtin_amdgcn_readlane(kn_wave_inclusive_scan(t), KN_WAVE - 1);
            if (user_counts && n <= N && blockIdx.x == 0) user_counts[n] = c;
        }
    }
    if (lane == 0) {
        s_sum[0][wv] = sum;
        s_sum[1][wv] = tile_sum;
    }
    __syncthreads();
    int32_t before = 0, tiles_before = 0, tiles_all = 0;
    for (int w = 0; w < PLACE_WAVES; ++w) {
        before += w < wv ? s_sum[0][w] : 0;
        tiles_before += w < wv ? s_sum[1][w] : 0;
        tiles_all += s_sum[1][w];
    }
    if (before)
        for (int s = 0; s < per; ++s) start[b0 + s * KN_WAVE] += before;
    if (blockIdx.x == 0 && threadIdx.x == 0) *n_tiles = tiles_all;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < PLACE_POINTS; ++r) {
        const int64_t i = i0 + r * PLACE_THREADS;
        if (i < M) perm[start[kr[r].x] + (int32_t)kr[r].y] = (int32_t)i;
    }
    // tiles: those of part u of wavefront w's networks are written by workgroup (w * parts + u) % gridDim.x.  A part is a step of 64 networks, or, with
    // one step only, PLACE_PART of them
    const int grid = (int)gridDim.x, lg_part = per == 1 && grid >= KN_WAVE / PLACE_PART ? __builtin_ctz(PLACE_PART) : __builtin_ctz(KN_WAVE);
    const int parts = per << (__builtin_ctz(KN_WAVE) - lg_part), first_u = ((int)blockIdx.x - wv * parts % grid + grid) % grid;
    for (int u = first_u; u < parts; u += grid) { // (uniform)
        const int s = u >> (__builtin_ctz(KN_WAVE) - lg_part);
        const bool mine = (u << lg_part) - (s << __builtin_ctz(KN_WAVE)) == (lane & -(1 << lg_part));
        const int32_t n = b0 + s * KN_WAVE, c = n <= N ? counts[n] : 0, t = n < N ? tiles_of(c, tile_len) : 0;
        const int32_t inc = kn_wave_inclusive_scan(t), in_front = tiles_before + step_tiles[wv * per + s];
        // a lane writes its own network's tiles, the wavefront together those of a network with many (one network after
        // the other for all 64 took 5 of this kernel's 14 us at 65,537 points)
        if (mine && t <= PLACE_OWN_TILES) {
            const int32_t first = n <= N ? start[n] : 0;
            for (int32_t k = 0; k < t; ++k) tiles[in_front + inc - t + k] = KnTile{n, first + k * tile_len, min(tile_len, c - k * tile_len), 0};
        }
        for (unsigned long long many = __ballot(mine && t > PLACE_OWN_TILES); many; many &= many - 1) { // (uniform)
            const int q = (int)__builtin_ctzll(many);
            const int32_t tq = __builtin_amdgcn_readlane(t, q), base = in_front + __builtin_amdgcn_readlane(inc, q) - tq;
            const int32_t nq = n - lane + q, cq = __builtin_amdgcn_readlane(c, q), first = start[nq];
            for (int32_t k = lane; k < tq; k += KN_WAVE) tiles[base + k] = KnTile{nq, first + k * tile_len, min(tile_len, cq - k * tile_len), 0};
        }
    }
}

// Order by counting with the samples themselves (kn_eval_grouped, large batches whose permutation nobody asks for): one
// trip of the samples instead of one per digit.  A workgroup takes `share` consecutive points, up to ROWS per thread.
//   k_keys_count    network of each point, the workgroup's count per network (LDS) -> row of the (workgroup, network) table
//   k_table_scan    per network exclusive prefix over the workgroups, totals
//   k_count_scatter the workgroup's samples into sorted order in LDS (a sample's rank comes from an LDS atomic), then to
//                   memory; every workgroup forms the networks' starts from the totals for itself and writes its share of
//                   the tiles
// A workgroup has about two samples per network with 4,096 networks, 32 bytes of each half side by side: the runs of one
// network follow each other by workgroup, so an XCD takes one contiguous part of the batch, and its workgroups, which go
// through the networks at the same pace, fill the lines in its L2 together.
// From COUNT_BACK_M points on a result goes to its sample's own place (k_results_back), and the two halves are 12 bytes each; 16 with the key and the
// result's place: 4 M points, 16^3 networks, scatter 72 us, MLP kernel 87 / 69, 80; 8 M skewed 127, 160 / 115, 148.
// Bound by memory traffic: 4 M points, 16^3 networks: count 20 us, scan 6 (11 with rows of N + 1 entries, whose lines two workgroups share; 8 M 17 -> 10), scatter 59 (118 MB read, 126 to be written),
// against 158 for the two radix passes and 10 for the search for the tiles.  Batches of less than a round of workgroups: by the chain of a workgroup's
// phases (300,000 points: some 10 us in the kernel, of which reading the points 1, ranks 1.4, starts 2.3, either half 1 to 2).
// Whole calls, width 32, fp16, against the radix passes: 4 M points 322 -> 180 us, 1 M 106 -> 63, 270,001 73 -> 36.
constexpr int CO_T = 1024;
// COUNT_MAX_N: the staging buffer of eight rows (128 KB) and the networks' starts are the LDS of a compute unit.
// COUNT_WIDE_M: four rows where they hold a 256th of the batch.  Against 512 threads of eight rows (twice the networks per thread): 300,007 points
// 48.8 -> 46.8 us, 1 M, width 64, bf16 82.5 -> 80.6.
// COUNT_FULL_M: shares are a 256th or a 512th of the batch (all compute units, one or two workgroups one after the other, all of one size) up to here, beyond
// as large as they can be, since short shares have short runs.  Shares of 4,096 / a 256th, 16^3 networks, fp16: 270,001 points 40.9 / 38.8 us, 560,001 51.7 / 49.6, 1.3 M
// 83 / 74.6; of 8,192 / a 512th: 2.1 M 127 / 114, 2.5 M 131 / 125, 3.2 M 151 / 151; of 8,192 / a 768th: 5 M 230 / 239.
// COUNT_MIN_M: ORDER_MAX_M_COUNTED, see kn_order_pays, which is asked first.  (Few networks, where the radix sort is one trip as well: 5x8x5, 270,000 points 50 -> 30 us, 1 M
// 67 -> 47, 4 M 219 -> 150; 2^3 with nine in ten points in one network, the most LDS atomics on one address, 4 M 279 -> 180.)
// COUNT_BACK_M: 16-bit scenes from here on, and all with eight rows: results go through k_results_back.  Width 32, fp16 / width 64, bf16,
// 16^3 networks, before / with it: 270,001 points 40.9 / 43.2, 55.9 / 58.7 us, 400,001 47.5 / 46.8, 59.6 / 61.0, 560,001 51.6 / 51.6, 67.2 / 67.3 (skewed, width 32, 46.6 / 44.1;
// 5x8x5 38.8 / 37.6), 1 M 72.7 / 69.9, 89.5 / 86.3; fp32, whose evaluation the scattered stores don't hold up, 1.3 M 186 / 190.
constexpr int64_t COUNT_BACK_M = 1 << 19;
constexpr int32_t COUNT_MAX_N = 6143;
constexpr int64_t COUNT_MIN_M = 5 << 15, COUNT_WIDE_M = 1 << 20, COUNT_FULL_M = 1 << 22;
typedef uint16_t h4_t __attribute__((ext_vector_type(4)));

// Non-temporal: what a workgroup reads once stays out of the way of the lines that the workgroups of an XCD fill and read together in its L2.  4 M points,
// 16^3 networks: k_count_scatter 68 -> 63 us, the MLP kernel 80 -> 77, k_results_back 40 -> 37; 8 M skewed 118 -> 108, 151 -> 147, 76 -> 73.  (With
// four rows, whose batches fit the caches, 0.3 us slower; non-temporal stores of the results 38 -> 67.)
template <bool STREAM, typename V> __device__ __forceinline__ V load_once(const V *p)
{
    if constexpr (STREAM) return __builtin_nontemporal_load(p);
    else return *p;
}
template <bool STREAM, typename V> __device__ __forceinline__ void store_once(V *p, V v)
{
    if constexpr (STREAM) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// (the same numbering in both kernels: row b of the table)
__device__ __forceinline__ int32_t xcd_block(int32_t nblk)
{
    const int32_t x = blockIdx.x & 7, each = nblk >> 3, more = nblk & 7;
    return x * each + min(x, more) + ((int32_t)blockIdx.x >> 3);
}

template <int ROWS>
__global__ void __launch_bounds__(CO_T)
    k_keys_count(const float *__restrict__ pts, int64_t M, KnGrid g, const int32_t *__restrict__ cell_net, int32_t *__restrict__ ids,
                 uint16_t *__restrict__ keys, int32_t N, int32_t nblk, int32_t share, int32_t *__restrict__ table)
{
    constexpr int T = CO_T;
    extern __shared__ int32_t hist[]; // N + 1
    for (int i = threadIdx.x; i <= N; i += T) hist[i] = 0;
    __syncthreads();
    const int32_t b = xcd_block(nblk);
    auto point = [&](int64_t i, float x, float y, float z) -> uint16_t {
        const int32_t id = kn_net_of_cell(cell_net, kn_grid_index(g, x, y, z));
        const int32_t key = id < 0 ? N : id;
        if (ids) ids[i] = id;
        atomicAdd(&hist[key], 1);
        return (uint16_t)key;
    };
    const int64_t base = (int64_t)b * share;
    const int32_t n_here = (int32_t)min((int64_t)share, M - base);
    if ((n_here & 3) == 0 && ((uintptr_t)pts & 15) == 0) { // (uniform) four points per thread and step, 16-byte loads
        float4 v[ROWS / 4][3];
#pragma unroll
        for (int r = 0; r < ROWS / 4; ++r)
#pragma unroll
            for (int c = 0; c < 3; ++c) v[r][c] = *(const float4 *)(pts + 3 * (base + min(4 * (r * T + (int)threadIdx.x), n_here - 4)) + 4 * c);
#pragma unroll
        for (int r = 0; r < ROWS / 4; ++r) {
            if (4 * (r * T + (int)threadIdx.x) >= n_here) break;
            const int64_t i = base + 4 * (r * T + (int)threadIdx.x);
            const float4 p = v[r][0], q = v[r][1], s = v[r][2];
            h4_t k;
            k[0] = point(i, p.x, p.y, p.z);
            k[1] = point(i + 1, p.w, q.x, q.y);
            k[2] = point(i + 2, q.z, q.w, s.x);
            k[3] = point(i + 3, s.y, s.z, s.w);
            *(h4_t *)(keys + i) = k;
        }
    } else {
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const int64_t i = base + r * T + threadIdx.x;
            if (i < base + n_here) keys[i] = point(i, pts[3 * i], pts[3 * i + 1], pts[3 * i + 2]);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i <= N; i += T) table[b * table_stride(N + 1) + i] = hist[i];
}

// 32 networks per workgroup (their places in a row of the table are a line of their own: table_stride), 32 shares of the table's rows, two to
// a wavefront
constexpr int TS_NETS = 32, TS_SHARES = 1024 / TS_NETS;
__global__ void __launch_bounds__(1024) k_table_scan(int32_t *__restrict__ table, int32_t bins, int32_t nblk, int32_t *__restrict__ totals)
{
    const int64_t stride = table_stride(bins);
    __shared__ int32_t part[1024 / KN_WAVE][TS_NETS];
    const int lane = threadIdx.x & (TS_NETS - 1), seg = threadIdx.x / TS_NETS, wv = threadIdx.x / KN_WAVE;
    const int32_t d = blockIdx.x * TS_NETS + lane;
    const int32_t each = (nblk + TS_SHARES - 1) / TS_SHARES, r0 = min(seg * each, nblk), r1 = min(r0 + each, nblk);
    const bool has = d < bins;
    int32_t *col = table + (has ? d : bins - 1);
    constexpr int KEPT = 32; // rows of a share that stay in registers between the two sweeps (all loads in flight together)
    int32_t v[KEPT], sum = 0;
#pragma unroll
    for (int k = 0; k < KEPT; ++k) v[k] = r0 + k < r1 ? col[(r0 + k) * stride] : 0;
#pragma unroll
    for (int k = 0; k < KEPT; ++k) sum += v[k];
    for (int32_t r = r0 + KEPT; r < r1; ++r) sum += col[r * stride];
    int32_t run = sum; // up to and with this share of the wavefront's
#pragma unroll
    for (int w = TS_NETS; w < KN_WAVE; w <<= 1) {
        const int32_t o = __shfl_up(run, w, KN_WAVE);
        if ((int)(threadIdx.x & (KN_WAVE - 1)) >= w) run += o;
    }
    if ((threadIdx.x & (KN_WAVE - 1)) >= KN_WAVE - TS_NETS) part[wv][lane] = run;
    __syncthreads();
    run -= sum;
    for (int q = 0; q < wv; ++q) run += part[q][lane];
    if (!has) return;
    if (seg == TS_SHARES - 1) totals[d] = run + sum;
#pragma unroll
    for (int k = 0; k < KEPT; ++k) {
        if (r0 + k < r1) col[(r0 + k) * stride] = run;
        run += v[k];
    }
    for (int32_t r = r0 + KEPT; r < r1; ++r) {
        const int32_t c = col[r * stride];
        col[r * stride] = run;
        run += c;
    }
}

// Dynamic LDS: CO_T * ROWS halves of 16 bytes (first the counts), then N + 1 ints.
// CO_LIST: networks whose tiles one workgroup writes, at most: network d is workgroup d % nblk's, and there are 250 workgroups or more (a share is
// less than 4 points more than a 256th of COUNT_MIN_M points or more, and at most a 512th of more than COUNT_FULL_M).
constexpr int CO_LIST = (COUNT_MAX_N + 249) / 250;
static_assert((COUNT_MAX_N + 1) * 4 <= CO_T * 4 * 16, "the counts share the staging buffer's place");
constexpr int LIST_LANES = 16, LIST_LONG = 512; // lanes that write one network's tiles; those of networks with more than LIST_LONG the whole workgroup writes
struct f3_t { float x, y, z; };
__device__ __forceinline__ int opaque(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}
// What a thread needs of its networks is requested with the points, all of it together, and a thread's place is made anew for each phase (left to
// itself the compiler keeps the addresses of all phases from the start on, which took the registers for that): one network after the other 24.6 us at
// 300,007 points, 23.8 at 1 M, 63 at 4 M; so, with the tiles by sixteen lanes per network, 13 / 19 / 59.
template <int ROWS, bool BACK>
__global__ void __launch_bounds__(CO_T)
    k_count_scatter(const uint16_t *__restrict__ keys, const float *__restrict__ pts, const float *__restrict__ dirs, void *__restrict__ pout,
                    void *__restrict__ dout, int64_t M, int32_t N, int32_t nblk, int32_t share, const int32_t *__restrict__ table,
                    const int32_t *__restrict__ totals, int32_t tile_len, int32_t *__restrict__ user_counts, KnTile *__restrict__ tiles,
                    int32_t *__restrict__ n_tiles, uint32_t *__restrict__ at, uint16_t *__restrict__ from, float *__restrict__ out4)
{
    constexpr int T = CO_T;
    constexpr bool STREAM = ROWS == 8;
    extern __shared__ u4 stage[];
    __shared__ int32_t s_sum[3][T / KN_WAVE];
    __shared__ int4 s_list[CO_LIST]; // (network, samples, first sample, first tile)
    __shared__ int32_t s_listed, s_long; // how many; whether one has more than LIST_LONG tiles
    int32_t *cnt = (int32_t *)stage, *delta = (int32_t *)(stage + T * ROWS);
    int tid = threadIdx.x;
    const int lane = tid & (KN_WAVE - 1), wv = tid / KN_WAVE;
    const int32_t b = xcd_block(nblk), bins = N + 1;
    const int64_t base = (int64_t)b * share;
    const int32_t n_here = (int32_t)min((int64_t)share, M - base);
    if (tid == 0) s_listed = s_long = 0;
    for (int i = tid; i < bins; i += T) cnt[i] = 0;
    uint32_t key[ROWS];
    float p[ROWS][3];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const int64_t i = base + min(r * T + tid, n_here - 1);
        key[r] = load_once<STREAM>(keys + i);
#pragma unroll
        for (int c = 0; c < 3; ++c) p[r][c] = load_once<STREAM>(pts + 3 * i + c);
    }
    // thread t: networks t * per ..
    const int32_t per = (bins + T - 1) / T, d0 = min(tid * per, bins), d1 = min(d0 + per, bins);
    constexpr int KEPT = (COUNT_MAX_N + T) / T;
    int32_t total[KEPT], in_front[KEPT], here[KEPT]; // all requested together
    const int32_t *const row = table + b * table_stride(bins);
    // (wavefronts without a network of their own do not wait for any, and so not for the points in front of them: 5 M points on 2^3 networks, the call, 208.3 -> 205.5 us)
    if (d0 < d1) {
#pragma unroll
        for (int j = 0; j < KEPT; ++j)
            if (j < per) total[j] = totals[min(d0 + j, N)];
#pragma unroll
        for (int j = 0; j < KEPT; ++j)
            if (j < per) in_front[j] = row[min(d0 + j, N)];
    }
    __syncthreads();
    int32_t lpos[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) lpos[r] = r * T + tid < n_here ? atomicAdd(&cnt[key[r]], 1) : 0;
    __syncthreads();
    // sums in front of a thread's networks of the workgroup's samples, of all samples and of tiles
    int32_t own[3] = {0, 0, 0}, run[3];
    if (d0 < d1) {
#pragma unroll
        for (int j = 0; j < KEPT; ++j)
            if (j < per) here[j] = cnt[min(d0 + j, N)];
#pragma unroll
        for (int j = 0; j < KEPT; ++j) {
            if (j >= per) break; // (uniform)
            if (d0 + j >= d1) here[j] = total[j] = 0; // (another thread's, or none)
            own[0] += here[j];
            own[1] += total[j];
            own[2] += d0 + j < N ? tiles_of(total[j], tile_len) : 0;
        }
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        run[q] = kn_wave_inclusive_scan(own[q]);
        if (lane == KN_WAVE - 1) s_sum[q][wv] = run[q];
        run[q] -= own[q];
    }
    __syncthreads();
    int32_t tiles_all = 0;
    for (int w = 0; w < T / KN_WAVE; ++w) {
#pragma unroll
        for (int q = 0; q < 3; ++q) run[q] += w < wv ? s_sum[q][w] : 0;
        tiles_all += s_sum[2][w];
    }
    if (b == 0 && tid == 0) *n_tiles = tiles_all;
    int32_t turn = d0 % nblk; // (network d's tiles are written by workgroup d % nblk)
    if (d0 < d1) {
#pragma unroll
        for (int j = 0; j < KEPT; ++j) {
            if (j >= per) break;
            const int32_t d = d0 + j, n_t = d < N ? tiles_of(total[j], tile_len) : 0;
            if (d < d1) {
                delta[d] = run[1] + in_front[j] - run[0];
                cnt[d] = run[0];
                if (user_counts && b == 0) user_counts[d] = total[j];
            }
            if (n_t > 0 && turn == b) {
                s_list[atomicAdd(&s_listed, 1)] = make_int4(d, total[j], run[1], run[2]);
                if (n_t > LIST_LONG) s_long = 1;
            }
            if (++turn == nblk) turn = 0;
            run[0] += here[j];
            run[1] += total[j];
            run[2] += n_t;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROWS; ++r) lpos[r] += cnt[key[r]];
    __syncthreads(); // the counts' place is the staging buffer's from here on
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
        if (r * T + tid < n_here)
            stage[lpos[r]] = (u4){__float_as_uint(p[r][0]), __float_as_uint(p[r][1]), __float_as_uint(p[r][2]), key[r]};
    tid = opaque(tid);
#pragma unroll
    for (int r = 0; r < ROWS; ++r) { // (the second halves are under way while the first ones are written)
        const int64_t i = base + min(r * T + tid, n_here - 1);
        if (!BACK && key[r] == (uint32_t)N) *(float4 *)(out4 + 4 * i) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
        for (int c = 0; c < 3; ++c) p[r][c] = load_once<STREAM>(dirs + 3 * i + c);
    }
    __syncthreads();
    // BACK: a sample's result goes to its own place, and its halves need no fourth word
    auto put = [&](void *half, int32_t i, u4 v) {
        if constexpr (BACK) ((f3_t *)half)[i] = (f3_t){__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2])};
        else ((u4 *)half)[i] = v;
    };
    tid = opaque(tid);
    int32_t dst[ROWS];
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
        const int32_t sp = k * T + tid;
        if (sp < n_here) {
            const u4 v = stage[sp];
            dst[k] = sp + delta[v[3]];
            put(pout, dst[k], v);
            if constexpr (BACK) store_once<STREAM>(at + base + sp, (uint32_t)dst[k]);
            // no network: the result is zero
            if (BACK && v[3] == (uint32_t)N) *(float4 *)(out4 + 4 * (int64_t)dst[k]) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
        if (r * T + tid < n_here)
            stage[lpos[r]] = (u4){__float_as_uint(p[r][0]), __float_as_uint(p[r][1]), __float_as_uint(p[r][2]), (uint32_t)(r * T + tid)};
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
        const int32_t sp = k * T + tid;
        if (sp < n_here) {
            u4 v = stage[sp];
            if constexpr (BACK) store_once<STREAM>(from + base + sp, (uint16_t)v[3]);
            else v[3] += (uint32_t)base; // the place in the caller's order
            put(dout, dst[k], v);
        }
    }
    // tiles: sixteen lanes per network, the whole workgroup for networks of many (a wavefront per network, and a look at the whole list for
    // those of more tiles than lanes: 3 of this kernel's 18 us at 300,000 points)
    const int32_t listed = s_listed;
    auto write_tiles = [&](const int4 &l, int32_t first, int32_t stride) {
        const int32_t n_t = tiles_of(l.y, tile_len);
        for (int32_t k = first; k < n_t; k += stride) tiles[l.w + k] = KnTile{l.x, l.z + k * tile_len, min(tile_len, l.y - k * tile_len), 0};
    };
    for (int e = tid / LIST_LANES; e < listed; e += T / LIST_LANES)
        if (const int4 l = s_list[e]; tiles_of(l.y, tile_len) <= LIST_LONG) write_tiles(l, tid & (LIST_LANES - 1), LIST_LANES);
    if (s_long) // (uniform)
        for (int e = 0; e < listed; ++e)
            if (const int4 l = s_list[e]; tiles_of(l.y, tile_len) > LIST_LONG) write_tiles(l, tid, T);
}

// Results in the order of the samples -> the caller's sigma and rgb arrays, by the workgroups of k_count_scatter: sample `sp` of
// a workgroup's sorted order is its point `from` and lies at `at`.  Through LDS, so that a workgroup reads runs of a few
// results, which its neighbours on the XCD read the rest of the lines of, and writes its points one after the other.
// Instead of one random 16-byte store per sample by the MLP kernel (one transaction each, 57 G/s): 4 M points, 16^3 networks,
// MLP kernel 120 -> 83 us, this kernel 40 (169 MB, 4.2 TB/s) against 25 for k_split_results.
template <int ROWS>
__global__ void __launch_bounds__(CO_T)
    k_results_back(const float *__restrict__ out4, const uint32_t *__restrict__ at, const uint16_t *__restrict__ from, int64_t M, int32_t nblk, int32_t share,
                   float *__restrict__ sigma, float *__restrict__ rgb)
{
    constexpr int T = CO_T;
    constexpr bool STREAM = ROWS == 8;
    extern __shared__ u4 stage[]; // T * ROWS results
    const int64_t base = (int64_t)xcd_block(nblk) * share;
    const int32_t n_here = (int32_t)min((int64_t)share, M - base);
    uint32_t a[ROWS], f[ROWS];
    u4 v[ROWS];
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
        const int64_t i = base + min(k * T + (int)threadIdx.x, n_here - 1);
        a[k] = load_once<STREAM>(at + i);
        f[k] = load_once<STREAM>(from + i);
    }
#pragma unroll
    for (int k = 0; k < ROWS; ++k) v[k] = *(const u4 *)(out4 + 4 * (int64_t)a[k]);
#pragma unroll
    for (int k = 0; k < ROWS; ++k) stage[f[k]] = v[k]; // (beyond the end: the last sample once more)
    __syncthreads();
    const float *res = (const float *)stage;
    const bool aligned = (((uintptr_t)sigma | (uintptr_t)rgb) & 15) == 0; // (base is a multiple of 4)
#pragma unroll
    for (int r = 0; r < ROWS / 4; ++r) {
        const int32_t q = 4 * (r * T + (int)threadIdx.x);
        if (q + 3 < n_here && aligned) {
            float4 o[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) o[k] = *(const float4 *)(res + 4 * (q + k));
            *(float4 *)(sigma + base + q) = make_float4(o[0].w, o[1].w, o[2].w, o[3].w);
            float4 *c = (float4 *)(rgb + 3 * (base + q));
            c[0] = make_float4(o[0].x, o[0].y, o[0].z, o[1].x);
            c[1] = make_float4(o[1].y, o[1].z, o[2].x, o[2].y);
            c[2] = make_float4(o[2].z, o[3].x, o[3].y, o[3].z);
        } else {
            for (int32_t j = q; j < n_here && j < q + 4; ++j) {
                const float4 o = *(const float4 *)(res + 4 * j);
                sigma[base + j] = o.w;
                rgb[3 * (base + j)] = o.x;
                rgb[3 * (base + j) + 1] = o.y;
                rgb[3 * (base + j) + 2] = o.z;
            }
        }
    }
}

// staging array (r, g, b, sigma per point, caller order) -> the caller's sigma and rgb arrays; 4 points per thread
__global__ void __launch_bounds__(256) k_split_results(const float *__restrict__ out4, int64_t M, float *__restrict__ sigma, float *__restrict__ rgb)
{
    const int64_t i = 4 * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
    if (i >= M) return;
    if (i + 3 < M && (((uintptr_t)sigma | (uintptr_t)rgb) & 15) == 0) {
        float4 v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = *(const float4 *)(out4 + 4 * (i + k));
        *(float4 *)(sigma + i) = make_float4(v[0].w, v[1].w, v[2].w, v[3].w);
        float4 *c = (float4 *)(rgb + 3 * i);
        c[0] = make_float4(v[0].x, v[0].y, v[0].z, v[1].x);
        c[1] = make_float4(v[1].y, v[1].z, v[2].x, v[2].y);
        c[2] = make_float4(v[2].z, v[3].x, v[3].y, v[3].z);
    } else {
        for (int64_t j = i; j < M && j < i + 4; ++j) {
            const float4 v = *(const float4 *)(out4 + 4 * j);
            sigma[j] = v.w;
            rgb[3 * j] = v.x;
            rgb[3 * j + 1] = v.y;
            rgb[3 * j + 2] = v.z;
        }
    }
}

struct ReorderWs {
    int32_t *keys, *keys_b, *table, *totals, *n_tiles, *counts, *offsets;
    u4 *pos_a, *dir_a, *pos_b, *dir_b; // the two halves of the records, before and after the second pass
    float *out4;
    KnTile *tiles;
    int64_t nblk;
};

// workgroups of k_offsets_tiles: OT_WAVES wavefronts of OT_NETS_PER_WAVE networks each, for the networks 0 .. N
int64_t offsets_tiles_blocks(int32_t N) { return kn_div_up(kn_div_up((int64_t)N + 1, OT_NETS_PER_WAVE), OT_WAVES); }

int key_bits(int32_t N)
{
    int bits = 1;
    while ((1ll << bits) < (int64_t)N + 1) ++bits;
    return bits;
}

void carve_reorder(KnCarver &c, int64_t M, int32_t N, ReorderWs &w)
{
    w.nblk = kn_div_up(M > 0 ? M : 1, RO_TILE);
    const bool two = key_bits(N) > 8;
    w.n_tiles = c.carve<int32_t>(1);
    w.table = c.carve<int32_t>(256 * w.nblk);
    w.totals = c.carve<int32_t>(256);
    w.keys = c.carve<int32_t>(M);
    w.keys_b = two ? c.carve<int32_t>(M) : nullptr;
    w.counts = c.carve<int32_t>(N + 1);
    w.offsets = c.carve<int32_t>(N + 2);
    w.tiles = c.carve<KnTile>(kn_max_tiles(M, N, 64));
    w.pos_a = c.carve<u4>(M);
    w.dir_a = c.carve<u4>(M);
    w.pos_b = two ? c.carve<u4>(M) : nullptr;
    w.dir_b = two ? c.carve<u4>(M) : nullptr;
    w.out4 = c.carve<float>(4 * M);
}

} // namespace

int64_t kn_reorder_ws_bytes(int64_t M, int32_t N)
{
    KnCarver c((void *)256, INT64_MAX / 2);
    ReorderWs w;
    carve_reorder(c, M, N, w);
    return c.used;
}

int kn_reorder_run(const kn_scene *sc, hipStream_t st, const float *points, const float *dirs, int64_t M, int32_t tile_len,
                   int32_t *user_ids, int32_t *user_counts, int32_t *user_perm, KnCarver &ws, KnBucketOut *out,
                   const uint32_t *records[2], float **out4, KnStageTimer *tm)
{
    const int32_t N = sc->N;
    if (M < 1 || M > (1ll << 30) || N < 1 || N > 65535 || tile_len < 64) return KN_E_INVALID_ARG;
    ReorderWs w;
    carve_reorder(ws, M, N, w);
    if (!ws.ok()) return KN_E_WORKSPACE;
    const int bits = key_bits(N); // <= 16
    const bool two = bits > 8;
    const int bits0 = two ? bits / 2 : bits, bits1 = bits - bits0; // (the last pass takes the larger digit: N itself is a key)
    const int32_t nblk = (int32_t)w.nblk;
    const dim3 grid((unsigned)nblk), block(RO_THREADS);

    hipLaunchKernelGGL(k_keys_hist, grid, block, 0, st, points, M, sc->net_grid, sc->cell_net, user_ids, w.keys, N, (1u << bits0) - 1u,
                       nblk, w.table, w.n_tiles, (int64_t)1, w.out4);
    KN_CHECK_LAUNCH();
    if (tm) tm->mark(KN_ST_CELL);
    hipLaunchKernelGGL(k_digit_scan, dim3(1u << bits0), block, 0, st, w.table, nblk, w.totals);
    KN_CHECK_LAUNCH();
    const u4 *sorted_pos = w.pos_a, *sorted_dir = w.dir_a;
    constexpr size_t stage_bytes = (size_t)RO_TILE * sizeof(u4);
    hipLaunchKernelGGL((k_reorder_scatter<false>), grid, block, stage_bytes, st, w.keys, points, dirs, (const u4 *)nullptr,
                       (const u4 *)nullptr, w.pos_a, w.dir_a, w.keys_b, two ? (int32_t *)nullptr : user_perm, M, 0, bits0, nblk, w.table,
                       w.totals);
    KN_CHECK_LAUNCH();
    if (two) {
        hipLaunchKernelGGL(k_key_hist, grid, block, 0, st, w.keys_b, M, bits0, (1u << bits1) - 1u, nblk, w.table, (int32_t *)nullptr,
                           (int64_t)0);
        KN_CHECK_LAUNCH();
        hipLaunchKernelGGL(k_digit_scan, dim3(1u << bits1), block, 0, st, w.table, nblk, w.totals);
        KN_CHECK_LAUNCH();
        hipLaunchKernelGGL((k_reorder_scatter<true>), grid, block, stage_bytes, st, w.keys_b, (const float *)nullptr,
                           (const float *)nullptr, w.pos_a, w.dir_a, w.pos_b, w.dir_b, (int32_t *)nullptr, user_perm, M, bits0, bits1,
                           nblk, w.table, w.totals);
        KN_CHECK_LAUNCH();
        sorted_pos = w.pos_b;
        sorted_dir = w.dir_b;
    }
    hipLaunchKernelGGL(k_offsets_tiles, dim3((unsigned)offsets_tiles_blocks(N)), dim3(OT_THREADS), 0, st,
                       (const uint32_t *)sorted_pos + 3, 4, M, N, tile_len, w.offsets, (int32_t *)nullptr, w.counts, user_counts, w.tiles,
                       w.n_tiles);
    KN_CHECK_LAUNCH();
    out->perm = nullptr; // the records are the sorted list
    out->counts = w.counts;
    out->offsets = w.offsets;
    out->tiles = w.tiles;
    out->n_tiles = w.n_tiles;
    records[0] = (const uint32_t *)sorted_pos;
    records[1] = (const uint32_t *)sorted_dir;
    *out4 = w.out4;
    return KN_OK;
}

// ---------------------------------------------------------------------------------------------
// order without passes
namespace {
struct OrderWs {
    int32_t *counts, *n_tiles, *perm, *table;
    uint2 *ranks;
    KnTile *tiles;
};
void carve_order(KnCarver &c, int64_t M, int32_t N, bool stable, OrderWs &w)
{
    w.n_tiles = c.carve<int32_t>(1);
    w.counts = c.carve<int32_t>(N + 1);
    w.ranks = c.carve<uint2>(M);
    w.perm = stable ? nullptr : c.carve<int32_t>(M); // (stable: the caller's)
    w.table = stable ? c.carve<int32_t>(kn_div_up(M, RANK_THREADS) * table_stride(N + 1)) : nullptr;
    w.tiles = c.carve<KnTile>(kn_max_tiles(M, N, 64));
}
int64_t order_ws_bytes(int64_t M, int32_t N, bool stable)
{
    KnCarver c((void *)256, INT64_MAX / 2);
    OrderWs w;
    carve_order(c, M, N, stable, w);
    return c.used;
}
// Every workgroup of k_place scans the counts of all networks, in steps of 1,024, and keeps their starts in LDS.
constexpr int32_t ORDER_MAX_N = 32768;
static_assert(place_lds((ORDER_MAX_N + PLACE_THREADS) / PLACE_THREADS) <= 150 * 1024, "the starts of the networks (k_place) fit the LDS of a compute unit");
constexpr int64_t ORDER_MAX_M = 1 << 18, ORDER_MAX_M_COUNTED = 5 << 15, ORDER_MAX_M_FEW = 3 << 16;
constexpr int32_t ORDER_FEW = PLACE_THREADS - 1, ORDER_STABLE_MAX_N = 24575;
} // namespace

int64_t kn_order_ws_bytes(int64_t M, int32_t N) { return order_ws_bytes(M, N, false); }

// For batches that do not fill the chip with the radix passes' workgroups: four launches instead of nine (six with up to 255
// networks), and kernels of many small workgroups.  The evaluation then gathers its points and scatters its results, which
// costs more than moving the samples does once a batch is far larger than the caches.  65,537 points, fp16, width 32, against the
// radix passes: 16^3 networks 66 us -> 29, 10x16x10 61 -> 28, 5x8x5 39 -> 25; fp32 (10x16x10) 77 -> 35; in random order over two
// cells of 16^3 60 -> 27. Against
// kn_count_run (100,001 / 140,001 / 160,001 / 180,001 / 196,001 points, us): 16^3 networks, fp16, 29 / 31 / 33 / 35 / 38 against 32 / 33 / 34 / 35 / 36,
// bf16, skewed (nine in ten points in a twentieth of the cells) 29 / 33 / 34 / 37 / 38 against 32 / 33 / 33 / 34 / 34, width 64 40 / 45 / 48 / 49 / 52 against
// 44 / 45 / 45 / 48 / 49, 10x16x10 22 / 26 / 27 / 29 / 31 against 26 / 28 / 28 / 29 / 29; fp32, whose tiles and not whose order decide, 160,001 / 220,001 / 260,001
// 51 / 67 / 72 against 53 / 68 / 70; 20^3 (radix passes, 150,001 / 220,001 / 270,001) 47 / 56 / 63 against 75 / 79 / 78.  Networks of one
// step of k_place (112,001 / 140,001 / 163,841 / 180,001 / 196,608): 5x8x5, fp16, 20 / 23 / 24 / 26 / 28 against 22 / 24 / 25 / 25 / 26, skewed 19 / 20 / 21 / 22 / 24
// against 22 / 24 / 25 / 25 / 27; 8^3, bf16, width 64, 22 / 26 / 26 / 27 / 29 against 25 / 29 / 29 / 30 / 31, skewed 23 / 24 / 25 / 27 / 28 against 27 / 28 / 29 / 30 / 30; 10^3, fp16, at
// 163,841 and beyond 27 / 28 / 30 against 27 / 28 / 29, skewed 25 / 26 / 27 against 27 / 28 / 28; fp32, 8^3, 98,305 / 131,072 / 200,001 / 262,144, 30 / 40 / 47 / 62 against
// 34 / 44 / 50 / 64.  Many networks, against the radix passes (28,000 / 65,000 / 260,000 points): 24x20x28, fp16, 50 / 56 /
// 78 against 80 / 83 / 91, skewed 35 / 42 / 76 against 65 / 71 / 89, fp32 94 / 108 / 131 against 119 / 132 / 149; 32^3, fp16, 83 / 110 / 144 against
// 99 / 123 / 152, skewed 57 / 64 / 110 against 72 / 79 / 110, bf16, width 64, 160 / 219 / 308 against 171 / 231 / 317.
bool kn_order_pays(const kn_scene *sc, int64_t M)
{
    const int64_t line = sc->desc.wdtype == KN_F32 ? ORDER_MAX_M : sc->N <= ORDER_FEW ? ORDER_MAX_M_FEW : ORDER_MAX_M_COUNTED;
    return sc->N <= ORDER_MAX_N && (M <= line || (M <= ORDER_MAX_M && !kn_count_pays(M, sc->N)));
}

// The stable order, against the radix passes (3,000 / 40,000 / 260,000 / 550,000 points, us, with the ids, the counts and the permutation): 16^3 networks, fp16,
// 25 / 31 / 47 / 83 against 57 / 66 / 75 / 87, skewed, bf16, 25 / 29 / 48 / 78 against 52 / 65 / 75 / 85; 10x16x10, fp32, 25 / 33 / 64 / 101 (1 M: 155) against
// 59 / 70 / 104 / 137 (186); 2^3, fp16, 24 / 25 / 29 / 49 against 34 / 36 / 48 / 57; 24x20x28, fp16, 38 / 59 / 79 / 120 (400,000: 94) against 61 / 86 / 95 / 105
// (100).  In no more workspace than the passes take, which is the limit for more than some 17,000 networks; 28^3 networks, 1,000 / 4,000 points 42 / 44
// against 51 / 67; 32^3, 200 points (not taken) 53 against 47.
bool kn_order_stable_pays(const kn_scene *sc, int64_t M)
{
    if (sc->N > ORDER_STABLE_MAX_N || order_ws_bytes(M, sc->N, true) > kn_reorder_ws_bytes(M, sc->N)) return false;
    return M <= (sc->N > 8191 ? 3 << 17 : sc->desc.wdtype == KN_F32 ? 1 << 20 : 1 << 19);
}

int kn_order_run(const kn_scene *sc, hipStream_t st, const float *points, int64_t M, int32_t tile_len, int32_t *user_ids,
                 int32_t *user_counts, int32_t *user_perm, float *sigma, float *rgb, KnCarver &ws, KnBucketOut *out, KnStageTimer *tm)
{
    const int32_t N = sc->N;
    if (M < 1 || M > (1ll << 30) || N < 1 || N > ORDER_MAX_N || tile_len < 64 || (tile_len & (tile_len - 1)) != 0) return KN_E_INVALID_ARG;
    OrderWs w;
    carve_order(ws, M, N, user_perm != nullptr, w);
    if (!ws.ok()) return KN_E_WORKSPACE;
    if (!user_perm) KN_TRY(kn_fill_i32(st, w.counts, N + 1, 0));
    const dim3 grid((unsigned)kn_div_up(M, RANK_THREADS)), block(RANK_THREADS);
    hipLaunchKernelGGL(user_perm ? k_rank<true> : k_rank<false>, grid, block, (size_t)(N + 1) * 4, st, points, M, sc->net_grid, sc->cell_net, user_ids, N, w.counts, w.table, w.ranks,
                       sigma, rgb);
    KN_CHECK_LAUNCH();
    if (tm) tm->mark(KN_ST_CELL);
    if (user_perm) {
        hipLaunchKernelGGL(k_table_scan, dim3((unsigned)kn_div_up(N + 1, TS_NETS)), dim3(1024), 0, st, w.table, N + 1, (int32_t)grid.x, w.counts);
        KN_CHECK_LAUNCH();
        w.perm = user_perm;
    }
    const int32_t per = (int32_t)kn_div_up(N + 1, PLACE_THREADS);
    hipLaunchKernelGGL(k_place, dim3((unsigned)kn_div_up(M, PLACE_THREADS * PLACE_POINTS)), dim3(PLACE_THREADS), (size_t)place_lds(per), st,
                       w.ranks, M, N, per, tile_len, w.counts, w.table, w.perm, user_counts, w.tiles, w.n_tiles);
    KN_CHECK_LAUNCH();
    out->perm = w.perm;
    out->counts = w.counts;
    out->offsets = nullptr;
    out->tiles = w.tiles;
    out->n_tiles = w.n_tiles;
    return KN_OK;
}

// ---------------------------------------------------------------------------------------------
// order by counting, samples moved
namespace {
struct CountWs {
    int32_t *n_tiles, *totals, *table;
    uint16_t *keys;
    KnTile *tiles;
    void *pos, *dir; // the samples' halves: 12 bytes each where the results come back, else 16
    uint32_t *at;
    uint16_t *from;
    float *out4;
    int32_t rows, share, nblk;
};
bool count_back(int64_t M, bool fp32) { return M > COUNT_WIDE_M || (!fp32 && M >= COUNT_BACK_M); }
void carve_count(KnCarver &c, int64_t M, int32_t N, bool back, CountWs &w)
{
    w.rows = M > COUNT_WIDE_M ? 8 : 4;
    w.share = (int32_t)(M <= COUNT_FULL_M ? kn_align_up(kn_div_up(M, M <= COUNT_FULL_M / 2 ? 256 : 512), 4) : CO_T * w.rows);
    w.nblk = (int32_t)kn_div_up(M, w.share);
    w.n_tiles = c.carve<int32_t>(1);
    w.totals = c.carve<int32_t>(N + 1);
    w.table = c.carve<int32_t>(w.nblk * table_stride(N + 1));
    w.keys = c.carve<uint16_t>(M);
    w.tiles = c.carve<KnTile>(kn_max_tiles(M, N, 64));
    const int64_t words = (back ? 3 : 4) * M;
    w.pos = c.carve<float>(words);
    w.dir = c.carve<float>(words);
    w.at = back ? c.carve<uint32_t>(M) : nullptr;
    w.from = back ? c.carve<uint16_t>(M) : nullptr;
    w.out4 = c.carve<float>(4 * M);
}
int64_t count_bytes(int64_t M, int32_t N)
{
    KnCarver c((void *)256, INT64_MAX / 2);
    CountWs w;
    carve_count(c, M, N, count_back(M, true), w); // (the two ways differ in 2 bytes per point; the larger one)
    return c.used;
}
} // namespace

// (in no more workspace than the passes take: the table is the larger part of it for many networks and few points)
bool kn_count_pays(int64_t M, int32_t N) { return N <= COUNT_MAX_N && M >= COUNT_MIN_M && count_bytes(M, N) <= kn_reorder_ws_bytes(M, N); }

int64_t kn_count_ws_bytes(int64_t M, int32_t N) { return kn_count_pays(M, N) ? count_bytes(M, N) : 0; }

int kn_count_run(const kn_scene *sc, hipStream_t st, const float *points, const float *dirs, int64_t M, int32_t tile_len,
                 int32_t *user_ids, int32_t *user_counts, KnCarver &ws, KnBucketOut *out, KnSampleSrc *src, KnCountBack *back,
                 KnStageTimer *tm)
{
    const int32_t N = sc->N;
    if (!kn_count_pays(M, N) || M > (1ll << 30) || tile_len < 64 || (tile_len & (tile_len - 1)) != 0) return KN_E_INVALID_ARG;
    CountWs w;
    carve_count(ws, M, N, count_back(M, sc->desc.wdtype == KN_F32), w);
    if (!ws.ok()) return KN_E_WORKSPACE;
    const dim3 grid((unsigned)w.nblk), block(CO_T);
    const size_t bins = (size_t)(N + 1) * 4;
    auto count = w.rows == 8 ? k_keys_count<8> : k_keys_count<4>;
    auto scatter = w.rows == 8 ? k_count_scatter<8, true> : w.at ? k_count_scatter<4, true> : k_count_scatter<4, false>;
    hipLaunchKernelGGL(count, grid, block, bins, st, points, M, sc->net_grid, sc->cell_net, user_ids, w.keys, N, w.nblk, w.share, w.table);
    KN_CHECK_LAUNCH();
    if (tm) tm->mark(KN_ST_CELL);
    hipLaunchKernelGGL(k_table_scan, dim3((unsigned)kn_div_up(N + 1, TS_NETS)), dim3(1024), 0, st, w.table, N + 1, w.nblk, w.totals);
    KN_CHECK_LAUNCH();
    hipLaunchKernelGGL(scatter, grid, block, (size_t)CO_T * w.rows * sizeof(u4) + bins, st, w.keys, points, dirs, w.pos, w.dir, M, N,
                       w.nblk, w.share, w.table, w.totals, tile_len, user_counts, w.tiles, w.n_tiles, w.at, w.from, w.out4);
    KN_CHECK_LAUNCH();
    out->perm = nullptr; // the records are the sorted list
    out->counts = w.totals;
    out->offsets = nullptr;
    out->tiles = w.tiles;
    out->n_tiles = w.n_tiles;
    if (w.at) {
        src->points = (const float *)w.pos;
        src->dirs = (const float *)w.dir;
    } else {
        src->records = (const uint32_t *)w.pos;
        src->records_dir = (const uint32_t *)w.dir;
    }
    src->out4 = w.out4;
    *back = KnCountBack{w.out4, w.at, w.from, w.nblk, w.rows, w.share};
    return KN_OK;
}

int kn_count_results(hipStream_t st, const KnCountBack &back, int64_t M, float *sigma, float *rgb)
{
    if (!back.at) return kn_reorder_split_results(st, back.out4, M, sigma, rgb);
    auto kernel = back.rows == 8 ? k_results_back<8> : k_results_back<4>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)back.nblk), dim3(CO_T), (size_t)CO_T * back.rows * sizeof(u4), st, back.out4, back.at,
                       back.from, M, back.nblk, back.share, sigma, rgb);
    KN_CHECK_LAUNCH();
    return KN_OK;
}

// ---------------------------------------------------------------------------------------------
// index sort
namespace {
struct BucketWs {
    int32_t *keys_b, *vals_a, *vals_b, *table, *totals, *n_tiles, *counts, *offsets;
    KnTile *tiles;
    int64_t nblk;
};
void carve_bucket(KnCarver &c, int64_t M, int32_t N, BucketWs &w)
{
    w.nblk = kn_div_up(M > 0 ? M : 1, RO_TILE);
    w.n_tiles = c.carve<int32_t>(1);
    w.table = c.carve<int32_t>(256 * w.nblk);
    w.totals = c.carve<int32_t>(256);
    w.keys_b = c.carve<int32_t>(M);
    w.vals_a = c.carve<int32_t>(M);
    w.vals_b = c.carve<int32_t>(M);
    w.counts = c.carve<int32_t>(N + 1);
    w.offsets = c.carve<int32_t>(N + 2);
    w.tiles = c.carve<KnTile>(kn_max_tiles(M, N, 64));
}
} // namespace

int64_t kn_bucket_ws_bytes(int64_t M, int32_t N)
{
    KnCarver c((void *)256, INT64_MAX / 2);
    BucketWs w;
    carve_bucket(c, M, N, w);
    return c.used;
}

int kn_bucket_run(hipStream_t st, int32_t *keys, int64_t M, int32_t N, int32_t tile_len, int32_t *user_counts, int32_t *user_offsets,
                  int32_t *user_perm, KnCarver &ws, KnBucketOut *out)
{
    if (M < 0 || M > (1ll << 30) || N < 1 || N > 65535 || tile_len < 64) return KN_E_INVALID_ARG;
    BucketWs w;
    carve_bucket(ws, M, N, w);
    if (!ws.ok()) return KN_E_WORKSPACE;
    const int bits = key_bits(N);
    const bool two = bits > 8;
    const int bits0 = two ? bits / 2 : bits, bits1 = bits - bits0;
    const int32_t nblk = (int32_t)w.nblk;
    const dim3 grid((unsigned)nblk), block(RO_THREADS);
    const int32_t *sorted_keys = keys;
    const int32_t *perm = w.vals_a;
    // the first kernel clears the tile counter (with no keys there are no passes: a fill does it)
    if (M == 0) KN_TRY(kn_fill_i32(st, w.n_tiles, 1, 0));
    if (M > 0) {
        hipLaunchKernelGGL(k_key_hist, grid, block, 0, st, keys, M, 0, (1u << bits0) - 1u, nblk, w.table, w.n_tiles, (int64_t)1);
        KN_CHECK_LAUNCH();
        hipLaunchKernelGGL(k_digit_scan, dim3(1u << bits0), block, 0, st, w.table, nblk, w.totals);
        KN_CHECK_LAUNCH();
        int32_t *v1 = (!two && user_perm) ? user_perm : w.vals_a;
        hipLaunchKernelGGL(k_index_scatter, grid, block, 0, st, keys, (const int32_t *)nullptr, w.keys_b, v1, M, 0, bits0, nblk, w.table,
                           w.totals);
        KN_CHECK_LAUNCH();
        sorted_keys = w.keys_b;
        perm = v1;
        if (two) {
            hipLaunchKernelGGL(k_key_hist, grid, block, 0, st, w.keys_b, M, bits0, (1u << bits1) - 1u, nblk, w.table, (int32_t *)nullptr,
                               (int64_t)0);
            KN_CHECK_LAUNCH();
            hipLaunchKernelGGL(k_digit_scan, dim3(1u << bits1), block, 0, st, w.table, nblk, w.totals);
            KN_CHECK_LAUNCH();
            int32_t *v2 = user_perm ? user_perm : w.vals_b;
            // (the caller's key array is free by now: it takes the keys in final order)
            hipLaunchKernelGGL(k_index_scatter, grid, block, 0, st, w.keys_b, v1, keys, v2, M, bits0, bits1, nblk, w.table, w.totals);
            KN_CHECK_LAUNCH();
            sorted_keys = keys;
            perm = v2;
        }
    }
    hipLaunchKernelGGL(k_offsets_tiles, dim3((unsigned)offsets_tiles_blocks(N)), dim3(OT_THREADS), 0, st,
                       (const uint32_t *)sorted_keys, 1, M, N, tile_len, w.offsets, user_offsets, w.counts, user_counts, w.tiles, w.n_tiles);
    KN_CHECK_LAUNCH();
    out->perm = perm;
    out->counts = w.counts;
    out->offsets = w.offsets;
    out->tiles = w.tiles;
    out->n_tiles = w.n_tiles;
    return KN_OK;
}

int kn_reorder_split_results(hipStream_t st, const float *out4, int64_t M, float *sigma, float *rgb)
{
    hipLaunchKernelGGL(k_split_results, dim3((unsigned)kn_div_up(kn_div_up(M, 4), 256)), dim3(256), 0, st, out4, M, sigma, rgb);
    KN_CHECK_LAUNCH();
    return KN_OK;
}

// the scatter's staging buffer is above the default limit of dynamic LDS (once per device, from kn_create)
int kn_reorder_configure()
{
    const int bytes = (int)(RO_TILE * sizeof(u4));
    KN_HIP(hipFuncSetAttribute((const void *)k_reorder_scatter<false>, hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
    KN_HIP(hipFuncSetAttribute((const void *)k_reorder_scatter<true>, hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
    const int counts = (COUNT_MAX_N + 1) * 4;
    KN_HIP(hipFuncSetAttribute((const void *)k_rank<false>, hipFuncAttributeMaxDynamicSharedMemorySize, (ORDER_MAX_N + 1) * 4));
    KN_HIP(hipFuncSetAttribute((const void *)k_rank<true>, hipFuncAttributeMaxDynamicSharedMemorySize, (ORDER_MAX_N + 1) * 4));
    KN_HIP(hipFuncSetAttribute((const void *)k_place, hipFuncAttributeMaxDynamicSharedMemorySize,
                               place_lds((int)kn_div_up(ORDER_MAX_N + 1, PLACE_THREADS))));
    constexpr int half = CO_T * 4 * 16, full = CO_T * 8 * 16;
    KN_HIP(hipFuncSetAttribute((const void *)k_results_back<4>, hipFuncAttributeMaxDynamicSharedMemorySize, half));
    KN_HIP(hipFuncSetAttribute((const void *)k_results_back<8>, hipFuncAttributeMaxDynamicSharedMemorySize, full));
    KN_HIP(hipFuncSetAttribute((const void *)k_count_scatter<4, false>, hipFuncAttributeMaxDynamicSharedMemorySize, half + counts));
    KN_HIP(hipFuncSetAttribute((const void *)k_count_scatter<4, true>, hipFuncAttributeMaxDynamicSharedMemorySize, half + counts));
    KN_HIP(hipFuncSetAttribute((const void *)k_count_scatter<8, true>, hipFuncAttributeMaxDynamicSharedMemorySize, full + counts));
    return KN_OK;
}
