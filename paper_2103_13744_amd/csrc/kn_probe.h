// Occupancy grid extraction (Sec. 3.4, "Empty Space Skipping"): the work, as all its kernels see it.
//
// Every voxel of the grid being filled is probed at the 27 sub-cell centres of a 3x3x3 subgrid,
// x = bmin + (v + c) * cell per axis with c in {1/6, 1/2, 5/6}, evaluated as fmaf((float)v + c, cell, bmin); the voxel
// is marked iff any probe's density is above tau.  A probe is evaluated by the network of the cell it lies in
// (Eq. 6).  Probe i = 3 v + s of an axis (s-th sub-cell centre of voxel v) sits at kn_probe_coord, whatever the other
// axes' probes are, and Eq. 6 is per axis as well: the probes of axis a that lie in network cell c are those from the first
// of cell c to the first of cell c + 1 (positions and Eq. 6 are non-decreasing in i), and the probes of a cell are the box of
// its three ranges, all of one network, whether or not the grids nest.
#pragma once

#include "kn_common.h"

struct KnProbeJob {
    KnGrid occ;              // the grid being filled
    int32_t net_res[3];      // the network grid
    int32_t per[3];          // occ.res / net_res (six divisions per wavefront took 5 of 54 us where a cell has eight probes, 24^3 of them)
    const int32_t *cell_net; // device, sparse network grids: cell -> network or -1; nullptr on a dense grid
    const int32_t *first[3]; // device, net_res[a] + 1 entries per axis: first probe of a cell, counted from kn_probe_base
    int32_t parts;           // workgroups per network cell
    int32_t sub[3], waves;   // fp32 kernel: probes per axis that a workgroup takes together, at most; its wavefronts
    float tau;
    uint8_t *occupancy;      // device, occ.res[0]*[1]*[2] bytes, zero before the launch
};

constexpr int KN_PROBES = 27;
// Largest number of voxels one network cell may own: keeps a cell's probe numbers inside int32.
constexpr int64_t KN_PROBE_MAX_BOX = 0x7fffffff / KN_PROBES - 64;

// near the first probe of network cell c (an axis has up to 3 (2^31 - 1) probes; the distance from here fits 32 bits)
__host__ __device__ __forceinline__ int64_t kn_probe_base(int32_t per, int32_t c) { return 3 * ((int64_t)c * per); }

// probe i of the axis, counted from the first one of voxel v0 (i >= 0)
__device__ __forceinline__ float kn_probe_coord(float cell, float bmin, int32_t v0, int32_t i)
{
    const int32_t v = (int32_t)((uint32_t)i / 3u), s = i - 3 * v;
    return fmaf((float)(v0 + v) + (s == 0 ? 1.0f / 6.0f : (s == 1 ? 0.5f : 5.0f / 6.0f)), cell, bmin);
}
__device__ __forceinline__ float kn_probe_coord(const KnGrid &occ, int axis, int32_t v0, int32_t i)
{
    return kn_probe_coord(occ.cell[axis], occ.bmin[axis], v0, i);
}

// The probes of a network cell: p0[a] .. p1[a] - 1 per axis, counted from the first one of voxel v0[a].  All values uniform.
struct KnProbeBox {
    int32_t v0[3], p0[3], p1[3];
};
// false: the cell holds no probe
__device__ __forceinline__ bool kn_probe_box(const KnProbeJob &job, int32_t cell, KnProbeBox &b)
{
    const int32_t q = cell / job.net_res[2], c[3] = {q / job.net_res[1], q % job.net_res[1], cell % job.net_res[2]};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int64_t lo = kn_probe_base(job.per[a], c[a]) + job.first[a][c[a]];
        const int64_t hi = kn_probe_base(job.per[a], c[a] + 1) + job.first[a][c[a] + 1];
        if (lo >= hi) return false;
        b.v0[a] = __builtin_amdgcn_readfirstlane((int32_t)((uint64_t)lo / 3u));
        b.p0[a] = __builtin_amdgcn_readfirstlane((int32_t)(lo - 3 * (int64_t)b.v0[a]));
        b.p1[a] = __builtin_amdgcn_readfirstlane((int32_t)(hi - 3 * (int64_t)b.v0[a]));
    }
    return true;
}
