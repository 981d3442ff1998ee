// Evaluation of small batches in the caller's order (kn_direct.hip; the fp32 kernel is in kn_mlp_f32.hip).
#pragma once

#include "kn_common.h"

#include <hip/hip_ext.h>
#include <math.h>

struct KnDirectJob {
    KnGrid net;
    const int32_t *cell_net;
    const float *points, *dirs;
    int64_t M;
    int32_t lg_points; // a wavefront takes 1 << lg_points consecutive points (at most 64)
    int32_t *ids;      // nullable
    float *sigma, *rgb;
};

// -1: the batch is better ordered by network first; else KnDirectJob::lg_points
int kn_direct_lg_points(const kn_scene *sc, int64_t M);
int kn_direct_launch(const kn_scene *sc, hipStream_t st, const KnDirectJob &job, hipEvent_t ev_start, hipEvent_t ev_stop);
int kn_direct_f32_launch(const kn_scene *sc, hipStream_t st, const KnDirectJob &job, unsigned blocks, hipEvent_t ev_start,
                         hipEvent_t ev_stop);

struct KnDirectPoint {
    float p[3], d[3];
    int32_t net; // -1: none
};

// The lane's point of the wavefront's share and its network (Eq. 6; the id is written out, and zero results of a point
// without a network); returns the lanes that have one.
__device__ __forceinline__ unsigned long long kn_direct_point(const KnDirectJob &job, int64_t first, int lane, KnDirectPoint &pt)
{
    const int64_t i = first + lane;
    const bool mine = lane < (1 << job.lg_points) && i < job.M;
    const int64_t at = 3 * (mine ? i : job.M - 1);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        pt.p[c] = job.points[at + c];
        pt.d[c] = job.dirs[at + c];
    }
    pt.net = kn_net_of_cell(job.cell_net, kn_grid_index(job.net, pt.p[0], pt.p[1], pt.p[2]));
    if (!mine) pt.net = -1;
    if (mine && job.ids) job.ids[i] = pt.net;
    if (mine && pt.net < 0) {
        job.sigma[i] = 0.0f;
        job.rgb[3 * i] = job.rgb[3 * i + 1] = job.rgb[3 * i + 2] = 0.0f;
    }
    return __ballot(pt.net >= 0);
}
