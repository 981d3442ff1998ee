// Interface between kn_render (kn_render.hip), which prepares a frame, and the kernel that renders it (kn_fused.hip).
#pragma once

#include "kn_common.h"

constexpr int KN_FUSED_CTL = 8; // control words of a frame: live rays, rays handed out beyond the first pools, -, -, two 64-bit counters

constexpr int64_t KN_FUSED_OWN_RAYS = 32767; // frames of up to so many rays need no list

struct KnFusedJob {
    const void *march; // MarchParams of the call (kn_march.h)
    const float *rays_o, *rays_d;
    int64_t R;
    const int4 *list;  // live rays (ray, first lattice index, end of the clipped range, -), ctl[0] of them; nullptr: the kernel sets the rays up itself
    int32_t *ctl;      // KN_FUSED_CTL words, zero behind the first
    float eps;
    const float *bg;
    float *rgb_out;
    unsigned long long *counters; // nullable
    bool strat;
};
int kn_fused_configure(); // once per device
int kn_fused_f32_configure();
bool kn_fused_supports(const kn_scene *sc);
int kn_fused_launch(const kn_scene *sc, hipStream_t st, const KnFusedJob &job, hipEvent_t ev_start, hipEvent_t ev_stop);
int kn_fused_f32_launch(const kn_scene *sc, hipStream_t st, const KnFusedJob &job, hipEvent_t ev_start, hipEvent_t ev_stop);
