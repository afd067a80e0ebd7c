// Two- and four-lane instantiations of the rollout kernels (see
// rollout_kernels.h) for launches of at most one wave per SIMD with one Euler
// step per interval: each node's terrain is requested a whole step ahead and
// the controls a trip of four intervals ahead; Runge-Kutta's stages request
// their terrain one stage ahead.
#define PLAN_REQUEST_AHEAD 1
#include "rollout_kernels.h"

namespace plan {
namespace {

template <int L, bool CHUNK, bool SAMPLED, bool FUSED>
hipError_t launch_lanes(const RolloutArgs &a, int block, hipStream_t s) {
    const unsigned grid = (unsigned)(((long long)a.K * L + block - 1) / block);
#define PLAN_LAUNCH(B, CMAP)                                                                    \
    if (block == B && (a.has_costmap != 0) == CMAP) {                                           \
        hipLaunchKernelGGL((rollout_srb<L, B, CHUNK, SAMPLED, FUSED, false, false, true, CMAP>), \
                           dim3(grid), dim3(B), 0, s, a);                                       \
        return hipGetLastError();                                                               \
    }
    PLAN_LAUNCH(64, false)
    PLAN_LAUNCH(64, true)
    PLAN_LAUNCH(256, false)
    PLAN_LAUNCH(256, true)
#undef PLAN_LAUNCH
    return hipErrorInvalidValue;
}

template <int L, bool CHUNK>
hipError_t launch_rk4(const RolloutArgs &a, int block, hipStream_t s) {
    const unsigned grid = (unsigned)(((long long)a.K * L + block - 1) / block);
#define PLAN_LAUNCH(B, CMAP)                                                                   \
    if (block == B && (a.has_costmap != 0) == CMAP) {                                          \
        hipLaunchKernelGGL((rollout_srb<L, B, CHUNK, false, false, true, false, false, CMAP>),  \
                           dim3(grid), dim3(B), 0, s, a);                                      \
        return hipGetLastError();                                                              \
    }
    PLAN_LAUNCH(64, false)
    PLAN_LAUNCH(64, true)
    PLAN_LAUNCH(256, false)
    PLAN_LAUNCH(256, true)
#undef PLAN_LAUNCH
    return hipErrorInvalidValue;
}

template <bool CHUNK, bool SAMPLED, bool FUSED>
hipError_t launch_any(const RolloutArgs &a, int lanes, int block, hipStream_t s) {
    if (a.S != 1 || a.method != 0) return hipErrorInvalidValue;
    if (lanes == 2) return launch_lanes<2, CHUNK, SAMPLED, FUSED>(a, block, s);
    if (lanes == 4) return launch_lanes<4, CHUNK, SAMPLED, FUSED>(a, block, s);
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_rollout_multi_1wave(const RolloutArgs &a, int lanes, int block, bool chunk,
                                      hipStream_t s) {
    if (a.method == 1 && lanes == 2)
        return chunk ? launch_rk4<2, true>(a, block, s) : launch_rk4<2, false>(a, block, s);
    if (a.method == 1 && lanes == 4)
        return chunk ? launch_rk4<4, true>(a, block, s) : launch_rk4<4, false>(a, block, s);
    return chunk ? launch_any<true, false, false>(a, lanes, block, s)
                 : launch_any<false, false, false>(a, lanes, block, s);
}

hipError_t launch_sampled_multi_1wave(const RolloutArgs &a, int lanes, int block, hipStream_t s) {
    return launch_any<false, true, false>(a, lanes, block, s);
}

hipError_t launch_argmin_multi_1wave(const RolloutArgs &a, int lanes, int block, bool sampled,
                                     hipStream_t s) {
    return sampled ? launch_any<false, true, true>(a, lanes, block, s)
                   : launch_any<false, false, true>(a, lanes, block, s);
}

hipError_t launch_ckpt_multi_1wave(const RolloutArgs &a, int lanes, int block, hipStream_t s) {
    const unsigned grid = (unsigned)(((long long)a.K * lanes + block - 1) / block);
#define PLAN_LAUNCH(L, B, CMAP)                                                                 \
    if (lanes == L && block == B && (a.has_costmap != 0) == CMAP) {                             \
        hipLaunchKernelGGL((rollout_srb<L, B, false, false, false, false, true, true, CMAP>),    \
                           dim3(grid), dim3(B), 0, s, a);                                       \
        return hipGetLastError();                                                               \
    }
    PLAN_LAUNCH(2, 64, false)
    PLAN_LAUNCH(2, 64, true)
    PLAN_LAUNCH(2, 256, false)
    PLAN_LAUNCH(2, 256, true)
    PLAN_LAUNCH(4, 64, false)
    PLAN_LAUNCH(4, 64, true)
    PLAN_LAUNCH(4, 256, false)
    PLAN_LAUNCH(4, 256, true)
#undef PLAN_LAUNCH
    return hipErrorInvalidValue;
}

// A tick of so few waves takes workgroups of 64.
hipError_t launch_slots_multi_1wave(const RolloutArgs *slots, const TickTable &t, int *bad,
                                    SelectOut *ring, uint32_t seq, int lanes, int block,
                                    hipStream_t s) {
    const unsigned grid = (unsigned)t.total_blocks;
#define PLAN_LAUNCH(L, CMAP)                                                                  \
    if (lanes == L && block == 64 && (t.costmap != 0) == CMAP) {                              \
        hipLaunchKernelGGL((rollout_slots<L, 64, true, CMAP>), dim3(grid), dim3(64), 0, s,    \
                           slots, t, bad, ring, seq);                                         \
        return hipGetLastError();                                                             \
    }
    PLAN_LAUNCH(2, false)
    PLAN_LAUNCH(2, true)
    PLAN_LAUNCH(4, false)
    PLAN_LAUNCH(4, true)
#undef PLAN_LAUNCH
    return hipErrorInvalidValue;
}

}  // namespace plan
