// Adjoint (reverse-mode) rollout: gradients of each candidate's cost J with
// respect to its control sequence, for gradient refinement of the best
// sampled candidates.
//
// The paper samples because its vehicle model is not analytically
// differentiable (section on the state of the art, and section "Real-Time
// Implementation"); the discretised model used here is differentiable almost
// everywhere, so this file differentiates exactly what the forward kernel
// computes. Conventions at the non-smooth points:
//   * max(a, b) and the clamps pass the gradient to the branch the forward
//     pass took (ties to the first argument / the unclamped value);
//   * the damper's switch at liftoff, the bilinear cell edges, |phi| at 0 and
//     the ESM sign change use the active branch's derivative;
//   * the goal test fixes the exit step: steps after it carry no gradient and
//     the exit time is not differentiated.
//
// Memory: states are checkpointed every C control intervals during the
// forward pass; the backward pass recomputes one segment at a time into a
// [C*S][14][M] scratch (13 state components plus an executed flag) and runs
// the step adjoints in reverse. One lane per candidate (LANES = 1 step code,
// the same arithmetic as the forward kernel).
// Launches of few candidates take adjoint_linear.hip instead.
#include "adjoint_step.h"

namespace plan {
namespace {

// Backward pass over checkpointed segments; LANES lanes per candidate, the
// wheels split over them as in the forward kernel.
//   ckpt:    [nseg+1][13][K]: state at the start of each segment of C
//            intervals (segment nseg: the final state)
//   weight:  [K] dJ/dJ_k seeds (NULL = 1)
//   cost:    [K] the forward costs (+inf rows get zero gradients)
//   scratch: [C*S][14][K] recomputed states plus an executed flag (every
//            lane of a group writes and reads back the same values)
//   grad:    [N][2][K] output dJ/du
template <int LANES>
__global__ __launch_bounds__(64) void adjoint_backward(const RolloutArgs a, int C,
                                                       const float *__restrict__ ckpt,
                                                       const float *__restrict__ weight,
                                                       float *__restrict__ scratch,
                                                       float *__restrict__ grad) {
    constexpr int WPL = 4 / LANES;
    const int gtid = blockIdx.x * 64 + threadIdx.x;
    const int sub = gtid & (LANES - 1);
    const int k = gtid / LANES;
    // whole lane groups past K leave together (64 is a multiple of LANES)
    if (k >= a.K) return;
    const size_t K = (size_t)a.K;
    const int N = a.N, S = a.S;
    const int nseg = (N + C - 1) / C;
    const float wJ = weight ? weight[k] : 1.0f;
    const float Jk = a.cost[k];
    const float *up = a.controls + k;
    if (!isfinite(Jk)) {
        if (sub == 0)
            for (int e = 0; e < 2 * N; ++e) grad[(size_t)e * K + k] = 0.0f;
        return;
    }
    // terminal cost Phi = w_g |(x, y) - goal| at the final state
    float lam[13];
#pragma unroll
    for (int q = 0; q < 13; ++q) lam[q] = 0.0f;
    {
        const float xf = ckpt[((size_t)nseg * 13 + 0) * K + k];
        const float yf = ckpt[((size_t)nseg * 13 + 1) * K + k];
        const float gdx = xf - a.goal_x, gdy = yf - a.goal_y;
        const float dist = sqrtf(fmaf(gdx, gdx, gdy * gdy));
        if (dist > 0.0f) {
            lam[0] = wJ * a.w_g * gdx / dist;
            lam[1] = wJ * a.w_g * gdy / dist;
        }
    }
    Arm arms[WPL];
#pragma unroll
    for (int q = 0; q < WPL; ++q) arms[q] = arm(a, sub * WPL + q);

    // Loads are issued one step ahead from inside the step (after its terrain
    // requests): the next interval's controls in the recomputation, the
    // previous step's recomputed state and controls in the reverse sweep.
    // Indices are clamped to the segment, so every load stays in bounds.
    for (int seg = nseg - 1; seg >= 0; --seg) {
        const int n0 = seg * C;
        const int n1 = min(N, n0 + C);
        // recompute the segment's states
        float st[13];
#pragma unroll
        for (int q = 0; q < 13; ++q) st[q] = ckpt[((size_t)seg * 13 + q) * K + k];
        float Jdummy = 0.0f;
        int idx = 0;
        float nu0 = up[(2 * (size_t)n0) * K], nu1 = up[(2 * (size_t)n0 + 1) * K];
        for (int n = n0; n < n1; ++n) {
            const float dd = clampf_nan(nu0, -a.drate_max, a.drate_max);
            const float ax = a.accel_max * clampf_nan(nu1, -1.0f, 1.0f);
            const size_t nn = (size_t)min(n + 1, n1 - 1);
            for (int s = 0; s < S; ++s, ++idx) {
                float *sl = scratch + ((size_t)idx * 14) * K + k;
#pragma unroll
                for (int q = 0; q < 13; ++q) sl[(size_t)q * K] = st[q];
                const float gdx = st[0] - a.goal_x, gdy = st[1] - a.goal_y;
                const bool live = !(fmaf(gdx, gdx, gdy * gdy) <= a.goal_r2);
                sl[(size_t)13 * K] = live ? 1.0f : 0.0f;
                // a step that is not live leaves the state frozen, so no later
                // step of this candidate is live and the stale controls are
                // never applied
                if (live)
                    euler_step<LANES>(a, arms, st, Jdummy, dd, ax, [&]() {
                        nu0 = up[(2 * nn) * K];
                        nu1 = up[(2 * nn + 1) * K];
                    });
            }
        }
        // reverse through the segment, one step at a time (flat index i)
        const int cnt = (n1 - n0) * S;
        float cur[14];
        {
            const float *sl = scratch + ((size_t)(cnt - 1) * 14) * K + k;
#pragma unroll
            for (int q = 0; q < 14; ++q) cur[q] = sl[(size_t)q * K];
        }
        float cu0 = up[(2 * (size_t)(n1 - 1)) * K], cu1 = up[(2 * (size_t)(n1 - 1) + 1) * K];
        float gdd = 0.0f, gax = 0.0f;
        // (n, s): interval and substep of flat index i, stepped down with i
        // (no divisions in the loop)
        int n = n1 - 1, s = S - 1;
        for (int i = cnt - 1; i >= 0; --i) {
            const float u0 = cu0, u1 = cu1;
            const float dd = clampf_nan(u0, -a.drate_max, a.drate_max);
            const float ax = a.accel_max * clampf_nan(u1, -1.0f, 1.0f);
            const int ip = max(i - 1, 0);
            const size_t np = (size_t)(i == 0 ? n0 : (s > 0 ? n : n - 1));
            const float *slp = scratch + ((size_t)ip * 14) * K + k;
            float nxt[14], nu0, nu1;
            auto prefetch = [&]() {
#pragma unroll
                for (int q = 0; q < 14; ++q) nxt[q] = slp[(size_t)q * K];
                nu0 = up[(2 * np) * K];
                nu1 = up[(2 * np + 1) * K];
            };
            if (cur[13] != 0.0f) {  // executed (not after the goal exit)
                float sti[13];
#pragma unroll
                for (int q = 0; q < 13; ++q) sti[q] = cur[q];
                float g1, g2;
                step_vjp<LANES>(a, arms, sti, dd, ax, wJ, lam, &g1, &g2, prefetch);
                gdd += g1;
                gax += g2;
            } else {
                prefetch();
            }
            if (s == 0) {
                // first substep of interval n: its gradient is complete;
                // through the admissible-set clamps (identity branch inside)
                const bool in0 = !(u0 < -a.drate_max) && !(u0 > a.drate_max);
                const bool in1 = !(u1 < -1.0f) && !(u1 > 1.0f);
                if (sub == 0) {
                    grad[(2 * (size_t)n) * K + k] = in0 ? gdd : 0.0f;
                    grad[(2 * (size_t)n + 1) * K + k] = in1 ? a.accel_max * gax : 0.0f;
                }
                gdd = 0.0f;
                gax = 0.0f;
            }
#pragma unroll
            for (int q = 0; q < 14; ++q) cur[q] = nxt[q];
            cu0 = nu0;
            cu1 = nu1;
            if (s == 0) {
                s = S - 1;
                --n;
            } else {
                --s;
            }
        }
    }
}

}  // namespace

hipError_t launch_adjoint_backward(const RolloutArgs &a, int C, const float *ckpt,
                                   const float *weight, float *scratch, float *grad, int lanes,
                                   hipStream_t s) {
    const unsigned grid = (unsigned)(((long long)a.K * lanes + 63) / 64);
    if (lanes == 1)
        hipLaunchKernelGGL(adjoint_backward<1>, dim3(grid), dim3(64), 0, s, a, C, ckpt, weight,
                           scratch, grad);
    else if (lanes == 2)
        hipLaunchKernelGGL(adjoint_backward<2>, dim3(grid), dim3(64), 0, s, a, C, ckpt, weight,
                           scratch, grad);
    else if (lanes == 4)
        hipLaunchKernelGGL(adjoint_backward<4>, dim3(grid), dim3(64), 0, s, a, C, ckpt, weight,
                           scratch, grad);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace plan
