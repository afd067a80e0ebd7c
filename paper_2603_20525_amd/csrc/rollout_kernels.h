// Rollout kernel templates (SRB model, stage cost, ESM constraint) and, per
// lane count, their launch dispatch. Four translation units instantiate
// them: rollout.hip (one lane per candidate) and rollout_multilane.hip (two
// and four lanes per candidate), and rollout_onelane_1wave.hip and
// rollout_multilane_1wave.hip for launches of at most one wave per SIMD. The
// arithmetic is the same in all, so results are identical for every launch
// shape.
#pragma once

#include "plan_internal.h"
#include "rollout_step.h"
#include "select_common.h"

namespace plan {
namespace {

// The kernels built with PLAN_REQUEST_AHEAD (rollout_onelane_1wave.hip and
// rollout_multilane_1wave.hip: launches of at most one wave per SIMD) have
// registers to spare: their Euler kernels with one substep per interval
// request each node's terrain a whole step ahead (euler_step_ahead), which
// holds two nodes' cell coefficients in registers at once. The kernels for
// more waves per SIMD need the registers for occupancy and hide the gathers
// behind each other's arithmetic.
#ifdef PLAN_REQUEST_AHEAD
constexpr bool REQUEST_AHEAD = true;
#else
constexpr bool REQUEST_AHEAD = false;
#endif

// One candidate k over control intervals [a.n0, a.n1), simulated by the
// LANES lanes of its group (this lane is number sub). CHUNK: start from and
// write back a.state / a.cost; otherwise start from a.s0 with zero cost and
// write a.cost / a.final_state. SAMPLED: draw the controls from a.smp (one
// generator block per four intervals, kept in registers) instead of reading
// a.controls. Lanes with store == false run a duplicate candidate only to
// keep their lane group complete.
template <int LANES, bool CHUNK, bool SAMPLED = false, bool RK4 = false, bool CKPT = false,
          bool S1 = false, bool CM = true>
__device__ __forceinline__ float simulate(const RolloutArgs &a, int k, int sub, bool store,
                                          const float *up) {
    constexpr int WPL = 4 / LANES;  // wheels per lane
    constexpr bool AHEAD = REQUEST_AHEAD && !RK4 && S1 && (!CKPT || LANES > 1);
    constexpr bool TRIPS = AHEAD && LANES > 1;  // the loop of four-interval trips below
    constexpr bool RK4_AHEAD = REQUEST_AHEAD && RK4 && LANES > 1;
    const size_t K = (size_t)a.K;

    float st0[13];
    float J;
    if constexpr (CHUNK) {
#pragma unroll
        for (int q = 0; q < 13; ++q) st0[q] = a.state[(size_t)q * K + k];
        J = a.cost[k];
    } else {
#pragma unroll
        for (int q = 0; q < 13; ++q) st0[q] = a.s0[q];
        J = 0.0f;
    }
    float (&st)[13] = st0;

    // materialised controls are read one interval ahead (the index is clamped
    // to [n0, n1)). The Euler step requests the next pair right after its
    // terrain gathers, so waiting for the texels does not wait for it and the
    // load stays in flight for the rest of the step; RK4 requests it at the
    // start of the interval.
    // up: this candidate's control column (interval n at up[2 n K], up[(2 n + 1) K])
    float nu0 = 0.0f, nu1 = 0.0f;
    // the pair requested during interval n: interval min(n + 1, n1 - 1)
    const float *unext = up + 2 * (size_t)max(min(a.n0 + 1, a.n1 - 1), 0) * K;
    if constexpr (!SAMPLED && !TRIPS) {
        if (a.n0 < a.n1) {
            nu0 = up[(2 * (size_t)a.n0) * K];
            nu1 = up[(2 * (size_t)a.n0 + 1) * K];
        }
    }
    PhiloxBlock blk{};
    int blk_n = -1;

    // SAMPLED at several lanes per candidate: a generator block and its four
    // draws cost more than a third of a step, so each lane of the group makes
    // a different block, and an interval's pair comes from the lane that has it
    // (drawn from intervals base .. base + 4 LANES - 1, lane i's the four from
    // base + 4 i), restricted to the admissible set there. Gaussian draws,
    // 12 000 x 60 at two lanes with a costmap: 74.9 -> 49.8 us (with the trips
    // below)
    float du0[4], du1[4];
    auto draw_shared = [&](int base) {
        const PhiloxBlock b = sample_block(a.smp, k, (base >> 2) + sub);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            draw_controls(a.smp, block_word(b, j), k, min(base + 4 * sub + j, a.N - 1), du0[j],
                          du1[j]);
            du0[j] = clampf_nan(du0[j], -a.drate_max, a.drate_max);
            du1[j] = a.accel_max * clampf_nan(du1[j], -1.0f, 1.0f);
        }
    };
    // byte index of lane ((n / 4) mod LANES) of this lane's group, for ds_bpermute
    auto owner = [&](int n) {
        return (((int)(threadIdx.x & 63) & ~(LANES - 1)) + ((n >> 2) & (LANES - 1))) << 2;
    };
    auto from_lane = [](int byte, float v) {
        return __int_as_float(__builtin_amdgcn_ds_bpermute(byte, __float_as_int(v)));
    };

    Arm arms[WPL];
#pragma unroll
    for (int q = 0; q < WPL; ++q) arms[q] = arm(a, sub * WPL + q);

    // CKPT: ckpt[b] = state at interval min(b C, N), the 13 stores spread over
    // the lane group; a candidate past its goal exit keeps its frozen state
    int ckpt_done = 0;
    auto write_ckpt = [&](int b, const float (&s)[13]) {
        if (!store) return;
        float *c = a.ckpt + (size_t)b * 13 * K + k;
#pragma unroll
        for (int q = 0; q < 13; ++q)
            if ((q & (LANES - 1)) == sub) c[(size_t)q * K] = s[q];
    };
    if constexpr (CKPT) write_ckpt(0, st);

    // Euler with one substep per interval in a request-ahead build: the
    // terrain of each node is requested a step ahead. The loop
    // takes two intervals per trip so that the two nodes' requests alternate
    // between two register sets (P, Q) instead of being copied from one to
    // the other, which would wait for the loads in flight. A candidate at its
    // goal skips the step and its requests; it stays frozen, so it never uses
    // a set again.
    if constexpr (TRIPS) {
        // Two and four lanes per candidate: the same two sets, in trips of four
        // intervals whose controls are requested a whole trip ahead (one pair
        // of loads brings LANES intervals, interval n + q in lane q % LANES of
        // the group), so that neither the cells nor the controls of a launch
        // whose inputs are not in the caches hold a step up. Every lane takes
        // every step, a candidate past its goal too, so that a trip is one
        // block in which the number of loads in flight is known (a step that
        // some path skips makes the compiler wait for a node's requests before
        // it issues the next one's); the state and cost with which a candidate
        // first stands at its goal are kept aside, in a branch that a wave
        // takes once or so per candidate, and put back at the end.
        // The branch is marked unlikely: a taken branch costs a lone wave the
        // fetch behind it (2 to 4 us in 100 steps).
        // Measured against the plain loop, each on inputs that change from
        // call to call: 10 007 candidates x 73 steps 58.5 -> 45.5 us, with the
        // softmin, costmap and final states 66.7 -> 55.5 us; 16 000 x 90 with
        // a costmap 69.4 -> 55.6 us; 25 000 x 100 at two lanes 81.0 -> 72.9
        // us; 4 096 x 100, whose cells stay in the L2, 1 to 2 % less (58.3 -> 57.1
        // us). Inputs that the L2 still holds from the call before gain nothing
        // from it beyond a wave per compute unit: 6 000 x 70 36.0 -> 38.5 us, with
        // eight sets of controls in turn 38.6 -> 34.3.
        bool done = false;
        float kept[14];
#pragma unroll
        for (int q = 0; q < 13; ++q) kept[q] = st[q];
        kept[13] = J;
        // the one at N is written below, with the final state
        int until_ckpt = CKPT ? a.ckpt_every : 0;
        auto interval = [&](float dd, float ax, const NodeRequest<LANES, CM> &cur,
                            NodeRequest<LANES, CM> &nxt) {
            // goal test at the node, written as in the other loops so that a
            // NaN position (never at the goal) keeps stepping there as here
            const float gdx = st[0] - a.goal_x, gdy = st[1] - a.goal_y;
            const bool arrives = fmaf(gdx, gdx, gdy * gdy) <= a.goal_r2 && !done;
            if (__builtin_expect(__any(arrives), 0)) {
#pragma unroll
                for (int q = 0; q < 13; ++q) kept[q] = arrives ? st[q] : kept[q];
                kept[13] = arrives ? J : kept[13];
                done = done || arrives;
            }
            euler_step_ahead<LANES, CM>(a, arms, st, J, dd, ax, cur, nxt);
            if constexpr (CKPT) {
                if (__builtin_expect(--until_ckpt == 0, 0)) {
                    until_ckpt = a.ckpt_every;
                    float s[13];
#pragma unroll
                    for (int q = 0; q < 13; ++q) s[q] = done ? kept[q] : st[q];
                    write_ckpt(++ckpt_done, s);
                }
            }
        };
        constexpr int PER = 4 / LANES;  // pairs of a trip that a lane holds
        float cu0[PER], cu1[PER], nu0[PER], nu1[PER];
        auto request_controls = [&](int n, float (&u0)[PER], float (&u1)[PER]) {
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const float *p = up + 2 * (size_t)min(n + q * LANES + sub, a.n1 - 1) * K;
                u0[q] = p[0];
                u1[q] = p[K];
            }
        };
        // the controls before the cells, here as in the loop, so that waiting
        // for them never waits for the cells behind them
        int n = a.n0;
        if constexpr (!SAMPLED) {
            if (n < a.n1) request_controls(n, cu0, cu1);
            __builtin_amdgcn_sched_barrier(0);
        }
        NodeRequest<LANES, CM> P, Q;
        request_node<LANES, CM>(a, arms, st[0], st[1], st[2], st[3], st[4], st[5], P);
        for (; n + 3 < a.n1; n += 4) {
            float u0[4], u1[4];
            if constexpr (SAMPLED) {
                if ((n & (4 * LANES - 1)) == 0) draw_shared(n);
                const int o = owner(n);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    u0[q] = from_lane(o, du0[q]);
                    u1[q] = from_lane(o, du1[q]);
                }
            } else {
                request_controls(n + 4, nu0, nu1);
                float cdd[PER], cax[PER];
#pragma unroll
                for (int q = 0; q < PER; ++q) {
                    cdd[q] = clampf_nan(cu0[q], -a.drate_max, a.drate_max);
                    cax[q] = a.accel_max * clampf_nan(cu1[q], -1.0f, 1.0f);
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    u0[q] = group_lane<LANES>(cdd[q / LANES], q % LANES);
                    u1[q] = group_lane<LANES>(cax[q / LANES], q % LANES);
                }
            }
            interval(u0[0], u1[0], P, Q);
            interval(u0[1], u1[1], Q, P);
            interval(u0[2], u1[2], P, Q);
            interval(u0[3], u1[3], Q, P);
            if constexpr (!SAMPLED) {
#pragma unroll
                for (int q = 0; q < PER; ++q) {
                    cu0[q] = nu0[q];
                    cu1[q] = nu1[q];
                }
            }
            n = __all(done) ? a.n1 : n;  // nothing left to step
        }
        // the last one to three intervals
        for (; n < a.n1; ++n) {
            float u0, u1;
            if constexpr (SAMPLED) {
                if ((n & (4 * LANES - 1)) == 0) draw_shared(n);
                const int o = owner(n), j = n & 3;
                u0 = from_lane(o, j == 0 ? du0[0] : j == 1 ? du0[1] : du0[2]);
                u1 = from_lane(o, j == 0 ? du1[0] : j == 1 ? du1[1] : du1[2]);
            } else {
                u0 = up[2 * (size_t)n * K];
                u1 = up[(2 * (size_t)n + 1) * K];
                u0 = clampf_nan(u0, -a.drate_max, a.drate_max);
                u1 = a.accel_max * clampf_nan(u1, -1.0f, 1.0f);
            }
            interval(u0, u1, P, Q);
            P = Q;
        }
        // nothing is taken from a step past the goal
#pragma unroll
        for (int q = 0; q < 13; ++q) st[q] = done ? kept[q] : st[q];
        J = done ? kept[13] : J;
    } else if constexpr (AHEAD) {
        auto interval = [&](int n, const NodeRequest<LANES, CM> &cur,
                            NodeRequest<LANES, CM> &nxt) {
            float u0, u1;
            if constexpr (SAMPLED) {
                if ((n >> 2) != blk_n) {
                    blk_n = n >> 2;
                    blk = sample_block(a.smp, k, blk_n);
                }
                draw_controls(a.smp, block_word(blk, n & 3), k, n, u0, u1);
            } else {
                u0 = nu0;
                u1 = nu1;
            }
            const float dd = clampf_nan(u0, -a.drate_max, a.drate_max);
            const float ax = a.accel_max * clampf_nan(u1, -1.0f, 1.0f);
            // goal test at the node, written as in the other loop so that a
            // NaN position (never at the goal) keeps stepping there as here
            const float gdx = st[0] - a.goal_x, gdy = st[1] - a.goal_y;
            if (!(fmaf(gdx, gdx, gdy * gdy) <= a.goal_r2)) {
                if constexpr (SAMPLED) {
                    euler_step_ahead<LANES, CM>(a, arms, st, J, dd, ax, cur, nxt);
                } else {
                    euler_step_ahead<LANES, CM>(a, arms, st, J, dd, ax, cur, nxt, [&]() {
                        nu0 = unext[0];
                        nu1 = unext[K];
                    });
                }
            }
            if (n + 2 < a.n1) unext += 2 * K;
        };
        NodeRequest<LANES, CM> P, Q;
        request_node<LANES, CM>(a, arms, st[0], st[1], st[2], st[3], st[4], st[5], P);
        int n = a.n0;
        for (; n + 1 < a.n1; n += 2) {
            interval(n, P, Q);
            interval(n + 1, Q, P);
        }
        if (n < a.n1) interval(n, P, Q);
    } else {
    // uniform trip counts: a candidate that reaches the goal stays in the
    // loop frozen (its lanes skip the steps), so the loops carry no
    // per-lane exit or done-flag bookkeeping
    NodeRequest<LANES, CM> node;
    if constexpr (RK4_AHEAD)
        request_node<LANES, CM>(a, arms, st[0], st[1], st[2], st[3], st[4], st[5], node);
    for (int n = a.n0; n < a.n1; ++n) {
        // zero-order hold: control n for the whole interval, restricted to the
        // admissible set (|delta_dot| <= limit, throttle in [-1, 1])
        float u0, u1;
        if constexpr (SAMPLED && LANES > 1) {
            if ((n & (4 * LANES - 1)) == 0) draw_shared(n);  // n0 = 0
            const int o = owner(n), j = n & 3;
            u0 = from_lane(o, j == 0 ? du0[0] : j == 1 ? du0[1] : j == 2 ? du0[2] : du0[3]);
            u1 = from_lane(o, j == 0 ? du1[0] : j == 1 ? du1[1] : j == 2 ? du1[2] : du1[3]);
        } else if constexpr (SAMPLED) {
            if ((n >> 2) != blk_n) {
                blk_n = n >> 2;
                blk = sample_block(a.smp, k, blk_n);
            }
            draw_controls(a.smp, block_word(blk, n & 3), k, n, u0, u1);
        } else {
            u0 = nu0;
            u1 = nu1;
            if constexpr (RK4) {
                if (n + 1 < a.n1) {
                    nu0 = up[(2 * (size_t)n + 2) * K];
                    nu1 = up[(2 * (size_t)n + 3) * K];
                }
            }
        }
        constexpr bool DRAWN = SAMPLED && LANES > 1;
        const float dd = DRAWN ? u0 : clampf_nan(u0, -a.drate_max, a.drate_max);
        const float ax = DRAWN ? u1 : a.accel_max * clampf_nan(u1, -1.0f, 1.0f);

        // S1: one Euler substep per interval, no substep loop
        const int S = S1 ? 1 : a.S;
        for (int s = 0; s < S; ++s) {
            // goal test at the Euler node, before the step; a candidate at
            // its goal is frozen, so the test stays true for it from then on
            {
                const float gdx = st[0] - a.goal_x, gdy = st[1] - a.goal_y;
                if (fmaf(gdx, gdx, gdy * gdy) <= a.goal_r2) continue;
            }
            if constexpr (RK4_AHEAD) {
                rk4_step_ahead<LANES, CM>(a, arms, st, J, dd, ax, node);
            } else if constexpr (RK4) {
                rk4_step<LANES, CM>(a, arms, st, J, dd, ax);
            } else if constexpr (SAMPLED) {
                euler_step<LANES, CM>(a, arms, st, J, dd, ax);
            } else {
                euler_step<LANES, CM>(a, arms, st, J, dd, ax, [&]() {
                    nu0 = unext[0];
                    nu1 = unext[K];
                });
            }
        }
        if (n + 2 < a.n1) unext += 2 * K;
        if constexpr (CKPT) {
            if ((n + 1) % a.ckpt_every == 0 && n + 1 < a.N) {
                ckpt_done = (n + 1) / a.ckpt_every;
                write_ckpt(ckpt_done, st);
            }
        }
    }
    }
    if constexpr (CKPT) {
        const int nseg = (a.N + a.ckpt_every - 1) / a.ckpt_every;
        for (int b = ckpt_done + 1; b <= nseg; ++b) write_ckpt(b, st);
    }

    if (a.finalize) {
        // terminal cost at the final (or goal-exit) state; a non-finite cost
        // or state scores +inf
        const float gdx = st[0] - a.goal_x, gdy = st[1] - a.goal_y;
        J = fmaf(a.w_g, sqrtf(fmaf(gdx, gdx, gdy * gdy)), J);
        bool fin = isfinite(J);
#pragma unroll
        for (int q = 0; q < 13; ++q) fin = fin && isfinite(st[q]);
        if (!fin) J = __builtin_inff();
    }

    if (store) {
        if (sub == 0) a.cost[k] = J;
        float *out = CHUNK ? a.state : a.final_state;
        if (out) {
            // spread the 13 stores over the lane group
#pragma unroll
            for (int q = 0; q < 13; ++q)
                if ((q & (LANES - 1)) == sub) out[(size_t)q * K + k] = st[q];
        }
    }
    return J;
}

// Fused argmin: every workgroup reduces its candidates' packed keys and
// folds the result into a.sel_key with an atomic minimum (order-independent,
// so the winner is the same as the separate selection kernel's); the last of
// the nblocks workgroups to arrive publishes (k*, J*) to a.sel_out and
// out_host, writes the plan and resets the key and the ticket for the next
// launch. bad (optional) is a flag to report in the result's status and
// clear.
template <int BLOCK, bool SAMPLED>
__device__ __forceinline__ void argmin_epilogue(const RolloutArgs &a, unsigned long long key,
                                                unsigned int nblocks, SelectOut *out_host,
                                                int *bad) {
    __shared__ unsigned long long red[BLOCK / 64];
    __shared__ int last_sh;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    key = wave_min(key);
    if (lane == 0) red[wv] = key;
    __syncthreads();
    if (tid == 0) {
        unsigned long long b = red[0];
#pragma unroll
        for (int q = 1; q < BLOCK / 64; ++q) b = red[q] < b ? red[q] : b;
        last_sh = fold_key_and_take_ticket(a.sel_key, a.sel_ticket, b, nblocks);
    }
    __syncthreads();
    if (!last_sh) return;
    if (tid == 0) {
        const unsigned long long m = take_key_and_reset(a.sel_key, a.sel_ticket);
        red[0] = m;
        const int32_t status = (bad && *bad) ? (int32_t)PLAN_EINVAL : 0;
        if (bad) *bad = 0;  // the slot's next request starts with a clear flag
        publish_result(a.sel_out, out_host, m, a.sel_seq, status);
    }
    __syncthreads();
    const unsigned long long m = red[0];
    const int kb = (m == ~0ull) ? -1 : (int)(unsigned int)(m & 0xffffffffu);
    write_plan<SAMPLED>(kb, a.N, a.K, a.controls, a.smp, a.drate_max, a.plan, tid, BLOCK);
}

// One-lane full-horizon launches with several Euler substeps per interval and
// no costmap (the paper's solver shape) are held to 128 VGPRs, four waves per
// SIMD, so its 204 288 candidates (3.1 waves per SIMD) run in one round
// instead of three full rounds and a tail: the materialised-control kernel
// fits in 126 registers, the in-kernel-sampled one spills 15-17 registers
// (its generator words, read once per interval) and is 4.7 % faster all the
// same (2.93 -> 2.79 ms per ordered plan).
// (The instantiation for launches of at most one wave per SIMD, built with
// PLAN_ONE_WAVE_PER_SIMD, has no use for the bound.)
#ifdef PLAN_ONE_WAVE_PER_SIMD
template <int LANES, bool CHUNK, bool RK4, bool CKPT, bool S1, bool CM>
constexpr bool ONE_LANE_4_WAVES = false;
#else
template <int LANES, bool CHUNK, bool RK4, bool CKPT, bool S1, bool CM>
constexpr bool ONE_LANE_4_WAVES = LANES == 1 && !CHUNK && !RK4 && !CKPT && !S1 && !CM;
#endif

template <int LANES, int BLOCK, bool CHUNK, bool SAMPLED = false, bool FUSED = false,
          bool RK4 = false, bool CKPT = false, bool S1 = false, bool CM = true>
__global__ __launch_bounds__(BLOCK, (ONE_LANE_4_WAVES<LANES, CHUNK, RK4, CKPT, S1, CM> ? 4 : 1))
void rollout_srb(const RolloutArgs a) {
    const int gtid = blockIdx.x * BLOCK + threadIdx.x;
    const int sub = gtid & (LANES - 1);
    int slot = gtid / LANES;
    const bool store = slot < a.K;
    // Lanes past K simulate the last candidate again so that every lane group
    // is complete for the DPP sums; they store nothing (and reach the fused
    // epilogue's barriers like every other lane).
    if (!store) slot = a.K - 1;
    int k = slot;
    const float *up = a.controls + slot;
    if constexpr (LANES == 1 && !CHUNK && !CKPT) {
        // ordered launches run one lane per candidate
        if (a.order) {
            // clamped so that a malformed order can only misassign, never
            // address outside the candidate arrays
            k = min(max(a.order[slot], 0), a.K - 1);
            up = a.controls_lane ? a.controls_lane + slot : a.controls + k;
        }
    }
    const float J = simulate<LANES, CHUNK, SAMPLED, RK4, CKPT, S1, CM>(a, k, sub, store, up);
    if constexpr (FUSED)
        argmin_epilogue<BLOCK, SAMPLED>(a, (store && sub == 0) ? cost_key(J, k) : ~0ull,
                                        gridDim.x, a.sel_out_host, nullptr);
}

// A one-lane full-horizon launch whose candidates fill R whole rounds of one
// wave per SIMD plus a small remainder (the paper's 204 288 candidates are
// 3.12 waves per SIMD): run one lane per candidate would give that remainder
// a fourth wave on a few SIMDs and make the whole launch wait for them.
// Here workgroups [0, split) run one lane per candidate on slots
// [0, split x BLOCK) and the rest run four lanes per candidate on the
// remaining slots, so the remainder's work (about half a one-lane wave per
// 16 candidates) spreads over four times as many SIMDs. Every candidate's
// arithmetic is the same at any lane count, so results equal the one-lane
// launch's bit for bit. Held to four waves per SIMD like the one-lane kernel
// of the same shape.
template <int BLOCK, bool SAMPLED, bool FUSED, bool S1, bool CM>
__global__ __launch_bounds__(BLOCK, 4) void rollout_balanced(const RolloutArgs a, int split) {
    const bool four = (int)blockIdx.x >= split;  // uniform over the workgroup
    int slot, sub;
    if (!four) {
        slot = (int)blockIdx.x * BLOCK + (int)threadIdx.x;
        sub = 0;
    } else {
        const int g = ((int)blockIdx.x - split) * BLOCK + (int)threadIdx.x;
        slot = split * BLOCK + (g >> 2);
        sub = g & 3;
    }
    const bool store = slot < a.K;
    if (!store) slot = a.K - 1;
    int k = slot;
    const float *up = a.controls + slot;
    if (a.order) {
        k = min(max(a.order[slot], 0), a.K - 1);
        up = a.controls_lane ? a.controls_lane + slot : a.controls + k;
    }
    float J;
    if (four)
        J = simulate<4, false, SAMPLED, false, false, S1, CM>(a, k, sub, store, up);
    else
        J = simulate<1, false, SAMPLED, false, false, S1, CM>(a, k, 0, store, up);
    if constexpr (FUSED)
        argmin_epilogue<BLOCK, SAMPLED>(a, (store && sub == 0) ? cost_key(J, k) : ~0ull,
                                        gridDim.x, a.sel_out_host, nullptr);
}

// Several independent plans in one launch (the serving loop's tick). Entry e
// of the table owns blocks [e.block_start, next block_start) and advances
// slot e.slot through intervals [e.n0, e.n1); every block belongs to exactly
// one slot, so the per-slot arguments are wave-uniform. An entry that ends
// its request's horizon also selects the request's plan: the entry's blocks
// run the fused argmin epilogue on the slot's own key and ticket, and the
// last of them writes the result to ring[slot] and the plan.
//
// The entries come with the most intervals first, and every second round of
// t.row workgroups takes its blocks in reverse: a compute unit that holds the
// longest of one round gets the shortest of the next. 64 requests of 40 to 160
// intervals and 512 to 8 192 candidates at once, 4.2 waves per SIMD: 475 us in
// the slots' order, where the unluckiest compute unit held half as much again as
// the average one, 377 us so; and 308 us with the cost channel left out (CM)
// where no resident request has a costmap.
template <int LANES, int BLOCK, bool S1, bool CM>
__global__ __launch_bounds__(BLOCK) void rollout_slots(const RolloutArgs *__restrict__ slots,
                                                       const TickTable t, int *bad,
                                                       SelectOut *ring, uint32_t seq) {
    int block = (int)blockIdx.x;
    const int round = block / t.row;
    if ((round & 1) && (round + 1) * t.row <= t.total_blocks)
        block = (2 * round + 1) * t.row - 1 - block;
    int lo = 0, hi = t.count - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (t.e[mid].block_start <= block)
            lo = mid;
        else
            hi = mid - 1;
    }
    const TickEntry te = t.e[lo];
    const int block_end = lo + 1 < t.count ? t.e[lo + 1].block_start : t.total_blocks;
    RolloutArgs a = slots[te.slot];
    a.n0 = te.n0;
    a.n1 = te.n1;
    a.finalize = te.finalize;
    a.sel_seq = seq;
    const int gtid = (block - te.block_start) * BLOCK + threadIdx.x;
    const int sub = gtid & (LANES - 1);
    int k = gtid / LANES;
    const bool store = k < a.K;
    if (!store) k = a.K - 1;
    const float J = simulate<LANES, true, false, false, false, S1, CM>(a, k, sub, store,
                                                                       a.controls + k);
    if (te.finalize)
        argmin_epilogue<BLOCK, false>(a, (store && sub == 0) ? cost_key(J, k) : ~0ull,
                                      (unsigned int)(block_end - te.block_start),
                                      ring + te.slot, bad + te.slot);
}

// Launch dispatch for one lane count L (block 64 or 256) and costmap flag CM
// (the context's a.has_costmap). Euler launches with one substep per interval
// (a.S == 1) use the S1 instantiations, which carry no substep loop.
template <int L, bool CM>
__forceinline__ hipError_t launch_rollout_cm(const RolloutArgs &a, int block, bool chunk,
                                             hipStream_t s) {
    const long long threads = (long long)a.K * L;
    const unsigned grid = (unsigned)((threads + block - 1) / block);
#define PLAN_LAUNCH(B, C)                                                                       \
    if (block == B && chunk == C) {                                                             \
        if (a.method == 1)                                                                      \
            hipLaunchKernelGGL((rollout_srb<L, B, C, false, false, true, false, false, CM>),     \
                               dim3(grid), dim3(B), 0, s, a);                                   \
        else if (a.S == 1)                                                                      \
            hipLaunchKernelGGL((rollout_srb<L, B, C, false, false, false, false, true, CM>),     \
                               dim3(grid), dim3(B), 0, s, a);                                   \
        else                                                                                    \
            hipLaunchKernelGGL((rollout_srb<L, B, C, false, false, false, false, false, CM>),    \
                               dim3(grid), dim3(B), 0, s, a);                                   \
        return hipGetLastError();                                                               \
    }
    PLAN_LAUNCH(64, false)
    PLAN_LAUNCH(256, false)
    PLAN_LAUNCH(64, true)
    PLAN_LAUNCH(256, true)
#undef PLAN_LAUNCH
    return hipErrorInvalidValue;
}

template <int L>
__forceinline__ hipError_t launch_rollout_lanes(const RolloutArgs &a, int block, bool chunk,
                                                hipStream_t s) {
    return a.has_costmap ? launch_rollout_cm<L, true>(a, block, chunk, s)
                         : launch_rollout_cm<L, false>(a, block, chunk, s);
}

template <int L, bool CM>
__forceinline__ hipError_t launch_sampled_cm(const RolloutArgs &a, int block, hipStream_t s) {
    const long long threads = (long long)a.K * L;
    const unsigned grid = (unsigned)((threads + block - 1) / block);
    if (block == 64)
        hipLaunchKernelGGL((rollout_srb<L, 64, false, true, false, false, false, false, CM>),
                           dim3(grid), dim3(64), 0, s, a);
    else if (block == 256)
        hipLaunchKernelGGL((rollout_srb<L, 256, false, true, false, false, false, false, CM>),
                           dim3(grid), dim3(256), 0, s, a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

template <int L>
__forceinline__ hipError_t launch_sampled_lanes(const RolloutArgs &a, int block, hipStream_t s) {
    return a.has_costmap ? launch_sampled_cm<L, true>(a, block, s)
                         : launch_sampled_cm<L, false>(a, block, s);
}

template <int L>
__forceinline__ hipError_t launch_ckpt_lanes(const RolloutArgs &a, int block, hipStream_t s) {
    const long long threads = (long long)a.K * L;
    const unsigned grid = (unsigned)((threads + block - 1) / block);
#define PLAN_LAUNCH(B)                                                                          \
    if (block == B) {                                                                           \
        if (a.S == 1)                                                                           \
            hipLaunchKernelGGL((rollout_srb<L, B, false, false, false, false, true, true>),      \
                               dim3(grid), dim3(B), 0, s, a);                                   \
        else                                                                                    \
            hipLaunchKernelGGL((rollout_srb<L, B, false, false, false, false, true>),            \
                               dim3(grid), dim3(B), 0, s, a);                                   \
        return hipGetLastError();                                                               \
    }
    PLAN_LAUNCH(64)
    PLAN_LAUNCH(256)
#undef PLAN_LAUNCH
    return hipErrorInvalidValue;
}

template <int L, bool CM>
__forceinline__ hipError_t launch_argmin_cm(const RolloutArgs &a, int block, bool sampled,
                                            hipStream_t s) {
    const long long threads = (long long)a.K * L;
    const unsigned grid = (unsigned)((threads + block - 1) / block);
#define PLAN_LAUNCH(B)                                                                          \
    if (block == B) {                                                                           \
        if (sampled)                                                                            \
            hipLaunchKernelGGL((rollout_srb<L, B, false, true, true, false, false, false, CM>),  \
                               dim3(grid), dim3(B), 0, s, a);                                   \
        else if (a.S == 1)                                                                      \
            hipLaunchKernelGGL((rollout_srb<L, B, false, false, true, false, false, true, CM>),  \
                               dim3(grid), dim3(B), 0, s, a);                                   \
        else                                                                                    \
            hipLaunchKernelGGL((rollout_srb<L, B, false, false, true, false, false, false, CM>), \
                               dim3(grid), dim3(B), 0, s, a);                                   \
        return hipGetLastError();                                                               \
    }
    PLAN_LAUNCH(64)
    PLAN_LAUNCH(256)
#undef PLAN_LAUNCH
    return hipErrorInvalidValue;
}

template <int L>
__forceinline__ hipError_t launch_argmin_lanes(const RolloutArgs &a, int block, bool sampled,
                                               hipStream_t s) {
    return a.has_costmap ? launch_argmin_cm<L, true>(a, block, sampled, s)
                         : launch_argmin_cm<L, false>(a, block, sampled, s);
}

// s1: every slot of the tick integrates with one substep per interval.
template <int L>
__forceinline__ hipError_t launch_slots_lanes(const RolloutArgs *slots, const TickTable &t,
                                              int *bad, SelectOut *ring, uint32_t seq, bool s1,
                                              int block, hipStream_t s) {
    const unsigned grid = (unsigned)t.total_blocks;
#define PLAN_LAUNCH(B, ONE, CMAP)                                                            \
    if (block == B && s1 == ONE && (t.costmap != 0) == CMAP) {                               \
        hipLaunchKernelGGL((rollout_slots<L, B, ONE, CMAP>), dim3(grid), dim3(B), 0, s,      \
                           slots, t, bad, ring, seq);                                        \
        return hipGetLastError();                                                            \
    }
    PLAN_LAUNCH(64, true, false)
    PLAN_LAUNCH(64, true, true)
    PLAN_LAUNCH(64, false, false)
    PLAN_LAUNCH(64, false, true)
    PLAN_LAUNCH(256, true, false)
    PLAN_LAUNCH(256, true, true)
    PLAN_LAUNCH(256, false, false)
    PLAN_LAUNCH(256, false, true)
#undef PLAN_LAUNCH
    return hipErrorInvalidValue;
}

}  // namespace

// One-lane dispatch for launches of at most one wave per SIMD, defined in
// rollout_onelane_1wave.hip.
hipError_t launch_rollout_1wave(const RolloutArgs &a, int block, bool chunk, hipStream_t s);
hipError_t launch_sampled_1wave(const RolloutArgs &a, int block, hipStream_t s);
hipError_t launch_argmin_1wave(const RolloutArgs &a, int block, bool sampled, hipStream_t s);

// Two- and four-lane dispatch of the launches of at most one wave per SIMD
// whose intervals are one Euler step, defined in rollout_multilane_1wave.hip.
hipError_t launch_rollout_multi_1wave(const RolloutArgs &a, int lanes, int block, bool chunk,
                                      hipStream_t s);
hipError_t launch_sampled_multi_1wave(const RolloutArgs &a, int lanes, int block, hipStream_t s);
hipError_t launch_argmin_multi_1wave(const RolloutArgs &a, int lanes, int block, bool sampled,
                                     hipStream_t s);
hipError_t launch_ckpt_multi_1wave(const RolloutArgs &a, int lanes, int block, hipStream_t s);
hipError_t launch_slots_multi_1wave(const RolloutArgs *slots, const TickTable &t, int *bad,
                                    SelectOut *ring, uint32_t seq, int lanes, int block,
                                    hipStream_t s);

// Two- and four-lane dispatch, defined in rollout_multilane.hip.
hipError_t launch_rollout_multi(const RolloutArgs &a, int lanes, int block, bool chunk,
                                hipStream_t s);
hipError_t launch_sampled_multi(const RolloutArgs &a, int lanes, int block, hipStream_t s);
hipError_t launch_ckpt_multi(const RolloutArgs &a, int lanes, int block, hipStream_t s);
hipError_t launch_argmin_multi(const RolloutArgs &a, int lanes, int block, bool sampled,
                               hipStream_t s);
hipError_t launch_slots_multi(const RolloutArgs *slots, const TickTable &t, int *bad,
                              SelectOut *ring, uint32_t seq, bool s1, int lanes, int block,
                              hipStream_t s);

}  // namespace plan
