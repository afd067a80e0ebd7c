// Rollout of the extended single-track (EST) baseline formulation: the
// paper's comparison model (appendix "Extended Single-Track Vehicle Dynamics
// Model": state eq. models:3dof:state, eqs. models:3dof:update and
// models:3dof:A, 1-2-3 rotation, virtual-tire slip angles, load transfer
// eq. models:3dof:Fz_lon, sigmoid tire eq. models:tire) with the
// lateral-acceleration soft constraint of section "OCP Formulation"
// (pi_ay = |a_y - g_y| - a_bar_y, a_bar_y = M g / (2 K_zy)), in place of the
// SRB model and the ESM.
//
// One lane per candidate: the 7-component state stays in VGPRs; each Euler
// step interpolates the slopes of the terrain cell under the CoM (they give
// roll and pitch) and, when a costmap is set, the cost at the four wheels.
// Arithmetic is fixed by the source (no contraction, explicit fmaf), as in
// the SRB kernel.
#include "handoff.h"
#include "plan_internal.h"
#include "rollout_step.h"

namespace plan {
namespace {

// Bilinear interpolant of channel ch (0 h, 1 f_x, 2 f_y, 3 cost) at the
// world point (Px, Py), clamp-to-edge; a NaN coordinate clamps to the grid
// origin, so every cell is inside the grid.
template <int CH>
__device__ __forceinline__ float lookup(const RolloutArgs &a, const CellPos &c) {
    return bil(load_coefs(cell_rsrc(a), c.off, CH), c.tx, c.ty);
}

__device__ __forceinline__ CellPos cell_at(const RolloutArgs &a, float Px, float Py) {
    return cell_pos(a, (Px - a.x0) * a.inv_res, (Py - a.y0) * a.inv_res);
}

// The terrain slopes at a node's CoM, requested a step before the step that
// starts there uses them.
struct Slopes {
    float4 fx, fy;
    float tx, ty;
};

__device__ __forceinline__ Slopes request_slopes(const RolloutArgs &a, float x, float y) {
    const CellPos c = cell_at(a, x, y);
    return Slopes{load_coefs(cell_rsrc(a), c.off, 1), load_coefs(cell_rsrc(a), c.off, 2), c.tx,
                  c.ty};
}

// A node's running cost whose wheel costs are still in flight: it is added to
// J during the next step, or by settle() at the end.
struct PendingCost {
    float L = 0.0f;
    float4 c[4] = {};
    float tx[4] = {}, ty[4] = {};
};

__device__ __forceinline__ void settle(const RolloutArgs &a, const PendingCost &p, float &J) {
    float c[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) c[w] = bil(p.c[w], p.tx[w], p.ty[w]);
    J = fmaf(a.h, p.L + ((c[0] + c[1]) + (c[2] + c[3])), J);
}

// One forward-Euler step of the EST formulation for one candidate: the
// running cost at the node is added to J and the state advanced in place.
// AHEAD: node holds the slopes at the state's position and receives those at
// the next one, which depends on the slopes, the heading and the velocity only,
// so that their request goes out before the tires are computed; and with a
// costmap the cost added to J is the previous node's, this one's is left in
// pend. FAST: slip ratios of at most 1, in every candidate of the wave, take the
// arctangent without its reciprocal and selections.
template <bool AHEAD, bool CM, bool FAST>
__device__ __forceinline__ void est_step(const RolloutArgs &a, float (&st)[7], float &J,
                                         float dd, float ax, Slopes &node_next, PendingCost &pend_next) {
    // without AHEAD nothing is carried from step to step
    Slopes own_node;
    PendingCost own_pend;
    Slopes &node = AHEAD ? node_next : own_node;
    PendingCost &pend = AHEAD ? pend_next : own_pend;
    const float h = a.h;
    float x = st[0], y = st[1], psi = st[2];
    float vy = st[3], wz = st[4], delta = st[5], vx = st[6];

    // Roll and pitch put b_z on the unit upward normal (-f_x, -f_y, 1)/s
    // under the CoM. With the 1-2-3 convention b_z = (sin th, -cos th sin ph,
    // cos ph cos th), so sin th = -f_x/s, cos th = sqrt(1 + f_y^2)/s,
    // sin ph = f_y/sqrt(1 + f_y^2), cos ph = 1/sqrt(1 + f_y^2).
    if constexpr (!AHEAD) node = request_slopes(a, x, y);
    const float Tfx = bil(node.fx, node.tx, node.ty), Tfy = bil(node.fy, node.tx, node.ty);
    const float q = fmaf(Tfy, Tfy, 1.0f);
    const float rq = frsq(q), rs = frsq(fmaf(Tfx, Tfx, q));
    const float sth = -Tfx * rs;
    const float cth = (q * rq) * rs;
    const float sph = Tfy * rq;
    const float cph = rq;
    float sps, cps;
    __sincosf(psi, &sps, &cps);
    // rows of the 1-2-3 rotation W <- B that the model uses
    const float R11 = cth * cps, R12 = -(cth * sps);
    const float R21 = fmaf(cps * sph, sth, cph * sps);
    const float R22 = fmaf(-(sph * sth), sps, cph * cps);
    const float R32 = fmaf(cph * sth, sps, cps * sph);
    const float R33 = cph * cth;

    // world velocity of the planar body velocity (v_x, v_y, 0)
    const float vWx = fmaf(R11, vx, R12 * vy);
    const float vWy = fmaf(R21, vx, R22 * vy);
    const float x_next = fmaf(h, vWx, x), y_next = fmaf(h, vWy, y);
    if constexpr (AHEAD) node = request_slopes(a, x_next, y_next);
    // costmap at the four wheels, P = p + R rho with the SRB lever arms
    auto request_costs = [&]() {
        const float R13 = sth, R23 = -(cth * sph);
        const float rz = -a.hR;
        const float bx = fmaf(R13, rz, x), by = fmaf(R23, rz, y);
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float rx = (w < 2) ? a.Lf : -a.Lr;
            const float ry = (w & 1) ? -a.half_e : a.half_e;
            const CellPos c = cell_at(a, fmaf(R11, rx, fmaf(R12, ry, bx)),
                                      fmaf(R21, rx, fmaf(R22, ry, by)));
            pend.c[w] = load_coefs(cell_rsrc(a), c.off, 3);
            pend.tx[w] = c.tx;
            pend.ty[w] = c.ty;
        }
    };
    if constexpr (AHEAD && CM) {
        settle(a, pend, J);
        request_costs();
    }
    if constexpr (AHEAD) __builtin_amdgcn_sched_barrier(0);
    // gravity in the body frame, R^T (0, 0, -g): lateral and normal parts
    const float gBy = -a.g * R32;
    const float gBz = -a.g * R33;

    // load transfer to the virtual tires from the longitudinal acceleration
    // a_x = vx_dot - omega_z v_y
    const float axb = fmaf(-wz, vy, ax);
    const float Fzf = fmaf(-a.Kzzf, gBz, -(a.Kzx * axb));
    const float Fzr = fmaf(-a.Kzzr, gBz, a.Kzx * axb);
    // virtual-tire slip angles (v_x >= vx_min > 0) and sigmoid tire
    const float ivx = frcp(vx);
    const float tf = fmaf(wz, a.Lf, vy) * ivx, tr = fmaf(-wz, a.Lr, vy) * ivx;
    // (a NaN is no reason for the long form: both give NaN)
    float af, ar;
    if (!FAST || __builtin_expect(__any(fmaxf(fabsf(tf), fabsf(tr)) > 1.0f), 0)) {
        af = atan_mm(tf);
        ar = atan_mm(tr);
    } else {
        af = atan_mm<false, true>(tf);
        ar = atan_mm<false, true>(tr);
    }
    af -= delta;
    const float Caf = a.C * af, Car = a.C * ar;
    const float Fyf = (Fzf * (-Caf * a.mu)) * frsq(fmaf(Caf, Caf, a.mu2));
    const float Fyr = (Fzr * (-Car * a.mu)) * frsq(fmaf(Car, Car, a.mu2));
    const float Fy = Fyf + Fyr;
    const float vyd = fmaf(Fy, a.invM, gBy) - wz * vx;
    const float wzd = fmaf(Fyf * a.Lf, __cosf(delta), -(Fyr * a.Lr)) * a.invJzz;

    // lateral-acceleration measure: a_y - g_y = (F_y,f + F_y,r) / M
    const float pi = fabsf(Fy * a.invM) - a.a_bar_y;
    const float mm = fmaxf(0.0f, fmaf(pi, a.inv_eps_ay, 1.0f));
    const float L = fmaf(a.w_c * dd, dd, a.w_t) + (a.sigma * mm) * mm;
    if constexpr (AHEAD && CM) {
        pend.L = L;
    } else if (!AHEAD && a.has_costmap) {
        // in a block of their own: issued among the tires' instructions they
        // cost 3 % (204 288 candidates x 800 steps, whose cells miss the L1)
        pend.L = L;
        request_costs();
        settle(a, pend, J);
    } else {
        J = fmaf(h, L, J);
    }

    // forward Euler and the steering / speed limits
    x = x_next;
    y = y_next;
    psi = fmaf(h, wz, psi);
    vy = fmaf(h, vyd, vy);
    wz = fmaf(h, wzd, wz);
    delta = clampf_nan(fmaf(h, dd, delta), -a.delta_max, a.delta_max);
    vx = fmaf(h, ax, vx);
    vx = maxn(vx, a.vx_min);
    st[0] = x;
    st[1] = y;
    st[2] = psi;
    st[3] = vy;
    st[4] = wz;
    st[5] = delta;
    st[6] = vx;
}

// Steps of one candidate; a candidate that reaches its goal stays frozen.
template <bool AHEAD, bool CM, bool FAST>
struct Stepper {
    const RolloutArgs &a;
    float (&st)[7];
    float &J;
    Slopes node;
    PendingCost pend;

    __device__ Stepper(const RolloutArgs &a_, float (&st_)[7], float &J_)
        : a(a_), st(st_), J(J_) {
        if constexpr (AHEAD) node = request_slopes(a, st[0], st[1]);
    }
    __device__ __forceinline__ void operator()(float u0, float u1) {
        const float dd = clampf_nan(u0, -a.drate_max, a.drate_max);
        const float ax = a.accel_max * clampf_nan(u1, -1.0f, 1.0f);
        const float gdx = st[0] - a.goal_x, gdy = st[1] - a.goal_y;
        // at the goal the test stays true
        if (!(fmaf(gdx, gdx, gdy * gdy) <= a.goal_r2))
            est_step<AHEAD, CM, FAST>(a, st, J, dd, ax, node, pend);
    }
    __device__ __forceinline__ void finish() {
        if constexpr (AHEAD && CM) settle(a, pend, J);
    }
};

// S1: one substep per interval; the controls are then requested four intervals
// ahead, else one. A step waits for its slopes, and with a costmap for the
// cells under the wheels after that, about as long as it computes; a launch of
// up to one wave per SIMD hides neither, so it requests both a step ahead: 64
// candidates x 60 steps 30 -> 22 us, 4 096 with a costmap 45 -> 31, 11 144 x
// 266 with one 249 -> 164, 65 536 x 800 329 -> 268. Without a costmap that pays
// with more waves too (131 072 x 800 402 -> 376 us, 204 288 x 800 712 -> 690);
// with one, several waves' requests a step ahead displace each other's cells
// (150 000 x 800: 2 460 us at the start of the step, 2 750 ahead).
// FAST where the vector instructions of several waves a SIMD are the bound:
// 204 288 x 800 690 -> 597 us, 131 072 x 800 376 -> 358; one wave loses as much
// by the branch (65 536 x 800 268 -> 274), and with a costmap the cells are the
// bound (204 288 x 800 2 390 -> 2 480).
// Steps [from, to) of the horizon's N S for the candidate whose controls start
// at up.
template <bool S1, bool AHEAD, bool CM, bool FAST>
__device__ __forceinline__ void est_steps(const RolloutArgs &a, const float *up, float (&st)[7],
                                          float &J, long long from, long long to) {
    const size_t K = (size_t)a.K;
    constexpr int PAIRS = S1 ? 4 : 1;
    float cu0[PAIRS], cu1[PAIRS], nu0[PAIRS], nu1[PAIRS];
    auto request = [&](int n, float (&u0)[PAIRS], float (&u1)[PAIRS]) {
#pragma unroll
        for (int q = 0; q < PAIRS; ++q) {
            const float *p = up + 2 * (size_t)min(n + q, a.N - 1) * K;
            u0[q] = p[0];
            u1[q] = p[K];
        }
    };
    int n = (int)(from / a.S);
    const int n_to = (int)(to / a.S);
    request(n, cu0, cu1);
    Stepper<AHEAD, CM, FAST> step(a, st, J);
    if constexpr (S1) {
        for (; n + PAIRS - 1 < n_to; n += PAIRS) {
            request(n + PAIRS, nu0, nu1);
#pragma unroll
            for (int q = 0; q < PAIRS; ++q) step(cu0[q], cu1[q]);
#pragma unroll
            for (int q = 0; q < PAIRS; ++q) {
                cu0[q] = nu0[q];
                cu1[q] = nu1[q];
            }
        }
#pragma unroll
        for (int q = 0; q < PAIRS - 1; ++q)
            if (n + q < n_to) step(cu0[q], cu1[q]);
    } else {
        int s = (int)(from - (long long)n * a.S);
        const int s_to = (int)(to - (long long)n_to * a.S);
        for (; n <= n_to; ++n, s = 0) {
            request(n + 1, nu0, nu1);
            const int end = n < n_to ? a.S : s_to;
            for (; s < end; ++s) step(cu0[0], cu1[0]);
            cu0[0] = nu0[0];
            cu1[0] = nu1[0];
        }
    }
    step.finish();
}

// Terminal cost and outputs of candidate k.
__device__ __forceinline__ void est_finish(const RolloutArgs &a, int k, const float (&st)[7],
                                           float J) {
    const float gdx = st[0] - a.goal_x, gdy = st[1] - a.goal_y;
    J = fmaf(a.w_g, sqrtf(fmaf(gdx, gdx, gdy * gdy)), J);
    bool fin = isfinite(J);
#pragma unroll
    for (int q = 0; q < 7; ++q) fin = fin && isfinite(st[q]);
    if (!fin) J = __builtin_inff();
    a.cost[k] = J;
    if (a.final_state) {
#pragma unroll
        for (int q = 0; q < 7; ++q) a.final_state[(size_t)q * a.K + k] = st[q];
    }
}

template <int BLOCK, bool S1, bool AHEAD, bool CM, bool FAST>
__global__ __launch_bounds__(BLOCK) void rollout_est(const RolloutArgs a) {
    const int slot = blockIdx.x * BLOCK + threadIdx.x;
    if (slot >= a.K) return;
    const int k = a.order ? min(max(a.order[slot], 0), a.K - 1) : slot;
    float st[7];
#pragma unroll
    for (int q = 0; q < 7; ++q) st[q] = a.s0[q];
    float J = 0.0f;
    const float *up = a.controls_lane ? a.controls_lane + slot : a.controls + k;
    est_steps<S1, AHEAD, CM, FAST>(a, up, st, J, 0, (long long)a.N * a.S);
    est_finish(a, k, st, J);
}

// A hand-off flag in device memory, written by a wave's first lane and known to
// all of them.
struct WaveFlag {
    int *p;
    __device__ __forceinline__ int load() const {
        return __builtin_amdgcn_readfirstlane(
            __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    }
    __device__ __forceinline__ void store(int v) const {
        if ((threadIdx.x & 63) == 0)
            __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // the first lane alone gets the value before (the others v)
    __device__ __forceinline__ int exchange(int v) const {
        if ((threadIdx.x & 63) == 0)
            v = __hip_atomic_exchange(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return v;
    }
    __device__ __forceinline__ int compare_exchange(int expected, int v) const {
        if ((threadIdx.x & 63) == 0)
            __hip_atomic_compare_exchange_strong(p, &expected, v, __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return __builtin_amdgcn_readfirstlane(expected);
    }
    __device__ __forceinline__ void pause() const { __builtin_amdgcn_s_sleep(32); }
};

// A launch of a few waves per SIMD and a remainder lasts as long as the SIMDs
// that take a wave more than the others (204 288 candidates: 120 of 1 024 SIMDs
// take four, the others three). Here exactly `rounds` waves per SIMD, the
// workers, share the groups of 64 candidates in equal parts of their steps:
// the groups' steps in a row, group after group, are cut every `part` steps
// (at least one horizon). A worker whose part ends inside a group
// first runs that group up to there and hands its state on, then the whole
// groups, and last the rest of the group that its part starts in, whose state
// the worker before it handed on long since: it ran that piece first, and all
// parts are as long. Were it not there in time (the workers of a launch need
// not all be running, or have started), the worker runs the piece itself.
// One flag a worker, as in handoff.h.
template <bool S1>
__global__ __launch_bounds__(256) void rollout_est_parts(const RolloutArgs a, long long part,
                                                         float *handoff, int *flag) {
    const int worker =
        __builtin_amdgcn_readfirstlane((int)blockIdx.x * 4 + (int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    const long long T = (long long)a.N * a.S;
    const long long total = (long long)((a.K + 63) / 64) * T;
    const long long lo = worker * part, hi = min(lo + part, total);
    if (lo >= hi) return;
    const int g_lo = (int)(lo / T), g_hi = (int)((hi - 1) / T);
    const long long o_lo = lo - g_lo * T, o_hi = hi - g_hi * T;
    const bool head = o_hi < T, tail = o_lo > 0;  // never both of one group: part >= T
    const int first = g_lo + tail, last = g_hi - head;  // whole groups
    const int pieces = (int)head + (last - first + 1) + (int)tail;
    for (int p = 0; p < pieces; ++p) {
        const bool is_head = head && p == 0, is_tail = tail && p == pieces - 1;
        const int g = is_head ? g_hi : is_tail ? g_lo : first + p - (int)head;
        const int slot = min(g * 64 + lane, a.K - 1);
        const int k = a.order ? min(max(a.order[slot], 0), a.K - 1) : slot;
        const float *up = a.controls_lane ? a.controls_lane + slot : a.controls + k;
        float st[7];
#pragma unroll
        for (int q = 0; q < 7; ++q) st[q] = a.s0[q];
        float J = 0.0f;
        long long from = 0;
        if (is_tail) {
            const WaveFlag theirs{&flag[worker - 1]};
            if (handoff_take(theirs, 1 << 14)) {
                asm volatile("" ::: "memory");  // the state after the flag
                float *h = handoff + (size_t)(worker - 1) * 512 + lane;
#pragma unroll
                for (int q = 0; q < 7; ++q)
                    st[q] = __hip_atomic_load(h + q * 64, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
                J = __hip_atomic_load(h + 7 * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                handoff_release(theirs);
                from = o_lo;
            }
        }
        est_steps<S1, true, false, true>(a, up, st, J, from, is_head ? o_hi : T);
        if (is_head) {
            float *h = handoff + (size_t)worker * 512 + lane;
#pragma unroll
            for (int q = 0; q < 7; ++q)
                __hip_atomic_store(h + q * 64, st[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(h + 7 * 64, J, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the flag after the state
            handoff_give(WaveFlag{&flag[worker]});
        } else if (g * 64 + lane < a.K) {
            est_finish(a, k, st, J);
        }
    }
}

}  // namespace

hipError_t launch_rollout_est(const RolloutArgs &a, int block, bool one_wave, hipStream_t s) {
    const unsigned grid = (unsigned)(((long long)a.K + block - 1) / block);
    const bool cm = a.has_costmap != 0;
#define PLAN_LAUNCH(B, ONE, NARROW, REQ, CMAP, FAST)                                         \
    if (block == B && (a.S == 1) == ONE && one_wave == NARROW && cm == CMAP) {               \
        hipLaunchKernelGGL((rollout_est<B, ONE, REQ, CMAP, FAST>), dim3(grid), dim3(B), 0, s, \
                           a);                                                               \
        return hipGetLastError();                                                            \
    }
#define PLAN_LAUNCHES(B, ONE)                        \
    PLAN_LAUNCH(B, ONE, false, true, false, true)    \
    PLAN_LAUNCH(B, ONE, false, false, true, false)
    // launches of up to one wave per SIMD take 64 threads
    PLAN_LAUNCH(64, false, true, true, false, false)
    PLAN_LAUNCH(64, false, true, true, true, false)
    PLAN_LAUNCH(64, true, true, true, false, false)
    PLAN_LAUNCH(64, true, true, true, true, false)
    PLAN_LAUNCHES(64, false)
    PLAN_LAUNCHES(64, true)
    PLAN_LAUNCHES(256, false)
    PLAN_LAUNCHES(256, true)
#undef PLAN_LAUNCHES
#undef PLAN_LAUNCH
    return hipErrorInvalidValue;
}

hipError_t launch_rollout_est_parts(const RolloutArgs &a, int rounds, int simds, float *handoff,
                                    int *flag, hipStream_t s) {
    const long long T = (long long)a.N * a.S, workers = (long long)rounds * simds;
    const long long total = (((long long)a.K + 63) / 64) * T;
    const long long share = (total + workers - 1) / workers;
    const long long part = share > T ? share : T;
    // no more workgroups of four waves fit a compute unit's 160 KB than rounds
    const unsigned lds = 160 * 1024 / (rounds + 1) + 1024;
    const dim3 grid((unsigned)(workers / 4));
    if (a.S == 1)
        hipLaunchKernelGGL((rollout_est_parts<true>), grid, dim3(256), lds, s, a, part,
                           handoff, flag);
    else
        hipLaunchKernelGGL((rollout_est_parts<false>), grid, dim3(256), lds, s, a, part,
                           handoff, flag);
    return hipGetLastError();
}

}  // namespace plan
