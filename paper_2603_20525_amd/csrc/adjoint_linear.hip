// Backward pass of the adjoint rollout for few candidates: the same gradient
// as adjoint.hip's, with every step linearised in parallel and only the
// products with the linearisations left in the serial chain over the steps.
//
// What bounds it: a candidate's steps are a chain, and at a few thousand
// candidates the chip has fewer waves than SIMDs, so a backward pass that
// recomputes, differentiates and pulls back one step after the other lasts as
// long as its instructions take one wave (2 us a step). Of these only the
// product lam <- A^T lam depends on the step after it. So a workgroup of five
// waves takes four candidates and, from the end of the horizon backwards,
//   1. recomputes up to 160 steps' states from the checkpoints into LDS,
//      twenty segments at a time (sixteen lanes a segment: four candidates of
//      four wheels);
//   2. linearises sixteen steps at a time (four waves of four steps of four
//      candidates of four wheels): the columns of A and the gradients of the
//      running cost, 16 x 12 floats a step and candidate, go to LDS;
//   3. pulls lam back through the sixteen steps before with the fifth wave,
//      sixteen lanes a candidate: lane j holds lam_j and column j, and a step
//      is a dozen multiply-adds whose other factor is broadcast along the row
//      of sixteen lanes by DPP.
//
// 1 024 candidates x 100 steps: 31 us (six rounds of it at 6 000: 167) against
// 204 us; of these 6 go to the start and the recomputation and 3.5 to each of
// seven batches. The linearisations' 700 vector instructions account for 1.4 of
// those; the rest are waits, a third of the waves' cycles, for LDS (1 971 cycles
// a wave of bank conflicts: candidates' columns are 768 bytes apart) and at the
// barrier between two batches. A chain step is 13 multiply-adds, five other
// vector instructions and four LDS
// reads, 160 cycles; read from LDS without the columns being fetched ahead and
// with the broadcasts as moves it took 600 and bound the kernel (40 us).
//
// Structure of a column: the wheels enter through two scalars, the load Fz and
// the lateral force fy, and a load's gradient with respect to the angles is a
// torque, P' x dFz/dP - n x (R dFz/dn), resolved about the three rotation axes
// (P' the arm in the world, n the terrain normal in the world).
//
// A candidate whose motion or adjoint comes near the end of float's range (its
// state has blown up numerically while its cost is still finite) is pulled back
// step by step, as adjoint.hip does, so that the products that overflow are the
// same ones. That is a chain as long as the serial kernel's, so it must not start
// after the rest: the final states tell such candidates beforehand, and the first
// workgroups of the launch take them, 32 candidates' worth each, while the others
// leave them out. What only shows on the way (the adjoint, or a state that the
// goal froze behind) is pulled back again by its own workgroup at its end. 4 096
// candidates x 100 steps on side slopes, where a few per cent blow up: 317 to 485
// us with all of them pulled back at the end, 217 to 243 now, 322 serially.
#include "adjoint_step.h"

namespace plan {
namespace {

constexpr int BATCH = 16;       // steps linearised at a time
constexpr int WAVES = 5;        // four linearise, the last one pulls back
// No product of a step's linearisation overflows below these: up to rates of 1e28
// the gradients of 1 300 blown-up candidates had the infinities and NaN of the
// serial pass (and its values, but for rounding).
constexpr float WILD_RATE = 1e18f;  // m/s or rad/s
constexpr float WILD_ADJOINT = 1e28f;
constexpr int FRONT = 32;  // candidates that a workgroup at the front looks at

// A - 1 and the gradient of the running cost, by columns: the thirteen states,
// dd, ax (column 15 is not used). Rows in quads (x, y, z, psi), (th, ph, vy,
// vz), (wx, wy, wz, running cost) and the pair (vx, delta), whose rows have two
// entries each. A step that was not taken has zeros.
struct Batch {
    float4 col[BATCH][4][3][16];
    float2 pair[BATCH][4][16];
};

struct Linear {
    Batch batch[2];
    float st[ADJOINT_LINEAR_STEPS][4][14];  // recomputed states and the executed flag
    float g[ADJOINT_LINEAR_STEPS][4][2];    // the steps' gradients by (dd, ax)
    int early[4], late[4];  // blown up by the final state; seen on the way
    int list[FRONT], listed;  // candidates to pull back step by step
};

struct Column {
    float4 q0, q1, q2;
    float2 pair;
};

// acc0 + acc1 + sum over the rows i of lam_i times row i's entry, lam_i from
// lane i of each row of sixteen lanes (a DPP operand of the multiply-add; the
// wait states it needs after lam's last write are the leading s_nop).
__device__ __forceinline__ float pull_back(float lam, float acc0, float acc1, const Column &r) {
    const float4 &q0 = r.q0, &q1 = r.q1, &q2 = r.q2;
    const float2 &pr = r.pair;
    float acc2;
#define PLAN_ROW(ACC, OP, V, I)                                                          \
    "v_" OP "_f32_dpp %" ACC ", %3, %" V " row_newbcast:" I " row_mask:0xf bank_mask:0xf\n\t"
    asm volatile(  //
        "s_nop 1\n\t"                                                     //
        PLAN_ROW("0", "fmac", "15", "6") PLAN_ROW("2", "mul", "4", "0")     //
        PLAN_ROW("1", "fmac", "5", "1") PLAN_ROW("0", "fmac", "16", "12")   //
        PLAN_ROW("2", "fmac", "6", "2") PLAN_ROW("1", "fmac", "7", "3")     //
        PLAN_ROW("0", "fmac", "8", "4") PLAN_ROW("2", "fmac", "9", "5")     //
        PLAN_ROW("1", "fmac", "10", "7") PLAN_ROW("0", "fmac", "11", "8")   //
        PLAN_ROW("2", "fmac", "12", "9") PLAN_ROW("1", "fmac", "13", "10")  //
        PLAN_ROW("0", "fmac", "14", "11")
        : "+&v"(acc0), "+&v"(acc1), "=&v"(acc2)
        : "v"(lam), "v"(q0.x), "v"(q0.y), "v"(q0.z), "v"(q0.w), "v"(q1.x), "v"(q1.y), "v"(q1.z),
          "v"(q1.w), "v"(q2.x), "v"(q2.y), "v"(q2.z), "v"(pr.x), "v"(pr.y));
#undef PLAN_ROW
    return acc0 + (acc1 + acc2);
}

__device__ __forceinline__ float sum4(float v) { return group_sum<4>(v); }

// What a step's linearisation reads: the state it starts from (and whether it
// was taken), its controls, and this lane's wheel's terrain.
struct StepIn {
    float st[13], flag, u0, u1;
    Attitude A;
    Gather g;
};

// Linearises one step of one candidate, this lane's wheel r of the four; the
// lane of the group that has `write` stores the columns at col and pair.
template <bool CM>
__device__ __forceinline__ void linearise(const RolloutArgs &a, const Arm &r, const StepIn &in,
                                          bool write, float4 (&col)[3][16], float2 (&pair)[16]) {
    const float (&st)[13] = in.st;
    const float u0 = in.u0, u1 = in.u1;
    const bool live = in.flag != 0.0f;
    const float h = live ? a.h : 0.0f;
    const float dd = clampf_nan(u0, -a.drate_max, a.drate_max);
    const float ax = a.accel_max * clampf_nan(u1, -1.0f, 1.0f);
    const float ph = st[5];
    const float vx = st[6], vy = st[7], vz = st[8];
    const float wx = st[9], wy = st[10], wz = st[11];
    const float delta = st[12];

    const Attitude &A = in.A;
    const Gather &g = in.g;
    const GridPos gp = grid_pos(a, st[0], st[1]);
    const Kin kn = kinematics(A, st);
    float sps, cps;
    __sincosf(st[3], &sps, &cps);

    // ---- this lane's wheel
    const float ur = fmaf(A.R11, r.gx, fmaf(A.R12, r.gy, fmaf(A.R13, r.gz, gp.xg)));
    const float vr = fmaf(A.R21, r.gx, fmaf(A.R22, r.gy, fmaf(A.R23, r.gz, gp.yg)));
    // per world metre; 0 where the lookup is clamped to the edge (NaN: clamped)
    const float su = (ur > 0.0f && ur < a.umax) ? a.inv_res : 0.0f;
    const float sv = (vr > 0.0f && vr < a.vmax) ? a.inv_res : 0.0f;
    const float px = fmaf(A.R11, r.rx, fmaf(A.R12, r.ry, A.R13 * r.rz));
    const float py = fmaf(A.R21, r.rx, fmaf(A.R22, r.ry, A.R23 * r.rz));
    const float pz = fmaf(A.R31, r.rx, fmaf(A.R32, r.ry, A.R33 * r.rz));
    const float vix = fmaf(wy, r.rz, fmaf(-wz, r.ry, vx));
    const float viy = fmaf(wz, r.rx, fmaf(-wx, r.rz, vy));
    const float viz = fmaf(wx, r.ry, fmaf(-wy, r.rx, vz));
    const float sind = __sinf(delta), cosd = __cosf(delta);
    const bool guard = vix == 0.0f && viy == 0.0f;
    const float ivx = frcp(vix);
    const float rr = guard ? 0.0f : viy * ivx;
    const float alpha = (guard ? 0.0f : atan_mm(rr)) - (r.front ? delta : 0.0f);
    const float Ca = a.C * alpha;
    const float q = frsq(fmaf(Ca, Ca, a.mu2));
    // slip angle's gradient: (al_x, al_y) by the contact velocity
    const float al_y = guard ? 0.0f : ivx / fmaf(rr, rr, 1.0f);
    const float al_x = -rr * al_y;

    const float hgt = bil(g.ch, g.tx, g.ty);
    const float fx = bil(g.cfx, g.tx, g.ty);
    const float fy = bil(g.cfy, g.tx, g.ty);
    const float nBx = fmaf(-A.R11, fx, fmaf(-A.R21, fy, A.R31));
    const float nBy = fmaf(-A.R12, fx, fmaf(-A.R22, fy, A.R32));
    const float nBz = fmaf(-A.R13, fx, fmaf(-A.R23, fy, A.R33));
    const float inz = frcp(nBz);
    const float gap = g.Pz - hgt;
    const float chi = gap * inz;
    const float relx = fmaf(-chi, wy, vix);
    const float rely = fmaf(chi, wx, viy);
    const float D = fmaf(nBx, relx, fmaf(nBy, rely, nBz * viz));
    const float chid = D * inz;
    const float k = r.front ? a.kf : a.kr;
    const float b = r.front ? a.bf : a.br;
    const float Fkr = fmaf(-k, chi, r.front ? a.Fsf : a.Fsr);
    const float Fk = fmaxf(Fkr, 0.0f);
    const bool damps = (-b * chid) >= -Fk;  // the damper's branch, not the liftoff's
    const float Fb = (Fk > 0.0f) ? fmaxf(-b * chid, -Fk) : 0.0f;
    const float Fz = Fk + Fb;
    const float tire = -Ca * a.mu;
    const float Fy = (Fz * tire) * q;

    // the load's gradient: by chi and chid, then by the terrain normal in the
    // body (n), the contact point (P) and the contact velocity (gv)
    const float by_chid = (Fk > 0.0f && damps) ? -b : 0.0f;
    const float by_chi = (Fkr >= 0.0f && !(Fk > 0.0f && !damps)) ? -k : 0.0f;
    const float LD = inz * by_chid;
    const float gvx = nBx * LD, gvy = nBy * LD, gvz = nBz * LD;
    const float Lchi = fmaf(wx, gvy, fmaf(-wy, gvx, by_chi));
    const float nx = relx * LD, ny = rely * LD;
    const float nz = fmaf(viz, LD, -(inz * inz) * fmaf(D, by_chid, gap * Lchi));
    const float Wx = fmaf(A.R11, nx, fmaf(A.R12, ny, A.R13 * nz));
    const float Wy = fmaf(A.R21, nx, fmaf(A.R22, ny, A.R23 * nz));
    const float Wz = fmaf(A.R31, nx, fmaf(A.R32, ny, A.R33 * nz));
    const float PZ = inz * Lchi;
    auto dtx = [&](const float4 &c) { return fmaf(g.ty, c.w, c.y); };
    auto dty = [&](const float4 &c) { return fmaf(g.tx, c.w, c.z); };
    const float PX = -su * fmaf(dtx(g.ch), PZ, fmaf(dtx(g.cfx), Wx, dtx(g.cfy) * Wy));
    const float PY = -sv * fmaf(dty(g.ch), PZ, fmaf(dty(g.cfx), Wx, dty(g.cfy) * Wy));
    const float mx = fmaf(py, PZ, fmaf(-pz, PY, fmaf(fy, Wz, Wy)));
    const float my = fmaf(pz, PX, fmaf(-px, PZ, -fmaf(fx, Wz, Wx)));
    const float mz = fmaf(px, PY, fmaf(-py, PX, fmaf(fx, Wy, -fy * Wx)));
    // about the axes of psi, th and ph
    auto by_th = [&](float x, float y) { return fmaf(cps, y, -sps * x); };
    auto by_ph = [&](float x, float y, float z) {
        return fmaf(A.R11, x, fmaf(A.R21, y, A.R31 * z));
    };
    const float rzc = r.rz - chi;
    const float Z[12] = {PX, PY, PZ, mz, by_th(mx, my), by_ph(mx, my, mz), gvx, gvy, gvz,
                         fmaf(r.ry, gvz, -rzc * gvy), fmaf(rzc, gvx, -r.rx * gvz),
                         fmaf(r.rx, gvy, -r.ry * gvx)};
    // lateral force fy = (cos delta) Fz tire q: by the load and the slip angle
    const float turn = r.front ? cosd : 1.0f;
    const float by_z = turn * (tire * q);
    const float by_a =
        turn * (a.C * fmaf(Fz * -a.mu, q, (-Ca * (q * q) * q) * (Fz * tire)));
    const float al[12] = {0, 0, 0, 0, 0, 0, al_x, al_y, 0,
                          -r.rz * al_y, r.rz * al_x, fmaf(r.rx, al_y, -r.ry * al_x)};

    // ---- chassis
    const float icth = frcp(A.cth);
    const float t1 = kn.psid * A.cth;
    const float ang = fabsf(ph) + a.phibar;
    const float sang = __sinf(ang), cang = __cosf(ang);
    const float MgR = (ang > 1.57079632679489662f) ? -a.MgRbar : a.MgRbar;
    const float mm_raw = fmaf(-(MgR * (1.0f - sang) * A.cth), a.inv_eps_esm, 1.0f);
    const float mm = fmaxf(0.0f, mm_raw);
    const float by_U = (mm_raw >= 0.0f) ? -a.inv_eps_esm * (2.0f * a.sigma * mm) : 0.0f;
    const float esm_th = -MgR * (1.0f - sang) * A.sth * by_U;
    const float esm_ph = (ph < 0.0f ? MgR : -MgR) * cang * A.cth * by_U;
    const float F2 = -2.0f * a.hR * a.Mhalf;  // the pitch moment per FxR / Mhalf
    const float hM = h * a.invM, hx = h * a.invJxx, hy = h * a.invJyy, hz = h * a.invJzz;

    // running cost of the terrain: by the position, and its torque
    float cX = 0.0f, cY = 0.0f, cpsi = 0.0f, cth = esm_th, cph = esm_ph;
    if constexpr (CM) {
        const float gx = su * dtx(g.cc), gy = sv * dty(g.cc);
        const float tx = -pz * gy, ty = pz * gx, tz = fmaf(px, gy, -py * gx);
        cX = sum4(gx);
        cY = sum4(gy);
        cpsi = sum4(tz);
        cth += sum4(by_th(tx, ty));
        cph += sum4(by_ph(tx, ty, tz));
    }
    const float hpi = h * icth;
    // what the wheels do not give of each column: the rows' chassis terms
    // (vy, vz before h; Mx, My, Mz before h / J) and the running cost
    struct Rest {
        float vy, vz, Mx, My, Mz, cost;
    };
    const Rest rest[12] = {
        {0, 0, 0, 0, 0, cX},
        {0, 0, 0, 0, 0, cY},
        {0, 0, 0, 0, 0, 0},
        {0, 0, 0, 0, 0, cpsi},
        {a.g * (A.sth * A.sph), a.g * (A.sth * A.cph), 0, F2 * (-a.g * A.cth), 0, cth},
        {-a.g * A.R33, a.g * A.R32, 0, 0, 0, cph},
        {-wz, wy, 0, 0, 0, 0},
        {0, -wx, 0, F2 * -wz, 0, 0},
        {wx, 0, 0, F2 * wy, 0, 0},
        {vz, -vy, 0, -a.dJxz * wz, a.dJxy * wy, 0},
        {0, vx, a.dJyz * wz, F2 * vz, a.dJxy * wx, 0},
        {-vx, 0, a.dJyz * wy, fmaf(F2, -vy, -a.dJxz * wx), 0, 0}};
    // kinematic rows x, y, z, psi and th, ph of each column (x, y, z have none)
    const float hsp = hpi * A.sph, hcp = hpi * A.cph, htd = hpi * kn.thd;
    const float4 kin0[12] = {
        {}, {}, {},
        {-h * kn.vWy, h * kn.vWx, 0, 0},
        {h * (cps * kn.vWz), h * (sps * kn.vWz), -h * fmaf(sps, kn.vWy, cps * kn.vWx),
         kn.psid * A.sth * hpi},
        {h * fmaf(A.R21, kn.vWz, -A.R31 * kn.vWy), h * fmaf(A.R31, kn.vWx, -A.R11 * kn.vWz),
         h * fmaf(A.R11, kn.vWy, -A.R21 * kn.vWx), htd},
        {h * A.R11, h * A.R21, h * A.R31, 0},
        {h * A.R12, h * A.R22, h * A.R32, 0},
        {h * A.R13, h * A.R23, h * A.R33, 0},
        {0, 0, 0, 0},
        {0, 0, 0, hsp},
        {0, 0, 0, hcp}};
    const float kin1[12][2] = {{0, 0}, {0, 0}, {0, 0}, {0, 0},
                               {0, kn.psid * hpi},
                               {-h * t1, A.sth * htd},
                               {0, 0}, {0, 0}, {0, 0},
                               {0, h},
                               {h * A.cph, A.sth * hsp},
                               {-h * A.sph, A.sth * hcp}};
#pragma unroll
    for (int j = 0; j < 12; ++j) {
        const float Y = (j >= 6 && j != 8) ? fmaf(by_a, al[j], by_z * Z[j]) : by_z * Z[j];
        const float SF = sum4(Y), SZ = sum4(Z[j]);
        const float SX = sum4(r.ry * Z[j]), ST = sum4(r.rx * Z[j]), SU = sum4(r.rx * Y);
        const Rest &c = rest[j];
        const float vyr = fmaf(hM, SF, h * c.vy), vzr = fmaf(hM, SZ, h * c.vz);
        const float wxr = hx * (fmaf(a.hR, SF, SX) + c.Mx);
        const float wyr = hy * (c.My - ST);
        const float wzr = hz * (SU + c.Mz);
        if (write) {
            // columns x, y, z have no kinematic rows: zeroed once by the kernel
            if (j >= 3) col[0][j] = kin0[j];
            col[1][j] = make_float4(kin1[j][0], kin1[j][1], vyr, vzr);
            col[2][j] = make_float4(wxr, wyr, wzr, h * c.cost);
        }
    }
    {
        const float Yd = r.front ? fmaf(-sind, Fy, -by_a) : 0.0f;
        const float SF = sum4(Yd), SU = sum4(r.rx * Yd);
        const float vx_new = fmaf(a.h, ax, vx), d_new = fmaf(a.h, dd, delta);
        const bool floor_v = live && vx_new < a.vx_min;
        const bool limit_d = live && (d_new < -a.delta_max || d_new > a.delta_max);
        if (write) {
            col[1][12] = make_float4(0, 0, hM * SF, 0);
            col[2][12] = make_float4(hx * (a.hR * SF), 0, hz * SU, 0);
            col[2][13] = make_float4(0, 0, 0, h * (2.0f * a.w_c * dd));
            col[2][14] = make_float4(0, hy * F2, 0, 0);
            pair[6].x = floor_v ? -1.0f : 0.0f;
            pair[12].y = limit_d ? -1.0f : 0.0f;
            pair[13].y = limit_d ? 0.0f : h;
            pair[14].x = floor_v ? 0.0f : h;
        }
    }
}

// The arguments are those of adjoint_backward in adjoint.hip; a segment has at
// most ADJOINT_LINEAR_STEPS steps. The first `front` workgroups take the blown-up
// candidates, the others four candidates each.
template <bool CM>
__global__ __launch_bounds__(64 * WAVES, 1) void adjoint_linear(
    const RolloutArgs a, int C, const float *__restrict__ ckpt,
    const float *__restrict__ weight, float *__restrict__ grad, int front) {
    __shared__ Linear L;
    const int t = threadIdx.x, lane = t & 63;
    const bool pulls = t >= 64 * (WAVES - 1);
    const size_t K = (size_t)a.K;
    const int N = a.N, S = a.S;
    const int nseg = (N + C - 1) / C;
    const int segs = ADJOINT_LINEAR_STEPS / (C * S);  // recomputed together

    // recompute and linearise: wheel t & 3 of candidate c
    const int wheel_i = t & 3, c = (t >> 2) & 3;
    const bool at_front = (int)blockIdx.x < front;
    const int k0 = at_front ? 0 : ((int)blockIdx.x - front) * 4;
    const size_t kc = (size_t)min(k0 + c, a.K - 1);
    const float *up = a.controls + kc;
    const Arm arms[1] = {arm(a, wheel_i)};
    const bool finite_c = isfinite(a.cost[kc]);
    const bool some = __any(finite_c);  // of the workgroup's four

    // the pull-back: lane j of candidate cj
    const int j = lane & 15, cj = lane >> 4;
    const size_t kjc = (size_t)min(k0 + cj, a.K - 1);
    const float wJ = weight ? weight[kjc] : 1.0f;
    float lam = 0.0f, peak = 0.0f;  // peak: largest |lam|, NaN if one is
    // terminal cost Phi = w_g |(x, y) - goal| at the final state
    auto terminal = [&](size_t k, float w, float &lx, float &ly) {
        const float gdx = ckpt[((size_t)nseg * 13 + 0) * K + k] - a.goal_x;
        const float gdy = ckpt[((size_t)nseg * 13 + 1) * K + k] - a.goal_y;
        const float dist = sqrtf(fmaf(gdx, gdx, gdy * gdy));
        lx = dist > 0.0f ? w * a.w_g * gdx / dist : 0.0f;
        ly = dist > 0.0f ? w * a.w_g * gdy / dist : 0.0f;
    };
    auto blown_up = [&](size_t k) {
        const float *fs = ckpt + ((size_t)nseg * 13 + 6) * K + k;
        float m = fabsf(fs[0]);
#pragma unroll
        for (int q = 1; q < 6; ++q) m = maxn(m, fabsf(fs[(size_t)q * K]));
        return isfinite(a.cost[k]) && !(m < WILD_RATE);
    };

    // The states at which candidate kc's steps of segments [lo, hi) start; one with
    // a cost that is not finite has gradient zero and takes none.
    auto recompute = [&](size_t kc, bool finite, int lo, int hi) {
        const float *up = a.controls + kc;
        const int n_lo = lo * C;
        for (int seg = lo + (t >> 4); seg < hi; seg += 4 * WAVES) {
            const int n0 = seg * C;
            const int n1 = min(N, n0 + C);
            float st[13];
#pragma unroll
            for (int q = 0; q < 13; ++q) st[q] = ckpt[((size_t)seg * 13 + q) * K + kc];
            float Jdummy = 0.0f;
            int idx = (n0 - n_lo) * S;
            float nu0 = up[(2 * (size_t)n0) * K], nu1 = up[(2 * (size_t)n0 + 1) * K];
            for (int n = n0; n < n1; ++n) {
                const float dd = clampf_nan(nu0, -a.drate_max, a.drate_max);
                const float ax = a.accel_max * clampf_nan(nu1, -1.0f, 1.0f);
                const size_t nn = (size_t)min(n + 1, n1 - 1);
                for (int s = 0; s < S; ++s, ++idx) {
                    const float gdx = st[0] - a.goal_x, gdy = st[1] - a.goal_y;
                    const bool live = finite && !(fmaf(gdx, gdx, gdy * gdy) <= a.goal_r2);
                    if (wheel_i == 0) {
                        float *sl = &L.st[idx][c][0];
#pragma unroll
                        for (int q = 0; q < 13; ++q) sl[q] = st[q];
                        sl[13] = live ? 1.0f : 0.0f;
                    }
                    // a candidate at its goal stays frozen, so the stale
                    // controls are never applied; the segment's last step
                    // leads to the next checkpoint
                    if (live && (n + 1 < n1 || s + 1 < S))
                        euler_step<4, false>(a, arms, st, Jdummy, dd, ax, [&]() {
                            nu0 = up[(2 * nn) * K];
                            nu1 = up[(2 * nn + 1) * K];
                        });
                }
            }
        }
    };

    if (t == 0) L.listed = 0;
    if (at_front) {
        __syncthreads();
        const int k = (int)blockIdx.x * FRONT + t;
        if (t < FRONT && k < a.K && blown_up(k)) L.list[atomicAdd(&L.listed, 1)] = k;
    } else {
        {
            float lx, ly;
            terminal(kjc, wJ, lx, ly);
            lam = j == 0 ? lx : j == 1 ? ly : 0.0f;
        }
        // entries no step writes
        for (int i = some ? t : 2 * BATCH * 4 * 16; i < 2 * BATCH * 4 * 16; i += 64 * WAVES) {
            Batch &B = L.batch[i / (BATCH * 4 * 16)];
            const int o = i % (BATCH * 4 * 16);
            float4 *cl = &B.col[0][0][0][0] + (o >> 4) * 48 + (o & 15);
            (&B.pair[0][0][0])[o] = make_float2(0, 0);
            cl[0] = cl[16] = cl[32] = make_float4(0, 0, 0, 0);
        }
        if (t < 4) {
            L.early[t] = blown_up((size_t)min(k0 + t, a.K - 1));
            L.late[t] = 0;
        }
        for (int hi = nseg; hi > 0; hi -= segs) {
            const int lo = max(hi - segs, 0);  // segments [lo, hi)
            const int n_lo = lo * C;
            const int count = min(N, hi * C) - n_lo;  // their intervals
            __syncthreads();
            if (some) recompute(kc, finite_c, lo, hi);
            __syncthreads();
            // Steps after the four have reached the goal leave lam as it is, and
            // those of a candidate whose cost is not finite do not count: the
            // batches end before them, as the serial pass skips them. 6 000
            // candidates x 100 that reach it within 0, 10 and 30 steps: 163, 173 and
            // 188 us with them, 63, 95 and 120 without, serially 86, 104 and 143; 516
            // x 210 on ground that turns nearly all of them over 133 serially, 170 and
            // 119. The test costs the others 1 % at most.
            const int steps = count * S;
            auto taken = [&](int i) {
                return L.st[i][0][13] + L.st[i][1][13] + L.st[i][2][13] + L.st[i][3][13] != 0.0f;
            };
            int cnt = some ? steps : 0;
            if (some && !__any(taken(steps - 1))) {
                cnt = 0;
                for (int i = 0; i < steps; i += 64)
                    cnt += __popcll(__ballot(i + lane < steps && taken(min(i + lane, steps - 1))));
            }
            const int batches = (cnt + BATCH - 1) / BATCH;
            // step `slot` of a batch that starts at `first`; past the end the last
            // one, as a step that was not taken
            const int slot = (t >> 4) & (BATCH - 1);
            auto fetch = [&](int first, StepIn &in) {
                const int i = min(first + slot, cnt - 1);
                const float *sl = &L.st[i][c][0];
#pragma unroll
                for (int q = 0; q < 13; ++q) in.st[q] = sl[q];
                in.flag = first + slot < cnt ? sl[13] : 0.0f;
                const size_t n = (size_t)(n_lo + i / S);
                in.A = attitude(in.st[3], in.st[4], in.st[5]);
                in.g = gather<CM>(a, in.A, grid_pos(a, in.st[0], in.st[1]), in.st[2], arms[0]);
                in.u0 = up[(2 * n) * K];
                in.u1 = up[(2 * n + 1) * K];
            };
            StepIn next;
            if (!pulls && batches > 0) fetch((batches - 1) * BATCH, next);
            for (int it = 0; it <= batches; ++it) {
                if (!pulls) {
                    if (it < batches) {
                        const int first = (batches - 1 - it) * BATCH;
                        const StepIn in = next;
                        fetch(max(first - BATCH, 0), next);
                        __builtin_amdgcn_sched_barrier(0);
                        Batch &B = L.batch[it & 1];
                        linearise<CM>(a, arms[0], in, wheel_i == 0, B.col[slot][c], B.pair[slot][c]);
                        float m = fabsf(in.st[6]);
#pragma unroll
                        for (int q = 7; q < 12; ++q) m = maxn(m, fabsf(in.st[q]));
                        if (wheel_i == 0 && finite_c && !(m < WILD_RATE)) L.late[c] = 1;
                    }
                } else if (it > 0) {
                    const Batch &B = L.batch[(it - 1) & 1];
                    float e[BATCH];
                    // columns are read two steps ahead
                    Column r[BATCH];
                    auto read = [&](int b) {
                        r[b] = Column{B.col[b][cj][0][j], B.col[b][cj][1][j], B.col[b][cj][2][j],
                                      B.pair[b][cj][j]};
                    };
                    read(BATCH - 1);
                    read(BATCH - 2);
#pragma unroll
                    for (int b = BATCH - 1; b >= 0; --b) {
                        if (b > 1) read(b - 2);
                        __builtin_amdgcn_sched_barrier(0);
                        lam = pull_back(lam, j < 13 ? lam : 0.0f, wJ * r[b].q2.w, r[b]);
                        e[b] = lam;
                        peak = maxn(peak, fabsf(lam));
                    }
                    if (j == 13 || j == 14) {
                        const int first = (batches - it) * BATCH;
#pragma unroll
                        for (int b = 0; b < BATCH; ++b) L.g[first + b][cj][j - 13] = e[b];
                    }
                }
                __syncthreads();
            }
            // the intervals' gradients, through the admissible-set clamps (identity
            // branch inside)
            for (int i = t; i < count * 8; i += 64 * WAVES) {
                const int n = i >> 3, cg = (i >> 1) & 3, x = i & 1;
                if (k0 + cg >= a.K || L.early[cg]) continue;  // the front's
                const size_t at = (2 * (size_t)(n_lo + n) + x) * K + k0 + cg;
                const float u = a.controls[at], lim = x ? 1.0f : a.drate_max;
                float gs = 0.0f;
                for (int s = min(S, batches * BATCH - n * S) - 1; s >= 0; --s)
                    gs += L.g[n * S + s][cg][x];
                const bool in = !(u < -lim) && !(u > lim) && isfinite(a.cost[k0 + cg]);
                grad[at] = in ? (x ? a.accel_max * gs : gs) : 0.0f;
            }
        }
        if (pulls && j < 15 && !(peak < WILD_ADJOINT) && isfinite(a.cost[kjc])) L.late[cj] = 1;
        __syncthreads();
        if (t < 4 && k0 + t < a.K && L.late[t] && !L.early[t])
            L.list[atomicAdd(&L.listed, 1)] = k0 + t;
    }
    __syncthreads();

    // step by step, four candidates at a time (the first sixteen lanes)
    const int listed = L.listed;
    // the gradients stored above are stored over (a fence in every workgroup
    // would cost 0.1 us each: they write back the same L2s)
    if (listed > 0) __threadfence();
    for (int from = 0; from < listed; from += 4) {
        const size_t kr = (size_t)L.list[min(from + c, listed - 1)];
        const float *ur = a.controls + kr;
        const float w = weight ? weight[kr] : 1.0f;
        const bool redo = t < 16 && from + c < listed;
        float lv[13];
#pragma unroll
        for (int q = 0; q < 13; ++q) lv[q] = 0.0f;
        terminal(kr, w, lv[0], lv[1]);
        for (int hi = nseg; hi > 0; hi -= segs) {
            const int lo = max(hi - segs, 0);
            const int n_lo = lo * C;
            __syncthreads();
            recompute(kr, true, lo, hi);
            __syncthreads();
            if (!redo) continue;
            float gdd = 0.0f, gax = 0.0f;
            for (int n = min(N, hi * C) - 1; n >= n_lo; --n) {
                const float u0 = ur[(2 * (size_t)n) * K], u1 = ur[(2 * (size_t)n + 1) * K];
                const float dd = clampf_nan(u0, -a.drate_max, a.drate_max);
                const float ax = a.accel_max * clampf_nan(u1, -1.0f, 1.0f);
                for (int s = S - 1; s >= 0; --s) {
                    const float *sl = &L.st[(n - n_lo) * S + s][c][0];
                    if (sl[13] != 0.0f) {
                        float st[13], g1, g2;
#pragma unroll
                        for (int q = 0; q < 13; ++q) st[q] = sl[q];
                        step_vjp<4>(a, arms, st, dd, ax, w, lv, &g1, &g2);
                        gdd += g1;
                        gax += g2;
                    }
                }
                const bool in0 = !(u0 < -a.drate_max) && !(u0 > a.drate_max);
                const bool in1 = !(u1 < -1.0f) && !(u1 > 1.0f);
                if (wheel_i == 0) {
                    grad[(2 * (size_t)n) * K + kr] = in0 ? gdd : 0.0f;
                    grad[(2 * (size_t)n + 1) * K + kr] = in1 ? a.accel_max * gax : 0.0f;
                }
                gdd = 0.0f;
                gax = 0.0f;
            }
        }
    }
}

}  // namespace

hipError_t launch_adjoint_linear(const RolloutArgs &a, int C, const float *ckpt,
                                 const float *weight, float *grad, hipStream_t s) {
    if ((long long)C * a.S > ADJOINT_LINEAR_STEPS) return hipErrorInvalidValue;
    const int front = (a.K + FRONT - 1) / FRONT;
    const dim3 grid((unsigned)((a.K + 3) / 4 + front));
    if (a.has_costmap)
        hipLaunchKernelGGL(adjoint_linear<true>, grid, dim3(64 * WAVES), 0, s, a, C, ckpt, weight,
                           grad, front);
    else
        hipLaunchKernelGGL(adjoint_linear<false>, grid, dim3(64 * WAVES), 0, s, a, C, ckpt,
                           weight, grad, front);
    return hipGetLastError();
}

}  // namespace plan
