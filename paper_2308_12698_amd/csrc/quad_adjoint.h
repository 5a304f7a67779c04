/*
 * quad_adjoint.h -- hand-written reverse mode (vector-Jacobian product) of
 * one quadrotor time step, FP32, one agent per lane.
 *
 * Forward step (quad_step.h): controller -> held rotor command dc; classical
 * RK4 over v, q, w, d (and p, J, which only integrate) with dc held;
 * quaternion renormalisation.  step_vjp() recomputes the RK4
 * stages of one step from its replayed start and then applies the
 * transposed derivatives in reverse order:
 *     renormalisation -> RK4 stages 4, 3, 2, 1 -> controller.
 * Non-smooth points take the derivative of the branch the forward pass
 * took: a clamp passes the cotangent inside its interval and stops it
 * outside; the error-quaternion sign is a constant; sqrt'(0) is taken as 0.
 * The branches are the forward's own decisions, recorded by the replay of
 * the forward from its checkpoints (the same bits), as is the rotor command
 * held through the step; the controller's integrals are the forward's too, bit
 * for bit (undo).  The reverse sweep does not decide any branch itself.  The
 * rounding carries of the forward integrator are not differentiated (the represented value is row + carry, so both have the
 * same cotangent).
 */
#pragma once

#include "kernels.h"
#include "quad_step.h"

namespace potato {

/* Cotangents of the 30 physical state rows. */
struct AgentAdj {
    float p[3], v[3], q[4], w[3], d[4], J;
    float ip[3], ia[3], ir[3], wprev[3];
};

/* Cotangent of a stage's rates of v, q and w, and of sum_i s_i's share in
 * the cost.  h is the cotangent of q o (0, w), i.e. half that of the
 * quaternion rate q o (0, w) / 2, so the kinematics need no factor. */
struct RateAdj {
    float v[3], h[4], w[3], J;
};

/* Dynamic part of a stage's state that the Jacobian reads (it does not
 * depend on the velocity: drag is linear). */
struct Dyn {
    float q[4], w[3], d[4];
};

/* Transpose of the Jacobian of the right-hand side (eqs. qd2-qd4, 2, 3) at y,
 * applied to mu (ssum: y's sum of s_i, as rates() returns it): adds the stage state's cotangent to (lq, lw) and sets lsd
 * to that of the stage's rotor deviations through thrust and torque (the
 * rotor lag's own part is in closed form, see step_vjp).  With FIRST, lq and
 * lw hold nothing yet.  The velocity's part is -(c_d/m) mu.v, left to the
 * caller.  Products with inverse inertia use the per-type constants of the
 * forward step: (I_z - I_y)/I_x = gx etc., k_f L sin(a)/I_x = ax etc. */
template <bool FIRST>
__device__ __forceinline__ void derivative_vjp(const TypeConst& c, const Dyn& y, float ssum, const RateAdj& mu,
                                               float lq[4], float lw[3], float lsd[4]) {
#pragma clang fp contract(off)
    const float *q = y.q, *w = y.w, *d = y.d, *h = mu.h;
    const float ftm2 = POTATO_FMA(c.kf_m2, ssum, c.F0_2);
    const float bx2 = POTATO_FMA(q[0], q[2], q[1] * q[3]);
    const float by2 = POTATO_FMA(q[2], q[3], -(q[0] * q[1]));
    const float x2y2 = POTATO_FMA(q[1], q[1], q[2] * q[2]);

    /* translational part: v' = ftm2 (bx2, by2, 1/2 - x2y2) - (c_d/m) v - g z */
    const float l_ftm2 = POTATO_FMA(-mu.v[2], x2y2, POTATO_FMA(mu.v[1], by2, mu.v[0] * bx2));
    const float l_ssum = POTATO_FMA(c.kf_m2, l_ftm2, POTATO_FMA(c.kf_m, mu.v[2], mu.J));
    const float m0 = ftm2 * mu.v[0], m1 = ftm2 * mu.v[1], m2 = (ftm2 + ftm2) * mu.v[2];
    auto first = [](float acc, float x, float y) { return FIRST ? x * y : POTATO_FMA(x, y, acc); };
    lq[0] = POTATO_FMA(-m1, q[1], first(lq[0], m0, q[2]));
    lq[1] = POTATO_FMA(-m2, q[1], POTATO_FMA(-m1, q[0], first(lq[1], m0, q[3])));
    lq[2] = POTATO_FMA(-m2, q[2], POTATO_FMA(m1, q[3], first(lq[2], m0, q[0])));
    lq[3] = POTATO_FMA(m1, q[2], first(lq[3], m0, q[1]));

    /* quaternion kinematics q o (0, w) */
    lq[0] = POTATO_FMA(w[2], h[3], POTATO_FMA(w[1], h[2], POTATO_FMA(w[0], h[1], lq[0])));
    lq[1] = POTATO_FMA(w[1], h[3], POTATO_FMA(-w[2], h[2], POTATO_FMA(-w[0], h[0], lq[1])));
    lq[2] = POTATO_FMA(-w[0], h[3], POTATO_FMA(w[2], h[1], POTATO_FMA(-w[1], h[0], lq[2])));
    lq[3] = POTATO_FMA(w[0], h[2], POTATO_FMA(-w[1], h[1], POTATO_FMA(-w[2], h[0], lq[3])));
    lw[0] = POTATO_FMA(-q[2], h[3], POTATO_FMA(q[3], h[2], POTATO_FMA(-q[1], h[0], first(lw[0], q[0], h[1]))));
    lw[1] = POTATO_FMA(-q[3], h[1], POTATO_FMA(q[1], h[3], POTATO_FMA(-q[2], h[0], first(lw[1], q[0], h[2]))));
    lw[2] = POTATO_FMA(-q[1], h[2], POTATO_FMA(q[2], h[1], POTATO_FMA(-q[3], h[0], first(lw[2], q[0], h[3]))));

    /* Euler's equations: w' = (ax (A + B), ay (P23 - P01), az (A - B)) - (gx w1 w2, gy w2 w0, gz w0 w1) */
    const float b0 = c.gx * mu.w[0], b1 = c.gy * mu.w[1], b2 = c.gz * mu.w[2];
    lw[0] = POTATO_FMA(-b2, w[1], POTATO_FMA(-b1, w[2], lw[0]));
    lw[1] = POTATO_FMA(-b0, w[2], POTATO_FMA(-b2, w[0], lw[1]));
    lw[2] = POTATO_FMA(-b1, w[0], POTATO_FMA(-b0, w[1], lw[2]));

    /* rotor model and allocation (eqs. 2, 3) through s_i = W_i^2 - w_ref^2 */
    const float tX = c.ax * mu.w[0], tY = c.ay * mu.w[1], tZ = c.az * mu.w[2];
    const float pz = l_ssum + tZ, mz = l_ssum - tZ, u = tX - tY, v = tX + tY;
    const float ls[4] = {pz + u, mz - v, pz - u, mz + v};
#pragma unroll
    for (int i = 0; i < 4; ++i) lsd[i] = ls[i] * POTATO_FMA(2.0f, d[i], c.two_w);
}

/* All ones where branch bit POS is set (a bit-field extract: the compiler
 * makes a comparison and a selection of every expression of it), and x there,
 * +0 elsewhere. */
template <int POS>
__device__ __forceinline__ int32_t bit_mask(uint32_t bits) {
    int32_t mask;
    asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(mask) : "v"(bits), "n"(POS));
    return mask;
}
__device__ __forceinline__ float where(int32_t mask, float x) {
    return __builtin_bit_cast(float, __builtin_bit_cast(int32_t, x) & mask);
}

/* What the reverse of one step reads of its forward: the step-start state,
 * the controller's integrals after their update, the change of the body
 * rates since the previous step, the rotor command held through the step
 * and the branch decisions (kBit*). */
struct Replay {
    float p[3], v[3], q[4], w[3], d[4], ip[3], ia[3], ir[3], dw[3], dc[4];
    uint32_t bits, off;                       /* kBit*, undo offsets */
};

/* Where the undo offsets are: five of the attitude and rate integrals' in a
 * word of their own, the sixth and the position's above the branch
 * decisions, and above those whether the tape holds the integrals themselves
 * in their place. */
constexpr int kUndoWord = 5;
constexpr int kUndoAt = 16, kUndoPosAt = kUndoAt + kUndoRate;
constexpr uint32_t kWholeBit = 1u << 31;
static_assert(kUndoWord * kUndoRate <= 32 && kUndoPosAt + 3 * kUndoPos <= 31, "the offsets' places");
__device__ __forceinline__ uint32_t field(uint32_t word, int at, int bits) { return word >> at & ((1u << bits) - 1u); }
/* of the position's integral i, of the attitude's (k = i) and the rate's (k = 3 + i) */
__device__ __forceinline__ uint32_t pos_offset(const Replay& a, int i) {
    return field(a.bits, kUndoPosAt + kUndoPos * i, kUndoPos);
}
__device__ __forceinline__ uint32_t rate_offset(const Replay& a, int k) {
    return k < kUndoWord ? field(a.off, kUndoRate * k, kUndoRate) : field(a.bits, kUndoAt, kUndoRate);
}

/*
 * Reverse of one step.  `a` is its replay, wp the waypoint of this step and
 * k the gains; on return a.ip, a.ia and a.ir are the integrals before the
 * step where the undo offsets hold them (not kWholeBit).  lam
 * holds the cotangent of
 * the step-end state on entry and of the step-start state on return; gk
 * accumulates the gain cotangents, the last one (kdr) times dt: gk[8] is
 * divided by dt once at the end of the sweep (kdr_from_sum).
 *
 * Bound by the tape's traffic and by instruction issue at the two waves per
 * SIMD its registers allow, so it is written for few instructions, every one
 * placed: sums accumulate in fused multiply-adds onto what is there already
 * (no zero-initialised temporaries), the last reversed stage accumulates
 * into lam itself, the rotor lag's cotangents come from its closed form
 * (d_stage = dc + (d - dc) c_stage) instead of through the stages, and masks
 * are bit-field extracts.  1,190 vector instructions became 980 (backward at
 * 1,048,576 agents, K = 50: 59.0 to 57.7 us per step; the integrals left off
 * the tape, 251 to 183 B per agent-step: 50.3).
 */
__device__ __forceinline__ void step_vjp(const TypeConst& c, const Limits& L, const Gains& k,
                                         Replay& a, const float wp[3], AgentAdj& lam, float gk[9]) {
#pragma clang fp contract(off)
    const float* const dc = a.dc;
    const uint32_t bits = a.bits;
    /* ---------------- RK4 forward, keeping the stage states ----------------
     * (the forward step's own arithmetic: rates() with the quaternion rate's
     * factor 1/2 on the step sizes, and the rotor lag's closed-form stage
     * values, so the stage states are the forward's bits) */
    const float z = -(L.dt * c.inv_tau);
    const float hz = 0.5f * z;
    const float c2 = 1.0f + hz;
    const float c3 = POTATO_FMA(hz, c2, 1.0f);
    const float c4 = POTATO_FMA(z, c3, 1.0f);
    const float zR = z * (1.0f / 6.0f), sR = ((1.0f + (c2 + c2)) + (c3 + c3)) + c4;
    Dyn y1, y2, y3, y4;
    float kv[3], kq[4], kw[3], aq[4];
#pragma unroll
    for (int i = 0; i < 3; ++i) y1.w[i] = a.w[i];
#pragma unroll
    for (int i = 0; i < 4; ++i) { y1.q[i] = a.q[i]; y1.d[i] = a.d[i]; }
    auto stage = [&](const Dyn& from, float hw, float hq, float cp, Dyn& to) {
        const float ssum = rates(c, a.v, from.q, from.w, from.d, kv, kq, kw);      /* kv is not used */
#pragma unroll
        for (int i = 0; i < 3; ++i) to.w[i] = POTATO_FMA(hw, kw[i], y1.w[i]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            to.q[i] = POTATO_FMA(hq, kq[i], y1.q[i]);
            to.d[i] = POTATO_FMA(a.d[i] - dc[i], cp, dc[i]);
        }
        return ssum;
    };
    const float ss1 = stage(y1, L.half_dt, L.quarter_dt, c2, y2);
#pragma unroll
    for (int i = 0; i < 4; ++i) aq[i] = kq[i];
    const float ss2 = stage(y2, L.half_dt, L.quarter_dt, c3, y3);
#pragma unroll
    for (int i = 0; i < 4; ++i) aq[i] = POTATO_FMA(2.0f, kq[i], aq[i]);
    const float ss3 = stage(y3, L.dt, L.half_dt, c4, y4);
#pragma unroll
    for (int i = 0; i < 4; ++i) aq[i] = POTATO_FMA(2.0f, kq[i], aq[i]);
    const float ss4 = rates(c, a.v, y4.q, y4.w, y4.d, kv, kq, kw);
    float qn[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) qn[i] = POTATO_FMA(L.dt12, aq[i] + kq[i], a.q[i]);

    /* ---------------- reverse: renormalisation ---------------- */
    {
        const float r = rsq(POTATO_FMA(qn[3], qn[3], POTATO_FMA(qn[2], qn[2], POTATO_FMA(qn[1], qn[1], qn[0] * qn[0]))));
        const float u[4] = {qn[0] * r, qn[1] * r, qn[2] * r, qn[3] * r};
        const float dot = POTATO_FMA(u[3], lam.q[3], POTATO_FMA(u[2], lam.q[2], POTATO_FMA(u[1], lam.q[1], u[0] * lam.q[0])));
#pragma unroll
        for (int i = 0; i < 4; ++i) lam.q[i] = r * POTATO_FMA(-u[i], dot, lam.q[i]);
    }

    /* ---------------- reverse: RK4 ----------------
     * lam (v, q, w) is the cotangent of the step-end dynamic state; the stage
     * rate cotangents are b_i * dt * lam + (stage offset) * (cotangent of the
     * next stage's state), with b = 1/6, 1/3, 1/3, 1/6.  Position and cost
     * only integrate, so their cotangents pass through unchanged and enter
     * each stage as b_i * dt * lam.p (on the stage velocity) and
     * b_i * dt * lam.J.  The rotor deviations are dc + (d - dc) c at the
     * stages and dc + (d - dc) R at the end, so the direct cotangents of the
     * stages sum, weighted by c, into that of d and, by 1 - c, into that of
     * dc. */
    const float R = POTATO_FMA(zR, sR, 1.0f);
    float ldc[4];
    RateAdj w6, w3;                           /* dt/6 and dt/3 times the step end's cotangent */
    float p6[3], p3[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        w6.v[i] = L.dt6 * lam.v[i]; w3.v[i] = w6.v[i] + w6.v[i];
        w6.w[i] = L.dt6 * lam.w[i]; w3.w[i] = w6.w[i] + w6.w[i];
        p6[i] = L.dt6 * lam.p[i]; p3[i] = p6[i] + p6[i];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        w6.h[i] = L.dt12 * lam.q[i]; w3.h[i] = w6.h[i] + w6.h[i];
        ldc[i] = -(zR * sR) * lam.d[i];
        lam.d[i] = R * lam.d[i];
    }
    w6.J = L.dt6 * lam.J; w3.J = w6.J + w6.J;
    float sv[3], sq[4], sw[3], lsd[4];
    /* the next earlier stage's rate cotangent: base + offset * this stage's
     * state cotangent */
    auto earlier = [&](const RateAdj& base, float off, float offh) {
        RateAdj mu;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            mu.v[i] = POTATO_FMA(off, sv[i], base.v[i]);
            mu.w[i] = POTATO_FMA(off, sw[i], base.w[i]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) mu.h[i] = POTATO_FMA(offh, sq[i], base.h[i]);
        mu.J = base.J;
        return mu;
    };
    auto reverse_stage = [&](const RateAdj& mu, const float lp[3], const Dyn& y, float ssum, float cp, float ncp) {
        derivative_vjp<true>(c, y, ssum, mu, sq, sw, lsd);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            sv[i] = POTATO_FMA(c.ncd_m, mu.v[i], lp[i]);
            lam.v[i] += sv[i];
            lam.w[i] += sw[i];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            lam.q[i] += sq[i];
            lam.d[i] = POTATO_FMA(cp, lsd[i], lam.d[i]);
            ldc[i] = POTATO_FMA(ncp, lsd[i], ldc[i]);
        }
    };
    reverse_stage(w6, p6, y4, ss4, c4, -(z * c3));
    reverse_stage(earlier(w3, L.dt, L.half_dt), p3, y3, ss3, c3, -(hz * c2));
    reverse_stage(earlier(w3, L.half_dt, L.quarter_dt), p3, y2, ss2, c2, -hz);
    {
        const RateAdj mu = earlier(w6, L.half_dt, L.quarter_dt);
#pragma unroll
        for (int i = 0; i < 3; ++i) lam.v[i] = POTATO_FMA(c.ncd_m, mu.v[i], lam.v[i] + p6[i]);
        derivative_vjp<false>(c, y1, ss1, mu, lam.q, lam.w, lsd);
#pragma unroll
        for (int i = 0; i < 4; ++i) lam.d[i] += lsd[i];
    }

    const int32_t in_ip[3] = {bit_mask<kBitIp>(bits), bit_mask<kBitIp - 1>(bits), bit_mask<kBitIp - 2>(bits)};
    const int32_t in_ia[3] = {bit_mask<kBitIa>(bits), bit_mask<kBitIa - 2>(bits), bit_mask<kBitIa - 4>(bits)};
    const int32_t in_ir[3] = {bit_mask<kBitIr>(bits), bit_mask<kBitIr - 2>(bits), bit_mask<kBitIr - 4>(bits)};
    const int32_t in_f[4] = {bit_mask<kBitRotor>(bits), bit_mask<kBitRotor - 1>(bits), bit_mask<kBitRotor - 2>(bits),
                             bit_mask<kBitRotor - 3>(bits)};

    /* ---------------- controller, forward with intermediates ----------------
     * (the values the reverse needs; the branches are the recorded ones) */
    const float er[3] = {wp[0] - a.p[0], wp[1] - a.p[1], wp[2] - a.p[2]};
    const float n2 = POTATO_FMA(er[2], er[2], POTATO_FMA(er[1], er[1], er[0] * er[0]));
    const bool sat = (bits >> kBitSat & 1u) != 0;
    const float rs = rsq(n2), sc = sat ? L.r_sat * rs : 1.0f;
    float e[3], acc[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        e[i] = er[i] * sc;
        acc[i] = POTATO_FMA(-k.kdp, a.v[i], POTATO_FMA(k.kip, a.ip[i], k.kpp * e[i]));
    }
    const bool az_cl = (bits >> kBitAz & 1u) != 0;
    acc[2] = az_cl ? L.az_min : acc[2] + L.g;
    float bz[3];
    body_z(a.q, bz);
    const float ra = rsq(POTATO_FMA(acc[2], acc[2], POTATO_FMA(acc[1], acc[1], acc[0] * acc[0])));
    const float nv[3] = {acc[0] * ra, acc[1] * ra, acc[2] * ra};
    const float qr0 = 1.0f + nv[2];
    const float rq = rsq(qr0 + qr0);
    const float qd[3] = {qr0 * rq, -(nv[1] * rq), nv[0] * rq};
    const float* q = a.q;
    const float sg = (bits >> kBitSgn & 1u) != 0 ? -2.0f : 2.0f;
    const float eatt[3] = {sg * POTATO_FMA(q[3], qd[2], POTATO_FMA(-q[1], qd[0], q[0] * qd[1])),
                           sg * POTATO_FMA(-q[3], qd[1], POTATO_FMA(-q[2], qd[0], q[0] * qd[2])),
                           sg * POTATO_FMA(-q[3], qd[0], POTATO_FMA(-q[1], qd[2], q[2] * qd[1]))};

    /* ---------------- reverse: controller ----------------
     * rotor speed W = sqrt(f / k_f) of the held command: dW/df = 1 / (2 k_f W),
     * zero where the thrust was clamped or W == 0 */
    float lf[4];
    const float hik = 0.5f * c.inv_kf;
#pragma unroll
    for (int i = 0; i < 4; ++i) lf[i] = where(in_f[i], ldc[i] * (hik * __builtin_amdgcn_rcpf(dc[i] + c.w_ref)));
    const float s02 = lf[0] + lf[2], s13 = lf[1] + lf[3], d02 = lf[0] - lf[2], d31 = lf[3] - lf[1];
    const float m0 = (0.25f * c.mass) * (s02 + s13);          /* cotangent of the thrust per mass */
    const float lal[3] = {c.Ix * (c.mix_x * (d02 + d31)), c.Iy * (c.mix_y * (d31 - d02)),
                          c.Iz * (c.mix_z * (s02 - s13))};
    /* gyroscopic feed-forward w x (I w): (I_z - I_y) ltx = gx I_x ltx */
    {
        const float g0 = c.gx * lal[0], g1 = c.gy * lal[1], g2 = c.gz * lal[2];
        lam.w[0] = POTATO_FMA(g2, a.w[1], POTATO_FMA(g1, a.w[2], lam.w[0]));
        lam.w[1] = POTATO_FMA(g0, a.w[2], POTATO_FMA(g2, a.w[0], lam.w[1]));
        lam.w[2] = POTATO_FMA(g1, a.w[0], POTATO_FMA(g0, a.w[1], lam.w[2]));
    }
    float le[3];
    const float kda1 = 1.0f + k.kda;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const float erate = POTATO_FMA(-k.kda, a.w[i], POTATO_FMA(k.kia, a.ia[i], k.kpa * eatt[i])) - a.w[i];
        /* rate loop, and w_prev <- w */
        gk[6] = POTATO_FMA(lal[i], erate, gk[6]);
        gk[7] = POTATO_FMA(lal[i], a.ir[i], gk[7]);
        a.ir[i] = undo<kUndoRate>(a.ir[i], erate, L.dt, rate_offset(a, 3 + i));
        gk[8] = POTATO_FMA(-lal[i], a.dw[i], gk[8]);
        const float l_dw = k.kdr_dt * lal[i];
        const float lw = (lam.w[i] + lam.wprev[i]) - l_dw;
        lam.wprev[i] = l_dw;
        lam.ir[i] = where(in_ir[i], POTATO_FMA(k.kir, lal[i], lam.ir[i]));
        const float l_er = POTATO_FMA(L.dt, lam.ir[i], k.kpr * lal[i]);
        /* attitude loop, erate = wdes - w */
        gk[3] = POTATO_FMA(l_er, eatt[i], gk[3]);
        gk[4] = POTATO_FMA(l_er, a.ia[i], gk[4]);
        a.ia[i] = undo<kUndoRate>(a.ia[i], eatt[i], L.dt, rate_offset(a, i));
        gk[5] = POTATO_FMA(-l_er, a.w[i], gk[5]);
        lam.w[i] = POTATO_FMA(-kda1, l_er, lw);
        lam.ia[i] = where(in_ia[i], POTATO_FMA(k.kia, l_er, lam.ia[i]));
        le[i] = sg * POTATO_FMA(L.dt, lam.ia[i], k.kpa * l_er);
    }
    /* error quaternion (the sign is a constant of the branch) */
    lam.q[0] = POTATO_FMA(le[1], qd[2], POTATO_FMA(le[0], qd[1], lam.q[0]));
    lam.q[1] = POTATO_FMA(-le[2], qd[2], POTATO_FMA(-le[0], qd[0], lam.q[1]));
    lam.q[2] = POTATO_FMA(le[2], qd[1], POTATO_FMA(-le[1], qd[0], lam.q[2]));
    lam.q[3] = POTATO_FMA(-le[2], qd[0], POTATO_FMA(-le[1], qd[1], POTATO_FMA(le[0], qd[2], lam.q[3])));
    const float lqd[3] = {-POTATO_FMA(le[2], q[3], POTATO_FMA(le[1], q[2], le[0] * q[1])),
                          POTATO_FMA(le[2], q[2], POTATO_FMA(-le[1], q[3], le[0] * q[0])),
                          POTATO_FMA(-le[2], q[1], POTATO_FMA(le[1], q[0], le[0] * q[3]))};
    /* normalisation of the desired-attitude quaternion (1 + n_z, -n_y, n_x, 0) */
    const float dqd = POTATO_FMA(qd[2], lqd[2], POTATO_FMA(qd[1], lqd[1], qd[0] * lqd[0]));
    const float ln[3] = {rq * POTATO_FMA(-qd[2], dqd, lqd[2]), -(rq * POTATO_FMA(-qd[1], dqd, lqd[1])),
                         rq * POTATO_FMA(-qd[0], dqd, lqd[0])};
    const float dn = POTATO_FMA(nv[2], ln[2], POTATO_FMA(nv[1], ln[1], nv[0] * ln[0]));
    float la[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) la[i] = POTATO_FMA(ra, POTATO_FMA(-nv[i], dn, ln[i]), m0 * bz[i]);
    /* body z axis used for the collective thrust */
    {
        const float t = m0 + m0;
        const float b0 = t * acc[0], b1 = t * acc[1], b2 = (t + t) * acc[2];
        lam.q[0] = POTATO_FMA(-q[1], b1, POTATO_FMA(q[2], b0, lam.q[0]));
        lam.q[1] = POTATO_FMA(-q[1], b2, POTATO_FMA(-q[0], b1, POTATO_FMA(q[3], b0, lam.q[1])));
        lam.q[2] = POTATO_FMA(-q[2], b2, POTATO_FMA(q[3], b1, POTATO_FMA(q[0], b0, lam.q[2])));
        lam.q[3] = POTATO_FMA(q[2], b1, POTATO_FMA(q[1], b0, lam.q[3]));
    }
    la[2] = az_cl ? 0.0f : la[2];
    /* position loop */
    float l_e[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        gk[0] = POTATO_FMA(la[i], e[i], gk[0]);
        gk[1] = POTATO_FMA(la[i], a.ip[i], gk[1]);
        a.ip[i] = undo<kUndoPos>(a.ip[i], e[i], L.dt, pos_offset(a, i));
        gk[2] = POTATO_FMA(-la[i], a.v[i], gk[2]);
        lam.v[i] = POTATO_FMA(-k.kdp, la[i], lam.v[i]);
        lam.ip[i] = where(in_ip[i], POTATO_FMA(k.kip, la[i], lam.ip[i]));
        l_e[i] = POTATO_FMA(L.dt, lam.ip[i], k.kpp * la[i]);
    }
    /* saturation e = r_sat * er / |er| */
    if (sat) {
        const float u[3] = {er[0] * rs, er[1] * rs, er[2] * rs};
        const float du = POTATO_FMA(u[2], l_e[2], POTATO_FMA(u[1], l_e[1], u[0] * l_e[0]));
#pragma unroll
        for (int i = 0; i < 3; ++i) l_e[i] = sc * POTATO_FMA(-u[i], du, l_e[i]);
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) lam.p[i] -= l_e[i];
}

/* gk[8] as summed by step_vjp to the cotangent of kdr. */
__device__ __forceinline__ void kdr_from_sum(const Limits& L, float gk[9]) { gk[8] *= L.inv_dt; }

/* Row accessors: `base` is row 0 of a [rows][ld] buffer, the same address
 * in every active lane, and `bo` the lane's byte offset (column index
 * times 4). */
template <typename T>
__device__ __forceinline__ T* row_ptr(T* base, int64_t ld, int k) {
    return uniform(base + k * ld);
}

__device__ __forceinline__ void load_rows(const float* base, int64_t ld, uint32_t bo, Agent& a, bool carries) {
    auto row = [&](int k) { return elem(row_ptr(base, ld, k), bo); };
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        a.p[k] = row(k); a.v[k] = row(3 + k); a.w[k] = row(10 + k);
        a.ip[k] = row(17 + k); a.ia[k] = row(20 + k);
        a.ir[k] = row(23 + k); a.wprev[k] = row(26 + k);
        a.p_lo[k] = carries ? row(30 + k) : 0.0f;
        a.v_lo[k] = carries ? row(33 + k) : 0.0f;
        a.ip_lo[k] = carries ? row(37 + k) : 0.0f;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) { a.q[k] = row(6 + k); a.d[k] = row(13 + k); }
    a.J = row(29);
    a.J_lo = carries ? row(36) : 0.0f;
}

__device__ __forceinline__ void load_adj(const float* base, int64_t ld, uint32_t bo, AgentAdj& l) {
    auto row = [&](int k) { return elem(row_ptr(base, ld, k), bo); };
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        l.p[k] = row(k); l.v[k] = row(3 + k); l.w[k] = row(10 + k);
        l.ip[k] = row(17 + k); l.ia[k] = row(20 + k);
        l.ir[k] = row(23 + k); l.wprev[k] = row(26 + k);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) { l.q[k] = row(6 + k); l.d[k] = row(13 + k); }
    l.J = row(29);
}

/* Cotangent of the initial state: rows 0-16 to x0 ([17][ld]), rows 17-29
 * to mem ([13][ld]) when it is given. */
__device__ __forceinline__ void store_adj(float* x0, float* mem, int64_t ld, uint32_t bo, const AgentAdj& l) {
    auto row = [&](int k) -> float& { return elem(row_ptr(x0, ld, k), bo); };
#pragma unroll
    for (int k = 0; k < 3; ++k) { row(k) = l.p[k]; row(3 + k) = l.v[k]; row(10 + k) = l.w[k]; }
#pragma unroll
    for (int k = 0; k < 4; ++k) { row(6 + k) = l.q[k]; row(13 + k) = l.d[k]; }
    if (mem) {
        auto mrow = [&](int k) -> float& { return elem(row_ptr(mem, ld, k), bo); };
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            mrow(k) = l.ip[k]; mrow(3 + k) = l.ia[k]; mrow(6 + k) = l.ir[k]; mrow(9 + k) = l.wprev[k];
        }
        mrow(12) = l.J;
    }
}

/* Tape slots: one block of kTapeRows x 64 floats per wave and step, a row
 * being 64 consecutive floats (one per lane).  Their traffic is what bounds
 * the sweep most: with every slot's address folded onto one (a timing run)
 * it took 27 % less time.  `slot` is the block's base,
 * the same for the whole wave; rows 0-15 and 16-30 are addressed from two
 * scalar bases at immediate offsets (k x 256 bytes, within the 4 KiB range
 * of the instruction's offset field), and `lb` is the lane's byte offset. */
template <typename T>
struct TapeRows {
    T* lo;
    T* hi;
    __device__ __forceinline__ explicit TapeRows(T* slot) : lo(uniform(slot)), hi(uniform(slot + 16 * 64)) {}
    __device__ __forceinline__ T* row(int k) const { return k < 16 ? lo + k * 64 : hi + (k - 16) * 64; }
};

/* A tape value's load.  STREAM: marked as not read again, so that it leaves
 * its cache line to the slots still to be written and read; for tapes that
 * do not fit the Infinity Cache (adjoint_streams). */
template <bool STREAM>
__device__ __forceinline__ float tape_load(const float& x) {
    return STREAM ? __builtin_nontemporal_load(&x) : x;
}

/* The integrals before a step are on the tape only where they are needed:
 * the reverse sweep knows those after the step, and undo() gives those before
 * it from them with a few bits each, exactly the forward's, as if they were
 * on the tape (23 rows per step instead of 30; backward of 300,007 agents
 * 16.6 to 14.3-14.9 us per step, of 1,048,576 56 to 51-52.6).  Where an agent's
 * offsets do not fit or it is at a clamp, the wave writes the nine rows
 * themselves, the first in the place of the offsets' word. */
constexpr uint32_t kBitInt = 7u << (kBitIp - 2) | 0x3fu << (kBitIr - 4);   /* inside all nine clamps */

/* A tape slot: the step-start state (rows 0-16: p, v, q, w, rotors), the
 * held command, the branch decisions, and the undo offsets or the integrals. */
__device__ __forceinline__ void store_tape(float* slot, uint32_t lb, const Agent& a, const float dc[4],
                                           const WayBack& b, const float before[9]) {
    const TapeRows<float> t(slot);
    auto row = [&](int k) -> float& { return elem(t.row(k), lb); };
    uint32_t wide = 0;
#pragma unroll
    for (int k = 0; k < 9; ++k) wide |= b.off[k] >> (k < 3 ? kUndoPos : kUndoRate);
    const bool whole = __ballot(wide != 0 || (b.bits & kBitInt) != kBitInt) != 0;
    uint32_t bits = b.bits, word = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) { row(k) = a.p[k]; row(3 + k) = a.v[k]; row(10 + k) = a.w[k]; }
#pragma unroll
    for (int k = 0; k < 4; ++k) { row(6 + k) = a.q[k]; row(13 + k) = a.d[k]; row(kTapeCmd + k) = dc[k]; }
    if (whole) {
        bits |= kWholeBit;
#pragma unroll
        for (int k = 0; k < 9; ++k) row(kTapeInt + k) = before[k];
    } else {
#pragma unroll
        for (int k = 0; k < 3; ++k) bits |= b.off[k] << (kUndoPosAt + kUndoPos * k);
#pragma unroll
        for (int k = 0; k < kUndoWord; ++k) word |= b.off[3 + k] << (kUndoRate * k);
        bits |= b.off[3 + kUndoWord] << kUndoAt;
        row(kTapeInt) = __uint_as_float(word);
    }
    row(kTapeBits) = __uint_as_float(bits);
}

/* The same without the body rates, which the step after has read already;
 * integrals on the tape come with load_tape_integrals. */
template <bool STREAM>
__device__ __forceinline__ void load_tape(const float* slot, uint32_t lb, Replay& a) {
    const TapeRows<const float> t(slot);
    auto row = [&](int k) { return tape_load<STREAM>(elem(t.row(k), lb)); };
#pragma unroll
    for (int k = 0; k < 3; ++k) { a.p[k] = row(k); a.v[k] = row(3 + k); }
#pragma unroll
    for (int k = 0; k < 4; ++k) { a.q[k] = row(6 + k); a.d[k] = row(13 + k); a.dc[k] = row(kTapeCmd + k); }
    a.bits = __float_as_uint(row(kTapeBits));
    a.off = __float_as_uint(row(kTapeInt));
}

/* The integrals before the step, where the tape holds them. */
__device__ __forceinline__ void load_tape_integrals(const float* slot, uint32_t lb, Replay& a) {
    const TapeRows<const float> t(slot);
    auto row = [&](int r) { return elem(t.row(kTapeInt + r), lb); };
#pragma unroll
    for (int r = 0; r < 3; ++r) { a.ip[r] = row(r); a.ia[r] = row(3 + r); a.ir[r] = row(6 + r); }
}

/* Body rates at the start of a step: rows 10-12 of a tape slot. */
template <bool STREAM>
__device__ __forceinline__ void load_tape_w(const float* slot, uint32_t lb, float w[3]) {
    const TapeRows<const float> t(slot);
#pragma unroll
    for (int k = 0; k < 3; ++k) w[k] = tape_load<STREAM>(elem(t.row(10 + k), lb));
}

/* w_prev of step s of a segment: the body rates of step s - 1 on the tape,
 * or, for the segment's first step, the checkpoint's rows 26-28. */
template <bool STREAM>
__device__ __forceinline__ void step_wprev(const float* tape, int64_t tape_step, uint32_t lb, int s,
                                           const float* ckpt_seg, int64_t ld, uint32_t bo, float wprev[3]) {
    if (s > 0) {
        load_tape_w<STREAM>(tape + (int64_t)(s - 1) * tape_step, lb, wprev);
    } else {
#pragma unroll
        for (int k = 0; k < 3; ++k) wprev[k] = elem(row_ptr(ckpt_seg, ld, 26 + k), bo);
    }
}

/* Recomputed forward step: what its reverse needs goes to the tape slot,
 * then the state advances (the forward pass's own arithmetic, carries
 * included, so the same bits). */
__device__ __forceinline__ void recompute_step(const TypeConst& c, const Limits& L, const Gains& g, Agent& a,
                                               const float wp[3], float* slot, uint32_t lb) {
    float dc[4], before[9];
    WayBack back;
#pragma unroll
    for (int r = 0; r < 3; ++r) { before[r] = a.ip[r]; before[3 + r] = a.ia[r]; before[6 + r] = a.ir[r]; }
    controller<true, true>(c, L, g, a, wp, dc, &back);
    store_tape(slot, lb, a, dc, back, before);
    rk4_step(c, L, a, dc);
}

/* Reverse of step s of a segment from the tape.  x
 * carries the integrals after the step and w the body rates at its start,
 * both from the step after it; they come back as those of the step before. */
template <bool STREAM>
__device__ __forceinline__ void reverse_step(const TypeConst& c, const Limits& L, const Gains& g, Replay& x,
                                             float w[3], int s, const float wp[3], const float* tape,
                                             int64_t tape_step, uint32_t lb, const float* ckpt_seg, int64_t ld,
                                             uint32_t bo, AgentAdj& lam, float gk[9]) {
    const float* const slot = tape + (int64_t)s * tape_step;
    float wprev[3];
    load_tape<STREAM>(slot, lb, x);
    step_wprev<STREAM>(tape, tape_step, lb, s, ckpt_seg, ld, bo, wprev);
#pragma unroll
    for (int r = 0; r < 3; ++r) { x.w[r] = w[r]; x.dw[r] = w[r] - wprev[r]; }
    step_vjp(c, L, g, x, wp, lam, gk);
#pragma unroll
    for (int r = 0; r < 3; ++r) w[r] = wprev[r];
    if (x.bits & kWholeBit) load_tape_integrals(slot, lb, x);
}

/*
 * Reverse sweep of one agent's closed-loop rollout of `steps` steps from
 * global step step0.  Checkpoint slot s (kCkptRows rows of stride ld: the
 * state, then its rounding carries; this agent's column at byte offset bo)
 * holds the state before call-relative step s*K.
 * Each segment is recomputed forward from its checkpoint with the
 * step-start states written to this wave's tape blocks (`tape` is the
 * wave's block of step 0, consecutive steps tape_step floats apart; lane
 * byte offset lb), then reversed step by step.
 * lam: cotangent of the final state on entry, of the initial state on
 * return; gk accumulates the gain cotangents.
 *
 * The loops run over the call's segments and slots (n_seg_all =
 * ceil(n_steps / K) and K, the same for every lane), and a lane skips the
 * iterations beyond its own step count.  All active lanes are therefore at
 * the same segment, slot and step, so checkpoint, tape and waypoint rows
 * are wave-uniform addresses even when step budgets differ between lanes.
 * Each reverse step loads its tape slot; the other resident wave covers
 * the load latency (holding the next slot in registers instead costs 22
 * registers and the second wave).
 */
template <bool STREAM>
__device__ __forceinline__ void agent_backward(const TypeConst& c, const Limits& L, const Gains& g,
                                               const float* ckpt, int64_t ld, uint32_t bo, int K,
                                               int n_seg_all, int steps, int64_t step0, const float* wp,
                                               int64_t cmd_ld, int n_epochs, int resample, float* tape,
                                               int64_t tape_step, uint32_t lb, AgentAdj& lam, float gk[9]) {
    const int n_seg = (steps + K - 1) / K;
    /* Waypoint epochs: global step k uses epoch min(k / resample, n_epochs - 1).
     * The epoch is divided out once per sweep of a segment and then tracked
     * across its boundaries, and the waypoint is reloaded only when the
     * (clamped) epoch changes. */
    const int64_t period = resample > 0 ? resample : INT64_MAX;
    int64_t cur_ep = -1;
    float wpv[3] = {0.0f, 0.0f, 0.0f};
    auto use_epoch = [&](int64_t e) {
        const int64_t ep = e < n_epochs - 1 ? e : (int64_t)n_epochs - 1;
        if (ep != cur_ep) {
#pragma unroll
            for (int i = 0; i < 3; ++i) wpv[i] = elem(uniform(wp + (ep * 3 + i) * cmd_ld), bo);
            cur_ep = ep;
        }
    };
    Replay x{};
    float w[3] = {0.0f, 0.0f, 0.0f};
    for (int seg = n_seg_all - 1; seg >= 0; --seg) {
        if (seg >= n_seg) continue;
        const int k_begin = seg * K;
        const int len = steps - k_begin < K ? steps - k_begin : K;
        const int64_t k0 = step0 + k_begin;        /* global index of the segment's first step */
        Agent a;
        load_rows(ckpt + (int64_t)seg * kCkptRows * ld, ld, bo, a, true);
        int64_t e = resample > 0 ? k0 / resample : 0;
        int64_t next = resample > 0 ? (e + 1) * period : INT64_MAX;   /* first step of epoch e + 1 */
        for (int s = 0; s < len; ++s) {
            if (k0 + s == next) { ++e; next += period; }
            use_epoch(e);
            recompute_step(c, L, g, a, wpv, tape + (int64_t)s * tape_step, lb);
        }
        /* reverse: start from the epoch of the segment's last step */
        e = resample > 0 ? (k0 + len - 1) / resample : 0;
        int64_t first = resample > 0 ? e * period : INT64_MIN;         /* first step of epoch e */
        const float* ck = ckpt + (int64_t)seg * kCkptRows * ld;
        if (seg == n_seg - 1) {
            /* the recomputation ended with the integrals after this lane's
             * last step and, as the w_prev of the step that would follow,
             * that step's body rates */
#pragma unroll
            for (int r = 0; r < 3; ++r) { x.ip[r] = a.ip[r]; x.ia[r] = a.ia[r]; x.ir[r] = a.ir[r]; w[r] = a.wprev[r]; }
        }
        for (int s = K - 1; s >= 0; --s) {
            if (s >= len) continue;
            if (k0 + s < first) { --e; first -= period; }
            use_epoch(e);
            reverse_step<STREAM>(c, L, g, x, w, s, wpv, tape, tape_step, lb, ck, ld, bo, lam, gk);
        }
    }
}

/* Waypoint row of the current epoch (clamped to the last one), reloaded
 * only when the epoch changes. */
struct WaypointCache {
    const float* wp;
    int64_t cmd_ld;
    int n_epochs;
    uint32_t bo;
    int64_t cur = -1;
    float v[3] = {0.0f, 0.0f, 0.0f};
    __device__ __forceinline__ void use(int64_t e) {
        const int64_t ep = e < n_epochs - 1 ? e : (int64_t)n_epochs - 1;
        if (ep != cur) {
#pragma unroll
            for (int i = 0; i < 3; ++i) v[i] = elem(uniform(wp + (ep * 3 + i) * cmd_ld), bo);
            cur = ep;
        }
    }
};

constexpr int kTailRows = 12;      /* the integrals and body rates that reverse_segment starts from */

/* The two halves of one segment of agent_backward, for a kernel that runs
 * them on different waves: the forward recomputation of segment `seg` from
 * its checkpoint into the tape, and the reverse sweep of a recomputed
 * segment.  Same operations, in the same order, as agent_backward. */
__device__ __forceinline__ void recompute_segment(const TypeConst& c, const Limits& L, const Gains& g,
                                                  const float* ckpt, int64_t ld, uint32_t bo, int K, int seg,
                                                  int steps, int64_t step0, int resample, WaypointCache& wc,
                                                  float* tape, int64_t tape_step, uint32_t lb, float* tail) {
    const int64_t period = resample > 0 ? resample : INT64_MAX;
    const int k_begin = seg * K;
    const int len = steps - k_begin < K ? steps - k_begin : K;
    const int64_t k0 = step0 + k_begin;
    Agent a;
    load_rows(ckpt + (int64_t)seg * kCkptRows * ld, ld, bo, a, true);
    int64_t e = resample > 0 ? k0 / resample : 0;
    int64_t next = resample > 0 ? (e + 1) * period : INT64_MAX;
    for (int s = 0; s < len; ++s) {
        if (k0 + s == next) { ++e; next += period; }
        wc.use(e);
        recompute_step(c, L, g, a, wc.v, tape + (int64_t)s * tape_step, lb);
    }
    if (k_begin + len == steps) {              /* this lane's last segment */
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            elem(tail + r * 64, lb) = a.ip[r];
            elem(tail + (3 + r) * 64, lb) = a.ia[r];
            elem(tail + (6 + r) * 64, lb) = a.ir[r];
            elem(tail + (9 + r) * 64, lb) = a.wprev[r];
        }
    }
}

template <bool STREAM>
__device__ __forceinline__ void reverse_segment(const TypeConst& c, const Limits& L, const Gains& g,
                                                const float* ckpt, int64_t ld, uint32_t bo, int K,
                                                int seg, int steps, int64_t step0, int resample,
                                                WaypointCache& wc, const float* tape, int64_t tape_step,
                                                uint32_t lb, const float* tail, Replay& x, float w[3],
                                                AgentAdj& lam, float gk[9]) {
    const int64_t period = resample > 0 ? resample : INT64_MAX;
    const int k_begin = seg * K;
    const int len = steps - k_begin < K ? steps - k_begin : K;
    const int64_t k0 = step0 + k_begin;
    int64_t e = resample > 0 ? (k0 + len - 1) / resample : 0;
    int64_t first = resample > 0 ? e * period : INT64_MIN;
    const float* ck = ckpt + (int64_t)seg * kCkptRows * ld;
    if (k_begin + len == steps) {              /* this lane's last segment */
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            x.ip[r] = elem(tail + r * 64, lb);
            x.ia[r] = elem(tail + (3 + r) * 64, lb);
            x.ir[r] = elem(tail + (6 + r) * 64, lb);
            w[r] = elem(tail + (9 + r) * 64, lb);
        }
    }
    for (int s = K - 1; s >= 0; --s) {
        if (s >= len) continue;
        if (k0 + s < first) { --e; first -= period; }
        wc.use(e);
        reverse_step<STREAM>(c, L, g, x, w, s, wc.v, tape, tape_step, lb, ck, ld, bo, lam, gk);
    }
}

}  // namespace potato
