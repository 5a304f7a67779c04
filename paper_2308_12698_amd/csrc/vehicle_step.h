/*
 * vehicle_step.h -- per-agent FP32 arithmetic of one time step of the two
 * other robot kinds the simulator batches with its quadrotors (the paper
 * names fixed-wing drones, quadrotors and cars, Sec. II-B, and writes out
 * only the quadrotor; the other two follow the works it cites for them):
 *   - car (kind 1): the kinematic bicycle model referenced at the centre of
 *     mass (Rajamani, Vehicle Dynamics and Control, 2nd ed., Sec. 2.2):
 *     side-slip beta = atan(l_r tan(delta) / L), position rate
 *     v (cos(psi + beta), sin(psi + beta)), yaw rate v cos(beta) tan(delta) / L,
 *     a first-order steering actuator and an acceleration input with
 *     linear drag;
 *   - fixed wing (kind 2): the kinematic guidance model of Beard and
 *     McLain (Small Unmanned Aircraft, Ch. 9) in still air: velocity V along
 *     course chi and flight-path angle gamma, coordinated-turn course rate
 *     g tan(phi) / V, first-order airspeed, roll and flight-path responses;
 *   - guidance of both in closed loop: the orbit-following vector field of
 *     the same book (Ch. 10) around the agent's waypoint, radius rho,
 *     direction lambda: course command
 *     atan2(y - c_y, x - c_x) + lambda (pi/2 + atan(k_orb (d - rho) / rho)),
 *     plus the steering or bank that holds the circle exactly, a speed hold
 *     (car) and a saturated altitude hold (aircraft).  These are the circle
 *     trajectories of the paper's first demonstration (Sec. IV).
 * State rows (of the simulator's [30][ld] layout; rows 7-29 are not
 * touched): 0-2 position, 3 speed, 4 heading (car yaw psi, aircraft course
 * chi), 5 actuator angle (steering delta, bank phi), 6 flight-path angle
 * gamma (aircraft only; a car leaves rows 2 and 6 unchanged).  Inputs, held
 * through the step: car (a_c, delta_c), aircraft (V_c, phi_c, gamma_c).
 *
 * Differences from a literal transcription, exact in real arithmetic or to
 * below FP32 rounding: cos(beta) and sin(beta) are 1/sqrt(1 + t^2) and
 * t/sqrt(1 + t^2) with t = tan(beta), and cos/sin(psi + beta) are expanded
 * by the angle-sum formulas, so a car's derivative takes no arctangent; the
 * trigonometric functions of the angles are evaluated once per step, at
 * the step-start state, and carried to each RK4 stage's angles by the
 * angle-sum formulas with short series for the stage's small offset
 * (veh_trig_near); the course error is the angle of one product of complex numbers
 * (one arctangent instead of two or three); divisions by
 * the time constants, the wheelbase and g rho are multiplications by
 * reciprocals precomputed per type; the car's steering feed-forward is a
 * per-type constant.  Every integrated row keeps a rounding carry
 * (Fast2Sum), as the quadrotor's position and velocity do.  Contraction is
 * off and fused multiply-adds are placed explicitly, so the plain and the
 * fused launches give the same bits.
 *
 * Bound by instruction issue, like the quadrotor's step.  The library's
 * sine, tangent, arctangent and division (large-argument branches, full
 * special-case sequences) made a step of several hundred instructions more
 * than the functions written here, which keep the library's as the rare
 * branch: a car's step is now 327 vector instructions and an aircraft's 439
 * (262,144 agents each), in straight lines (a quadrotor's 525).  Mixed kinds
 * in the type order, us per step before and after: 2.57 and 1.72 at 3,000
 * agents, 6.03 and 5.37 at 524,288, 11.4 and 9.8 at 1,048,576.
 */
#pragma once

#include "quad_step.h"

namespace potato {

constexpr float kPi = 3.14159265358979323846f;
constexpr float kTwoPi = 6.28318530717958647692f;
constexpr float kInvTwoPi = 0.159154943091895335769f;

/* Angle a moved into [-pi, pi] by whole turns. */
__device__ __forceinline__ float wrap_pi(float a) {
    return POTATO_FMA(-kTwoPi, rintf(a * kInvTwoPi), a);
}

/* n / d: reciprocal, quotient and one correction by its exact residual, four
 * instructions where the full sequence takes eleven, with the division's own
 * rounding (4 million random pairs without a difference).  For a finite n
 * and |d| from 1e-37 to 1e37: v_rcp_f32 makes infinity of a subnormal and
 * zero of a number whose reciprocal would be one, and the correction then
 * has no residual to work with. */
__device__ __forceinline__ float quotient(float n, float d) {
#pragma clang fp contract(off)
    const float r = __builtin_amdgcn_rcpf(d);
    const float q = n * r;
    return POTATO_FMA(POTATO_FMA(-d, q, n), r, q);
}

/* Airspeeds that quotient() divides by; the speeds at the step's stages are
 * then zero or normal numbers too (a sum of products of such numbers with a
 * time step does not come below 1e-35). */
__device__ __forceinline__ bool ordinary_speed(float v) { return fabsf(v) >= 1e-20f && fabsf(v) <= 1e20f; }

/* Taylor polynomials of the sine and cosine of r, at most pi/4 and a little:
 * sin r = r + r^3 ps, cos r = 1 + r^2 pc (through r^9 and r^10: truncation
 * below 3e-9 and 2e-9).  Returns r^2. */
__device__ __forceinline__ float sincos_series(float r, float& ps, float& pc) {
#pragma clang fp contract(off)
    const float r2 = r * r;
    ps = POTATO_FMA(r2, POTATO_FMA(r2, POTATO_FMA(r2, 1.0f / 362880.0f, -1.0f / 5040.0f), 1.0f / 120.0f), -1.0f / 6.0f);
    pc = POTATO_FMA(r2, POTATO_FMA(r2, POTATO_FMA(r2, POTATO_FMA(r2, -1.0f / 3628800.0f, 1.0f / 40320.0f), -1.0f / 720.0f), 1.0f / 24.0f), -0.5f);
    return r2;
}

/* sin and cos of a, |a| <= kTrigMax: a - k pi/2 for the nearest k with pi/2
 * in three parts (Cody and Waite, Software Manual for the Elementary
 * Functions, 1980; each step a fused multiply-add, the first one exact),
 * then the series of the remainder.  Against 64 bits, 4 million angles
 * within 6 rad: 1.42 ulp at most, 0.28 and 0.31 in the mean (the library's
 * sincosf: 1.45 and 1.54, 0.29 and 0.32). */
constexpr float kTrigMax = 1e5f;
__device__ __forceinline__ void sincos_near(float a, float& s, float& c) {
#pragma clang fp contract(off)
    const float k = rintf(a * 0.6366197466850281f);
    float r = POTATO_FMA(-k, 1.5707963705062866f, a);
    r = POTATO_FMA(-k, -4.371138828673793e-08f, r);
    r = POTATO_FMA(-k, -1.7151245100058819e-15f, r);
    float ps, pc;
    const float r2 = sincos_series(r, ps, pc);
    const float sr = POTATO_FMA(r * r2, ps, r), cr = POTATO_FMA(r2, pc, 1.0f);
    const uint32_t q = (uint32_t)(int32_t)k;
    const bool odd = (q & 1u) != 0;
    const uint32_t ss = (q & 2u) << 30, cs = ((q + 1u) & 2u) << 30;
    s = __uint_as_float(__float_as_uint(odd ? cr : sr) ^ ss);
    c = __uint_as_float(__float_as_uint(odd ? sr : cr) ^ cs);
}

/* tan a, |a| <= kTrigMax, with one division, numerator and denominator being
 * the sine and cosine of the remainder as sums of two numbers each: 1.32 ulp
 * at most, 0.26 in the mean (tanf: 1.32 and 0.28; the quotient of the rounded
 * sine and cosine: 2.2 and 0.42). */
__device__ __forceinline__ float tan_near(float a) {
#pragma clang fp contract(off)
    const float k = rintf(a * 0.6366197466850281f);
    const float t = POTATO_FMA(-k, 1.5707963705062866f, a);
    const float r = POTATO_FMA(-k, -4.371138828673793e-08f, t);
    const float lo = POTATO_FMA(-k, -1.7151245100058819e-15f, POTATO_FMA(-k, -4.371138828673793e-08f, t - r));
    float ps, pc;
    const float r2 = sincos_series(r, ps, pc);
    const float ds = POTATO_FMA(r * r2, ps, lo), dc = POTATO_FMA(r2, pc, -(r * lo));
    const float s = r + ds, c = 1.0f + dc;
    const float s_lo = (r - s) + ds, c_lo = (1.0f - c) + dc;
    const bool odd = ((uint32_t)(int32_t)k & 1u) != 0;
    const float n = odd ? -c : s, n_lo = odd ? -c_lo : s_lo, d = odd ? s : c, d_lo = odd ? s_lo : c_lo;
    const float rd = __builtin_amdgcn_rcpf(d);
    const float q = n * rd;
    return POTATO_FMA(POTATO_FMA(-q, d_lo, POTATO_FMA(-d, q, n) + n_lo), rd, q);
}

/* Angle of the vector (x, y), as atan2(y, x), for a vector other than
 * (0, 0) with the larger coordinate from 1e-37 to 1e37: the smaller
 * coordinate over the larger, moved by pi/4 where it exceeds tan(pi/8) (both
 * within one division), and the arctangent's series through r^17 (truncation
 * below 3e-9 for |r| <= tan(pi/8)).  NaN for a NaN coordinate.  2.27 ulp at
 * most, 0.38 in the mean (atan2f: 2.76 and 0.43). */
__device__ __forceinline__ float vector_angle(float y, float x) {
#pragma clang fp contract(off)
    const float ax = fabsf(x), ay = fabsf(y);
    const bool steep = ay > ax;
    const float mx = steep ? ay : ax, mn = steep ? ax : ay;
    const bool big = mn > 0.41421356f * mx;
    const float r = quotient(big ? mn - mx : mn, big ? mn + mx : mx);
    const float r2 = r * r;
    float p = POTATO_FMA(r2, 1.0f / 17.0f, -1.0f / 15.0f);
    p = POTATO_FMA(r2, p, 1.0f / 13.0f);
    p = POTATO_FMA(r2, p, -1.0f / 11.0f);
    p = POTATO_FMA(r2, p, 1.0f / 9.0f);
    p = POTATO_FMA(r2, p, -1.0f / 7.0f);
    p = POTATO_FMA(r2, p, 1.0f / 5.0f);
    p = POTATO_FMA(r2, p, -1.0f / 3.0f);
    const float a0 = POTATO_FMA(r * r2, p, r);
    const float a1 = big ? a0 + 0.25f * kPi : a0;
    const float a2 = steep ? 0.5f * kPi - a1 : a1;
    const float a3 = x < 0.0f ? kPi - a2 : a2;
    return copysignf(a3, y);
}

/* Rows a kind integrates (the car has no altitude or flight-path dynamics). */
template <int KIND>
__device__ __forceinline__ constexpr bool veh_row(int k) {
    return KIND == KIND_WING || (k != 2 && k != 6);
}

/* Trigonometric functions of the angles of a state: heading (sh, ch),
 * tangent of the actuator angle (ta), flight-path angle (sg, cg; aircraft). */
struct VehTrig {
    float sh, ch, ta, sg, cg;
};

/* Angles beyond kTrigMax (and NaN) take the library's functions, which
 * reduce any argument. */
template <int KIND>
__device__ __forceinline__ void veh_trig(const float x[7], VehTrig& T) {
    const float far = KIND == KIND_WING ? fmaxf(fmaxf(fabsf(x[4]), fabsf(x[5])), fabsf(x[6]))
                                        : fmaxf(fabsf(x[4]), fabsf(x[5]));
    const bool nan = !(x[4] == x[4]) || !(x[5] == x[5]) || (KIND == KIND_WING && !(x[6] == x[6]));
    if (far <= kTrigMax && !nan) {
        sincos_near(x[4], T.sh, T.ch);
        T.ta = tan_near(x[5]);
        if (KIND == KIND_WING) sincos_near(x[6], T.sg, T.cg);
    } else {
        sincosf(x[4], &T.sh, &T.ch);
        T.ta = tanf(x[5]);
        if (KIND == KIND_WING) sincosf(x[6], &T.sg, &T.cg);
    }
}

/* The angles' functions at a stage state x0 + offsets d (h k of the previous
 * stage's rates) from those at x0: sin and cos by the angle-sum formulas,
 * tan(a0 + d) as (t0 + tan d) / (1 - t0 tan d), with sin d, cos d - 1 and
 * tan d from their Taylor series through d^5, d^6 and d^7: truncation below
 * 2e-11, 3e-13 and 3e-11 at kNearOffset, past FP32 rounding.  False when an
 * offset is larger. */
constexpr float kNearOffset = 0.1f;
template <int KIND>
__device__ __forceinline__ bool veh_trig_near(const VehTrig& T0, float d4, float d5, float d6, VehTrig& T) {
#pragma clang fp contract(off)
    auto shift = [](float s0, float c0, float d, float& s, float& c) {
        const float d2 = d * d;
        const float sd = POTATO_FMA(d * d2, POTATO_FMA(d2, 1.0f / 120.0f, -1.0f / 6.0f), d);
        const float cm = d2 * POTATO_FMA(d2, POTATO_FMA(d2, -1.0f / 720.0f, 1.0f / 24.0f), -0.5f);
        s = POTATO_FMA(c0, sd, POTATO_FMA(s0, cm, s0));
        c = POTATO_FMA(-s0, sd, POTATO_FMA(c0, cm, c0));
    };
    shift(T0.sh, T0.ch, d4, T.sh, T.ch);
    if (KIND == KIND_WING) shift(T0.sg, T0.cg, d6, T.sg, T.cg);
    const float q2 = d5 * d5;
    const float td = d5 * POTATO_FMA(q2, POTATO_FMA(q2, POTATO_FMA(q2, 17.0f / 315.0f, 2.0f / 15.0f), 1.0f / 3.0f), 1.0f);
    const float den = POTATO_FMA(-T0.ta, td, 1.0f);
    T.ta = quotient(T0.ta + td, den);
    const float far = fmaxf(fmaxf(fabsf(d4), fabsf(d5)), KIND == KIND_WING ? fabsf(d6) : 0.0f);
    return far <= kNearOffset && den >= 0.5f;
}

/* Rates of rows 0-6 at state x (its angles' functions in T) with inputs u
 * held. */
template <int KIND, bool ANY_SPEED>
__device__ __forceinline__ void veh_rates(const VehConst& c, const float x[7], const VehTrig& T, const float u[3],
                                          float dx[7]) {
#pragma clang fp contract(off)
    if (KIND == KIND_CAR) {
        const float td = T.ta;
        const float tb = c.lr_L * td;                         /* tan(beta) */
        const float cb = rsq(POTATO_FMA(tb, tb, 1.0f));       /* cos(beta) > 0 */
        const float sb = tb * cb;                             /* sin(beta) */
        const float cc = POTATO_FMA(T.ch, cb, -(T.sh * sb));  /* cos(psi + beta) */
        const float sc = POTATO_FMA(T.sh, cb, T.ch * sb);     /* sin(psi + beta) */
        dx[0] = x[3] * cc;
        dx[1] = x[3] * sc;
        dx[2] = 0.0f;
        dx[3] = POTATO_FMA(-c.cd_m, x[3], u[0]);
        dx[4] = (x[3] * cb) * (td * c.inv_L);
        dx[5] = (u[1] - x[5]) * c.inv_tau[0];
        dx[6] = 0.0f;
    } else {
        const float vh = x[3] * T.cg;                         /* horizontal speed */
        dx[0] = vh * T.ch;
        dx[1] = vh * T.sh;
        dx[2] = x[3] * T.sg;
        dx[3] = (u[0] - x[3]) * c.inv_tau[0];
        const float turn = c.g * T.ta;
        dx[4] = ANY_SPEED && !ordinary_speed(x[3]) ? turn / x[3] : quotient(turn, x[3]);
        dx[5] = (u[1] - x[5]) * c.inv_tau[1];
        dx[6] = (u[2] - x[6]) * c.inv_tau[2];
    }
}

/* Closed-loop inputs from the step-start state x (its angles' functions in
 * T) around orbit centre wp. */
template <int KIND>
__device__ __forceinline__ void veh_guidance(const VehConst& c, const float x[7], const VehTrig& T, const float wp[3],
                                             float u[3]) {
#pragma clang fp contract(off)
    const float ex = x[0] - wp[0], ey = x[1] - wp[1];
    /* distance from the orbit's centre: the square root with one correction
     * by its exact residual, the library's rounding (NaN at the centre and at
     * infinity, which take the general form below) */
    const float d2 = POTATO_FMA(ey, ey, ex * ex);
    const float rd = rsq(d2), d0 = d2 * rd;
    const float u0 = c.k_orb_rho * (POTATO_FMA(POTATO_FMA(-d0, d0, d2), 0.5f * rd, d0) - c.rho);
    /* course error: course command minus the car's course (its yaw plus the
     * side-slip angle) or the aircraft's, in [-pi, pi]: the angle of the
     * product of the complex numbers whose angles add up to it, ex + i ey,
     * i lam, 1 + i lam u0, cos - i sin of the heading and 1 - i tan(beta) */
    const float lu = c.lam * u0;
    const float ar = -c.lam * ey, ai = c.lam * ex;
    const float br = POTATO_FMA(-ai, lu, ar), bi = POTATO_FMA(ar, lu, ai);
    float cr = POTATO_FMA(bi, T.sh, br * T.ch), ci = POTATO_FMA(-br, T.sh, bi * T.ch);
    if (KIND == KIND_CAR) {
        const float tb = c.lr_L * T.ta;
        const float dr = POTATO_FMA(ci, tb, cr), di = POTATO_FMA(-cr, tb, ci);
        cr = dr;
        ci = di;
    }
    const float size = fabsf(cr) + fabsf(ci);
    float e;
    if (fabsf(c.lam) == 1.0f && size >= 1e-30f && size <= 1e37f) {
        e = vector_angle(ci, cr);
    } else {
        /* another lambda, the orbit's centre, very far, infinities: angle by angle
         * (the heading without its whole turns, whose rounding would be that
         * of the difference) */
        const float uf = c.k_orb_rho * (sqrtf(d2) - c.rho);
        const float chi_d = POTATO_FMA(c.lam, atanf(uf), atan2f(ey, ex) + c.lam_half_pi);
        const float course = atan2f(T.sh, T.ch);
        e = wrap_pi(chi_d - (KIND == KIND_CAR ? course + atanf(c.lr_L * T.ta) : course));
    }
    if (KIND == KIND_CAR) {
        u[0] = clampf_(POTATO_FMA(c.k_hold, c.cruise - x[3], c.cd_m * x[3]), -c.lim[0], c.lim[0]);
        u[1] = clampf_(POTATO_FMA(c.k_head, e, c.ff), -c.lim[1], c.lim[1]);
        u[2] = 0.0f;
    } else {
        /* bank that holds the circle: tan(phi) = V^2 / (g rho) */
        const float tb = (x[3] * x[3]) * c.inv_g_rho;
        const float ff = c.lam * vector_angle(tb > 1e30f ? 1e30f : tb, 1.0f);
        u[0] = c.cruise;
        u[1] = clampf_(POTATO_FMA(c.k_head, e, ff), -c.lim[1], c.lim[1]);
        u[2] = clampf_(c.k_hold * (wp[2] - x[2]), -c.lim[2], c.lim[2]);
    }
}

constexpr float kNearStep = 0.06f;

/* Classical RK4 over rows 0-6 with the inputs held, from the step-start
 * state x whose angles' functions are T; CARRY: every integrated row keeps
 * its rounding carry in lo (the heading matters most: it grows by nearly
 * equal increments every step, and a rounding bias of its updates would be
 * cancelled by a steady steering or bank offset).  The increment dt/6 times
 * the sum of the rates is not rounded before it meets the carry, and dt/6 is
 * taken in two parts: its rounding alone moves an aircraft by half an ulp of
 * the way flown.  Mean position error after 500 steps of 1 ms, against 64
 * bits: aircraft 2.1e-7 -> 0.8e-7 m, cars 4.8e-8 -> 1.3e-8 (at the cost of
 * the multiplication and addition that the two fused ones replace). */
template <int KIND, bool CARRY>
__device__ __forceinline__ void veh_rk4(const VehConst& c, const Limits& L, float dt6_lo, float x[7], const VehTrig& T,
                                        float lo[7], const float u[3]) {
#pragma clang fp contract(off)
    float k[7], acc[7], xs[7];
    VehTrig Ts;
    auto start = [&]() {
#pragma unroll
        for (int i = 0; i < 7; ++i) acc[i] = k[i];
    };
    auto advance = [&](float h) {
#pragma unroll
        for (int i = 0; i < 7; ++i) xs[i] = veh_row<KIND>(i) ? POTATO_FMA(h, k[i], x[i]) : x[i];
    };
    auto add = [&](float weight) {
#pragma unroll
        for (int i = 0; i < 7; ++i) acc[i] = POTATO_FMA(weight, k[i], acc[i]);
    };
    /* Straight through, the stages' functions from those of the step's start.
     * An agent with an offset too large for that, or an aircraft nearly at
     * rest, takes the step again, every stage's functions from its own angles
     * (one copy of that code), and so do all agents at once where the time
     * step makes such offsets common: a step of both forms takes 1.5 of
     * either.  us per step of 500,000 cars and aircraft turning towards their
     * orbits: 4.0 and 5.2 at steps of 1 to 20 ms, 4.1 and 5.9 at 50 ms, 5.6
     * and 7.3 at 250 ms (with series for offsets of 0.02 rad at most, the
     * three stages twice beyond: 3.9 and 5.1 at 1 ms, but 5.9 and 6.4 at 20
     * ms and 7.0 and 9.9 at 250 ms; with the library's functions throughout
     * 4.9 and 6.3, 5.8 and 7.5 at 250 ms). */
    bool near = L.dt <= kNearStep;
    if (near) {
        veh_rates<KIND, false>(c, x, T, u, k);
        start();
#pragma unroll
        for (int st = 0; st < 3; ++st) {
            const float h = st < 2 ? L.half_dt : L.dt;
            advance(h);
            near = veh_trig_near<KIND>(T, h * k[4], h * k[5], h * k[6], Ts) && near;
            veh_rates<KIND, false>(c, xs, Ts, u, k);
            add(st < 2 ? 2.0f : 1.0f);
        }
        if (KIND == KIND_WING) near = near && ordinary_speed(x[3]);
    }
    if (!near) {
        veh_rates<KIND, true>(c, x, T, u, k);
        start();
#pragma unroll 1
        for (int st = 0; st < 3; ++st) {
            const float h = st < 2 ? L.half_dt : L.dt;
            advance(h);
            veh_trig<KIND>(xs, Ts);
            veh_rates<KIND, true>(c, xs, Ts, u, k);
            add(st < 2 ? 2.0f : 1.0f);
        }
    }
#pragma unroll
    for (int i = 0; i < 7; ++i) {
        if (!veh_row<KIND>(i)) continue;
        if (CARRY) {
            const float y = POTATO_FMA(L.dt6, acc[i], POTATO_FMA(dt6_lo, acc[i], lo[i]));
            const float s = x[i] + y;
            lo[i] = y - (s - x[i]);
            x[i] = s;
        } else {
            x[i] = POTATO_FMA(L.dt6, acc[i], x[i]);
        }
    }
}

}  // namespace potato
