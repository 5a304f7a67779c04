/*
 * quad_lanes.h -- one quadrotor time step on four lanes per agent, for swarms
 * that leave most of the chip idle with one agent per lane.
 *
 * Lanes 0-2 of an agent's four hold the x, y and z components of its
 * vectors, lanes 0-3 the four rotors; the attitude sits with its scalar part
 * on lane 3 (lane 0: q1, 1: q2, 2: q3, 3: q0).  Scalars (squared-speed sum,
 * cost, thrust) are computed by all four lanes alike.  Operands of another
 * lane come through DPP quad permutations, most of them folded into the
 * multiplication or addition that uses them; a sign that differs between the
 * lanes rides on a +-1 factor.  Lane 3 of a three-vector holds a value that
 * no other lane reads.
 *
 * Every operation is one of quad_step.h's, with the same operands in the
 * same order (up to the order of a product's or a sum's two operands and
 * sign flips, neither of which changes a rounding), so the results are those
 * of one agent per lane bit for bit.
 */
#pragma once

#include "quad_step.h"

namespace potato {

/* x of lane A of the agent in lane 0, of lane B in lane 1, and so on. */
template <int A, int B, int C, int D>
__device__ __forceinline__ float quad_perm(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), A | B << 2 | C << 4 | D << 6,
                                                              0xf, 0xf, true));
}
template <int A>
__device__ __forceinline__ float quad_bcast(float x) {
    return quad_perm<A, A, A, A>(x);
}

/* A lane's share of a type's constants, gains and limits. */
struct LaneConst {
    float ncd_m, kf_m, kf_m2, F0_2, F0_g, two_w, four_w2, w_ref, inv_tau, mass, f_max, inv_kf;
    float a, g, I, mix;          /* of the lane's axis: ax/-ay/az, gx.., Ix.., mix_x.. */
    float kpp, kip, kdp, kpa, kia, kda, kpr, kir, kdr_dt;
    float sT, sY, s3, sQa, sQc, sX, sYr, sZ, kz, oz;   /* signs, see their uses */
    bool odd, isz;
};

/* Agent on four lanes: one component of each vector per lane. */
struct LaneAgent {
    float p, v, q, w, d, J, ip, ia, ir, wprev, p_lo, v_lo, J_lo, ip_lo;
};

__device__ __forceinline__ LaneConst lane_const(const TypeConst& c, const Gains& k, int l) {
    LaneConst r;
    r.ncd_m = c.ncd_m; r.kf_m = c.kf_m; r.kf_m2 = c.kf_m2; r.F0_2 = c.F0_2; r.F0_g = c.F0_g;
    r.two_w = c.two_w; r.four_w2 = c.four_w2; r.w_ref = c.w_ref; r.inv_tau = c.inv_tau;
    r.mass = c.mass; r.f_max = c.f_max; r.inv_kf = c.inv_kf;
    auto axis = [&](float x, float y, float z) { return l == 0 ? x : l == 1 ? y : l == 2 ? z : 0.0f; };
    auto sign = [&](int minus) { return minus >> l & 1 ? -1.0f : 1.0f; };
    r.a = axis(c.ax, -c.ay, c.az);
    r.g = axis(c.gx, c.gy, c.gz);
    r.I = axis(c.Ix, c.Iy, c.Iz);
    r.mix = axis(c.mix_x, c.mix_y, c.mix_z);
    r.kpp = k.kpp; r.kip = k.kip; r.kdp = k.kdp; r.kpa = k.kpa; r.kia = k.kia; r.kda = k.kda;
    r.kpr = k.kpr; r.kir = k.kir; r.kdr_dt = k.kdr_dt;
    r.sT = sign(0b0011);
    r.sY = sign(0b0010);
    r.s3 = sign(0b1000);
    r.sQa = sign(0b0101);
    r.sQc = sign(0b0100);
    r.sX = sign(0b0110);
    r.sYr = sign(0b0011);
    r.sZ = sign(0b1010);
    r.kz = l == 2 ? -2.0f : 2.0f;
    r.oz = l == 2 ? 1.0f : -0.0f;
    r.odd = (l & 1) != 0;
    r.isz = l == 2;
    return r;
}

/* Lane's share of body_z's products: lane 0 q0 q2 + q1 q3, lane 1 q2 q3 -
 * q0 q1, lane 2 q1^2 + q2^2. */
__device__ __forceinline__ float lane_tilt(const LaneConst& c, float q) {
#pragma clang fp contract(off)
    const float x4 = quad_perm<2, 0, 1, 2>(q) * c.sY;
    const float pr = quad_perm<0, 3, 1, 0>(q) * x4;
    return POTATO_FMA((quad_perm<3, 1, 0, 0>(q)), (quad_perm<1, 2, 0, 1>(q)), pr);
}

/* rates() of quad_step.h. */
__device__ __forceinline__ float lane_rates(const LaneConst& c, float v, float q, float w, float d, float& dv,
                                            float& dq, float& dw) {
#pragma clang fp contract(off)
    const float s = POTATO_FMA(d, d, c.two_w * d);
    /* even lanes: u = s0 - s1 (= A), s2 - s3 (= -B); odd lanes: P01, P23 */
    const float sn = quad_perm<1, 0, 3, 2>(s);
    const float P = s + sn;
    const float ssum = P + quad_perm<2, 3, 0, 1>(P);
    const float m = c.odd ? P : s - sn;
    /* lane 0: A + B, lane 1: P01 - P23 (a holds -ay), lane 2: A - B */
    const float T = POTATO_FMA((quad_perm<2, 3, 0, 1>(m)), c.sT, m);
    const float ftm2 = POTATO_FMA(c.kf_m2, ssum, c.F0_2);
    const float b = lane_tilt(c, q);
    const float G = POTATO_FMA(c.kf_m, ssum, c.F0_g);
    const float vxy = POTATO_FMA(ftm2, b, c.ncd_m * v);
    const float vz = POTATO_FMA(c.ncd_m, v, POTATO_FMA(-ftm2, b, G));
    dv = c.isz ? vz : vxy;
    /* lane 3 holds the scalar part -(q1 w0 + q2 w1 + q3 w2) */
    const float w1 = quad_perm<1, 2, 0, 2>(w);
    const float w2 = quad_perm<2, 0, 1, 1>(w) * c.s3;
    const float w3 = quad_perm<0, 1, 2, 0>(w) * c.s3;
    dq = POTATO_FMA((-quad_perm<2, 0, 1, 2>(q)), w1,
                    POTATO_FMA((quad_perm<1, 2, 0, 1>(q)), w2, (quad_perm<3, 3, 3, 0>(q) * w3)));
    dw = POTATO_FMA(-c.g, w1 * w2, c.a * T);
    return ssum;
}

/* controller() of quad_step.h: the lane's rotor command. */
template <bool CARRY>
__device__ __forceinline__ float lane_controller(const LaneConst& c, const Limits& L, LaneAgent& a, float wp) {
#pragma clang fp contract(off)
    float e = wp - a.p;
    const float e0 = quad_bcast<0>(e), e1 = quad_bcast<1>(e), e2 = quad_bcast<2>(e);
    const float n2 = POTATO_FMA(e2, e2, POTATO_FMA(e1, e1, e0 * e0));
    const float sc = n2 > L.r_sat2 ? L.r_sat * rsq(n2) : 1.0f;
    e *= sc;
    const float y = CARRY ? POTATO_FMA(e, L.dt, a.ip_lo) : e * L.dt;
    const float s = a.ip + y;
    const float cl = clampf_(s, -L.ipos_max, L.ipos_max);
    if (CARRY) {
        const float lo = y - (s - a.ip);
        a.ip_lo = cl == s ? lo : 0.0f;
    }
    a.ip = cl;
    float acc = POTATO_FMA(-c.kdp, a.v, POTATO_FMA(c.kip, cl, c.kpp * e));
    const float accz = fmaxf(acc + L.g, L.az_min);
    acc = c.isz ? accz : acc;
    const float a0 = quad_bcast<0>(acc), a1 = quad_bcast<1>(acc), a2 = quad_bcast<2>(acc);
    const float bz = POTATO_FMA(c.kz, lane_tilt(c, a.q), c.oz);
    const float fc = c.mass * POTATO_FMA(a2, quad_bcast<2>(bz), POTATO_FMA(a1, quad_bcast<1>(bz), a0 * quad_bcast<0>(bz)));
    const float ra = rsq(POTATO_FMA(a2, a2, POTATO_FMA(a1, a1, a0 * a0)));
    const float n = acc * ra;
    const float qr0 = 1.0f + quad_bcast<2>(n);
    const float rq = rsq(qr0 + qr0);
    /* lane 0: qd2, lane 1: -qd1, lane 2: qd0 */
    const float D = (c.isz ? qr0 : n) * rq;
    const float Da = quad_perm<1, 0, 1, 2>(D) * c.sQa;
    const float Db = quad_perm<2, 2, 0, 1>(D);
    const float Dc = quad_perm<0, 1, 2, 0>(D) * c.sQc;
    /* lanes 0-2: vector part of conj(q) o q_des, lane 3 its scalar part */
    const float q = a.q;
    const float E = POTATO_FMA((quad_perm<2, 2, 2, 1>(q)), Dc,
                               POTATO_FMA((-quad_perm<0, 1, 0, 0>(q)), Db, (quad_perm<3, 3, 1, 3>(q) * Da)));
    const float sg = quad_bcast<3>(E) < 0.0f ? -2.0f : 2.0f;
    const float eatt = sg * E;
    a.ia = clampf_(POTATO_FMA(eatt, L.dt, a.ia), -L.iatt_max, L.iatt_max);
    const float wdes = POTATO_FMA(-c.kda, a.w, POTATO_FMA(c.kia, a.ia, c.kpa * eatt));
    const float erate = wdes - a.w;
    a.ir = clampf_(POTATO_FMA(erate, L.dt, a.ir), -L.irate_max, L.irate_max);
    const float alpha = POTATO_FMA(-c.kdr_dt, a.w - a.wprev, POTATO_FMA(c.kir, a.ir, c.kpr * erate));
    a.wprev = a.w;
    const float Iw = c.I * a.w;
    const float w1 = quad_perm<1, 2, 0, 2>(a.w), w2 = quad_perm<2, 0, 1, 1>(a.w);
    const float t = POTATO_FMA(c.I, alpha, POTATO_FMA((quad_perm<2, 0, 1, 2>(Iw)), w1, (-(quad_perm<1, 2, 0, 1>(Iw) * w2))));
    const float X = t * c.mix;
    const float f4 = 0.25f * fc;
    const float fz = f4 + quad_bcast<2>(X) * c.sZ;
    const float fxy = POTATO_FMA(quad_bcast<1>(X), c.sYr, quad_bcast<0>(X) * c.sX);
    const float f = clampf_(fz + fxy, 0.0f, c.f_max);
    return sqrt_fast(f * c.inv_kf) - c.w_ref;
}

/* rk4_step() of quad_step.h. */
template <bool CARRY>
__device__ __forceinline__ void lane_rk4(const LaneConst& c, const Limits& L, LaneAgent& a, float dc) {
#pragma clang fp contract(off)
    const float z = -(L.dt * c.inv_tau);
    const float hz = 0.5f * z;
    const float c2 = 1.0f + hz;
    const float c3 = POTATO_FMA(hz, c2, 1.0f);
    const float c4 = POTATO_FMA(z, c3, 1.0f);
    const float cR = POTATO_FMA(z * (1.0f / 6.0f), ((1.0f + (c2 + c2)) + (c3 + c3)) + c4, 1.0f);
    const float e = a.d - dc;
    float kv, kq, kw, ss;
    ss = lane_rates(c, a.v, a.q, a.w, a.d, kv, kq, kw);
    float av = kv, aw = kw, A3 = kv, aq = kq, ass = ss;
    auto stage = [&](float h, float hq, float cp) {
        const float sv = POTATO_FMA(h, kv, a.v), sw = POTATO_FMA(h, kw, a.w);
        const float sq = POTATO_FMA(hq, kq, a.q), sd = POTATO_FMA(e, cp, dc);
        ss = lane_rates(c, sv, sq, sw, sd, kv, kq, kw);
    };
    auto add = [&]() {
        av = POTATO_FMA(2.0f, kv, av);
        aw = POTATO_FMA(2.0f, kw, aw);
        A3 += kv;
        aq = POTATO_FMA(2.0f, kq, aq);
        ass = POTATO_FMA(2.0f, ss, ass);
    };
    stage(L.half_dt, L.quarter_dt, c2);
    add();
    stage(L.half_dt, L.quarter_dt, c3);
    add();
    stage(L.dt, L.half_dt, c4);
    ass += ss;
    add_carry<CARRY>(a.p, a.p_lo, POTATO_FMA(L.dt2_6, A3, L.dt * a.v));
    add_carry<CARRY>(a.v, a.v_lo, L.dt6 * (av + kv));
    a.w = POTATO_FMA(L.dt6, aw + kw, a.w);
    a.q = POTATO_FMA(L.dt12, aq + kq, a.q);
    a.d = POTATO_FMA(e, cR, dc);
    add_carry<CARRY>(a.J, a.J_lo, POTATO_FMA(L.dt6, ass, L.dt * c.four_w2));
    const float q0 = quad_bcast<3>(a.q), q1 = quad_bcast<0>(a.q), q2 = quad_bcast<1>(a.q), q3 = quad_bcast<2>(a.q);
    a.q *= rsq(POTATO_FMA(q3, q3, POTATO_FMA(q2, q2, POTATO_FMA(q1, q1, q0 * q0))));
}

}  // namespace potato
