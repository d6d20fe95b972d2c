// One drone on the four lanes of a DPP quad, for batches with fewer waves than the
// GPU has SIMDs. A drone's steps are one dependent chain, and a lone wave issues
// one instruction in about five cycles whatever it does, so the chain's time is
// its instruction count: 64 drones of 4096 behind the attitude controller kept 64
// of the 1024 SIMDs busy for 1.13 us a step. Here lane j of a quad holds component
// j of each of the drone's vectors (position, quaternion or Euler angle, velocity,
// rate, rotor j), every vector operation is one instruction for all its components
// and the other components come through DPP operands, which cost no instruction of
// their own in most places. The maps are those of the structured RK4 steps
// (cf_device.hpp: reduced variants only), with the drone's sums taken over the quad,
// and the forward maps round as theirs do: states come out bit for bit the same.
//
// Lane 3 has no third component of 3-vectors: its constants are zero there, its
// slots stay zero or are never read.
#pragma once
#include "cf_device.hpp"

namespace cfk {

template <int A, int B, int C, int D>
__device__ __forceinline__ float qperm(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), A | B << 2 | C << 4 | D << 6,
                                                              0xf, 0xf, true));
}
template <int I>
__device__ __forceinline__ float qb(float v) { return qperm<I, I, I, I>(v); }
// sum over the quad, the same bits in all four lanes
__device__ __forceinline__ float qsum(float v) {
    v += qperm<1, 0, 3, 2>(v);
    return v + qperm<2, 3, 0, 1>(v);
}
__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// the lane's byte offset of component j of a row group in an [S][D] array; rows
// counted from the array's start. Quad launches keep S * D * 4 bytes below 2^32.
struct QLane {
    int j;
    uint32_t d, D;
    __device__ __forceinline__ uint32_t row(int first) const { return ((uint32_t)(first + j) * D + d) * 4u; }
};
__device__ __forceinline__ float q_load(const float* base, uint32_t off) {
    return *(const float*)((const char*)base + off);
}
__device__ __forceinline__ void q_store(float* base, uint32_t off, float v) { *(float*)((char*)base + off) = v; }

// ---------------------------------------------------------------------------
// first principles

struct QFp {
    float k1, k2, a2r, m0, m1, m2, m3, tr, dj;   // wrench: row j of the torque mixing (lane 3: zero)
    float p2, p4, pf, l1, l2, l4, g, wr;
    float sgn, sb, sd, c0;                       // signs of the lane's products
};
struct QFpBack {
    float t0, t1, t2;                            // column j of the torque mixing (rotor j)
    float q2, q4, qf;
    float sq;                                    // lanes 0, 1: 1 (rows with the -2 (x^2 + y^2) term), else 0
    float sx;                                    // -1, 1, 1, -1
};

template <class R>
__device__ __forceinline__ QFp q_load_fp(const R& rec, int j) {
    QFp P;
    const bool v3 = j < 3;
    P.k1 = rec(F_K1); P.k2 = rec(F_K2); P.a2r = rec(F_A2R);
    const int jj = v3 ? j : 2;
    P.m0 = v3 ? rec(F_TX + 4 * jj) : 0.f;
    P.m1 = v3 ? rec(F_TX + 4 * jj + 1) : 0.f;
    P.m2 = v3 ? rec(F_TX + 4 * jj + 2) : 0.f;
    P.m3 = v3 ? rec(F_TX + 4 * jj + 3) : 0.f;
    P.tr = v3 ? rec(F_TR + jj) : 0.f;
    P.dj = v3 ? rec(F_DJ + jj) : 0.f;
    P.p2 = rec(F_P2); P.p4 = rec(F_P4); P.pf = rec(F_PF);
    P.l1 = rec(F_L1); P.l2 = rec(F_L2); P.l4 = rec(F_L4);
    P.g = j == 2 ? rec(P_GRAVITY) : 0.f;
    P.wr = rec(D_WR);
    P.sgn = v3 ? 1.f : -1.f;
    P.sb = j < 2 ? 1.f : (j == 2 ? -1.f : 0.f);
    P.sd = j == 0 ? 1.f : (v3 ? -1.f : 0.f);
    P.c0 = j == 2 ? 0.5f : 0.f;
    return P;
}
template <class R>
__device__ __forceinline__ QFpBack q_load_fp_back(const R& rec, int j) {
    QFpBack B;
    B.t0 = rec(F_TX + j); B.t1 = rec(F_TY + j); B.t2 = rec(F_TZ + j);
    B.q2 = rec(F_Q2); B.q4 = rec(F_Q4); B.qf = rec(F_QF);
    B.sq = j < 2 ? 1.f : 0.f;
    B.sx = (j == 0 || j == 3) ? -1.f : 1.f;
    return B;
}

// state of a first-principles drone: rotor rows as deviations from W_r
struct QFpState {
    float p, v, q, w, r, cp, cv;   // cp, cv: lost low parts of p and v
};

// {2 F / m - 2 F_r / m (all lanes), torque j / J_j} of the rotor deviation r
__device__ __forceinline__ void q_wrench(float r, const QFp& P, float* a, float* t) {
    const float d = r * fma_(P.k2, r, P.k1);
    *a = qsum(d);
    *t = fma_(qb<3>(d), P.m3, fma_(qb<2>(d), P.m2, fma_(qb<1>(d), P.m1, fma_(qb<0>(d), P.m0, P.tr))));
}
struct QWrench {
    float a[4], t[4];
};
__device__ __forceinline__ void q_wrenches(float r, float rc, const QFp& P, QWrench& W) {
    const float e = r - rc;
    q_wrench(r, P, &W.a[0], &W.t[0]);
    q_wrench(fma_(e, P.p2, rc), P, &W.a[1], &W.t[1]);
    q_wrench(fma_(e, P.p4, rc), P, &W.a[3], &W.t[3]);
    W.a[2] = fma_(P.l1, W.a[0], fma_(P.l4, W.a[3], P.l2 * W.a[1]));
    W.t[2] = fma_(P.l1, W.t[0], fma_(P.l4, W.t[3], P.l2 * W.t[1]));
#pragma unroll
    for (int s = 0; s < 4; ++s) W.a[s] += P.a2r;
}

// half the body z axis (lane 3: 0)
__device__ __forceinline__ float q_half_ez(float q, const QFp& P) {
    const float b = qperm<2, 2, 0, 3>(q) * P.sb, d = qperm<1, 0, 1, 3>(q) * P.sd;
    return fma_(qperm<3, 3, 1, 3>(q), d, fma_(qperm<0, 1, 0, 3>(q), b, P.c0));
}
// the body rate as the quaternion product and Euler's equations use it
struct QRate {
    float w1, w2, w3;
};
__device__ __forceinline__ QRate q_rate(float w, const QFp& P) {
    return {qperm<0, 1, 2, 0>(w) * P.sgn, qperm<2, 0, 1, 1>(w) * P.sgn, qperm<1, 2, 0, 2>(w)};
}
// twice the quaternion rate, q (x) [w, 0]
__device__ __forceinline__ float q_quat_rate(float q, const QRate& w) {
    return fma_(-qperm<2, 0, 1, 2>(q), w.w3, fma_(qperm<1, 2, 0, 1>(q), w.w2, qperm<3, 3, 3, 0>(q) * w.w1));
}
__device__ __forceinline__ float q_body_rate(const QRate& w, float t, float dj) { return fma_(-dj, w.w2 * w.w3, t); }

__device__ __forceinline__ void q_advance_pv(float* p, float* v, float* cp, float* cv, float h, float a1, float a2,
                                             float a3, float a4) {
    const float h6 = h * (1.0f / 6.0f);
    const float s = a2 + a3;
    const float dp = h * fma_(h6, a1 + s, *v);
    const float dv = h6 * fma_(2.f, s, a1 + a4);
    comp_add(p, cp, dp);
    comp_add(v, cv, dv);
}

// one step under the rotor command rc (this lane's rotor); n1 = q_half_ez of x.q
__device__ __forceinline__ void q_fp_step(QFpState& x, float rc, float n1, const QFp& P, float h, int renorm) {
    const float h2 = 0.5f * h, h4 = 0.25f * h, h6 = h * (1.0f / 6.0f), h12 = 0.5f * h6;
    QWrench W;
    q_wrenches(x.r, rc, P, W);
    x.r = fma_(x.r - rc, P.pf, rc);
    QRate w = q_rate(x.w, P);
    const float a1 = fma_(W.a[0], n1, -P.g);
    const float tq = q_quat_rate(x.q, w), tw = q_body_rate(w, W.t[0], P.dj);
    float q = fma_(h4, tq, x.q);
    w = q_rate(fma_(h2, tw, x.w), P);
    const float a2 = fma_(W.a[1], q_half_ez(q, P), -P.g);
    float sq = q_quat_rate(q, w), sw = q_body_rate(w, W.t[1], P.dj);
    q = fma_(h4, sq, x.q);
    w = q_rate(fma_(h2, sw, x.w), P);
    const float a3 = fma_(W.a[2], q_half_ez(q, P), -P.g);
    const float kq3 = q_quat_rate(q, w), kw3 = q_body_rate(w, W.t[2], P.dj);
    sq += kq3;
    sw += kw3;
    q = fma_(h2, kq3, x.q);
    w = q_rate(fma_(h, kw3, x.w), P);
    const float a4 = fma_(W.a[3], q_half_ez(q, P), -P.g);
    x.q = fma_(h12, fma_(2.f, sq, tq + q_quat_rate(q, w)), x.q);
    x.w = fma_(h6, fma_(2.f, sw, tw + q_body_rate(w, W.t[3], P.dj)), x.w);
    q_advance_pv(&x.p, &x.v, &x.cp, &x.cv, h, a1, a2, a3, a4);
    if (renorm) x.q *= rsqrt_hw(qsum(x.q * x.q));
}

// adjoints of the state rows a lane holds
struct QFpAdj {
    float p, v, q, w, r;
};

// one stage: given the adjoints kq (of twice the quaternion rate), kw and ga, the
// adjoints of the stage's quaternion, rate and wrench
__device__ __forceinline__ void q_fp_stage_vjp(float q, float w, float a2, const QFp& P, const QFpBack& B, float kq,
                                               float kw, float ga, float* qo, float* wo, float* ao) {
    *ao = qsum(ga * q_half_ez(q, P));
    const float b = a2 * ga;
    const float b0 = qb<0>(b), b1 = qb<1>(b) * B.sx, b2 = qb<2>(b) * (-2.f * B.sq);
    const QRate W = q_rate(w, P);
    float t = fma_(b2, q, fma_(qperm<3, 2, 1, 0>(q), b1, qperm<2, 3, 0, 1>(q) * b0));
    t = fma_(-qperm<3, 3, 3, 0>(kq), W.w1, t);
    t = fma_(-qperm<1, 2, 0, 1>(kq), W.w2, t);
    *qo = fma_(qperm<2, 0, 1, 2>(kq), W.w3, t);
    const float k3 = qb<3>(kq), k1 = qperm<1, 2, 0, 3>(kq), k2 = qperm<2, 0, 1, 3>(kq);
    float s = qb<3>(q) * kq;
    s = fma_(-q, k3, s);
    s = fma_(qperm<2, 0, 1, 3>(q), k1, s);
    s = fma_(-qperm<1, 2, 0, 3>(q), k2, s);
    const float u = P.dj * kw;
    s = fma_(-qperm<1, 2, 0, 3>(u), W.w2, s);
    *wo = fma_(-qperm<2, 0, 1, 3>(u), W.w3, s);
}

// VJP of q_fp_step (with its renormalisation): y the adjoint of the new state, out
// the state's; rcb accumulates the rotor command's
__device__ __forceinline__ void q_fp_step_vjp(const QFpState& x, float rc, const QFp& P, const QFpBack& B, float h,
                                              int renorm, const QFpAdj& y, QFpAdj& out, float* rcb) {
    const float h2 = 0.5f * h, h4 = 0.25f * h, h6 = h * (1.0f / 6.0f), h12 = 0.5f * h6;
    QWrench W;
    q_wrenches(x.r, rc, P, W);
    QRate wr = q_rate(x.w, P);
    const float kq1 = q_quat_rate(x.q, wr), kw1 = q_body_rate(wr, W.t[0], P.dj);
    const float q2 = fma_(h4, kq1, x.q), w2 = fma_(h2, kw1, x.w);
    wr = q_rate(w2, P);
    const float kq2 = q_quat_rate(q2, wr), kw2 = q_body_rate(wr, W.t[1], P.dj);
    const float q3 = fma_(h4, kq2, x.q), w3 = fma_(h2, kw2, x.w);
    wr = q_rate(w3, P);
    const float kq3 = q_quat_rate(q3, wr), kw3 = q_body_rate(wr, W.t[2], P.dj);
    const float q4 = fma_(h2, kq3, x.q), w4 = fma_(h, kw3, x.w);
    float lq = y.q;
    if (renorm) {
        const float kq4 = q_quat_rate(q4, q_rate(w4, P));
        const float yq = fma_(h12, fma_(2.f, kq2 + kq3, kq1 + kq4), x.q);
        const float inv = rsqrt_hw(qsum(yq * yq));
        const float qn = yq * inv;
        lq = (lq - qn * qsum(qn * lq)) * inv;
    }
    // accelerations: a1 gets h/6 lv + h^2/6 lp, a2 and a3 h/3 lv + h^2/6 lp, a4 h/6 lv
    const float g4 = h6 * y.v, g1 = fma_(h * h6, y.p, g4), g23 = g1 + g4;
    out.p = y.p;
    out.v = fma_(h, y.p, y.v);
    const float qh = h12 * lq, wh = h6 * y.w;
    float kq = qh, kw = wh, qo, wo, ab[4], tb[4];
    tb[3] = kw;
    q_fp_stage_vjp(q4, w4, W.a[3], P, B, kq, kw, g4, &qo, &wo, &ab[3]);
    out.q = lq + qo;
    out.w = y.w + wo;
    kq = fma_(h2, qo, qh + qh);
    kw = fma_(h, wo, wh + wh);
    tb[2] = kw;
    q_fp_stage_vjp(q3, w3, W.a[2], P, B, kq, kw, g23, &qo, &wo, &ab[2]);
    out.q += qo;
    out.w += wo;
    kq = fma_(h4, qo, qh + qh);
    kw = fma_(h2, wo, wh + wh);
    tb[1] = kw;
    q_fp_stage_vjp(q2, w2, W.a[1], P, B, kq, kw, g23, &qo, &wo, &ab[1]);
    out.q += qo;
    out.w += wo;
    kq = fma_(h4, qo, qh);
    kw = fma_(h2, wo, wh);
    tb[0] = kw;
    q_fp_stage_vjp(x.q, x.w, W.a[0], P, B, kq, kw, g1, &qo, &wo, &ab[0]);
    out.q += qo;
    out.w += wo;
    // stage 3's wrench back to stages 1, 2, 4; then rotor j's thrust difference
    const float l[4] = {P.l1, P.l2, 0.f, P.l4};
    const float e = x.r - rc, k22 = 2.f * P.k2;
    const auto back = [&](int s, float r) {
        const float a = fma_(l[s], ab[2], ab[s]), t = fma_(l[s], tb[2], tb[s]);
        const float f = fma_(qb<0>(t), B.t0, fma_(qb<1>(t), B.t1, fma_(qb<2>(t), B.t2, a)));
        return f * fma_(k22, r, P.k1);
    };
    const float r1 = back(0, x.r), r2 = back(1, fma_(e, P.p2, rc)), r4 = back(3, fma_(e, P.p4, rc));
    out.r = fma_(P.pf, y.r, fma_(P.p2, r2, fma_(P.p4, r4, r1)));
    *rcb = fma_(B.qf, y.r, fma_(B.q2, r2, fma_(B.q4, r4, *rcb)));
}

// ---- attitude controller: axis j in lane j (yaw rate in lane 2), rotor j's
// allocation in lane j, the commanded thrust in lane 3's command
struct QPid {
    float akp, aki, dta, rkp, rki, rkd, inv_dt, jc, dtr;   // lanes without the term: 0
    float a0, a1, a2, a3, lo, hi, fr, k4, disc, k1w, vtx;
    float sp;                                      // 1, -1, 0, 0
};
struct QPidBack {
    float c0, c1, c2, c3;                          // column of the allocation: torque j, lane 3 thrust
};
struct QPidState {
    float ia, ir, wp;
};
struct QPidTrace {
    float y, x, disc;
    bool pass;
};

template <class R>
__device__ __forceinline__ QPid q_load_pid(const R& rec, int j, float dt, float inv_dt) {
    QPid C;
    const int j2 = j < 2 ? j : 1, j3 = j < 3 ? j : 2;
    const float m2 = j < 2 ? 1.f : 0.f, m3 = j < 3 ? 1.f : 0.f;
    C.akp = m2 * rec(P_ANG_KP + j2);
    C.aki = m2 * rec(P_ANG_KI + j2);
    C.dta = m2 * dt;
    C.rkp = m3 * rec(P_RATE_KP + j3);
    C.rki = m3 * rec(P_RATE_KI + j3);
    C.rkd = m3 * rec(P_RATE_KD + j3);
    C.inv_dt = inv_dt;
    C.jc = m3 * rec(P_J_CTRL + j3);
    C.dtr = m3 * dt;
    C.a0 = rec(P_ALLOC + 4 * j); C.a1 = rec(P_ALLOC + 4 * j + 1);
    C.a2 = rec(P_ALLOC + 4 * j + 2); C.a3 = rec(P_ALLOC + 4 * j + 3);
    C.fr = rec(D_FR);
    C.lo = -C.fr;
    C.hi = rec(P_F_MAX) - C.fr;
    C.k4 = 4.f * rec(P_THRUST + 2);
    C.disc = rec(D_DISC_R);
    C.k1w = rec(D_K1W);
    C.vtx = rec(D_VTX);
    C.sp = j == 0 ? 1.f : (j == 1 ? -1.f : 0.f);
    return C;
}
template <class R>
__device__ __forceinline__ QPidBack q_load_pid_back(const R& rec, int j) {
    const int c = j < 3 ? j + 1 : 0;
    return {rec(P_ALLOC + c), rec(P_ALLOC + 4 + c), rec(P_ALLOC + 8 + c), rec(P_ALLOC + 12 + c)};
}

// rotor j's command, the controller's state advanced in c; n = q_half_ez(q)
__device__ __forceinline__ float q_pid(float q, float w, float n, float u, QPidState& c, const QPid& C, int j,
                                       QPidTrace& tr) {
    // lane 0: roll = atan2(s1, c1); lane 1: pitch = asin(s2) = atan2(s2, sqrt(1 - s2^2))
    float y = 2.f * fma_(qperm<1, 2, 2, 3>(q), qperm<2, 0, 2, 3>(q) * C.sp, qb<3>(q) * q);
    const float yc = fminf(fmaxf(y, -1.f), 1.f);
    tr.y = y;
    y = j == 1 ? yc : y;
    const float x = j == 1 ? sqrt_hw((1.f - yc) * (1.f + yc)) : 2.f * qb<2>(n);
    tr.x = x;
    const float at = atan2_poly(y, x);
    const float ea = u - (j < 2 ? at : 0.f);
    c.ia = fma_(ea, C.dta, c.ia);
    // (lane 2: the yaw-rate command itself; zero times an infinite one would be NaN)
    const float er = (j < 2 ? fma_(C.akp, ea, C.aki * c.ia) : ea) - w;
    c.ir = fma_(er, C.dtr, c.ir);
    const float tq = C.jc * fma_(-(C.rkd * (w - c.wp)), C.inv_dt, fma_(C.rkp, er, C.rki * c.ir));
    c.wp = w;
    const float dfr = fma_(C.a0, qb<3>(u), -C.fr) + fma_(qb<2>(tq), C.a3, fma_(qb<1>(tq), C.a2, qb<0>(tq) * C.a1));
    const float df = fminf(fmaxf(dfr, C.lo), C.hi);
    tr.disc = fma_(C.k4, df, C.disc);
    tr.pass = dfr >= C.lo && dfr <= C.hi && tr.disc > 0.f;
    return tr.disc > 0.f ? 2.f * df * rcp_hw(sqrt_hw(tr.disc) + C.k1w) : C.vtx;
}

// VJP: rcb rotor j's, cb the new controller state's adjoints; adds to xq, xw and ub,
// writes the old controller state's adjoints to co
__device__ __forceinline__ void q_pid_vjp(float q, const QPid& C, const QPidBack& CB, const QPidTrace& tr, int j,
                                          float rcb, const QPidState& cb, float* xq, float* xw, float* ub,
                                          QPidState& co) {
    const float f = tr.pass ? rcb * rsqrt_hw(tr.disc) : 0.f;
    const float wv = fma_(qb<3>(f), CB.c3, fma_(qb<2>(f), CB.c2, fma_(qb<1>(f), CB.c1, qb<0>(f) * CB.c0)));
    const float al = C.jc * wv;
    co.ir = fma_(C.rki, al, cb.ir);
    const float er = fma_(C.rkp, al, co.ir * C.dtr);
    co.wp = C.rkd * al * C.inv_dt;
    *xw += (cb.wp - er) - co.wp;
    co.ia = fma_(C.aki, er, cb.ia);
    const float ea = j < 2 ? fma_(C.akp, er, co.ia * C.dta) : er;
    *ub += j == 3 ? wv : ea;
    // lane 0: adjoints of s1 and c1; lane 1: of s2
    const float i2 = rcp_hw(fma_(tr.y, tr.y, tr.x * tr.x));
    const float in = fabsf(tr.y) <= 1.f ? rsqrt_hw(fma_(-tr.y, tr.y, 1.f)) : 0.f;
    const float sb = -2.f * ea * (j == 1 ? in : tr.x * i2);
    const float cb1 = -4.f * ea * tr.y * i2;   // minus four times c1's adjoint, -(-roll) y / (x^2 + y^2)
    const float s1 = qb<0>(sb), c1 = qb<0>(cb1) * (j < 2 ? 1.f : 0.f), s2 = qb<1>(sb) * (j & 1 ? 1.f : -1.f);
    *xq = fma_(qperm<3, 2, 1, 0>(q), s1, fma_(qperm<2, 3, 0, 1>(q), s2, fma_(q, c1, *xq)));
}

// ---------------------------------------------------------------------------
// identified model: angle j, rate j, position j in lanes 0..2, the thrust in all

struct QId {
    float c1, c2, c3, al, be, ga, de, a4, b4;   // lane 3: zero
    float p[4], pf, cf_m, g, f_hover;
    float sy;                                   // 1, -1, 0, 0
    bool direct;                                // no thrust dynamics
};
struct QIdBack {
    float q[4], qf;
};
struct QIdState {
    float p, a, v, w, f, cp, cv;
};
struct QIdBase {
    float a0, s0, c0;
};

template <class R>
__device__ __forceinline__ QId q_load_id(const R& rec, int j) {
    QId P;
    const bool v3 = j < 3;
    const int i = v3 ? j : 2;
    const float m = v3 ? 1.f : 0.f;
    P.c1 = m * rec(P_CPSI1 + i); P.c2 = m * rec(P_CPSI2 + i); P.c3 = m * rec(P_CPSI3 + i);
    P.al = m * rec(I_AL + i); P.be = m * rec(I_BE + i); P.ga = m * rec(I_GA + i); P.de = m * rec(I_DE + i);
    P.a4 = m * rec(I_A4 + i); P.b4 = m * rec(I_B4 + i);
#pragma unroll
    for (int s = 0; s < 4; ++s) P.p[s] = rec(I_P + s);
    P.pf = rec(I_PF);
    P.cf_m = rec(D_CF_M);
    P.g = j == 2 ? rec(P_GRAVITY) : 0.f;
    P.f_hover = rec(D_F_HOVER);
    P.direct = rec(P_CTAU) == 0.f;
    P.sy = j == 0 ? 1.f : (j == 1 ? -1.f : 0.f);
    return P;
}
template <class R>
__device__ __forceinline__ QIdBack q_load_id_back(const R& rec) {
    QIdBack B;
#pragma unroll
    for (int s = 0; s < 4; ++s) B.q[s] = rec(I_Q + s);
    B.qf = rec(I_QF);
    return B;
}

__device__ __forceinline__ void q_sincos(float a, float* s, float* c) {
    sincos_cw(a, s, c);
    if (__builtin_expect(fabsf(a) > 32768.f, 0)) sincosf(a, s, c);
}

// sines and cosines at N offsets from the base angle; beyond 1/16 rad on any axis in
// full (as one lane per drone decides)
template <int N>
__device__ __forceinline__ void q_sincos_off(const float* d, const QIdBase& b, float* s, float* c) {
    float m = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        m = fmaxf(m, fabsf(d[i]));
        const float d2 = d[i] * d[i];
        const float sd = fma_(d[i] * d2, fma_(d2, 1.f / 120.f, -1.f / 6.f), d[i]);
        const float cm1 = d2 * fma_(d2, fma_(d2, -1.f / 720.f, 1.f / 24.f), -0.5f);
        s[i] = fma_(b.s0, cm1, fma_(b.c0, sd, b.s0));
        c[i] = fma_(b.c0, cm1, fma_(-b.s0, sd, b.c0));
    }
    m = fmaxf(m, qperm<1, 0, 3, 2>(m));
    m = fmaxf(m, qperm<2, 3, 0, 1>(m));
    if (__builtin_expect(m > 0.0625f, 0)) {
        float r[N];
#pragma unroll
        for (int i = 0; i < N; ++i) r[i] = b.a0 + d[i];
        sincos_slow<N>(r, s, c);
    }
}
__device__ __forceinline__ void q_id_base(float a, QIdBase& b) {
    b.a0 = a;
    q_sincos(a, &b.s0, &b.c0);
}
__device__ __forceinline__ void q_id_rebase(float a, QIdBase& b) {
    const float d = a - b.a0;
    float s, c;
    q_sincos_off<1>(&d, b, &s, &c);
    b.a0 = a;
    b.s0 = s;
    b.c0 = c;
}

// component j of a R(Psi) e_z - g e_z from the lane's sine and cosine
__device__ __forceinline__ float q_id_acc(float s, float c, float a, const QId& P, int j) {
    // lane 0: cps (sth cph) + sps sph, lane 1: sps (sth cph) - cps sph, lane 2: cth cph
    // (whose zero factor of sps may not meet a yaw that is not finite: sph takes its place)
    const float c2 = qperm<2, 2, 1, 3>(c), s2 = qperm<2, 2, 0, 3>(s);
    const float al = j == 1 ? s2 : c2, be = j == 1 ? c2 : s2;
    const float X = qb<0>(c) * (j == 2 ? 1.f : qb<1>(s)), Y = qb<0>(s) * P.sy;
    return fma_(a, fma_(al, X, be * Y), -P.g);
}

struct QIdStages {
    float d2, off[3], a[4], df;
};
__device__ __forceinline__ void q_id_stages(const QIdState& x, float u, const QId& P, float h, QIdStages& T) {
    const float h2 = 0.5f * h;
    T.d2 = fma_(P.c1, x.a, fma_(P.c2, x.w, P.c3 * u));
    T.off[0] = h2 * x.w;
    T.off[1] = fma_(h2 * h2, T.d2, T.off[0]);
    T.off[2] = fma_(P.b4, T.d2, P.a4 * x.w);
    const float u3 = qb<3>(u);
    T.df = P.direct ? 0.f : x.f - u3;
    const float fu = P.cf_m * u3, fe = P.cf_m * T.df;
#pragma unroll
    for (int s = 0; s < 4; ++s) T.a[s] = fma_(fe, P.p[s], fu);
}

__device__ __forceinline__ void q_id_step(QIdState& x, float u, const QId& P, float h, const QIdBase& B, int j) {
    QIdStages T;
    q_id_stages(x, u, P, h, T);
    float s[3], c[3];
    q_sincos_off<3>(T.off, B, s, c);
    const float a1 = q_id_acc(B.s0, B.c0, T.a[0], P, j), a2 = q_id_acc(s[0], c[0], T.a[1], P, j),
                a3 = q_id_acc(s[1], c[1], T.a[2], P, j), a4 = q_id_acc(s[2], c[2], T.a[3], P, j);
    x.a += fma_(P.al, x.w, P.be * T.d2);
    x.w += fma_(P.ga, x.w, P.de * T.d2);
    x.f = fma_(T.df, P.pf, qb<3>(u));
    q_advance_pv(&x.p, &x.v, &x.cp, &x.cv, h, a1, a2, a3, a4);
}

struct QIdAdj {
    float p, a, v, w, f;   // f in all lanes
};

// adjoints of one stage's angles (lanes 0..2) and specific thrust (lane 3) given
// the acceleration's, ga
__device__ __forceinline__ float q_id_stage_vjp(float s, float c, float a, float ga, int j) {
    const float cps = qb<2>(c), sps = qb<2>(s), cth = qb<1>(c), sth = qb<1>(s);
    const float G = fma_(qb<1>(ga), sps, qb<0>(ga) * cps);
    const float H = fma_(-qb<1>(ga), cps, qb<0>(ga) * sps);
    const float g2 = qb<2>(ga);
    const float Q = fma_(sth, G, cth * g2), K = fma_(cth, G, -(sth * g2));
    const float ya = j < 2 ? (j == 0 ? H : K) : (j == 2 ? -(sth * H) : Q);
    const float yb = j < 2 ? (j == 0 ? -Q : 0.f) : (j == 2 ? G : H);
    const float t = fma_(qb<0>(s), yb, qb<0>(c) * ya);
    return j == 3 ? t : a * t;
}

// VJP of q_id_step; ub accumulates the command's adjoint (lane 3: thrust)
__device__ __forceinline__ void q_id_step_vjp(const QIdState& x, float u, const QId& P, const QIdBack& K, float h,
                                              const QIdBase& B, int j, const QIdAdj& y, QIdAdj& out, float* ub) {
    const float h2 = 0.5f * h, hh4 = h2 * h2, h6 = h * (1.0f / 6.0f);
    QIdStages T;
    q_id_stages(x, u, P, h, T);
    float s[3], c[3];
    q_sincos_off<3>(T.off, B, s, c);
    const float g4 = h6 * y.v, g1 = fma_(h * h6, y.p, g4), g23 = g1 + g4;
    out.p = y.p;
    out.v = fma_(h, y.p, y.v);
    const float t1 = q_id_stage_vjp(B.s0, B.c0, T.a[0], g1, j), t2 = q_id_stage_vjp(s[0], c[0], T.a[1], g23, j),
                t3 = q_id_stage_vjp(s[1], c[1], T.a[2], g23, j), t4 = q_id_stage_vjp(s[2], c[2], T.a[3], g4, j);
    const float t23 = t2 + t3;
    const float D = fma_(P.de, y.w, fma_(P.be, y.a, fma_(hh4, t3, P.b4 * t4)));
    const float wv = fma_(P.ga, y.w, fma_(P.al, y.a, fma_(h2, t23, P.a4 * t4)));
    out.a = y.a + fma_(P.c1, D, (t1 + t23) + t4);
    out.w = y.w + fma_(P.c2, D, wv);
    // lane 3's t1..t4 are the specific thrusts' adjoints
    const float fx = qb<3>(fma_(P.p[0], t1, fma_(P.p[1], t2, fma_(P.p[2], t3, P.p[3] * t4))));
    const float fu = fma_(K.q[0], t1, fma_(K.q[1], t2, fma_(K.q[2], t3, K.q[3] * t4)));
    out.f = P.direct ? 0.f : fma_(P.pf, y.f, P.cf_m * fx);
    *ub += j == 3 ? fma_(K.qf, y.f, P.cf_m * fu) : P.c3 * D;
}

}  // namespace cfk
