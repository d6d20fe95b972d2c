// Kernels with one drone on four lanes (cf_quad.hpp): held steps, the forward
// rollout and its adjoint, for handles of one model in the reduced variants under
// RK4 with the controller on every step.
#include "cf_internal.hpp"
#include "cf_quad.hpp"
#include "cf_rollout_impl.hpp"

namespace cfk {

// One model's state, parameters and step on a quad, with the same member names for
// both: slots e0..e3 are the lane's components of the state rows 0..12 that the
// feedback sees.
template <int MODEL, int CTRL>
struct QDrone;

template <int CTRL>
struct QDrone<MODEL_FP, CTRL> {
    static constexpr bool PID = CTRL == CTRL_PID;
    struct State {
        QFpState x;
        QPidState c;
    };
    QFp P;
    QPid C;

    template <class R>
    __device__ __forceinline__ QDrone(const R& rec, int j, float dt, float inv_dt) {
        P = q_load_fp(rec, j);
        if constexpr (PID) C = q_load_pid(rec, j, dt, inv_dt);
    }
    // rows of an [S][D] array; ABS: rotor rows hold absolute speeds
    template <bool ABS>
    __device__ __forceinline__ void load(const float* b, const QLane& L, State& s) const {
        const bool v3 = L.j < 3;
        s.x.p = v3 ? q_load(b, L.row(0)) : 0.f;
        s.x.q = q_load(b, L.row(3));
        s.x.v = v3 ? q_load(b, L.row(7)) : 0.f;
        s.x.w = v3 ? q_load(b, L.row(10)) : 0.f;
        s.x.r = q_load(b, L.row(13));
        if constexpr (PID) {
            s.c.ia = L.j < 2 ? q_load(b, L.row(17)) : 0.f;
            s.c.ir = v3 ? q_load(b, L.row(19)) : 0.f;
            s.c.wp = v3 ? q_load(b, L.row(22)) : 0.f;
        }
        if constexpr (ABS) s.x.r -= P.wr;
        s.x.cp = 0.f;
        s.x.cv = 0.f;
    }
    template <bool ABS>
    __device__ __forceinline__ void store(float* b, const QLane& L, const State& s) const {
        const bool v3 = L.j < 3;
        if (v3) {
            q_store(b, L.row(0), s.x.p);
            q_store(b, L.row(7), s.x.v);
            q_store(b, L.row(10), s.x.w);
        }
        q_store(b, L.row(3), s.x.q);
        q_store(b, L.row(13), ABS ? s.x.r + P.wr : s.x.r);
        if constexpr (PID) {
            if (L.j < 2) q_store(b, L.row(17), s.c.ia);
            if (v3) {
                q_store(b, L.row(19), s.c.ir);
                q_store(b, L.row(22), s.c.wp);
            }
        }
    }
    __device__ __forceinline__ bool finite(const State& s) const {
        bool ok = isfinite(s.x.p) && isfinite(s.x.q) && isfinite(s.x.v) && isfinite(s.x.w) && isfinite(s.x.r);
        if constexpr (PID) ok = ok && isfinite(s.c.ia) && isfinite(s.c.ir) && isfinite(s.c.wp);
        return ok;
    }
    __device__ __forceinline__ void begin(const State&) {}
    __device__ __forceinline__ void step(State& s, float u, float h, int renorm, int j, int) {
        const float n = q_half_ez(s.x.q, P);
        float rc;
        if constexpr (PID) {
            QPidTrace tr;
            rc = q_pid(s.x.q, s.x.w, n, u, s.c, C, j, tr);
        } else {
            rc = u - P.wr;
        }
        q_fp_step(s.x, rc, n, P, h, renorm);
    }
    // deviations from the reference state (rp, rv: reference position and velocity)
    __device__ __forceinline__ void error(const State& s, float rp, float rv, int j, float* e) const {
        e[0] = s.x.p - rp;
        e[1] = s.x.q - (j == 3 ? 1.f : 0.f);
        e[2] = s.x.v - rv;
        e[3] = s.x.w;
    }
    static __device__ __forceinline__ float dot13(const float* g, const float* e) {
        float o = g[0] * qb<0>(e[0]);
        o = fma_(qb<1>(e[0]), g[1], o); o = fma_(qb<2>(e[0]), g[2], o);
        o = fma_(qb<0>(e[1]), g[3], o); o = fma_(qb<1>(e[1]), g[4], o);
        o = fma_(qb<2>(e[1]), g[5], o); o = fma_(qb<3>(e[1]), g[6], o);
        o = fma_(qb<0>(e[2]), g[7], o); o = fma_(qb<1>(e[2]), g[8], o); o = fma_(qb<2>(e[2]), g[9], o);
        o = fma_(qb<0>(e[3]), g[10], o); o = fma_(qb<1>(e[3]), g[11], o); o = fma_(qb<2>(e[3]), g[12], o);
        return o;
    }
    static __device__ __forceinline__ void outer13(float b, const float* e, float* g) {
        g[0] = fma_(qb<0>(e[0]), b, g[0]); g[1] = fma_(qb<1>(e[0]), b, g[1]); g[2] = fma_(qb<2>(e[0]), b, g[2]);
        g[3] = fma_(qb<0>(e[1]), b, g[3]); g[4] = fma_(qb<1>(e[1]), b, g[4]);
        g[5] = fma_(qb<2>(e[1]), b, g[5]); g[6] = fma_(qb<3>(e[1]), b, g[6]);
        g[7] = fma_(qb<0>(e[2]), b, g[7]); g[8] = fma_(qb<1>(e[2]), b, g[8]); g[9] = fma_(qb<2>(e[2]), b, g[9]);
        g[10] = fma_(qb<0>(e[3]), b, g[10]); g[11] = fma_(qb<1>(e[3]), b, g[11]); g[12] = fma_(qb<2>(e[3]), b, g[12]);
    }
    // the state column of slot k in lane j, -1 where it has none
    static __device__ __forceinline__ int column(int k, int j) {
        if (k == 1) return 3 + j;
        if (j == 3) return -1;
        return k == 0 ? j : (k == 2 ? 7 + j : 10 + j);
    }
    static __device__ __forceinline__ float pos(const State& s) { return s.x.p; }

    // adjoint: the same rows
    struct Back {
        QFpBack B;
        QPidBack CB;
        template <class R>
        __device__ __forceinline__ Back(const R& rec, int j) {
            B = q_load_fp_back(rec, j);
            if constexpr (PID) CB = q_load_pid_back(rec, j);
        }
    };
    struct Adj {
        QFpAdj x;
        QPidState c;
    };
    static __device__ __forceinline__ void zero(Adj& a) {
        a.x = {0.f, 0.f, 0.f, 0.f, 0.f};
        a.c = {0.f, 0.f, 0.f};
    }
    static __device__ __forceinline__ void add_pos(Adj& a, float v) { a.x.p += v; }
    static __device__ __forceinline__ void add_slots(Adj& a, const float* v, int) {
        a.x.p += v[0]; a.x.q += v[1]; a.x.v += v[2]; a.x.w += v[3];
    }
    __device__ __forceinline__ void vjp(const Back& K, const State& s, float u, float h, int renorm, int j, Adj& lam,
                                        float* ub) const {
        float rc;
        QPidTrace tr;
        if constexpr (PID) {
            QPidState c = s.c;
            rc = q_pid(s.x.q, s.x.w, q_half_ez(s.x.q, P), u, c, C, j, tr);
        } else {
            rc = u - P.wr;
        }
        Adj o;
        float rcb = 0.f;
        q_fp_step_vjp(s.x, rc, P, K.B, h, renorm, lam.x, o.x, &rcb);
        if constexpr (PID) q_pid_vjp(s.x.q, C, K.CB, tr, j, rcb, lam.c, &o.x.q, &o.x.w, ub, o.c);
        else *ub += rcb;
        lam = o;
    }
    __device__ __forceinline__ void store_adj(float* b, const QLane& L, const Adj& a) const {
        State s;
        s.x = {a.x.p, a.x.v, a.x.q, a.x.w, a.x.r, 0.f, 0.f};
        s.c = a.c;
        store<false>(b, L, s);
    }
};

template <int CTRL>
struct QDrone<MODEL_ID, CTRL> {
    struct State {
        QIdState x;
    };
    QId P;
    QIdBase B;

    template <class R>
    __device__ __forceinline__ QDrone(const R& rec, int j, float, float) { P = q_load_id(rec, j); }
    template <bool ABS>
    __device__ __forceinline__ void load(const float* b, const QLane& L, State& s) const {
        const bool v3 = L.j < 3;
        s.x.p = v3 ? q_load(b, L.row(0)) : 0.f;
        s.x.a = v3 ? q_load(b, L.row(3)) : 0.f;
        s.x.v = v3 ? q_load(b, L.row(6)) : 0.f;
        s.x.w = v3 ? q_load(b, L.row(9)) : 0.f;
        s.x.f = q_load(b, (12u * L.D + L.d) * 4u);
        s.x.cp = 0.f;
        s.x.cv = 0.f;
    }
    template <bool ABS>
    __device__ __forceinline__ void store(float* b, const QLane& L, const State& s) const {
        if (L.j < 3) {
            q_store(b, L.row(0), s.x.p);
            q_store(b, L.row(3), s.x.a);
            q_store(b, L.row(6), s.x.v);
            q_store(b, L.row(9), s.x.w);
        } else {
            q_store(b, (12u * L.D + L.d) * 4u, s.x.f);
        }
    }
    __device__ __forceinline__ bool finite(const State& s) const {
        return isfinite(s.x.p) && isfinite(s.x.a) && isfinite(s.x.v) && isfinite(s.x.w) && isfinite(s.x.f);
    }
    __device__ __forceinline__ void begin(const State& s) { q_id_base(s.x.a, B); }
    // n: the step's number since begin(); the sines and cosines are exact every 8th
    __device__ __forceinline__ void step(State& s, float u, float h, int, int j, int n) {
        if ((n & 7) == 0) q_id_base(s.x.a, B);
        else q_id_rebase(s.x.a, B);
        q_id_step(s.x, u, P, h, B, j);
    }
    __device__ __forceinline__ void error(const State& s, float rp, float rv, int j, float* e) const {
        e[0] = j == 3 ? s.x.f - P.f_hover : s.x.p - rp;
        e[1] = s.x.a;
        e[2] = s.x.v - rv;
        e[3] = s.x.w;
    }
    static __device__ __forceinline__ float dot13(const float* g, const float* e) {
        float o = g[0] * qb<0>(e[0]);
        o = fma_(qb<1>(e[0]), g[1], o); o = fma_(qb<2>(e[0]), g[2], o);
        o = fma_(qb<0>(e[1]), g[3], o); o = fma_(qb<1>(e[1]), g[4], o); o = fma_(qb<2>(e[1]), g[5], o);
        o = fma_(qb<0>(e[2]), g[6], o); o = fma_(qb<1>(e[2]), g[7], o); o = fma_(qb<2>(e[2]), g[8], o);
        o = fma_(qb<0>(e[3]), g[9], o); o = fma_(qb<1>(e[3]), g[10], o); o = fma_(qb<2>(e[3]), g[11], o);
        return fma_(qb<3>(e[0]), g[12], o);
    }
    static __device__ __forceinline__ void outer13(float b, const float* e, float* g) {
        g[0] = fma_(qb<0>(e[0]), b, g[0]); g[1] = fma_(qb<1>(e[0]), b, g[1]); g[2] = fma_(qb<2>(e[0]), b, g[2]);
        g[3] = fma_(qb<0>(e[1]), b, g[3]); g[4] = fma_(qb<1>(e[1]), b, g[4]); g[5] = fma_(qb<2>(e[1]), b, g[5]);
        g[6] = fma_(qb<0>(e[2]), b, g[6]); g[7] = fma_(qb<1>(e[2]), b, g[7]); g[8] = fma_(qb<2>(e[2]), b, g[8]);
        g[9] = fma_(qb<0>(e[3]), b, g[9]); g[10] = fma_(qb<1>(e[3]), b, g[10]); g[11] = fma_(qb<2>(e[3]), b, g[11]);
        g[12] = fma_(qb<3>(e[0]), b, g[12]);
    }
    static __device__ __forceinline__ int column(int k, int j) {
        if (j == 3) return k == 0 ? 12 : -1;
        return 3 * k + j;
    }
    static __device__ __forceinline__ float pos(const State& s) { return s.x.p; }

    struct Back {
        QIdBack K;
        template <class R>
        __device__ __forceinline__ Back(const R& rec, int) { K = q_load_id_back(rec); }
    };
    struct Adj {
        QIdAdj x;
    };
    static __device__ __forceinline__ void zero(Adj& a) { a.x = {0.f, 0.f, 0.f, 0.f, 0.f}; }
    static __device__ __forceinline__ void add_pos(Adj& a, float v) { a.x.p += v; }
    static __device__ __forceinline__ void add_slots(Adj& a, const float* v, int) {
        a.x.p += v[0]; a.x.a += v[1]; a.x.v += v[2]; a.x.w += v[3];
        a.x.f += qb<3>(v[0]);
    }
    __device__ __forceinline__ void vjp(const Back& K, const State& s, float u, float h, int, int j, Adj& lam,
                                        float* ub) const {
        QIdBase b;
        q_id_base(s.x.a, b);
        QIdAdj o;
        q_id_step_vjp(s.x, u, P, K.K, h, b, j, lam.x, o, ub);
        lam.x = o;
    }
    __device__ __forceinline__ void store_adj(float* b, const QLane& L, const Adj& a) const {
        State s;
        s.x = {a.x.p, a.x.a, a.x.v, a.x.w, a.x.f, 0.f, 0.f};
        store<false>(b, L, s);
    }
};

// ---------------------------------------------------------------------------
// held steps
template <int MODEL, int CTRL>
__global__ __launch_bounds__(64) void k_quad_step(StepArgs a) {
    const uint32_t d = blockIdx.x * 16u + threadIdx.x / 4u;
    if (d >= (uint32_t)a.D) return;
    const QLane L{(int)(threadIdx.x & 3u), d, (uint32_t)a.D};
    const int w = a.drone_world[d];
    using Q = QDrone<MODEL, CTRL>;
    Q m(LaneRec{a.par_aos + (size_t)w * NREC}, L.j, a.dt, a.inv_dtc);
    typename Q::State s;
    m.template load<true>(a.st, L, s);
    const float u = q_load(a.cmd, L.row(0));
    m.begin(s);
    for (int k = 0; k < a.K; ++k) m.step(s, u, a.dt, a.renorm, L.j, k);
    m.template store<true>(a.st, L, s);
    if (a.nonfinite && !m.finite(s)) atomicOr(a.nonfinite + w, 1u);
}

// ---------------------------------------------------------------------------
// rollouts

// this lane's component of the figure-eight rows [p(3), v(3)] and its offset
struct QRef {
    const float* tab;
    float off;
    int j;
    bool on;
    __device__ __forceinline__ void at(int t, float* p, float* v) const {
        *p = 0.f;
        *v = 0.f;
        if (on) {
            const float* r = tab + (size_t)t * 6 + j;
            *p = r[0] + off;
            *v = r[3];
        }
    }
};
__device__ __forceinline__ QRef q_ref(const RollArgs& a, const QLane& L) {
    QRef r{a.ref_tab, 0.f, L.j, a.has_obj && L.j < 3};
    if (r.on && a.ref_off) r.off = q_load(a.ref_off, L.row(0));
    return r;
}

// the lane's row of the world's gain
__device__ __forceinline__ void q_gain_row(const float* G, int j, float* g) {
#pragma unroll
    for (int i = 0; i < 13; ++i) g[i] = G[j * 13 + i];
}

template <int MODEL, int CTRL>
__global__ __launch_bounds__(64) void k_quad_fwd(RollArgs a) {
    rollout_priority();
    const uint32_t d = blockIdx.x * 16u + threadIdx.x / 4u;
    if (d >= (uint32_t)a.D) return;
    const QLane L{(int)(threadIdx.x & 3u), d, (uint32_t)a.D};
    const int w = a.drone_world[d];
    const size_t D = (size_t)a.D, SD = (size_t)a.S_h * D;
    using Q = QDrone<MODEL, CTRL>;
    Q m(LaneRec{a.par_aos + (size_t)w * NREC}, L.j, a.dt, a.inv_dtc);
    typename Q::State s;
    m.template load<true>(a.x0, L, s);
    m.begin(s);
    const bool fb = a.has_obj && a.gain;
    float g[13];
    if (fb) q_gain_row(a.gain + (size_t)a.gidx[w] * NG, L.j, g);
    const QRef ref = q_ref(a, L);
    float rp, rv, loss = 0.f;
    ref.at(0, &rp, &rv);
    const uint32_t uo = L.row(0);
    const float* cmd = a.cmds;
    float ubar = q_load(cmd, uo);
    float* ck = a.ckpt;
    float* tj = a.traj;
    if (ck) m.template store<true>(ck, L, s);
    if (tj) m.template store<true>(tj, L, s);
    int left = a.K;   // steps to the next checkpoint
    for (int t = 0; t < a.T; ++t) {
        // the next step's command and reference, issued early
        cmd += 4 * D;
        float un = 0.f, rpn, rvn;
        if (t + 1 < a.T) un = q_load(cmd, uo);
        ref.at(t + 1, &rpn, &rvn);
        float u = ubar;
        if (fb) {
            float e[4];
            m.error(s, rp, rv, L.j, e);
            u += Q::dot13(g, e);
        }
        if (a.has_obj) loss = fma_(a.w_u, u * u, loss);
        m.step(s, u, a.dt, a.renorm, L.j, t);
        if (a.has_obj && L.j < 3) {
            const float e = Q::pos(s) - rpn;
            loss = fma_(e, e, loss);
        }
        if (--left == 0) {
            left = a.K;
            if (ck && t + 1 < a.T) {
                ck += SD;
                m.template store<true>(ck, L, s);
            }
        }
        if (tj) {
            tj += SD;
            m.template store<true>(tj, L, s);
        }
        ubar = un;
        rp = rpn;
        rv = rvn;
    }
    if (a.xT) m.template store<true>(a.xT, L, s);
    if (a.loss) {
        loss = qsum(loss);
        if (L.j == 0) a.loss[d] = loss;
    }
}

template <int MODEL, int CTRL>
__global__ __launch_bounds__(64) void k_quad_bwd(RollArgs a) {
    rollout_priority();
    const uint32_t d = blockIdx.x * 16u + threadIdx.x / 4u;
    if (d >= (uint32_t)a.D) return;
    const QLane L{(int)(threadIdx.x & 3u), d, (uint32_t)a.D};
    if (!ckpt_tag_intact(a)) {
        if (L.j == 0) poison_gradients(a, d);
        return;
    }
    const int w = a.drone_world[d], j = L.j;
    const size_t D = (size_t)a.D, SD = (size_t)a.S_h * D;
    using Q = QDrone<MODEL, CTRL>;
    const LaneRec rec{a.par_aos + (size_t)w * NREC};
    Q m(rec, j, a.dt, a.inv_dtc);
    const typename Q::Back back(rec, j);
    const bool fb = a.has_obj && a.gain;
    float g[13], gt[4][4], gg[13];
#pragma unroll
    for (int i = 0; i < 13; ++i) gg[i] = 0.f;
    if (fb) {
        const float* G = a.gain + (size_t)a.gidx[w] * NG;
        q_gain_row(G, j, g);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int c = Q::column(k, j);
#pragma unroll
            for (int i = 0; i < 4; ++i) gt[k][i] = c >= 0 ? G[i * 13 + (c >= 0 ? c : 0)] : 0.f;
        }
    }
    const QRef ref = q_ref(a, L);
    const float two_seed = 2.f * (a.dloss ? a.dloss[d] : 1.f);
    const uint32_t uo = L.row(0);
    const auto command = [&](const typename Q::State& s, float ubar, float rp, float rv, float* e) {
        if (!fb) return ubar;
        m.error(s, rp, rv, j, e);
        return ubar + Q::dot13(g, e);
    };
    typename Q::Adj lam;
    Q::zero(lam);
    const int nseg = (a.T + a.K - 1) / a.K;
    float pn = 0.f;   // position of x_{t+1} of the step being reversed
    float rp, rv, rpn, rvn;
    ref.at(a.T, &rpn, &rvn);
    typename Q::State xq;   // state and command of the next step to reverse, loaded one step ahead
    float uq = 0.f;
    bool have_q = false;
    for (int sg = nseg - 1; sg >= 0; --sg) {
        const int t0 = sg * a.K;
        const int t1 = min(a.T, t0 + a.K);
        const float* ck = a.ckpt_in + (size_t)sg * SD;
        // recompute x_{t0+1} .. x_{t1-1} into segment slots 1..; slot 0 is the
        // checkpoint. The last segment steps once more for the final position.
        const int n_re = (sg == nseg - 1) ? (t1 - t0) : (t1 - t0 - 1);
        if (n_re > 0) {
            typename Q::State x;
            m.template load<true>(ck, L, x);
            m.begin(x);
            float* slot = a.seg;
            const float* cmd = a.cmds + (size_t)t0 * 4 * D;
            for (int i = 0; i < n_re; ++i) {
                float e[4], p, v;
                ref.at(t0 + i, &p, &v);
                const float u = command(x, q_load(cmd, uo), p, v, e);
                m.step(x, u, a.dt, a.renorm, j, i);
                cmd += 4 * D;
                slot += SD;
                if (i + 1 < t1 - t0) m.template store<false>(slot, L, x);
            }
            if (sg == nseg - 1) pn = Q::pos(x);
        }
        typename Q::State xc;
        float uc;
        if (have_q) {
            xc = xq;
            uc = uq;
        } else {
            if (t1 - 1 > t0) m.template load<false>(a.seg + (size_t)(t1 - 1 - t0) * SD, L, xc);
            else m.template load<true>(ck, L, xc);
            uc = q_load(a.cmds + (size_t)(t1 - 1) * 4 * D, uo);
        }
        for (int t = t1 - 1; t >= t0; --t) {
            have_q = false;
            const bool more = t > t0 || (a.K == 1 && sg > 0);
            if (more) {
                if (t - 1 > t0) m.template load<false>(a.seg + (size_t)(t - 1 - t0) * SD, L, xq);
                else m.template load<true>(t > t0 ? ck : ck - SD, L, xq);
                uq = q_load(a.cmds + (size_t)(t - 1) * 4 * D, uo);
                have_q = true;
            }
            ref.at(t, &rp, &rv);
            if (a.has_obj && j < 3) Q::add_pos(lam, two_seed * (pn - rpn));
            float e[4], ub = 0.f;
            const float u = command(xc, uc, rp, rv, e);
            m.vjp(back, xc, u, a.dt, a.renorm, j, lam, &ub);
            if (a.has_obj) ub = fma_(two_seed * a.w_u, u, ub);
            if (a.g_cmds) q_store(a.g_cmds + (size_t)t * 4 * D, uo, ub);
            if (fb) {
                float v[4];
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    v[k] = fma_(qb<3>(ub), gt[k][3], fma_(qb<2>(ub), gt[k][2], fma_(qb<1>(ub), gt[k][1], qb<0>(ub) * gt[k][0])));
                Q::add_slots(lam, v, j);
                Q::outer13(ub, e, gg);
            }
            pn = Q::pos(xc);
            rpn = rp;
            if (t > t0) {
                xc = xq;
                uc = uq;
            }
        }
    }
    if (a.g_x0) m.store_adj(a.g_x0, L, lam);
    if (a.ggc) {
#pragma unroll
        for (int i = 0; i < 13; ++i) a.ggc[(size_t)(j * 13 + i) * D + d] = gg[i];
    }
}

template <int MODEL, int CTRL>
static hipError_t launch_step_q(const StepArgs& a, hipStream_t s) {
    hipLaunchKernelGGL((k_quad_step<MODEL, CTRL>), dim3((unsigned)((a.D + 15) / 16)), dim3(64), 0, s, a);
    return hipGetLastError();
}
template <int MODEL, int CTRL>
static hipError_t launch_roll_q(const RollArgs& a, bool bwd, hipStream_t s) {
    const dim3 grid((unsigned)((a.D + 15) / 16));
    if (bwd) hipLaunchKernelGGL((k_quad_bwd<MODEL, CTRL>), grid, dim3(64), 0, s, a);
    else hipLaunchKernelGGL((k_quad_fwd<MODEL, CTRL>), grid, dim3(64), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_step_quad(const KernelSel& ks, const StepArgs& a, hipStream_t s) {
    if (ks.models == MS_ID) return launch_step_q<MODEL_ID, CTRL_ROTOR>(a, s);
    if (ks.ctrl == CTRL_PID) return launch_step_q<MODEL_FP, CTRL_PID>(a, s);
    return launch_step_q<MODEL_FP, CTRL_ROTOR>(a, s);
}

hipError_t launch_rollout_quad(const KernelSel& ks, const RollArgs& a, bool bwd, hipStream_t s) {
    if (ks.models == MS_ID) return launch_roll_q<MODEL_ID, CTRL_ROTOR>(a, bwd, s);
    if (ks.ctrl == CTRL_PID) return launch_roll_q<MODEL_FP, CTRL_PID>(a, bwd, s);
    return launch_roll_q<MODEL_FP, CTRL_ROTOR>(a, bwd, s);
}

}  // namespace cfk
