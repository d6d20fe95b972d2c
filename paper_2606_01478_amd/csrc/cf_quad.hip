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
    // of the rows that store writes from lane j: lane 3's slots of 3-vectors may hold
    // anything (0 inf for an infinite thrust command)
    __device__ __forceinline__ bool finite(const State& s, int j) const {
        bool ok = isfinite(s.x.q) && isfinite(s.x.r);
        if (j < 3) ok = ok && isfinite(s.x.p) && isfinite(s.x.v) && isfinite(s.x.w);
        if constexpr (PID) {
            if (j < 2) ok = ok && isfinite(s.c.ia);
            if (j < 3) ok = ok && isfinite(s.c.ir) && isfinite(s.c.wp);
        }
        return ok;
    }
    __device__ __forceinline__ void step(State& s, float u, float h, int renorm, int j) {
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
    __device__ __forceinline__ void held_step(State& s, float u, float h, int renorm, int j, int) {
        step(s, u, h, renorm, j);
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
    __device__ __forceinline__ bool finite(const State& s, int j) const {
        return j < 3 ? isfinite(s.x.p) && isfinite(s.x.a) && isfinite(s.x.v) && isfinite(s.x.w) : isfinite(s.x.f);
    }
    // the start angle's sine and cosine in full, or (held step n of a launch) as
    // id_begin_step does
    __device__ __forceinline__ void step(State& s, float u, float h, int, int j) {
        q_id_base(s.x.a, B);
        q_id_step(s.x, u, P, h, B, j);
    }
    __device__ __forceinline__ void held_step(State& s, float u, float h, int, int j, int n) {
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
    for (int k = 0; k < a.K; ++k) m.held_step(s, u, a.dt, a.renorm, L.j, k);
    m.template store<true>(a.st, L, s);
    if (a.nonfinite && !m.finite(s, L.j)) atomicOr(a.nonfinite + w, 1u);
}

// ---------------------------------------------------------------------------
// rollouts

// this lane's component of the figure-eight rows [p(3), v(3)], moved by the drone's
// time shift in the extended kernels (x runs at w, y at 2 w: see RefLane) and its offset
template <bool EXT>
struct QRef {
    const float* tab;   // lane 3 reads lane 2's column (zeros)
    float off, c, s, w, iw;
    bool on;
    __device__ __forceinline__ QRef(const RollArgs& a, const QLane& L)
        : tab(a.ref_tab + (L.j < 3 ? L.j : 2)), off(0.f), c(1.f), s(0.f), w(0.f), iw(0.f), on(a.has_obj) {
        if (on && a.ref_off && L.j < 3) off = q_load(a.ref_off, L.row(0));
        if constexpr (EXT) {
            if (on && a.ref_shift && L.j < 2) {
                float s1, c1;
                sincosf(a.ref_w * a.ref_shift[L.d], &s1, &c1);
                c = L.j == 0 ? c1 : c1 * c1 - s1 * s1;
                s = L.j == 0 ? s1 : 2.f * s1 * c1;
                w = L.j == 0 ? a.ref_w : 2.f * a.ref_w;
                iw = L.j == 0 ? a.ref_inv_w : 0.5f * a.ref_inv_w;
            }
        }
    }
    __device__ __forceinline__ void at(int t, float* p, float* v) const {
        *p = 0.f;
        *v = 0.f;
        if (on) {
            const float* r = tab + (size_t)t * 6;
            if constexpr (EXT) {
                const float p0 = r[0], v0 = r[3];
                *p = fma_(p0, c, (v0 * iw) * s) + off;
                *v = fma_(v0, c, -(w * p0) * s);
            } else {
                *p = r[0] + off;
                *v = r[3];
            }
        }
    }
};

// the lane's row of the world's gain
__device__ __forceinline__ void q_gain_row(const float* G, int j, float* g) {
#pragma unroll
    for (int i = 0; i < 13; ++i) g[i] = G[j * 13 + i];
}

// The small-MLP policy on a quad: lane j holds hidden units j U .. j U + U - 1 of each
// layer (U = ceil(H / 4) rounded to 2, 4 or 8; units beyond H have zero weights) and
// output j. The weights lie in LDS in the order each product reads them, zero padded,
// rows 4 words apart beyond their length so that the four lanes' rows start in
// different banks; the backward adds the transposes.
template <int U>
struct QMlp {
    static constexpr int H = 4 * U;
    static constexpr int S1 = 20, S2 = H + 4;
    // every offset and stride is a multiple of 4 words
    static constexpr int W1 = 0, W2 = W1 + H * S1, W3 = W2 + H * S2, B1 = W3 + 4 * S2, B2 = B1 + H, B3 = B2 + H,
                         FWD = B3 + 4;
    static constexpr int T1 = FWD, T2 = T1 + 14 * S2, T3 = T2 + H * S2, BWD = T3 + H * 4;

    // stage one policy theta (CF_MLP_PARAMS(h) packing) at m
    template <bool BACK>
    static __device__ void stage(const float* th, int h, float* m) {
        const int n = BACK ? BWD : FWD;
        for (int i = threadIdx.x; i < n; i += blockDim.x) m[i] = 0.f;
        __syncthreads();
        const float *w1 = th, *b1 = w1 + 13 * h, *w2 = b1 + h, *b2 = w2 + h * h, *w3 = b2 + h, *b3 = w3 + 4 * h;
        // walk each matrix by row: the row index advances without a division
        for (int i = threadIdx.x, r = threadIdx.x / 13, c = threadIdx.x % 13; i < 13 * h; i += 64) {
            m[W1 + r * S1 + c] = w1[i];
            if constexpr (BACK) m[T1 + c * S2 + r] = w1[i];
            c += 64 % 13;
            r += 64 / 13;
            if (c >= 13) { c -= 13; ++r; }
        }
        for (int i = threadIdx.x; i < h * h; i += 64) {
            const int r = i / h, c = i - r * h;
            m[W2 + r * S2 + c] = w2[i];
            if constexpr (BACK) m[T2 + c * S2 + r] = w2[i];
        }
        for (int i = threadIdx.x; i < 4 * h; i += 64) {
            const int r = i / h, c = i - r * h;
            m[W3 + r * S2 + c] = w3[i];
            if constexpr (BACK) m[T3 + c * 4 + r] = w3[i];
        }
        for (int i = threadIdx.x; i < h; i += 64) {
            m[B1 + i] = b1[i];
            m[B2 + i] = b2[i];
        }
        if (threadIdx.x < 4) m[B3 + threadIdx.x] = b3[threadIdx.x];
    }
};

// the staged policy is read through LDS pointers (the generic ones of a hidden base
// would make flat loads), four words at a time
typedef __attribute__((address_space(3))) const float lds_float;
typedef float vec4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) const vec4 lds_vec4;

template <int N>
__device__ __forceinline__ void q_row(lds_float* p, float* w) {
#pragma unroll
    for (int i = 0; i < N / 4; ++i) {
        const vec4 v = ((lds_vec4*)p)[i];
        w[4 * i] = v.x; w[4 * i + 1] = v.y; w[4 * i + 2] = v.z; w[4 * i + 3] = v.w;
    }
}
// the policy's base hidden from the optimiser: its weights are read again at every
// step rather than held in registers
__device__ __forceinline__ lds_float* q_again(lds_float* p) {
    asm volatile("" : "+v"(p));
    return p;
}

// sum of w[l U + q] v_l[q] over the four lanes' values v, w a row in LDS
template <int U>
__device__ __forceinline__ float q_dot_all(lds_float* row, const float* v, float s) {
    float w[4 * U];
    q_row<4 * U>(row, w);
#pragma unroll
    for (int q = 0; q < U; ++q) s = fma_(qb<0>(v[q]), w[q], s);
#pragma unroll
    for (int q = 0; q < U; ++q) s = fma_(qb<1>(v[q]), w[U + q], s);
#pragma unroll
    for (int q = 0; q < U; ++q) s = fma_(qb<2>(v[q]), w[2 * U + q], s);
#pragma unroll
    for (int q = 0; q < U; ++q) s = fma_(qb<3>(v[q]), w[3 * U + q], s);
    return s;
}
// g[l U + q] += b v_l[q]
template <int U>
__device__ __forceinline__ void q_outer_all(float b, const float* v, float* g) {
#pragma unroll
    for (int q = 0; q < U; ++q) {
        g[q] = fma_(qb<0>(v[q]), b, g[q]);
        g[U + q] = fma_(qb<1>(v[q]), b, g[U + q]);
        g[2 * U + q] = fma_(qb<2>(v[q]), b, g[2 * U + q]);
        g[3 * U + q] = fma_(qb<3>(v[q]), b, g[3 * U + q]);
    }
}

// (units beyond the policy's H stay zero also where the input is infinite, which their zero
// weights would make NaN)
template <class Q, int U>
__device__ __forceinline__ float q_mlp_forward(lds_float* m, int H, const float* e, int j, float* h1, float* h2) {
    using M = QMlp<U>;
    float b1[U < 4 ? 4 : U], b2[U < 4 ? 4 : U];
#pragma unroll
    for (int r = 0; r < U; ++r) { b1[r] = m[M::B1 + j * U + r]; b2[r] = m[M::B2 + j * U + r]; }
#pragma unroll
    for (int r = 0; r < U; ++r) {
        float w[16];
        q_row<16>(m + M::W1 + (j * U + r) * M::S1, w);
        const float h = tanhf(Q::dot13(w, e) + b1[r]);
        h1[r] = j * U + r < H ? h : 0.f;
    }
#pragma unroll
    for (int r = 0; r < U; ++r) h2[r] = tanhf(q_dot_all<U>(m + M::W2 + (j * U + r) * M::S2, h1, b2[r]));
    return q_dot_all<U>(m + M::W3 + j * M::S2, h2, m[M::B3 + j]);
}

// what the lane sums of its drone's weight gradient over the steps (U <= 4)
template <int U>
struct QMlpGrad {
    float w1[U][13], b1[U], w2[U][4 * U], b2[U], w3[4 * U], b3;
};

// hover command, component j
template <class Q>
__device__ __forceinline__ float q_hover(const Q& m, int j) { return j == 3 ? m.P.f_hover : 0.f; }

template <int MODEL, int CTRL, bool EXT, int U>
__global__ __launch_bounds__(64) void k_quad_fwd(RollArgs a) {
    rollout_priority();
    extern __shared__ __align__(16) float q_lds[];
    if constexpr (U > 0) {
        for (int k = 0; k < a.n_pol; ++k)
            QMlp<U>::template stage<false>(a.gain + (size_t)k * a.mlp_P, a.mlp_H, q_lds + k * QMlp<U>::FWD);
        __syncthreads();
    }
    const uint32_t d = blockIdx.x * 16u + threadIdx.x / 4u;
    if (d >= (uint32_t)a.D) return;
    const QLane L{(int)(threadIdx.x & 3u), d, (uint32_t)a.D};
    const int w = a.drone_world[d];
    const size_t D = (size_t)a.D, SD = (size_t)a.S_h * D;
    using Q = QDrone<MODEL, CTRL>;
    Q m(LaneRec{a.par_aos + (size_t)w * NREC}, L.j, a.dt, a.inv_dtc);
    typename Q::State s;
    m.template load<true>(a.x0, L, s);
    const bool fb = U == 0 && a.has_obj && a.gain;
    float g[13];
    if (fb) q_gain_row(a.gain + (size_t)a.gidx[w] * NG, L.j, g);
    lds_float* pol = U > 0 ? (lds_float*)q_lds + a.gidx[w] * QMlp<U == 0 ? 2 : U>::FWD : nullptr;
    const QRef<EXT> ref(a, L);
    const bool rew = EXT && a.has_obj && a.obj_kind == 1;
    float rp, rv, loss = 0.f, uprev = 0.f, ah = 0.f;
    if constexpr (EXT) uprev = ah = q_hover(m, L.j);
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
        if (fb || U > 0) {
            float e[4], o;
            m.error(s, rp, rv, L.j, e);
            if constexpr (U > 0) {
                float h1[U], h2[U];
                o = q_mlp_forward<Q, U>(q_again(pol), a.mlp_H, e, L.j, h1, h2);
            } else {
                o = Q::dot13(g, e);
            }
            if (EXT && a.squash) u = fma_(a.act_s[L.j], tanhf(o), u);
            else u += o;
        }
        if (rew) {
            const float da = u - ah, dd = u - uprev;
            loss += fma_(a.w_act[L.j] * da, da, a.w_dact[L.j] * dd * dd);
            uprev = u;
            // kept for the backward, which needs the neighbours of every command
            if (a.ubuf) q_store(a.ubuf + (size_t)t * 4 * D, uo, u);
        } else if (a.has_obj) {
            loss = fma_(a.w_u, u * u, loss);
        }
        m.step(s, u, a.dt, a.renorm, L.j);
        if (a.has_obj) {
            const float e = L.j < 3 ? Q::pos(s) - rpn : 0.f;
            if (rew) {
                if constexpr (EXT) {
                    const float d2 = qsum(e * e);
                    const float at[4] = {qb<0>(s.x.a), qb<1>(s.x.a), 0.f, 0.f};
                    const float r = a.w_tilt * tilt_of<MODEL_ID>(at) - expf(-2.f * sqrtf(d2));
                    loss += L.j == 0 ? r : 0.f;
                }
            } else {
                loss = fma_(e, e, loss);
            }
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

// The applied command of the adjoint's recompute and reverse sweeps; e: the policy's
// input, h1, h2: its activations, o: its output.
template <class Q, bool EXT, int U>
__device__ __forceinline__ float q_command(const RollArgs& a, const Q& m, bool fb, const float* g, lds_float* pol,
                                           const typename Q::State& s, int j, float ubar, float rp, float rv, float* e,
                                           float* h1, float* h2, float* o) {
    if (!fb && U == 0) return ubar;
    m.error(s, rp, rv, j, e);
    if constexpr (U > 0) *o = q_mlp_forward<Q, U>(q_again(pol), a.mlp_H, e, j, h1, h2);
    else *o = Q::dot13(g, e);
    if (EXT && a.squash) return fma_(a.act_s[j], tanhf(*o), ubar);
    return ubar + *o;
}

// Recompute steps t0 .. t0 + n of a segment from its checkpoint, storing the states of
// all but the last into the slots after `slot`; the last too where `last`.
template <class Q, bool EXT, int U>
__device__ __forceinline__ void q_recompute(const RollArgs& a, Q& m, const QLane& L, bool fb, const float* g,
                                            lds_float* pol, const QRef<EXT>& ref, const float* ck, int t0, int n,
                                            int n_store, float* slot, typename Q::State& x) {
    const size_t D = (size_t)a.D, SD = (size_t)a.S_h * D;
    constexpr int UM = U == 0 ? 2 : U;
    const uint32_t uo = L.row(0);
    m.template load<true>(ck, L, x);
    const float* cmd = a.cmds + (size_t)t0 * 4 * D;
    float ubar = q_load(cmd, uo), rp, rv;
    ref.at(t0, &rp, &rv);
    for (int i = 0; i < n; ++i) {
        cmd += 4 * D;
        float un = 0.f, rpn = 0.f, rvn = 0.f;
        if (i + 1 < n) {   // the next step's, issued early
            un = q_load(cmd, uo);
            ref.at(t0 + i + 1, &rpn, &rvn);
        }
        float e[4], h1[UM], h2[UM], o;
        const float u = q_command<Q, EXT, U>(a, m, fb, g, pol, x, L.j, ubar, rp, rv, e, h1, h2, &o);
        m.step(x, u, a.dt, a.renorm, L.j);
        slot += SD;
        if (i < n_store) m.template store<false>(slot, L, x);
        ubar = un;
        rp = rpn;
        rv = rvn;
    }
}

// The states between the checkpoints, every segment at once: blockIdx.y is the
// segment. One drone's segments are independent given their checkpoints, and a small
// batch leaves the SIMDs to run them side by side: the adjoint's chain is then the
// reverse sweep alone (1024 identified drones, 500 steps, checkpoint every 50: 836 ->
// 560 us). Slot t of a.seg receives x_t; slot T the final state.
template <int MODEL, int CTRL, bool EXT, int U>
__global__ __launch_bounds__(64) void k_quad_segments(RollArgs a) {
    extern __shared__ __align__(16) float q_lds[];
    if constexpr (U > 0) {
        for (int k = 0; k < a.n_pol; ++k)
            QMlp<U>::template stage<false>(a.gain + (size_t)k * a.mlp_P, a.mlp_H, q_lds + k * QMlp<U>::FWD);
        __syncthreads();
    }
    const uint32_t d = blockIdx.x * 16u + threadIdx.x / 4u;
    if (d >= (uint32_t)a.D || !ckpt_tag_intact(a)) return;
    const QLane L{(int)(threadIdx.x & 3u), d, (uint32_t)a.D};
    const int w = a.drone_world[d];
    const size_t SD = (size_t)a.S_h * a.D;
    using Q = QDrone<MODEL, CTRL>;
    Q m(LaneRec{a.par_aos + (size_t)w * NREC}, L.j, a.dt, a.inv_dtc);
    const bool fb = U == 0 && a.has_obj && a.gain;
    float g[13];
    if (fb) q_gain_row(a.gain + (size_t)a.gidx[w] * NG, L.j, g);
    lds_float* pol = U > 0 ? (lds_float*)q_lds + a.gidx[w] * QMlp<U == 0 ? 2 : U>::FWD : nullptr;
    const QRef<EXT> ref(a, L);
    const int t0 = blockIdx.y * a.K, t1 = min(a.T, t0 + a.K);
    const int n = t1 == a.T ? t1 - t0 : t1 - t0 - 1;
    typename Q::State x;
    q_recompute<Q, EXT, U>(a, m, L, fb, g, pol, ref, a.ckpt_in + (size_t)blockIdx.y * SD, t0, n, n,
                           a.seg + (size_t)t0 * SD, x);
}

template <int MODEL, int CTRL, bool EXT, int U>
__global__ __launch_bounds__(64) void k_quad_bwd(RollArgs a) {
    rollout_priority();
    extern __shared__ __align__(16) float q_lds[];
    if constexpr (U > 0) {
        for (int k = 0; k < a.n_pol; ++k)
            QMlp<U>::template stage<true>(a.gain + (size_t)k * a.mlp_P, a.mlp_H, q_lds + k * QMlp<U>::BWD);
        __syncthreads();
    }
    const uint32_t d = blockIdx.x * 16u + threadIdx.x / 4u;
    if (d >= (uint32_t)a.D) return;
    const QLane L{(int)(threadIdx.x & 3u), d, (uint32_t)a.D};
    if (!ckpt_tag_intact(a)) {
        if (L.j == 0) {
            constexpr bool SUMS = U > 0 && U <= 4;   // (below)
            poison_gradients(a, DroneAt{blockIdx.x * 16u, threadIdx.x & ~3u}, !SUMS);
            if constexpr (SUMS) {
                if (a.mlp_rec)
                    for (int i = 0; i < a.mlp_P; ++i) a.mlp_rec[(size_t)i * a.D + d] = __builtin_nanf("");
            }
        }
        return;
    }
    const int w = a.drone_world[d], j = L.j;
    const size_t D = (size_t)a.D, SD = (size_t)a.S_h * D;
    using Q = QDrone<MODEL, CTRL>;
    constexpr int UM = U == 0 ? 2 : U;
    using M = QMlp<UM>;
    const LaneRec rec{a.par_aos + (size_t)w * NREC};
    Q m(rec, j, a.dt, a.inv_dtc);
    const typename Q::Back back(rec, j);
    const bool fb = U == 0 && a.has_obj && a.gain;
    float g[13], gt[4][4], gg[13];
    int col[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) col[k] = Q::column(k, j);
#pragma unroll
    for (int i = 0; i < 13; ++i) gg[i] = 0.f;
    if (fb) {
        const float* G = a.gain + (size_t)a.gidx[w] * NG;
        q_gain_row(G, j, g);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
#pragma unroll
            for (int i = 0; i < 4; ++i) gt[k][i] = col[k] >= 0 ? G[i * 13 + (col[k] >= 0 ? col[k] : 0)] : 0.f;
        }
    }
    lds_float* pol = U > 0 ? (lds_float*)q_lds + a.gidx[w] * M::BWD : nullptr;
    constexpr bool SUM = U > 0 && U <= 4;   // the weight gradient is summed in registers
    QMlpGrad<SUM ? UM : 1> mg;
    if constexpr (SUM) {
#pragma unroll
        for (int r = 0; r < U; ++r) {
#pragma unroll
            for (int i = 0; i < 13; ++i) mg.w1[r][i] = 0.f;
#pragma unroll
            for (int i = 0; i < 4 * U; ++i) mg.w2[r][i] = 0.f;
            mg.b1[r] = mg.b2[r] = 0.f;
        }
#pragma unroll
        for (int i = 0; i < 4 * U; ++i) mg.w3[i] = 0.f;
        mg.b3 = 0.f;
    }
    const QRef<EXT> ref(a, L);
    const bool rew = EXT && a.has_obj && a.obj_kind == 1;
    const float seed = a.dloss ? a.dloss[d] : 1.f, two_seed = 2.f * seed;
    float ah = 0.f;
    if constexpr (EXT) ah = q_hover(m, j);
    const uint32_t uo = L.row(0);
    typename Q::Adj lam;
    Q::zero(lam);
    const int nseg = (a.T + a.K - 1) / a.K;
    float pn = 0.f, an = 0.f;   // position and (identified) angle of x_{t+1} of the step being reversed
    float rp, rv, rpn, rvn;
    ref.at(a.T, &rpn, &rvn);
    float ub1 = 0.f, ub2 = 0.f;   // reward: the forward's u_t and u_{t+1}
    if (rew) ub1 = q_load(a.ubuf + (size_t)(a.T - 1) * 4 * D, uo);
    typename Q::State xq;   // state and command of the next step to reverse, loaded one step ahead
    float uq = 0.f;
    bool have_q = false;
    for (int sg = nseg - 1; sg >= 0; --sg) {
        const int t0 = sg * a.K;
        const int t1 = min(a.T, t0 + a.K);
        const float* ck = a.ckpt_in + (size_t)sg * SD;
        float* const slots = a.seg_all ? a.seg + (size_t)t0 * SD : a.seg;
        // recompute x_{t0+1} .. x_{t1-1} into segment slots 1..; slot 0 is the
        // checkpoint. The last segment steps once more for the final position.
        const int n_re = (sg == nseg - 1) ? (t1 - t0) : (t1 - t0 - 1);
        if (a.seg_all) {
            if (sg == nseg - 1) {   // done by k_quad_segments
                typename Q::State x;
                m.template load<false>(slots + (size_t)(t1 - t0) * SD, L, x);
                pn = Q::pos(x);
                if constexpr (EXT) an = x.x.a;
            }
        } else if (n_re > 0) {
            typename Q::State x;
            q_recompute<Q, EXT, U>(a, m, L, fb, g, pol, ref, ck, t0, n_re, t1 - t0 - 1, slots, x);
            if (sg == nseg - 1) {
                pn = Q::pos(x);
                if constexpr (EXT) an = x.x.a;
            }
        }
        typename Q::State xc;
        float uc;
        if (have_q) {
            xc = xq;
            uc = uq;
        } else {
            if (t1 - 1 > t0) m.template load<false>(slots + (size_t)(t1 - 1 - t0) * SD, L, xc);
            else m.template load<true>(ck, L, xc);
            uc = q_load(a.cmds + (size_t)(t1 - 1) * 4 * D, uo);
        }
        for (int t = t1 - 1; t >= t0; --t) {
            have_q = false;
            // (across a segment's start too, where the states before it are there)
            const bool more = t > t0 || ((a.K == 1 || a.seg_all) && sg > 0);
            if (more) {
                const bool in_slot = t > t0 ? t - 1 > t0 : a.K > 1;
                if (in_slot) m.template load<false>(slots + (ptrdiff_t)(t - 1 - t0) * (ptrdiff_t)SD, L, xq);
                else m.template load<true>(t > t0 ? ck : ck - SD, L, xq);
                uq = q_load(a.cmds + (size_t)(t - 1) * 4 * D, uo);
                have_q = true;
            }
            ref.at(t, &rp, &rv);
            float up = ah;
            if (rew && t > 0) up = q_load(a.ubuf + (size_t)(t - 1) * 4 * D, uo);
            if (a.has_obj) {
                const float ep = j < 3 ? pn - rpn : 0.f;
                if (rew) {
                    if constexpr (EXT) {
                        const float dn = sqrtf(qsum(ep * ep));
                        const float gp = dn > 0.f ? seed * 2.f * expf(-2.f * dn) / dn : 0.f;
                        Q::add_pos(lam, gp * ep);
                        const float at[4] = {qb<0>(an), qb<1>(an), 0.f, 0.f};
                        float tb[7] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                        tilt_vjp<MODEL_ID>(at, seed * a.w_tilt, tb);
                        lam.x.a += j == 0 ? tb[3] : (j == 1 ? tb[4] : 0.f);
                    }
                } else {
                    Q::add_pos(lam, two_seed * ep);
                }
            }
            float e[4], h1[UM], h2[UM], o = 0.f, ub = 0.f;
            const float u = q_command<Q, EXT, U>(a, m, fb, g, pol, xc, j, uc, rp, rv, e, h1, h2, &o);
            m.vjp(back, xc, u, a.dt, a.renorm, j, lam, &ub);
            if (rew) {
                // (u_t - u_hover)^2, (u_t - u_{t-1})^2 and, from the next step, (u_{t+1} - u_t)^2
                const float un = t + 1 < a.T ? ub2 : u;
                ub = fma_(two_seed, fma_(a.w_act[j], u - ah, a.w_dact[j] * ((u - up) - (un - u))), ub);
                ub2 = ub1;
                ub1 = up;
            } else if (a.has_obj) {
                ub = fma_(two_seed * a.w_u, u, ub);
            }
            if (a.g_cmds) q_store(a.g_cmds + (size_t)t * 4 * D, uo, ub);
            if (fb || U > 0) {
                float ob = ub;   // adjoint of the policy's output
                if (EXT && a.squash) {
                    const float th = tanhf(o);
                    ob = ub * a.act_s[j] * fma_(-th, th, 1.f);
                }
                float v[4];
                if constexpr (U > 0) {
                    lds_float* const wl = q_again(pol);
                    float z2[U], z1[U];
#pragma unroll
                    for (int r = 0; r < U; ++r) {
                        float c[4];
                        q_row<4>(wl + M::T3 + (j * U + r) * 4, c);
                        const float q = fma_(qb<3>(ob), c[3], fma_(qb<2>(ob), c[2], fma_(qb<1>(ob), c[1], qb<0>(ob) * c[0])));
                        z2[r] = q * fma_(-h2[r], h2[r], 1.f);
                    }
#pragma unroll
                    for (int r = 0; r < U; ++r)
                        z1[r] = q_dot_all<U>(wl + M::T2 + (j * U + r) * M::S2, z2, 0.f) * fma_(-h1[r], h1[r], 1.f);
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        v[k] = q_dot_all<U>(wl + M::T1 + (col[k] >= 0 ? col[k] : 13) * M::S2, z1, 0.f);
                    if constexpr (SUM) {
#pragma unroll
                        for (int r = 0; r < U; ++r) {
                            Q::outer13(z1[r], e, mg.w1[r]);
                            q_outer_all<U>(z2[r], h1, mg.w2[r]);
                            mg.b1[r] += z1[r];
                            mg.b2[r] += z2[r];
                        }
                        q_outer_all<U>(ob, h2, mg.w3);
                        mg.b3 += ob;
                    } else if (a.mlp_rec) {
                        const size_t TD = (size_t)a.T * D, base = (size_t)t * D + d;
                        const int H = a.mlp_H;
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            if (col[k] >= 0) a.mlp_rec[col[k] * TD + base] = e[k];
#pragma unroll
                        for (int r = 0; r < U; ++r) {
                            const int n = j * U + r;
                            if (n < H) {
                                a.mlp_rec[(13 + n) * TD + base] = h1[r];
                                a.mlp_rec[(13 + H + n) * TD + base] = h2[r];
                                a.mlp_rec[(13 + 2 * H + n) * TD + base] = z1[r];
                                a.mlp_rec[(13 + 3 * H + n) * TD + base] = z2[r];
                            }
                        }
                        a.mlp_rec[(13 + 4 * H + j) * TD + base] = ob;
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        v[k] = fma_(qb<3>(ob), gt[k][3], fma_(qb<2>(ob), gt[k][2], fma_(qb<1>(ob), gt[k][1], qb<0>(ob) * gt[k][0])));
                    Q::outer13(ob, e, gg);
                }
                Q::add_slots(lam, v, j);
            }
            pn = Q::pos(xc);
            if constexpr (EXT) an = xc.x.a;
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
    if constexpr (SUM) {
        if (a.mlp_rec) {   // [P][D], the policy's packing
            const int H = a.mlp_H;
            const auto put = [&](int i, float v) { a.mlp_rec[(size_t)i * D + d] = v; };
#pragma unroll
            for (int r = 0; r < U; ++r) {
                const int n = j * U + r;
                if (n < H) {
#pragma unroll
                    for (int i = 0; i < 13; ++i) put(n * 13 + i, mg.w1[r][i]);
                    put(13 * H + n, mg.b1[r]);
#pragma unroll
                    for (int k = 0; k < 4 * U; ++k)
                        if (k < H) put(14 * H + n * H + k, mg.w2[r][k]);
                    put(14 * H + H * H + n, mg.b2[r]);
                }
            }
#pragma unroll
            for (int k = 0; k < 4 * U; ++k)
                if (k < H) put(15 * H + H * H + j * H + k, mg.w3[k]);
            put(19 * H + H * H + j, mg.b3);
        }
    }
}

template <int MODEL, int CTRL>
static hipError_t launch_step_q(const StepArgs& a, hipStream_t s) {
    hipLaunchKernelGGL((k_quad_step<MODEL, CTRL>), dim3((unsigned)((a.D + 15) / 16)), dim3(64), 0, s, a);
    return hipGetLastError();
}
template <int MODEL, int CTRL, bool EXT, int U>
static hipError_t launch_roll_q(const RollArgs& a, bool bwd, hipStream_t s) {
    const dim3 grid((unsigned)((a.D + 15) / 16));
    const size_t lds = U == 0 ? 0 : sizeof(float) * a.n_pol * (bwd ? QMlp<U == 0 ? 2 : U>::BWD : QMlp<U == 0 ? 2 : U>::FWD);
    if (bwd) {
        if (a.seg_all) {
            const size_t fwd_lds = U == 0 ? 0 : sizeof(float) * a.n_pol * QMlp<U == 0 ? 2 : U>::FWD;
            const dim3 segments(grid.x, (unsigned)((a.T + a.K - 1) / a.K));
            hipLaunchKernelGGL((k_quad_segments<MODEL, CTRL, EXT, U>), segments, dim3(64), fwd_lds, s, a);
        }
        hipLaunchKernelGGL((k_quad_bwd<MODEL, CTRL, EXT, U>), grid, dim3(64), lds, s, a);
    }
    else hipLaunchKernelGGL((k_quad_fwd<MODEL, CTRL, EXT, U>), grid, dim3(64), lds, s, a);
    return hipGetLastError();
}

hipError_t launch_step_quad(const KernelSel& ks, const StepArgs& a, hipStream_t s) {
    if (ks.models == MS_ID) return launch_step_q<MODEL_ID, CTRL_ROTOR>(a, s);
    if (ks.ctrl == CTRL_PID) return launch_step_q<MODEL_FP, CTRL_PID>(a, s);
    return launch_step_q<MODEL_FP, CTRL_ROTOR>(a, s);
}

static int mlp_units(int H) { return H <= 8 ? 2 : (H <= 16 ? 4 : 8); }

size_t quad_policy_lds(int H, int n_pol) {
    const int u = mlp_units(H);
    const size_t n = u == 2 ? QMlp<2>::BWD : (u == 4 ? QMlp<4>::BWD : QMlp<8>::BWD);
    return n * n_pol * sizeof(float);
}
bool quad_sums_policy(int H) { return mlp_units(H) <= 4; }

hipError_t launch_rollout_quad(const KernelSel& ks, const RollArgs& a, bool bwd, hipStream_t s) {
    if (ks.models == MS_ID) {
        if (a.mlp_H > 0) {
            switch (mlp_units(a.mlp_H)) {
                case 2: return launch_roll_q<MODEL_ID, CTRL_ROTOR, true, 2>(a, bwd, s);
                case 4: return launch_roll_q<MODEL_ID, CTRL_ROTOR, true, 4>(a, bwd, s);
                default: return launch_roll_q<MODEL_ID, CTRL_ROTOR, true, 8>(a, bwd, s);
            }
        }
        if (a.has_obj && (a.obj_kind == 1 || a.ref_shift || a.squash))
            return launch_roll_q<MODEL_ID, CTRL_ROTOR, true, 0>(a, bwd, s);
        return launch_roll_q<MODEL_ID, CTRL_ROTOR, false, 0>(a, bwd, s);
    }
    if (ks.ctrl == CTRL_PID) return launch_roll_q<MODEL_FP, CTRL_PID, false, 0>(a, bwd, s);
    return launch_roll_q<MODEL_FP, CTRL_ROTOR, false, 0>(a, bwd, s);
}

}  // namespace cfk
