// Sampled-rollout controller (the iCEM / MPPI hybrid of the paper's obstacle
// avoidance showcase): every lane is one sample of one controller. It draws its
// temporally correlated command noise from a counter-based generator on the
// fly (nothing is stored), rolls the sample through the model and writes only
// its cost. A workgroup per controller then selects and sorts the elites by (cost,
// sample index); workgroups of 64 elites regenerate their commands from the counters
// and sum them with their exponential weights; a last kernel adds those sums up in a
// fixed order. (One workgroup per controller for all of it took 131 us of a control
// step with 5 x 100 000 samples: 1000 elites on 16 waves, 25 steps one after the other.)
#include "cf_device.hpp"
#include "cf_dispatch.hpp"
#include "cf_internal.hpp"

namespace cfk {

constexpr int MPPI_PARTS = 2;

// ---- Philox4x64-10 (Salmon, Moraes, Dror, Shaw, SC'11) ------------------------
constexpr uint64_t PH_M0 = 0xD2E7470EE14C6C93ull, PH_M1 = 0xCA5A826395121157ull;
constexpr uint64_t PH_W0 = 0x9E3779B97F4A7C15ull, PH_W1 = 0xBB67AE8584CAA73Bull;

__device__ __forceinline__ void philox4x64(uint64_t x[4], uint64_t k0, uint64_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r) {
            k0 += PH_W0;
            k1 += PH_W1;
        }
        const unsigned __int128 p0 = (unsigned __int128)PH_M0 * x[0], p1 = (unsigned __int128)PH_M1 * x[2];
        const uint64_t hi0 = (uint64_t)(p0 >> 64), lo0 = (uint64_t)p0, hi1 = (uint64_t)(p1 >> 64), lo1 = (uint64_t)p1;
        const uint64_t y0 = hi1 ^ x[1] ^ k0, y2 = hi0 ^ x[3] ^ k1;
        x[0] = y0;
        x[1] = lo1;
        x[2] = y2;
        x[3] = lo0;
    }
}

// open-interval uniform from the top 23 bits, exact in binary32
__device__ __forceinline__ float unit_open(uint32_t u) { return ((float)(u >> 9) + 0.5f) * 0x1p-23f; }

// eight standard normals of block b of sample (k, c) at iteration `iter`:
// each 64-bit word gives one Box-Muller pair from its (low, high) halves;
// the hardware sine and cosine take their argument in revolutions, so
// sin(2 pi u2) is one instruction with no range reduction (u2 in (0, 1))
__device__ __forceinline__ void normals8(uint64_t b, uint64_t k, uint64_t c, const MppiArgs& a, float z[8]) {
    uint64_t x[4] = {b, k, c, a.iter};
    philox4x64(x, a.seed, 0ull);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const float u1 = unit_open((uint32_t)x[w]);
        const float u2 = unit_open((uint32_t)(x[w] >> 32));
        const float r = sqrt_hw(-2.f * logf(u1));
        z[2 * w] = r * __builtin_amdgcn_cosf(u2);
        z[2 * w + 1] = r * __builtin_amdgcn_sinf(u2);
    }
}

// Sequential generator of one sample's correlated noise eps_t (t = 0, 1, ...):
// first-order autoregressive filter with unit stationary variance; sample 0
// is the noise-free mean.
struct NoiseSeq {
    uint64_t k, c;
    float eps[4], z[8];
    float scale;  // 0 for sample 0
    __device__ __forceinline__ void init(uint64_t k_, uint64_t c_) {
        k = k_;
        c = c_;
        scale = k_ == 0 ? 0.f : 1.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) eps[i] = 0.f;
    }
    // advance to step t (called with t = 0, 1, 2, ... in order); even steps draw
    // a new block, odd steps use its second half (selected, not indexed, so z
    // stays in registers)
    __device__ __forceinline__ void next(int t, const MppiArgs& a) {
        if ((t & 1) == 0) normals8((uint64_t)(t >> 1), k, c, a, z);
        const bool odd = (t & 1) != 0;
        float zi[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) zi[i] = odd ? z[4 + i] : z[i];
        if (t == 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) eps[i] = zi[i];
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) eps[i] = a.beta * eps[i] + a.beta_c * zi[i];
        }
    }
    // sampled command at step t: clip(mean + sigma eps)
    __device__ __forceinline__ void command(int t, const MppiArgs& a, float u[4]) const {
        const int ts = min(t + a.shift, a.H - 1);
        const float* m = a.mean + ((size_t)c * a.H + ts) * 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) u[i] = fminf(fmaxf(m[i] + a.sigma[i] * (scale * eps[i]), a.u_lo[i]), a.u_hi[i]);
    }
};

// ---- rollout + cost: one lane per sample ---------------------------------------
// MR: variant for an onboard controller slower than the physics
// ONE: a single physics step per command (no inner loop, whose exit copies the state)
template <int MODEL, int CTRL, int INTEG, bool AERO, bool MR, bool ONE>
__global__ __launch_bounds__(256) void k_mppi_rollout(MppiArgs a) {
    const int c = blockIdx.y;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= a.N) return;
    const VecRec rec(a.par);
    constexpr int S = MODEL == MODEL_ID ? S_ID : (CTRL == CTRL_PID ? S_PID : S_FP);
    constexpr int V = MODEL == MODEL_ID ? 6 : 7;  // first velocity row
    float x[S], comp[S];
#pragma unroll
    for (int i = 0; i < S; ++i) {
        x[i] = a.x_now[i];
        comp[i] = 0.f;
    }
    FpParams P;
    PidParams Cp;
    IdParams Pi;
    if constexpr (MODEL == MODEL_FP) {
        P = load_fp<AERO>(rec);
        if constexpr (CTRL != CTRL_ROTOR) Cp = load_pid(rec, CTRL == CTRL_POSITION);
        rotors_to_dev(x, P);
    } else {
        Pi = load_id<AERO>(rec);
    }
    NoiseSeq ns;
    ns.init((uint64_t)k, (uint64_t)c);
    float J = 0.f;
    float rc[4] = {0.f, 0.f, 0.f, 0.f};   // held rotor commands
    int phase = 0;                        // physics step within the controller period
    for (int t = 0; t < a.H; ++t) {
        ns.next(t, a);
        float u[4];
        ns.command(t, a, u);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float du = u[i] - a.u_ref[i];
            J += a.r_u[i] * du * du;
        }
        const int sub = ONE ? 1 : a.sub;
        for (int s = 0; s < sub; ++s) {
            if constexpr (MODEL == MODEL_FP) {
                fp_step<CTRL, INTEG>(x, comp, u, P, Cp, a.dt, a.dtc, a.inv_dtc, a.renorm, rc, MR ? phase == 0 : true);
                if constexpr (MR) {
                    if (++phase == a.ctrl_every) phase = 0;
                }
            } else {
                id_step<INTEG>(x, comp, u, Pi, a.dt);
            }
        }
        const float ex = x[0] - a.goal[0], ey = x[1] - a.goal[1], ez = x[2] - a.goal[2];
        J += a.q_p * (ex * ex + ey * ey + ez * ez) +
             a.q_v * (x[V] * x[V] + x[V + 1] * x[V + 1] + x[V + 2] * x[V + 2]);
#pragma unroll 4
        for (int o = 0; o < a.n_obs; ++o) {
            const float dx = x[0] - a.obs[o][0], dy = x[1] - a.obs[o][1], dz = x[2] - a.obs[o][2];
            const float pen = fmaxf(1.f - (dx * dx + dy * dy + dz * dz) * a.obs[o][3], 0.f);
            J += a.w_obs * pen * pen;
        }
    }
    a.cost[(size_t)c * a.N + k] = isfinite(J) ? J : __builtin_inff();
}

#if CF_PART == 0
// correlated noise only (eps, before sigma and clipping), [C][N][H][4]
__global__ __launch_bounds__(256) void k_mppi_noise(MppiArgs a) {
    const int c = blockIdx.y;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= a.N) return;
    NoiseSeq ns;
    ns.init((uint64_t)k, (uint64_t)c);
    float* out = a.eps_out + ((size_t)c * a.N + k) * a.H * 4;
    for (int t = 0; t < a.H; ++t) {
        ns.next(t, a);
#pragma unroll
        for (int i = 0; i < 4; ++i) out[t * 4 + i] = ns.scale * ns.eps[i];
    }
}

// ---- elite selection and weighted mean: one workgroup per controller ------------
// order-preserving map of a binary32 to an unsigned key
__device__ __forceinline__ uint32_t ordered_bits(float f) {
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float from_ordered(uint32_t o) {
    return __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// the value of lane ^ S
template <int S>
__device__ __forceinline__ uint32_t xor_lane32(uint32_t v) {
    const int i = (int)v;
    if constexpr (S == 1) return (uint32_t)__builtin_amdgcn_mov_dpp(i, 0xB1, 0xf, 0xf, true);         // quad 1,0,3,2
    else if constexpr (S == 2) return (uint32_t)__builtin_amdgcn_mov_dpp(i, 0x4E, 0xf, 0xf, true);    // quad 2,3,0,1
    else if constexpr (S == 4)   // i ^ 7 (mirror of 8), then ^ 3 (quad reversed)
        return (uint32_t)__builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp(i, 0x141, 0xf, 0xf, true), 0x1B, 0xf, 0xf, true);
    else if constexpr (S == 8) return (uint32_t)__builtin_amdgcn_mov_dpp(i, 0x128, 0xf, 0xf, true);   // rotate 16 by 8
    else return (uint32_t)__shfl_xor(i, S, 64);
}
template <int S>
__device__ __forceinline__ uint64_t xor_lane(uint64_t v) {
    return ((uint64_t)xor_lane32<S>((uint32_t)(v >> 32)) << 32) | xor_lane32<S>((uint32_t)v);
}

__global__ __launch_bounds__(MPPI_SELECT_THREADS) void k_mppi_select(MppiArgs a) {
    constexpr int BS = MPPI_SELECT_THREADS;
    __shared__ unsigned hist[256], bins[2 * MPPI_SELECT_THREADS];
    __shared__ int wave_sums[MPPI_SELECT_THREADS / 64];
    __shared__ uint64_t keys[MPPI_MAX_ELITE];
    __shared__ uint64_t s_prefix, s_mask;
    __shared__ int s_need, s_eq, s_count, s_in;
    __shared__ uint32_t s_last;
    const int c = blockIdx.x;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const float* J = a.cost + (size_t)c * a.N;
    // visit every sample's key; loads are issued UNR at a time so their
    // latencies overlap (one workgroup per controller has few waves to hide them)
    constexpr int UNR = 24;
    auto for_each_key = [&](auto&& fn) {
        for (int64_t k0 = tid; k0 < a.N; k0 += BS * UNR) {
            float v[UNR];
#pragma unroll
            for (int j = 0; j < UNR; ++j) {
                const int64_t k = k0 + j * BS;
                v[j] = k < a.N ? J[k] : 0.f;
            }
#pragma unroll
            for (int j = 0; j < UNR; ++j) {
                const int64_t k = k0 + j * BS;
                if (k < a.N) fn(((uint64_t)ordered_bits(v[j]) << 32) | (uint32_t)k);
            }
        }
    };

    // Ascending bitonic sort of keys[0, P2), 128 <= P2 <= MPPI_MAX_ELITE a power of two (all
    // threads). A wave takes 128 consecutive keys into registers, two per lane, for
    // every stage with a stride of at most 64 (56 of the 66 of 2048 keys): those through
    // LDS move 32 KiB a stage and took 0.3 us each.
    auto in_wave = [&](int P2, int first, int last) __attribute__((always_inline)) {   // sizes first .. last, strides from min(size / 2, 64)
        for (int g = wave; g < P2 / 128; g += BS / 64) {
            uint64_t* const q = keys + 128 * g;
            uint64_t x = q[lane], y = q[64 + lane];
            for (int size = first; size <= last; size <<= 1) {
                if (size >= 128 && (x > y) == ((128 * g & size) == 0)) {
                    const uint64_t s = x;
                    x = y;
                    y = s;
                }
                const bool up_x = ((128 * g + lane) & size) == 0, up_y = ((128 * g + 64 + lane) & size) == 0;
                const auto stage = [&](uint64_t px, uint64_t py, int stride) {
                    const bool low = (lane & stride) == 0;
                    x = (px < x) == (low == up_x) ? px : x;
                    y = (py < y) == (low == up_y) ? py : y;
                };
                if (size > 32) stage(xor_lane<32>(x), xor_lane<32>(y), 32);
                if (size > 16) stage(xor_lane<16>(x), xor_lane<16>(y), 16);
                if (size > 8) stage(xor_lane<8>(x), xor_lane<8>(y), 8);
                if (size > 4) stage(xor_lane<4>(x), xor_lane<4>(y), 4);
                if (size > 2) stage(xor_lane<2>(x), xor_lane<2>(y), 2);
                stage(xor_lane<1>(x), xor_lane<1>(y), 1);
            }
            q[lane] = x;
            q[64 + lane] = y;
        }
        __syncthreads();
    };
    auto bitonic = [&](int P2) __attribute__((always_inline)) {
        in_wave(P2, 2, 128);
        for (int size = 256; size <= P2; size <<= 1) {
            for (int stride = size >> 1; stride > 64; stride >>= 1) {
                for (int i = tid; i < P2 / 2; i += BS) {
                    const int lo = 2 * i - (i & (stride - 1));
                    const int hi = lo + stride;
                    const bool up = (lo & size) == 0;
                    const uint64_t x = keys[lo], y = keys[hi];
                    if ((x > y) == up) {
                        keys[lo] = y;
                        keys[hi] = x;
                    }
                }
                __syncthreads();
            }
            in_wave(P2, size, size);
        }
    };

    // Common case: a threshold just above the n_e-th smallest cost, from a sample of the
    // costs (its r-th smallest to 22 bits, by two histograms); one pass collects every
    // key at or below it and the candidates are sorted. Costs that agree in those bits all
    // become candidates: where the sample says that they would fill three quarters of the
    // list or more, the threshold is taken to the last bit and, among equal costs, to the
    // sample's index (a control step with 5 x 100 000 samples whose costs lie within 7e-5 of
    // each other: 543 -> 293 us, all equal: 888 -> 290; farther apart 289 either way). The
    // radix select below is the fallback when the candidates are too few or too many.
    bool selected = false;
    if (2 * a.n_e <= MPPI_MAX_ELITE) {
        constexpr int SAMPLE = 2 * BS;
        const int ns = (int)(a.N < SAMPLE ? a.N : SAMPLE);
        uint32_t o[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int i = tid + j * BS;
            o[j] = i < ns ? ordered_bits(J[ns == SAMPLE ? (int64_t)i * a.N / SAMPLE : i]) : 0xffffffffu;
        }
        int r = (ns == a.N) ? a.n_e - 1
                            : (int)ceilf((float)ns * (float)a.n_e / (float)a.N * 1.25f) + 8;
        r = r < ns - 1 ? r : ns - 1;
        const int rank = r;
        uint32_t prefix = 0;   // the bits found: 11, 11 and, where needed, 10
        bool narrow = false;
        for (int pass = 0; pass < (narrow ? 3 : 2); ++pass) {
            const int sh = pass == 0 ? 21 : (pass == 1 ? 10 : 0), known = sh + (pass == 2 ? 10 : 11);
            const uint32_t mask = pass == 2 ? 1023u : 2047u;
            bins[2 * tid] = 0;
            bins[2 * tid + 1] = 0;
            if (tid == 0) s_count = 0;
            __syncthreads();
#pragma unroll
            for (int j = 0; j < 2; ++j)
                if (tid + j * BS < ns && (pass == 0 || o[j] >> known == prefix)) atomicAdd(&bins[(o[j] >> sh) & mask], 1u);
            __syncthreads();
            const int b0 = (int)bins[2 * tid], b1 = (int)bins[2 * tid + 1];
            int incl = b0 + b1;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int u = __shfl_up(incl, off, 64);
                if (lane >= off) incl += u;
            }
            if (lane == 63) wave_sums[wave] = incl;
            __syncthreads();
            int before = incl - b0 - b1;
            for (int w = 0; w < wave; ++w) before += wave_sums[w];
            // the bin that holds rank r (one thread's)
            if (r >= before && r < before + b0 + b1) {
                const int second = r >= before + b0 ? 1 : 0;
                s_need = r - before - (second ? b0 : 0);
                s_eq = 2 * tid + second;
                s_in = second ? b1 : b0;
            }
            __syncthreads();
            prefix = (prefix << (pass == 2 ? 10 : 11)) | (uint32_t)s_eq;
            r = s_need;
            // samples at or below the bin, scaled to all
            if (pass == 1) narrow = (int64_t)(rank - r + s_in) * a.N > (int64_t)ns * (MPPI_MAX_ELITE * 3 / 4);
            __syncthreads();
        }
        uint32_t last = 0xffffffffu;   // largest index taken of the threshold's cost
        if (narrow) {
            // the r-th of the samples with that cost, in index order: first tid, then tid + BS
            const bool eq0 = tid < ns && o[0] == prefix, eq1 = tid + BS < ns && o[1] == prefix;
            const uint64_t m0 = __ballot(eq0), m1 = __ballot(eq1), below = (1ull << lane) - 1ull;
            if (lane == 0) {
                bins[wave] = (unsigned)__popcll(m0);
                bins[BS / 64 + wave] = (unsigned)__popcll(m1);
            }
            __syncthreads();
            int at0 = __popcll(m0 & below), at1 = __popcll(m1 & below);
            for (int w = 0; w < BS / 64; ++w) {
                at0 += w < wave ? (int)bins[w] : 0;
                at1 += (int)bins[w] + (w < wave ? (int)bins[BS / 64 + w] : 0);
            }
            const auto index = [&](int i) { return (uint32_t)(ns == SAMPLE ? (int64_t)i * a.N / SAMPLE : i); };
            if (eq0 && at0 == r) s_last = index(tid);
            if (eq1 && at1 == r) s_last = index(tid + BS);
            __syncthreads();
            last = s_last;
        } else {
            prefix = (prefix << 10) | 1023u;
        }
        // a wave takes the matches of UNR keys per lane to the list with one atomic
        const uint32_t tau = prefix;
        for (int64_t k0 = tid; k0 - tid < a.N; k0 += (int64_t)BS * UNR) {
            float v[UNR];
            uint32_t hit = 0;
#pragma unroll
            for (int j = 0; j < UNR; ++j) {
                const int64_t k = k0 + j * BS;
                v[j] = k < a.N ? J[k] : 0.f;
            }
#pragma unroll
            for (int j = 0; j < UNR; ++j) {
                const int64_t k = k0 + j * BS;
                if (k < a.N && ordered_bits(v[j]) <= tau) hit |= 1u << j;
            }
            if (narrow) {
#pragma unroll
                for (int j = 0; j < UNR; ++j)
                    if (ordered_bits(v[j]) == tau && (uint32_t)(k0 + j * BS) > last) hit &= ~(1u << j);
            }
            const int mine = __popc(hit);
            int incl = mine;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int u = __shfl_up(incl, off, 64);
                if (lane >= off) incl += u;
            }
            const int all = __shfl(incl, 63, 64);
            if (all) {
                int base = 0;
                if (lane == 0) base = atomicAdd(&s_count, all);
                int pos = __shfl(base, 0, 64) + incl - mine;
#pragma unroll
                for (int j = 0; j < UNR; ++j) {
                    if (hit >> j & 1u) {
                        if (pos < MPPI_MAX_ELITE)
                            keys[pos] = ((uint64_t)ordered_bits(v[j]) << 32) | (uint32_t)(k0 + j * BS);
                        ++pos;
                    }
                }
            }
        }
        __syncthreads();
        const int cnt = s_count;
        if (cnt >= a.n_e && cnt <= MPPI_MAX_ELITE) {
            int P2 = 128;
            while (P2 < cnt) P2 <<= 1;
            for (int i = cnt + tid; i < P2; i += BS) keys[i] = ~0ull;
            __syncthreads();
            bitonic(P2);
            selected = true;
        }
        __syncthreads();
    }
    if (!selected) {
        // radix select of the n_e-th smallest key, 8 bits per pass from the top;
        // stops once every key left in the chosen bucket is taken
        if (tid == 0) {
            s_prefix = 0;
            s_mask = 0;
            s_need = a.n_e;
        }
        __syncthreads();
        for (int pass = 0; pass < 8; ++pass) {
            const int sh = 56 - 8 * pass;
            if (tid < 256) hist[tid] = 0;
            __syncthreads();
            const uint64_t prefix = s_prefix, mask = s_mask;
            for_each_key([&](uint64_t key) {
                if ((key & mask) == prefix) atomicAdd(&hist[(key >> sh) & 255u], 1u);
            });
            __syncthreads();
            if (wave == 0) {
                const int need = s_need;
                const unsigned h0 = hist[4 * lane], h1 = hist[4 * lane + 1], h2 = hist[4 * lane + 2],
                               h3 = hist[4 * lane + 3];
                const unsigned tot = h0 + h1 + h2 + h3;
                unsigned incl = tot;
    #pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const unsigned v = __shfl_up(incl, off, 64);
                    if (lane >= off) incl += v;
                }
                const unsigned excl = incl - tot;
                const bool here = excl < (unsigned)need && (unsigned)need <= incl;
                if (here) {
                    unsigned cum = excl;
                    const unsigned hh[4] = {h0, h1, h2, h3};
                    int dig = 0;
    #pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (cum + hh[j] >= (unsigned)need) {
                            dig = 4 * lane + j;
                            s_need = need - (int)cum;
                            s_eq = (int)hh[j];
                            break;
                        }
                        cum += hh[j];
                    }
                    s_prefix = prefix | ((uint64_t)dig << sh);
                    s_mask = mask | (255ull << sh);
                }
            }
            __syncthreads();
            if (s_eq == s_need) break;
        }
        // collect the n_e keys with (key & mask) <= prefix, then sort them
        const uint64_t prefix = s_prefix, mask = s_mask;
        int P2 = 128;
        while (P2 < a.n_e) P2 <<= 1;
        for (int i = tid; i < P2; i += BS) keys[i] = ~0ull;
        if (tid == 0) s_count = 0;
        __syncthreads();
        for_each_key([&](uint64_t key) {
            if ((key & mask) <= prefix) {
                const int pos = atomicAdd(&s_count, 1);
                if (pos < a.n_e) keys[pos] = key;
            }
        });
        __syncthreads();
        bitonic(P2);
    }
    const float jmin = from_ordered((uint32_t)(keys[0] >> 32));
    for (int i = tid; i < a.n_e; i += BS) {
        a.elite_idx[(size_t)c * a.n_e + i] = (int32_t)(uint32_t)keys[i];
        a.elite_cost[(size_t)c * a.n_e + i] = from_ordered((uint32_t)(keys[i] >> 32));
    }
    if (tid == 0) a.cost_min[c] = jmin;
}

// Weighted sums of 64 elites' commands, one elite per lane: part[c][b][t * 4 + j] =
// sum_i w_i u_i(t, j), w_i = exp(-(J_i - J_min) / lambda), and the sum of the weights
// last. The normals of all steps are independent, so the waves draw them side by side
// into LDS, MEAN_STEPS steps at a time; one wave per component then runs the filter
// along the steps, and one thread per row sums the 64 elites (rows 65 words apart:
// the threads' banks differ).
constexpr int MEAN_STEPS = 32, MEAN_THREADS = 512;
__global__ __launch_bounds__(MEAN_THREADS) void k_mppi_mean(MppiArgs a) {
    __shared__ float z[MEAN_STEPS * 4][65];
    const int b = blockIdx.x, nb = gridDim.x, c = blockIdx.y;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = b * 64 + lane;
    const bool on = i < a.n_e;
    const uint64_t k = on ? (uint64_t)(uint32_t)a.elite_idx[(size_t)c * a.n_e + i] : 0;
    float w = 0.f;
    if (on) w = expf(-(a.elite_cost[(size_t)c * a.n_e + i] - a.cost_min[c]) * a.inv_lambda);
    const float scale = k == 0 ? 0.f : 1.f;
    const int rows = a.H * 4 + 1;
    float* part = a.mean_part + ((size_t)c * nb + b) * rows;
    float eps = 0.f;   // waves 0..3: component `wave` of this lane's elite
    for (int t0 = 0; t0 < a.H; t0 += MEAN_STEPS) {
        const int n = min(MEAN_STEPS, a.H - t0);
        for (int q = wave; 2 * q < n; q += MEAN_THREADS / 64) {
            float v[8];
            normals8((uint64_t)(t0 / 2 + q), k, (uint64_t)c, a, v);
#pragma unroll
            for (int j = 0; j < 8; ++j) z[8 * q + j][lane] = v[j];
        }
        __syncthreads();
        if (wave < 4) {
            for (int t = 0; t < n; ++t) {
                const float xi = z[4 * t + wave][lane];
                eps = t0 + t == 0 ? xi : a.beta * eps + a.beta_c * xi;
                const int ts = min(t0 + t + a.shift, a.H - 1);
                const float m = a.mean[((size_t)c * a.H + ts) * 4 + wave];
                const float u = fminf(fmaxf(m + a.sigma[wave] * (scale * eps), a.u_lo[wave]), a.u_hi[wave]);
                z[4 * t + wave][lane] = on ? w * u : 0.f;
            }
        }
        __syncthreads();
        for (int r = threadIdx.x; r < 4 * n; r += MEAN_THREADS) {
            float s = 0.f;
#pragma unroll 16
            for (int l = 0; l < 64; ++l) s += z[r][l];
            part[t0 * 4 + r] = s;
        }
        __syncthreads();
    }
    if (wave == 0) {
        w = wave_sum(w);
        if (lane == 0) part[rows - 1] = w;
    }
}

// the new plans, and the command of the controller with the lowest elite cost (ties to
// the lower index)
__global__ __launch_bounds__(256) void k_mppi_finish(MppiArgs a, int nb) {
    __shared__ int beaten;
    const int c = blockIdx.x, rows = a.H * 4 + 1;
    const float* part = a.mean_part + (size_t)c * nb * rows;
    if (threadIdx.x == 0) beaten = 0;
    __syncthreads();
    const float mine = a.cost_min[c];
    bool lost = false;
    for (int i = threadIdx.x; i < a.C; i += 256) {
        const float o = a.cost_min[i];
        lost = lost || o < mine || (o == mine && i < c);
    }
    if (lost) beaten = 1;
    float ws = 0.f;
#pragma unroll 8
    for (int b = 0; b < nb; ++b) ws += part[(size_t)b * rows + rows - 1];
    const float inv = 1.f / ws;
    __syncthreads();
    const bool best = beaten == 0;
    for (int r = threadIdx.x; r < rows - 1; r += 256) {
        float s = 0.f;
#pragma unroll 8
        for (int b = 0; b < nb; ++b) s += part[(size_t)b * rows + r];
        const float m = s * inv;
        a.mean_out[(size_t)c * a.H * 4 + r] = m;
        if (best && r < 4 && a.u_apply) a.u_apply[r] = m;
    }
    if (best && threadIdx.x == 0 && a.best) a.best[0] = c;
}

#endif  // CF_PART == 0

template <int MODEL, int CTRL, int INTEG, bool AERO>
static hipError_t launch_roll(const KernelSel&, const MppiArgs& a, hipStream_t s) {
    const dim3 grid((unsigned)((a.N + 255) / 256), (unsigned)a.C);
    if constexpr (MODEL == MODEL_FP && CTRL != CTRL_ROTOR) {
        if (a.ctrl_every > 1) {
            hipLaunchKernelGGL((k_mppi_rollout<MODEL, CTRL, INTEG, AERO, true, false>), grid, dim3(256), 0, s, a);
            return hipGetLastError();
        }
    }
    if (a.sub == 1)
        hipLaunchKernelGGL((k_mppi_rollout<MODEL, CTRL, INTEG, AERO, false, true>), grid, dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL((k_mppi_rollout<MODEL, CTRL, INTEG, AERO, false, false>), grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

template <int P>
hipError_t launch_mppi_part(const KernelSel& ks, const MppiArgs& a, hipStream_t s);

template <>
hipError_t launch_mppi_part<CF_PART>(const KernelSel& ks, const MppiArgs& a, hipStream_t s) {
    return dispatch<MPPI_PARTS>(ks, [&](auto m, auto c, auto i, auto e) {
        if constexpr (m() == MS_BOTH) return hipErrorInvalidValue;   // one world
        else return launch_roll<m() == MS_FP ? MODEL_FP : MODEL_ID, c(), i(), e() != 0>(ks, a, s);
    });
}

#if CF_PART == 0
template <> hipError_t launch_mppi_part<1>(const KernelSel&, const MppiArgs&, hipStream_t);

hipError_t launch_mppi_rollout(const KernelSel& ks, const MppiArgs& a, hipStream_t s) {
    return in_part<MPPI_PARTS>(ks, [&](auto p) { return launch_mppi_part<p()>(ks, a, s); });
}

hipError_t launch_mppi_noise(const MppiArgs& a, hipStream_t s) {
    const dim3 grid((unsigned)((a.N + 255) / 256), (unsigned)a.C);
    hipLaunchKernelGGL(k_mppi_noise, grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_mppi_select(const MppiArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(k_mppi_select, dim3((unsigned)a.C), dim3(MPPI_SELECT_THREADS), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int nb = mppi_mean_blocks(a.n_e);
    hipLaunchKernelGGL(k_mppi_mean, dim3((unsigned)nb, (unsigned)a.C), dim3(MEAN_THREADS), 0, s, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_mppi_finish, dim3((unsigned)a.C), dim3(256), 0, s, a, nb);
    return hipGetLastError();
}
#endif

}  // namespace cfk
