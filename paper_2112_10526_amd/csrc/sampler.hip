// Metropolis-Hastings sampling with a persistent per-chain wave (paper,
// Monte Carlo samplers section; local and exchange rules).
//
// A wave64 owns one chain, or two (32 lanes each) when the chains pair up.
// Lane l of a chain's L lanes keeps tanh(theta_j) for hidden units j = l + L q
// in registers for the whole launch, and the chain's configuration sits in
// LDS.  Random draws are made L at a time: lane l evaluates the Philox block
// of proposal p0 + l and leaves its site/bond and uniform in LDS.
//
// Single flip of site i (local rule):
//   psi(s')/psi(s) = K_i(s_i) prod_j f_j,  f_j = 1 - s_i t_j T_ij,
//   T_ij = tanh(2 W_ji),  K_i(s) = exp(-2 a_i s) prod_j cosh(2 W_ji),
// from cosh(theta - x)/cosh(theta) = cosh x (1 - tanh(theta) tanh x) with
// x = 2 s_i W_ji; after acceptance t_j <- (t_j - s_i T_ij) / f_j (tanh
// subtraction formula; f_j is the denominator already computed).
// Exchange of an antiparallel pair (a, b) (s_b = -s_a):
//   psi(s'')/psi(s) = K_a(s_a) K_b(s_b) prod_j g_j,
//   g_j = 1 - T_ja T_jb - s_a t_j (T_ja - T_jb),
//   t_j <- (t_j (1 - T_ja T_jb) - s_a (T_ja - T_jb)) / g_j.
// FP64: the product is formed directly and u < r^2 is tested.  FP32: each
// lane's partial product goes through ln, the wave sums the logs, and
// ln u < 2 ln r is tested.
#include "kernels.h"

namespace nqs {

// 1/x: hardware reciprocal refined by two Newton steps (FP64), or the FP32
// hardware reciprocal.  The factors are in (0, 2), away from zero.
__device__ __forceinline__ double recip(double x) {
    double y = __builtin_amdgcn_rcp(x);
    y = fma(fma(-x, y, 1.0), y, y);
    y = fma(fma(-x, y, 1.0), y, y);
    return y;
}
__device__ __forceinline__ float recip(float x) { return __builtin_amdgcn_rcpf(x); }

// The reciprocals of f[0 .. Q-1], in FP64 from their running products, of which
// pre[q] = f[0] .. f[q] are at hand: one reciprocal for eight factors, two or three
// products and one Newton step each, where the instruction takes four times as long as
// a product and needs two Newton steps (4 sweeps of 4,096 chains, 10x10, 200 hidden
// units, 315 -> 289 us).  The running products alone would leave up to 8 units of 2^-53;
// the step gives the value found one by one (the same bits in 3 million factors).
// Eight, because a factor is a multiple of 2^-106 (1 less a product of two 53-bit
// numbers) and not 0 in an accepted move: their product can be inverted, which that of
// 32 need not be.  FP32: one by one.
constexpr int RC_G = 8;
template <int Q>
__device__ __forceinline__ void recips(const double (&f)[Q], const double (&pre)[Q], double (&r)[Q]) {
    if constexpr (Q == 1) {
        r[0] = recip(f[0]);
        return;
    }
#pragma unroll
    for (int q0 = 0; q0 < Q; q0 += RC_G) {
        constexpr int G = Q < RC_G ? Q : RC_G;
        double p[G];
#pragma unroll
        for (int q = 0; q < G; ++q)
            p[q] = Q <= RC_G ? pre[q] : (q > 0 ? p[q > 0 ? q - 1 : 0] * f[q0 + q] : f[q0]);
        double inv = recip(p[G - 1]);
#pragma unroll
        for (int q = G - 1; q >= 0; --q) {
            const double y = q > 0 ? inv * p[q > 0 ? q - 1 : 0] : inv;
            r[q0 + q] = fma(fma(-f[q0 + q], y, 1.0), y, y);
            inv *= f[q0 + q];
        }
    }
}
template <int Q>
__device__ __forceinline__ void recips(const float (&f)[Q], const float (&)[Q], float (&r)[Q]) {
#pragma unroll
    for (int q = 0; q < Q; ++q) r[q] = recip(f[q]);
}

// Sum / product over the chain's lanes, in every lane of the chain: rows of 16 lanes,
// then pairs of rows, then (one chain per wave) the two halves.  With two chains per
// wave (64 / CPW consecutive lanes each) one cross-lane reduction and one
// accept/update sequence serve two proposals.
__device__ __forceinline__ void swap16(float v, float& a, float& b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_int(v), __float_as_int(v), false, false);
    a = __int_as_float(r[0]);
    b = __int_as_float(r[1]);
}
__device__ __forceinline__ void swap32(float v, float& a, float& b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_int(v), __float_as_int(v), false, false);
    a = __int_as_float(r[0]);
    b = __int_as_float(r[1]);
}
__device__ __forceinline__ void swap16(double v, double& a, double& b) {
    const int lo = __double2loint(v), hi = __double2hiint(v);
    const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto u = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    a = __hiloint2double(u[0], l[0]);
    b = __hiloint2double(u[1], l[1]);
}
__device__ __forceinline__ void swap32(double v, double& a, double& b) {
    const int lo = __double2loint(v), hi = __double2hiint(v);
    const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto u = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    a = __hiloint2double(u[0], l[0]);
    b = __hiloint2double(u[1], l[1]);
}
template <int CPW, typename T>
__device__ __forceinline__ T chain_sum(T v) {
    T a, b;
    swap16(row16_sum(v), a, b);
    v = a + b;
    if constexpr (CPW == 1) {
        swap32(v, a, b);
        v = a + b;
    }
    return v;
}
template <int CPW, typename T>
__device__ __forceinline__ T chain_prod(T v) {
    T a, b;
    swap16(row16_prod(v), a, b);
    v = a * b;
    if constexpr (CPW == 1) {
        swap32(v, a, b);
        v = a * b;
    }
    return v;
}

// One proposal's random draw: site(s) and the uniform, or its logarithm (FP32)
template <typename R> struct alignas(16) Draw;
template <> struct alignas(16) Draw<float> {
    int ia, ib;
    float u, pad;
};
template <> struct alignas(16) Draw<double> {
    int ia, ib;
    double u;
};
template <typename R, int V> struct alignas(V * sizeof(R)) Vec {
    R v[V];
};

// QMAX: hidden units per lane at one chain per wave (the row covers 64 QMAX).
//
// A proposal is a chain of some hundred dependent operations, and with two waves per
// SIMD (4,096 chains in pairs) the chain's length and its instructions count alike:
// the draws go through LDS, two proposals ahead, so that a chain's own site and
// uniform take one read; its table row comes in 16-byte loads and the spins are read
// while the proposal before is decided, and corrected if that one flips them; sums
// cross the rows of 16 lanes with lane swaps.  10x10, 200 hidden
// units, 100 proposals of 4,096 chains, FP32: 46.6 us (58.7 with the draws read out of
// the lanes, single-word rows and spins read when needed).
template <typename R, int QMAX, int RULE, int CPW>
__global__ __launch_bounds__(256) void k_sample(Dims d, const R* __restrict__ Tt,
                                                const R* __restrict__ Ks, SampleArgs a) {
    constexpr int LPC = 64 / CPW;  // lanes per chain
    constexpr int Q = QMAX * CPW;  // hidden units per lane
    constexpr int V = sampler_vec(Q, sizeof(R));
    typedef Vec<R, V> vec;
    __shared__ Draw<R> draws[4 * 64];
    extern __shared__ int8_t lds_s[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int h = lane / LPC, hl = lane % LPC;
    const int c0 = (blockIdx.x * 4 + wave) * CPW;
    if (c0 >= a.C) return;  // uniform per wave (the launcher makes C a multiple of CPW)
    const int c = c0 + h;
    const int N = d.N, Mw = d.Mw;
    int8_t* s = lds_s + (wave * CPW + h) * round_up(N, 16);
    Draw<R>* dr = draws + wave * 64 + h * LPC;  // this chain's
    int8_t* sg = a.s + (size_t)c * N;
    for (int i = hl; i < N; i += LPC) s[i] = sg[i];
    __builtin_amdgcn_wave_barrier();

    const R* tc = (const R*)a.tch + (size_t)c * Mw;
    R t[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) t[q] = tc[hl + LPC * q];

    // (byte offsets in 32 bits: at most 4,096 rows of 16 KiB)
    const uint32_t rowb = (uint32_t)Mw * sizeof(R), lofs = hl * V * sizeof(R);
    uint32_t n_acc = 0;
    for (int p0 = 0; p0 < a.K; p0 += LPC) {
        const uint64_t pidx = a.prop_base + (uint64_t)(p0 + hl);
        const uint4 x = philox10(make_uint4((uint32_t)pidx, (uint32_t)(pidx >> 32), (uint32_t)c,
                                            TAG_METROPOLIS), a.seed);
        {
            Draw<R> w{};
            if (RULE == 0) {
                w.ia = w.ib = mulshift(x.x, N);
            } else {
                const int k = mulshift(x.x, a.n_bonds);
                w.ia = a.bonds[2 * k];
                w.ib = a.bonds[2 * k + 1];
            }
            const double u = unit53(x.y, x.z);
            // FP32 path compares logarithms; u = 0 gives -inf and always accepts
            w.u = sizeof(R) == 8 ? (R)u : (R)logf((float)u);
            dr[hl] = w;
        }
        __builtin_amdgcn_wave_barrier();
        const int np = min(LPC, a.K - p0);
        Draw<R> cur = dr[0], nxt = dr[min(1, np - 1)];
        vec Ta[Q / V], Tb[Q / V];  // the next proposal's table rows and site factors
        Vec<R, 2> ka_n, kb_n;
        auto fetch = [&](const Draw<R>& w) {
            const uint32_t ra = lofs + __umul24(w.ia, rowb), rb = lofs + __umul24(w.ib, rowb);
#pragma unroll
            for (int g = 0; g < Q / V; ++g) {
                constexpr int step = LPC * V * sizeof(R);
                Ta[g] = *(const vec*)((const char*)Tt + ra + g * step);
                if (RULE == 1) Tb[g] = *(const vec*)((const char*)Tt + rb + g * step);
            }
            ka_n = *(const Vec<R, 2>*)((const char*)Ks + (uint32_t)w.ia * (2 * sizeof(R)));
            if (RULE == 1)
                kb_n = *(const Vec<R, 2>*)((const char*)Ks + (uint32_t)w.ib * (2 * sizeof(R)));
        };
        fetch(cur);
        int sa = s[cur.ia], sb = RULE == 1 ? s[cur.ib] : 0;
        for (int q = 0; q < np; ++q) {
            R Tv[Q], Tw[Q];
#pragma unroll
            for (int qq = 0; qq < Q; ++qq) {
                Tv[qq] = Ta[qq / V].v[qq % V];
                Tw[qq] = RULE == 1 ? Tb[qq / V].v[qq % V] : (R)0;
            }
            const Vec<R, 2> ka_c = ka_n, kb_c = RULE == 1 ? kb_n : ka_n;
            fetch(nxt);  // (the last proposal's again at the end)
            int sa_n = s[nxt.ia], sb_n = RULE == 1 ? s[nxt.ib] : 0;
            const Draw<R> nn = dr[min(q + 2, np - 1)];
            __builtin_amdgcn_sched_barrier(0);  // (the reads stay ahead of the decision)
            bool accept;
            if (RULE == 0) {
                R f[Q], pre[Q];
                R prod = (R)1;
#pragma unroll
                for (int qq = 0; qq < Q; ++qq) {
                    f[qq] = (R)1 - (R)sa * t[qq] * Tv[qq];
                    prod *= f[qq];
                    pre[qq] = prod;
                }
                const R kf = sa < 0 ? ka_c.v[1] : ka_c.v[0];
                if constexpr (sizeof(R) == 8) {
                    const double r = chain_prod<CPW>(prod) * kf;
                    accept = cur.u < r * r;
                } else {
                    const float lr = chain_sum<CPW>(__logf(prod)) + kf;
                    accept = cur.u < 2.0f * lr;
                }
                if (accept) {
                    R r[Q];
                    recips(f, pre, r);
#pragma unroll
                    for (int qq = 0; qq < Q; ++qq) t[qq] = (t[qq] - (R)sa * Tv[qq]) * r[qq];
                    s[cur.ia] = (int8_t)-sa;  // every lane of the chain stores the same value
                    if (nxt.ia == cur.ia) sa_n = -sa;
                }
            } else {
                // the ratio is formed for every chain of the wave (the cross-lane
                // reduction runs outside divergent code); a bond with equal spins
                // is the identity move, accepted with ratio 1
                R g[Q], pre[Q], TT[Q], Td[Q];
                R prod = (R)1;
#pragma unroll
                for (int qq = 0; qq < Q; ++qq) {
                    const R ta = Tv[qq], tb = Tw[qq];
                    TT[qq] = (R)1 - ta * tb;
                    Td[qq] = (R)sa * (ta - tb);
                    g[qq] = TT[qq] - t[qq] * Td[qq];
                    prod *= g[qq];
                    pre[qq] = prod;
                }
                const R ka = sa < 0 ? ka_c.v[1] : ka_c.v[0], kb = sb < 0 ? kb_c.v[1] : kb_c.v[0];
                bool take;
                if constexpr (sizeof(R) == 8) {
                    const double r = chain_prod<CPW>(prod) * ka * kb;
                    take = cur.u < r * r;
                } else {
                    const float lr = chain_sum<CPW>(__logf(prod)) + ka + kb;
                    take = cur.u < 2.0f * lr;
                }
                const bool ident = sa == sb;
                accept = ident || take;
                if (!ident && take) {
                    R r[Q];
                    recips(g, pre, r);
#pragma unroll
                    for (int qq = 0; qq < Q; ++qq) t[qq] = (t[qq] * TT[qq] - Td[qq]) * r[qq];
                    s[cur.ia] = (int8_t)sb;
                    s[cur.ib] = (int8_t)sa;
                    sa_n = nxt.ia == cur.ia ? sb : nxt.ia == cur.ib ? sa : sa_n;
                    sb_n = nxt.ib == cur.ia ? sb : nxt.ib == cur.ib ? sa : sb_n;
                }
            }
            n_acc += accept ? 1u : 0u;
            if (a.acc_log && hl == 0)
                a.acc_log[(size_t)c * a.log_stride + a.log_offset + p0 + q] = accept ? 1 : 0;
            cur = nxt;
            nxt = nn;
            sa = sa_n;
            sb = sb_n;
        }
        __builtin_amdgcn_wave_barrier();
    }
    __builtin_amdgcn_wave_barrier();
    for (int i = hl; i < N; i += LPC) {
        sg[i] = s[i];
        if (a.record) a.rec[(size_t)c * a.rec_stride + i] = s[i];
    }
    if (a.acc_count && hl == 0) a.acc_count[c] += n_acc;
}

// Two chains per wave when the chains pair up and a lane's registers allow (FP32 up to
// 8 x 2 hidden units per lane, FP64 up to 4 x 2).  FP64 takes one chain per wave below
// 2,048 chains, where the shorter chain of operations counts and not their number
// (10x10, 200 hidden units, 4 sweeps with theta: 1,024 chains 157 us, 193 in pairs;
// 2,048 209, 207; 4,096 341, 302); in FP32 the grouping fixes the rounding, so it stays.
int sampler_lanes(int QM, int prec, int C) {
    const bool pair = prec == 0 ? QM <= 4 && C >= 2048 : QM <= 8;
    return pair && C % 2 == 0 ? 32 : 64;
}

template <typename R, int QMAX>
static void launch_q(hipStream_t st, const Dims& d, int rule, const Tables& t,
                     const SampleArgs& a) {
    constexpr bool PAIR = QMAX <= (sizeof(R) == 4 ? 8 : 4);
    const int cpw = 64 / d.lpc;
    const dim3 grid((a.C + 4 * cpw - 1) / (4 * cpw));
    const size_t lds = 4 * cpw * (size_t)round_up(d.N, 16);
    if constexpr (PAIR) {
        if (cpw == 2) {
            if (rule == 0)
                k_sample<R, QMAX, 0, 2><<<grid, 256, lds, st>>>(d, (const R*)t.Tt, (const R*)t.Ks, a);
            else
                k_sample<R, QMAX, 1, 2><<<grid, 256, lds, st>>>(d, (const R*)t.Tt, (const R*)t.Ks, a);
            return;
        }
    }
    if (rule == 0)
        k_sample<R, QMAX, 0, 1><<<grid, 256, lds, st>>>(d, (const R*)t.Tt, (const R*)t.Ks, a);
    else
        k_sample<R, QMAX, 1, 1><<<grid, 256, lds, st>>>(d, (const R*)t.Tt, (const R*)t.Ks, a);
}

template <typename R>
static void launch_r(hipStream_t st, const Dims& d, int rule, const Tables& t,
                     const SampleArgs& a) {
    if (d.QM <= 1) launch_q<R, 1>(st, d, rule, t, a);
    else if (d.QM <= 2) launch_q<R, 2>(st, d, rule, t, a);
    else if (d.QM <= 4) launch_q<R, 4>(st, d, rule, t, a);
    else if (d.QM <= 8) launch_q<R, 8>(st, d, rule, t, a);
    else if (d.QM <= 16) launch_q<R, 16>(st, d, rule, t, a);
    else launch_q<R, 32>(st, d, rule, t, a);
}

// Caller guarantees d.QM <= 32 (M <= 2048).
void launch_sample(hipStream_t st, const Dims& d, int prec, int rule, const Tables& t,
                   const SampleArgs& a) {
    if (a.C <= 0 || a.K <= 0) return;
    if (prec == 0) launch_r<double>(st, d, rule, t, a);
    else launch_r<float>(st, d, rule, t, a);
}

}  // namespace nqs
