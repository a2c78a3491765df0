// Local energies (paper, local-estimator equation)
//   E(s) = sum_{s'} <s|H|s'> psi(s') / psi(s)
// with the connected configurations enumerated implicitly on the device:
//   TFIM:       diagonal J sum_b s_a s_b, and -h for each of the N single flips;
//   Heisenberg: diagonal J sum_b s_a s_b, and 2J (-1)^(l_a + l_b) (Marshall
//               labels, or +2J without them) for each antiparallel bond swap.
// The amplitude ratios use the product form of the sampler (see sampler.hip)
// with tanh(theta) of each sample taken from the activation rows written by
// the theta contraction.
//
// Layout: a wave handles SB samples and lanes run over sites (TFIM) or bonds
// (Heisenberg), ICH chunks of 64 at a time: an item group.  The 4 waves of a block
// are IW item groups of each of 4 / IW sample groups; with more item groups than IW,
// each wave takes every IW-th.  The table T = tanh(2W) is staged in LDS JC hidden
// units at a time and shared by the block, JU hidden units of a site together (one
// 16-byte read); the samples' tanh(theta_j) are wave-uniform and come through the
// scalar cache, JU at a time.
// Bound by the vector ALU: a factor is three operations in this order (the sign times
// the activation, the fused multiply-add, the product), so what a hidden unit costs
// besides is spread over SB samples and ICH chunks, and the waves of a compute unit
// come from item groups too.  16,384 samples, this kernel alone: Heisenberg 16x16,
// 1,024 hidden units, FP32: 787 us (1,340 with one wave over all bonds of 8 samples and
// activations read out of the lanes; its 2.6e10 operations alone take 470 at the
// measured rate of FP32 multiply-adds; at most 128 registers for four waves per
// SIMD, 842 with 138 and three); TFIM 10x10, 200 hidden units, FP64: 77 us (91).
#include "kernels.h"

namespace nqs {

constexpr int LOGCHUNK = 64;  // FP32: fold partial products into logs this often

template <typename R>
__device__ __forceinline__ double ratio_from(R prod, R logacc, R kfac) {
    if constexpr (sizeof(R) == 8) return (double)(kfac * prod);
    else return (double)__expf(kfac + logacc + __logf(prod));
}

template <typename R> struct Quad;  // 16 bytes: JU hidden units
template <> struct Quad<float> {
    float v[4];
};
template <> struct Quad<double> {
    double v[2];
};

// Stage table rows [j0, j0 + jn) (all Nw columns, jn a multiple of JU) into LDS as
// [jn / JU][Nw][JU].
template <typename R>
__device__ __forceinline__ void stage_rows(R* __restrict__ dst, const R* __restrict__ Tj, int j0,
                                           int jn, int Nw) {
    constexpr int JU = 16 / sizeof(R), U = sizeof(R) == 4 ? 2 : 4;
    const int total = jn / JU * Nw;
    const R* src = Tj + (size_t)j0 * Nw;
    for (int base = 0; base < total; base += 256 * U) {
        Quad<R> q[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = min(base + u * 256 + (int)threadIdx.x, total - 1);
            const int g = e / Nw, i = e - g * Nw;
#pragma unroll
            for (int k = 0; k < JU; ++k) q[u].v[k] = src[(size_t)(g * JU + k) * Nw + i];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = base + u * 256 + threadIdx.x;
            if (e < total) ((Quad<R>*)dst)[e] = q[u];
        }
    }
}

template <typename R, int KIND, int SB, int ICH>
__global__ __launch_bounds__(256, sizeof(R) == 4 ? 4 : 1) void k_eloc(Dims d, const R* __restrict__ Tj,
                                              const R* __restrict__ Ks, HamDev H,
                                              const int8_t* __restrict__ s,
                                              const R* __restrict__ tact, long n,
                                              double* __restrict__ out, int JC, int IW) {
    constexpr int JU = 16 / sizeof(R);
    extern __shared__ __align__(16) char lds_raw[];
    R* Ts = (R*)lds_raw;  // [JC / JU][Nw][JU]
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int iw = wave % IW;
    const long k0 = ((long)blockIdx.x * (4 / IW) + wave / IW) * SB;
    const int N = d.N, M = d.M, Mw = d.Mw, Nw = d.Nw;
    const int n_items = KIND == 0 ? N : H.n_bonds;
    long kr[SB];
#pragma unroll
    for (int r = 0; r < SB; ++r) kr[r] = min(k0 + r, n - 1);
    double acc[SB];
#pragma unroll
    for (int r = 0; r < SB; ++r) acc[r] = 0.0;

    for (int gb = 0; gb < n_items; gb += 64 * ICH * IW) {
        const int g0 = gb + 64 * ICH * iw;  // (past the items: staging only)
        int ia[ICH], ib[ICH];
        R sa[ICH][SB], prod[ICH][SB], lacc[ICH][SB];
#pragma unroll
        for (int c = 0; c < ICH; ++c) {
            const int it = g0 + 64 * c + lane;
            const bool valid = it < n_items;
            ia[c] = KIND == 0 ? (valid ? it : 0) : (valid ? H.bonds[2 * it] : 0);
            ib[c] = KIND == 0 ? 0 : (valid ? H.bonds[2 * it + 1] : 0);
#pragma unroll
            for (int r = 0; r < SB; ++r) {
                const int xa = s[kr[r] * N + ia[c]];
                sa[c][r] = (R)xa;
                if (KIND == 1) {
                    const int x = xa * s[kr[r] * N + ib[c]];
                    if (valid) acc[r] += H.J * (double)x;
                }
                prod[c][r] = (R)1;
                lacc[c][r] = (R)0;
            }
        }
        for (int j0 = 0; j0 < M; j0 += JC) {
            // (the table's rows past M are zero, the activations there finite: factors 1)
            const int jn = min(JC, (M - j0 + JU - 1) / JU * JU);
            __syncthreads();
            stage_rows<R>(Ts, Tj, j0, jn, Nw);
            __syncthreads();
            if (k0 >= n || g0 >= n_items) continue;
            // the table entries and activations of the next JU hidden units are read
            // while these ones' products are formed (the last ones' again at the end:
            // the reads stay unconditional)
            Quad<R> na[ICH], nb[ICH], nt[SB];
            auto fetch = [&](int jl) {
                const Quad<R>* row = (const Quad<R>*)Ts + jl / JU * Nw;
#pragma unroll
                for (int c = 0; c < ICH; ++c) {
                    na[c] = row[ia[c]];
                    if (KIND == 1) nb[c] = row[ib[c]];
                }
#pragma unroll
                for (int r = 0; r < SB; ++r) nt[r] = *(const Quad<R>*)(tact + kr[r] * Mw + j0 + jl);
            };
            fetch(0);
            for (int jl = 0; jl < jn; jl += JU) {
                Quad<R> ca[ICH], cb[ICH], ct[SB];
#pragma unroll
                for (int c = 0; c < ICH; ++c) {
                    ca[c] = na[c];
                    if (KIND == 1) cb[c] = nb[c];
                }
#pragma unroll
                for (int r = 0; r < SB; ++r) ct[r] = nt[r];
                fetch(min(jl + JU, jn - JU));
#pragma unroll
                for (int u = 0; u < JU; ++u)
#pragma unroll
                    for (int c = 0; c < ICH; ++c) {
                        if (KIND == 0) {
                            const R Tv = ca[c].v[u];
#pragma unroll
                            for (int r = 0; r < SB; ++r)
                                prod[c][r] *= (R)1 - sa[c][r] * ct[r].v[u] * Tv;
                        } else {
                            const R ta = ca[c].v[u], tb = cb[c].v[u];
                            const R TT = (R)1 - ta * tb, Td = ta - tb;
#pragma unroll
                            for (int r = 0; r < SB; ++r)
                                prod[c][r] *= TT - sa[c][r] * ct[r].v[u] * Td;
                        }
                    }
                if constexpr (sizeof(R) == 4) {
                    const int j = j0 + jl + JU;
                    if (j % LOGCHUNK == 0 && j <= M) {
#pragma unroll
                        for (int c = 0; c < ICH; ++c)
#pragma unroll
                            for (int r = 0; r < SB; ++r) {
                                lacc[c][r] += __logf(prod[c][r]);
                                prod[c][r] = (R)1;
                            }
                    }
                }
            }
        }
        // fold the item contributions
#pragma unroll
        for (int c = 0; c < ICH; ++c) {
            const int it = g0 + 64 * c + lane;
            if (it >= n_items) continue;
            if (KIND == 0) {
#pragma unroll
                for (int r = 0; r < SB; ++r) {
                    const R kf = Ks[2 * ia[c] + (sa[c][r] < 0)];
                    acc[r] -= H.h * ratio_from<R>(prod[c][r], lacc[c][r], kf);
                }
            } else {
                double elem = 2.0 * H.J;
                if (H.sub && ((H.sub[ia[c]] + H.sub[ib[c]]) & 1)) elem = -elem;
#pragma unroll
                for (int r = 0; r < SB; ++r) {
                    const int xa = (int)sa[c][r];
                    const int xb = s[kr[r] * N + ib[c]];
                    if (xa != xb) {
                        const R kab = sizeof(R) == 8 ? Ks[2 * ia[c] + (xa < 0)] * Ks[2 * ib[c] + (xb < 0)]
                                                     : Ks[2 * ia[c] + (xa < 0)] + Ks[2 * ib[c] + (xb < 0)];
                        acc[r] += elem * ratio_from<R>(prod[c][r], lacc[c][r], kab);
                    }
                }
            }
        }
    }
    if (KIND == 0) {
        for (int b = 64 * iw + lane; b < H.n_bonds; b += 64 * IW) {
            const int a0 = H.bonds[2 * b], b0 = H.bonds[2 * b + 1];
#pragma unroll
            for (int r = 0; r < SB; ++r)
                acc[r] += H.J * (double)(s[kr[r] * N + a0] * s[kr[r] * N + b0]);
        }
    }
    __syncthreads();
    double* es = (double*)lds_raw;  // [4 waves][SB]
#pragma unroll
    for (int r = 0; r < SB; ++r) {
        const double e = wave_sum(acc[r]);
        if (lane == 0) es[wave * SB + r] = e;
    }
    __syncthreads();
    if (iw == 0 && lane < SB && k0 + lane < n) {
        double e = es[wave * SB + lane];
        for (int w = 1; w < IW; ++w) e += es[(wave + w) * SB + lane];
        out[k0 + lane] = e;
    }
}

template <typename R, int KIND, int SB, int ICH>
static void launch_k(hipStream_t st, const Dims& d, const Tables& t, const HamDev& H,
                     const int8_t* s, const void* tact, long n, double* out, int IW) {
    constexpr int JU = 16 / sizeof(R);
    // hidden rows of the table staged per chunk: at most 32 KiB, so that five blocks
    // fit a compute unit (Heisenberg 16x16 with three waves per SIMD: 842 us, 1,029
    // with 64 KiB); at least JU,
    // which for the most sites, 4,096, are 64 KiB
    int JC = 64;
    while (JC > JU && (size_t)JC * d.Nw * sizeof(R) > 32768) JC /= 2;
    const size_t rows = (size_t)JC * d.Nw * sizeof(R), sums = 8 * 4 * SB;
    const int per = 4 / IW * SB;
    k_eloc<R, KIND, SB, ICH><<<(unsigned)((n + per - 1) / per), 256, rows > sums ? rows : sums, st>>>(
        d, (const R*)t.Tj, (const R*)t.Ks, H, s, (const R*)tact, n, out, JC, IW);
}

// Samples and chunks per wave.  One chunk where the items fit it (7x7 TFIM, FP64: 44
// us, 53 with room for two); eight samples only where the waves still fill every SIMD
// eight deep (Heisenberg 16x16, FP32: 16,384 samples 787 us, 918 with four; 8,192
// samples 526, 503 with four; 10x10, 2,000 samples with theta 57, 40 with four).
template <typename R, int KIND>
static void launch_items(hipStream_t st, const Dims& d, const Tables& t, const HamDev& H,
                         const int8_t* s, const void* tact, long n, double* out) {
    const int items = KIND == 0 ? d.N : H.n_bonds;
    const int groups = (items + 127) / 128, IW = groups <= 1 ? 1 : groups == 2 ? 2 : 4;
    if (items <= 64) launch_k<R, KIND, 4, 1>(st, d, t, H, s, tact, n, out, 1);
    else if (n / 8 * IW >= 8192) launch_k<R, KIND, 8, 2>(st, d, t, H, s, tact, n, out, IW);
    else launch_k<R, KIND, 4, 2>(st, d, t, H, s, tact, n, out, IW);
}

void launch_eloc(hipStream_t st, const Dims& d, int prec, const Tables& t, const HamDev& H,
                 const int8_t* s, const void* tact, long n, double* out) {
    if (n <= 0) return;
    if (prec == 0) {
        if (H.kind == 0) launch_items<double, 0>(st, d, t, H, s, tact, n, out);
        else launch_items<double, 1>(st, d, t, H, s, tact, n, out);
    } else {
        if (H.kind == 0) launch_items<float, 0>(st, d, t, H, s, tact, n, out);
        else launch_items<float, 1>(st, d, t, H, s, tact, n, out);
    }
}

}  // namespace nqs
