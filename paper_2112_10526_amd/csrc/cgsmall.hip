// The whole on-the-fly CG of a small FP64 system in one launch of one workgroup.
//
// For a handful of sites the three kernels of a CG iteration (qgt.hip) last 5 us
// each, nearly all of it launch and round trips to memory.  Here everything an
// iteration touches stays on one compute unit: the batch's activations in
// registers, its spins and the residual in LDS, the CG vectors one entry per thread,
// and three barriers per iteration.  The arithmetic is that of
// the iteration kernels (same rearranged CG, FP64 throughout, FP64 matrix cores):
//   w = J r + beta w_old;  z = (w - mean w) / n;  G p = J^T z;
//   alpha = r.r / (sum z (w - mean w) + shift p.p);  x, r, and r.r, r.p, p.p.
// Bound by the FP64 matrix cores of that one unit (n Ma Na / 32 cycles an iteration)
// and the chain of reductions between them: 5.9 us an iteration at 10 sites, 10 hidden
// units and 1,024 samples, where the three kernels take 15 us and their gaps.
#include "kernels.h"

namespace nqs {

// waves, of 256 registers each: the activations fit (with two hidden tiles 20 registers
// pass through scratch)
constexpr int CS_NW = 8;
constexpr long CS_LIMIT = 1L << 18;

// Sum over the four 16-lane rows of a wave with the result scattered: lane 16 q + r
// gets the sum of v[q] over the lanes 16 q' + r.
__device__ __forceinline__ void swap_rows(double& a, double& b, bool half) {
    uint32_t al = (uint32_t)__double2loint(a), ah = (uint32_t)__double2hiint(a);
    uint32_t bl = (uint32_t)__double2loint(b), bh = (uint32_t)__double2hiint(b);
    if (half) {
        const auto l = __builtin_amdgcn_permlane32_swap(al, bl, false, false);
        const auto h = __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
        a = __hiloint2double((int)h[0], (int)l[0]);
        b = __hiloint2double((int)h[1], (int)l[1]);
    } else {
        const auto l = __builtin_amdgcn_permlane16_swap(al, bl, false, false);
        const auto h = __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
        a = __hiloint2double((int)h[0], (int)l[0]);
        b = __hiloint2double((int)h[1], (int)l[1]);
    }
}
__device__ __forceinline__ double row4_scatter_sum(double (&v)[4]) {
    swap_rows(v[0], v[2], true);   // lower lanes: row 0's terms, upper: row 2's
    swap_rows(v[1], v[3], true);
    double a = v[0] + v[2], b = v[1] + v[3];
    swap_rows(a, b, false);
    return a + b;
}

// A hidden tiles x B site tiles (16 each); group g of wave w: samples (8 g + w) 64 ..
// + 63, lane l holding w of sample l.
template <int A, int B, int GR>
__global__ __launch_bounds__(64 * CS_NW) void k_cg_small(
    Dims d, const int8_t* __restrict__ Sp, const int8_t* __restrict__ St, long Nsp,
    const double* __restrict__ tact, int n, const double* __restrict__ f, double* __restrict__ x_out,
    double tol, int maxiter, double shift, CgScalars* sc, volatile int32_t* host_flag) {
    constexpr int NA = 16 * B, TOT = 256 * A * B;   // row of a CG vector, its entries
    constexpr int NS = 64 * CS_NW * GR;             // samples, padded
    constexpr int PL = NA + 1;                      // LDS row of the residual
    constexpr int SL = NS + 16;                     // LDS row of the site-major spins
    extern __shared__ __align__(16) char lds[];
    double* part = (double*)lds;                    // [CS_NW][TOT]
    double* R = part + CS_NW * TOT;                 // [16 A][PL]
    double* zs = R + 16 * A * PL;                   // [NS]
    double* red = zs + NS;                          // [2][CS_NW], [3][TOT / 64]
    double* red3 = red + 2 * CS_NW;
    int8_t* s1 = (int8_t*)(red3 + 3 * (TOT / 64) + (3 * (TOT / 64) & 1));  // [NS][NA]
    int8_t* s2 = s1 + NS * NA;                      // [NA][SL]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lk = lane >> 4;
    constexpr int NT = 64 * CS_NW;
    // spins, sample-major and site-major, in 16-byte pieces (zero past n: Sp and St are)
    for (int e = tid; e < NS * B; e += NT) {
        const int k = e / B, b = e - k * B;
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (k < Nsp) v = *(const uint4*)(Sp + (long)k * d.Kq + 16 * b);
        *(uint4*)(s1 + k * NA + 16 * b) = v;
    }
    for (int e = tid; e < NA * (NS / 16); e += NT) {
        const int i = e / (NS / 16), k = 16 * (e - i * (NS / 16));
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (k < Nsp) v = *(const uint4*)(St + (long)i * Nsp + k);
        *(uint4*)(s2 + i * SL + k) = v;
    }
    // this thread's CG entry
    const bool own = tid < TOT;
    const int ej = tid / NA, ei = tid - ej * NA;
    const bool keep = own && ((ej < d.M && ei < d.N) || (d.hb && ej < d.M && ei == d.N) ||
                              (d.vb && ej == d.M && ei < d.N));
    double r = own ? f[tid] : 0.0, p = 0.0, x = 0.0;
    auto sums = [&](double a, double b, double c) {  // block sums of the entries' terms
        if (64 * wave < TOT) {
            a = wave_sum(a);
            b = wave_sum(b);
            c = wave_sum(c);
            if (lane == 0) {
                red3[wave] = a;
                red3[TOT / 64 + wave] = b;
                red3[2 * (TOT / 64) + wave] = c;
            }
            if (own) R[ej * PL + ei] = r;
        }
    };
    sums(r * r, 0.0, 0.0);
    double w[GR];
#pragma unroll
    for (int g = 0; g < GR; ++g) w[g] = 0.0;
    // activations: t1 as weights of contraction 1 (sample 16 q + lr, hidden 4 i + lk),
    // t2 as operand of contraction 2 (sample 4 s + lk, hidden lr); kept in registers
    // for the whole solve (A GR <= 2)
    double t1[16 * A * GR], t2[16 * A * GR];
#pragma unroll
    for (int h = 0; h < A * GR; ++h) {
        const double* th = tact + 16 * (h % A);
        const int k0 = (CS_NW * (h / A) + wave) * 64;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            t1[16 * h + q] = th[(long)min(k0 + 16 * (q / 4) + lr, n - 1) * d.Mw + 4 * (q % 4) + lk];
            t2[16 * h + q] = th[(long)min(k0 + 4 * q + lk, n - 1) * d.Mw + lr];
        }
    }
    __syncthreads();
    const double inv_n = 1.0 / (double)n;
    double rr0 = 0.0, tol2 = 0.0, rr_prev = 0.0, rr = 0.0;
    int it = 0, bad = 0;
#pragma unroll 1
    for (;; ++it) {
        double rp = 0.0, pp = 0.0;
        rr = 0.0;
#pragma unroll
        for (int q = 0; q < TOT / 64; ++q) {
            rr += red3[q];
            rp += red3[TOT / 64 + q];
            pp += red3[2 * (TOT / 64) + q];
        }
        if (it == 0) {
            rr0 = rr;
            tol2 = tol * tol * rr0;
        }
        if (!isfinite(rr)) bad = 1;
        if (!(rr > tol2) || it >= maxiter || bad) break;  // (the same in every thread)
        const double beta = it == 0 ? 0.0 : rr / rr_prev;
        pp = rr + 2.0 * beta * rp + beta * beta * pp;
        // ---- w = J r + beta w: blocks P S^T with the hidden index as the row, so that
        // a lane sums its four hidden rows of one sample in its own registers
        double sw = 0.0;
#pragma unroll
        for (int g = 0; g < GR; ++g) {
            double v[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int a = 0; a < A; ++a) {
                v4d acc[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[q] = v4d{0, 0, 0, 0};
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    uint4 sp[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        sp[q] = *(const uint4*)(s1 + ((CS_NW * g + wave) * 64 + 16 * q + lr) * NA + 16 * b);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const double pr = R[(16 * a + lr) * PL + 16 * b + 4 * e + lk];
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const uint32_t u = e == 0 ? sp[q].x : e == 1 ? sp[q].y : e == 2 ? sp[q].z : sp[q].w;
                            const double s = (double)(int)__builtin_amdgcn_sbfe((int)u, 8 * lk, 8);
                            acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(pr, s, acc[q], 0, 0, 0);
                        }
                    }
                }
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        v[q] = fma(t1[16 * (g * A + a) + 4 * q + i], acc[q][i], v[q]);
            }
            w[g] = row4_scatter_sum(v) + beta * w[g];
            if ((CS_NW * g + wave) * 64 + lane < n) sw += w[g];
        }
        sw = wave_sum(sw);
        if (lane == 0) red[wave] = sw;
        __syncthreads();
        double mean = 0.0;
#pragma unroll
        for (int q = 0; q < CS_NW; ++q) mean += red[q];
        mean *= inv_n;
        // ---- z, and J^T z (the wave's own samples; z passes through its part of LDS)
        double zw = 0.0;
        v4d acc[A][B];
#pragma unroll
        for (int a = 0; a < A; ++a)
#pragma unroll
            for (int b = 0; b < B; ++b) acc[a][b] = v4d{0, 0, 0, 0};
#pragma unroll
        for (int g = 0; g < GR; ++g) {
            const int k0 = (CS_NW * g + wave) * 64;
            const double z = k0 + lane < n ? (w[g] - mean) * inv_n : 0.0;
            zw = fma(z, k0 + lane < n ? w[g] - mean : 0.0, zw);
            zs[k0 + lane] = z;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int c = 0; c < 4; ++c) {  // 16 samples: four k-steps
                uint4 sp[B];
#pragma unroll
                for (int b = 0; b < B; ++b)
                    sp[b] = *(const uint4*)(s2 + (16 * b + lr) * SL + k0 + 16 * c);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double z1 = zs[k0 + 16 * c + 4 * e + lk];
#pragma unroll
                    for (int a = 0; a < A; ++a) {
                        const double tz = t2[16 * (g * A + a) + 4 * c + e] * z1;
#pragma unroll
                        for (int b = 0; b < B; ++b) {
                            const uint32_t u = e == 0 ? sp[b].x : e == 1 ? sp[b].y : e == 2 ? sp[b].z : sp[b].w;
                            const double s = (double)(int)__builtin_amdgcn_sbfe((int)u, 8 * lk, 8);
                            acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(tz, s, acc[a][b], 0, 0, 0);
                        }
                    }
                }
            }
        }
#pragma unroll
        for (int a = 0; a < A; ++a)
#pragma unroll
            for (int b = 0; b < B; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    part[wave * TOT + (16 * a + acc_row<double>(lk, q)) * NA + 16 * b + lr] = acc[a][b][q];
        zw = wave_sum(zw);
        if (lane == 0) red[CS_NW + wave] = zw;
        __syncthreads();
        double pap = 0.0;
#pragma unroll
        for (int q = 0; q < CS_NW; ++q) pap += red[CS_NW + q];
        pap += shift * pp;
        const double alpha = rr / pap;
        if (!(pap > 0.0) || !isfinite(alpha)) {
            bad = 1;
            break;  // (the same in every thread)
        }
        double pn = 0.0;
        if (own) {
            double g = 0.0;
#pragma unroll
            for (int q = 0; q < CS_NW; ++q) g += part[q * TOT + tid];
            pn = r + beta * p;
            const double ap = keep ? g + shift * pn : 0.0;
            x += alpha * pn;
            r -= alpha * ap;
            p = pn;
        }
        sums(r * r, r * pn, pn * pn);
        rr_prev = rr;
        __syncthreads();
    }
    if (own) x_out[tid] = x;
    if (tid == 0) {
        sc->rr = rr;
        sc->rr0 = rr0;
        sc->tol2 = tol2;
        sc->iters = it;
        sc->done = 1;
        sc->bad = bad;
        if (host_flag) *host_flag = 1;
    }
}

// One tile: up to 1,024 samples; two: up to 512.  Measured against the iteration
// kernels (whole gradient and direction, tolerance 1e-10): 10 sites 1,024 samples
// 954 -> 458 us, 15 sites 300 samples 1,313 -> 420 us; at twice the limit (10 sites,
// 2,048 samples; 15 sites, 30 hidden units, 1,000 samples) this form was 15 to 20 %
// slower, its matrix-core work on one compute unit outgrowing the launches saved.
bool cg_small_fits(const Dims& d, int prec, long n) {
    return prec == 0 && d.Ma * d.Na <= 512 && n * d.Ma * d.Na <= CS_LIMIT;
}

template <int A, int B, int GR>
static void cg_small(hipStream_t st, const Dims& d, const QgtBatch& q, const double* tact, long n,
                     const double* f, double* x, double tol, int maxiter, double shift,
                     CgScalars* sc, int32_t* host_flag) {
    constexpr int NA = 16 * B, TOT = 256 * A * B, NS = 64 * CS_NW * GR;
    constexpr size_t lds = 8 * ((size_t)CS_NW * TOT + 16 * A * (NA + 1) + NS + 2 * CS_NW +
                                3 * (TOT / 64) + (3 * (TOT / 64) & 1)) +
                           (size_t)NS * NA + (size_t)NA * (NS + 16);
    (void)hipFuncSetAttribute((const void*)k_cg_small<A, B, GR>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    k_cg_small<A, B, GR><<<1, 64 * CS_NW, lds, st>>>(d, (const int8_t*)q.Sp, q.St, q.Nsp, tact,
                                                     (int)n, f, x, tol, maxiter, shift, sc,
                                                     host_flag);
}

void launch_cg_small(hipStream_t st, const Dims& d, const QgtBatch& q, const void* tact, long n,
                     const double* f, double* x, double tol, int maxiter, double shift,
                     CgScalars* sc, int32_t* host_flag) {
    const int A = d.Ma / 16, B = d.Na / 16;
    const double* t = (const double*)tact;
#define CGS(A, B, GR) \
    cg_small<A, B, GR>(st, d, q, t, n, f, x, tol, maxiter, shift, sc, host_flag)
    if (A * B == 1 && n <= 64 * CS_NW) CGS(1, 1, 1);
    else if (A * B == 1) CGS(1, 1, 2);
    else if (A == 2) CGS(2, 1, 1);
    else CGS(1, 2, 1);
#undef CGS
}

}  // namespace nqs
