// Energy statistics, the dense-form conjugate gradients and the parameter update.
// Every reduction (means, dot products) is a fixed-order two-level sum, so results
// do not depend on timing or on what else runs on the device.
#include "kernels.h"

namespace nqs {

// ---------------------------------------------------------------------------
// block-level helpers
// ---------------------------------------------------------------------------
template <int NT>
__device__ __forceinline__ double block_sum(double v, double* sh) {
    v = wave_sum(v);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) sh[wave] = v;
    __syncthreads();
    double r = 0.0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) r += sh[w];
    __syncthreads();
    return r;
}

// true in exactly one block: the last to arrive; its earlier writes and all
// other blocks' writes before their arrival are visible to it afterwards.
__device__ __forceinline__ bool arrive_last(uint32_t* counter) {
    __shared__ int last;
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t v = atomicAdd(counter, 1u);
        last = (v == gridDim.x - 1) ? 1 : 0;
    }
    __syncthreads();
    if (last) __threadfence();
    return last != 0;
}

__device__ __forceinline__ double vload(const double* p) { return *(const volatile double*)p; }

// Fixed-order sum of nb block partials by one 256-thread block.
__device__ __forceinline__ double final_sum(const double* dpart, int nb, double* sh) {
    double a = 0.0;
    for (int b = threadIdx.x; b < nb; b += 256) a += vload(&dpart[b]);
    return block_sum<256>(a, sh);
}

// ---------------------------------------------------------------------------
// statistics: mean, variance (1/n) and error of the mean; one block
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void k_stats(const double* __restrict__ E, long n,
                                                double* __restrict__ out) {
    __shared__ double sh[16];
    double a = 0.0;
    for (long k = threadIdx.x; k < n; k += 1024) a += E[k];
    const double mean = block_sum<1024>(a, sh) / (double)n;
    double b = 0.0;
    for (long k = threadIdx.x; k < n; k += 1024) {
        const double d = E[k] - mean;
        b += d * d;
    }
    const double var = block_sum<1024>(b, sh) / (double)n;
    if (threadIdx.x == 0) {
        out[0] = mean;
        out[1] = var;
        out[2] = sqrt(var / (double)n);
    }
}

// v_k = scale * (E_k - mean)
__global__ void k_center(const double* __restrict__ E, const double* __restrict__ stats,
                         double scale, long n, double* __restrict__ v) {
    const long k = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) v[k] = scale * (E[k] - stats[0]);
}

// Dense-form CG, one iteration in three kernels (product, update, direction);
// each sums the block partials of the kernel before it in a fixed order (the
// same in every block), so no kernel needs a cross-block step:
//   update:    p.Ap from the product's partials, alpha = r.r / p.Ap,
//              x += alpha p, r -= alpha Ap, block partials of the new r.r;
//   direction: r.r from the update's partials, beta = r.r / r.r_prev,
//              p = r + beta p; block 0 advances the iteration and the stop flag
//              (also stored to a pinned host word when asked: the last
//              iteration of a batch, so a batch can be replayed from a graph).
// The diagonal shift is taken from the scalars (set by k_cg_init).
// Every scalar is written by a different kernel from the one that reads it.
__device__ __forceinline__ double sum_partials(const double* part, int np, double* sh) {
    double a = 0.0;
    for (int b = threadIdx.x; b < np; b += 256) a += part[b];
    return block_sum<256>(a, sh);
}
__global__ __launch_bounds__(256) void k_cg_update(int total, double* __restrict__ x,
                                                   double* __restrict__ r,
                                                   const double* __restrict__ p,
                                                   const double* __restrict__ Ap,
                                                   const double* __restrict__ pap_part, int npap,
                                                   double* __restrict__ rr_part, CgScalars* sc) {
    if (sc->done) return;
    __shared__ double sh[4];
    const int e = blockIdx.x * 256 + threadIdx.x;
    const double rr = sc->rr;
    const double pAp = sum_partials(pap_part, npap, sh);
    const double alpha = rr / pAp;
    if (!(pAp > 0.0) || !isfinite(alpha)) {  // the same decision in every block
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            sc->bad = 1;
            sc->done = 1;
        }
        return;
    }
    double rn = 0.0;
    if (e < total) {
        x[e] += alpha * p[e];
        const double re = r[e] - alpha * Ap[e];
        r[e] = re;
        rn = re * re;
    }
    rn = block_sum<256>(rn, sh);
    if (threadIdx.x == 0) rr_part[blockIdx.x] = rn;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sc->alpha = alpha;
        sc->pAp = pAp;
        sc->rr_prev = rr;
    }
}

__global__ __launch_bounds__(256) void k_cg_p(int total, const double* __restrict__ r,
                                              double* __restrict__ p,
                                              const double* __restrict__ rr_part, int nrr,
                                              CgScalars* sc, volatile int32_t* host_flag) {
    const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
    if (sc->done) {
        if (host_flag && lead) *host_flag = 1;
        return;
    }
    __shared__ double sh[4];
    const double rr = sum_partials(rr_part, nrr, sh);
    const double beta = rr / sc->rr_prev;
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e < total) p[e] = r[e] + beta * p[e];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sc->beta = beta;
        sc->rr = rr;
        sc->iters += 1;
        if (!isfinite(rr)) {
            sc->bad = 1;
            sc->done = 1;
        }
        if (rr <= sc->tol2 || sc->iters >= sc->maxiter) sc->done = 1;
        if (host_flag) *host_flag = sc->done;
    }
}

// x = 0, r = p = f, rr = f.f, thresholds.
__global__ __launch_bounds__(256) void k_cg_init(int total, const double* __restrict__ f,
                                                 double* __restrict__ x, double* __restrict__ r,
                                                 double* __restrict__ p, double* __restrict__ dpart,
                                                 CgScalars* sc, double tol, int maxiter,
                                                 double shift) {
    __shared__ double sh[4];
    const int e = blockIdx.x * 256 + threadIdx.x;
    double ff = 0.0;
    if (e < total) {
        const double fe = f[e];
        x[e] = 0.0;
        r[e] = fe;
        p[e] = fe;
        ff = fe * fe;
    }
    ff = block_sum<256>(ff, sh);
    if (threadIdx.x == 0) dpart[blockIdx.x] = ff;
    if (arrive_last(&sc->counter[2])) {
        const double s = final_sum(dpart, gridDim.x, sh);
        if (threadIdx.x == 0) {
            sc->rr = s;
            sc->rr0 = s;
            sc->beta = 0.0;
            sc->tol2 = tol * tol * s;
            sc->iters = 0;
            sc->maxiter = maxiter;
            sc->shift = shift;
            sc->bad = isfinite(s) ? 0 : 1;
            sc->done = (s <= sc->tol2 || maxiter <= 0 || !isfinite(s)) ? 1 : 0;
            sc->counter[2] = 0;
        }
    }
}

// Pm -= lr * delta (delta is zero outside parameter entries); flags non-finite.
__global__ void k_axpy_update(int total, double* __restrict__ Pm, const double* __restrict__ delta,
                              double lr, CgScalars* sc) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    const double v = Pm[e] - lr * delta[e];
    Pm[e] = v;
    if (!isfinite(v)) sc->bad = 2;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static inline int nblk(long n, int b) { return (int)((n + b - 1) / b); }

void launch_stats(hipStream_t st, const double* E, long n, double* out3) {
    k_stats<<<1, 1024, 0, st>>>(E, n, out3);
}
void launch_center(hipStream_t st, const double* E, const double* stats, double scale, long n,
                   double* v) {
    k_center<<<nblk(n, 256), 256, 0, st>>>(E, stats, scale, n, v);
}
void launch_cg_init(hipStream_t st, int total, const double* f, double* x, double* r, double* p,
                    double* dpart, CgScalars* sc, double tol, int maxiter, double shift) {
    k_cg_init<<<nblk(total, 256), 256, 0, st>>>(total, f, x, r, p, dpart, sc, tol, maxiter, shift);
}
void launch_cg_update(hipStream_t st, int total, double* x, double* r, double* p,
                      const double* Ap, double* dpart, int npap, CgScalars* sc,
                      int32_t* host_flag) {
    const int nb = nblk(total, 256);
    double* rr_part = dpart + npap;  // after the product's partials
    k_cg_update<<<nb, 256, 0, st>>>(total, x, r, p, Ap, dpart, npap, rr_part, sc);
    k_cg_p<<<nb, 256, 0, st>>>(total, r, p, rr_part, nb, sc, host_flag);
}
void launch_axpy_update(hipStream_t st, int total, double* x, const double* delta, double lr,
                        CgScalars* sc) {
    k_axpy_update<<<nblk(total, 256), 256, 0, st>>>(total, x, delta, lr, sc);
}

}  // namespace nqs
