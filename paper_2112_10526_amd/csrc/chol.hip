// Dense direct solve of (A + shift I) x = f for a symmetric positive-definite A
// (paper: solving the SR / TDVP linear system with a dense QGT; the jVMC
// comparison's dense-solver rows): blocked Cholesky A + shift I = L L^T from the
// lower triangle of A, then L y = f and L^T x = y.  Panels of CH_NB = 32 columns,
// one launch each (k_chol_step): every block factors the panel's 32 x 32 diagonal
// block for itself, solves its own panel rows against it, and subtracts their outer
// product from its 64 x 64 tile of the trailing triangle.  As the blocks still read
// the panel while others finish, the solved rows go to the mirrored place in the
// upper triangle; k_chol_mirror puts them into the lower one.  L y = f rides on the panels: the right-hand side is one more
// row of each.  L^T x = y walks the diagonal blocks from the last: x_k from the
// stored inverse, then its part out of the columns before it, whose entries of L
// are loaded ahead (they do not depend on x): one workgroup for systems of up to
// 1,024, one launch per block above.
// The steps are a chain of dependent latencies (32 pivots at about 0.15 us each,
// one panel after the other), so launches and passes were what could go.  n = 880:
// 28 steps of 13.5 us (some 5 us of them the elimination, 3 us the loads behind the
// previous launch) and 72 us backward, 0.45 ms; a panel and an update launch per
// step (28 + 11 us) with a left-looking backward solve took 1.31 ms.  n = 8,448 (the
// 64-site complex model): 43 -> 33 ms.
// A pivot that is not positive (A + shift I not positive definite) sets *bad.
#include "kernels.h"

namespace nqs {

constexpr int CH_NB = 32;
constexpr int CH_XD = 33;   // LDS row of a 32-column matrix

// Cholesky elimination of the 32 x 32 block next to the identity, one wave, all in
// registers: lane c < 32 holds column c of the (symmetric) block, lane 32 + c column c
// of the identity, register i row i.  Step j scales row j by 1 / sqrt(d_j) (hardware
// estimate, two Newton steps, the second with the product's low part: half a unit) and
// takes l_i times it out of every row i > j, l_i being the scaled row's entry in lane i
// (readlane).  That leaves L^T on the left and L^-1 on the right.  A_ic and A_ci lose
// the same product l_i l_c, so the block stays symmetric to the bit: with A_ij times
// (A_jc / d_j) its halves part by roundings that the multipliers of a nearly singular
// block blow up (48 parameters, 30 samples, shift 1e-10: mean residual of the solve 134
// x 2^-53 |A| |x|, 7 here).
// Returns false if a pivot is not positive.
__device__ __forceinline__ bool chol_block32(double (&a)[CH_NB]) {
    bool ok = true;
#pragma unroll
    for (int j = 0; j < CH_NB; ++j) {
        double d = readlane(a[j], j);
        const bool pos = d > 0.0 && isfinite(d);
        ok = ok && pos;
        d = pos ? d : 1.0;
        double h = __builtin_amdgcn_rsq(d), t = d * h;
        h = fma(0.5 * h, fma(-t, h, 1.0), h);
        t = d * h;
        const double e = fma(-fma(d, h, -t), h, fma(-t, h, 1.0));  // 1 - d h^2
        a[j] *= fma(0.5 * h, e, h);
        // (scalars in groups: one at a time, each product waits for its own readlane)
#pragma unroll
        for (int i0 = j + 1; i0 < CH_NB; i0 += 8) {
            double l[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (i0 + u < CH_NB) l[u] = readlane(a[j], i0 + u);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (i0 + u < CH_NB) a[i0 + u] = fma(-l[u], a[j], a[i0 + u]);
        }
    }
    return ok;
}

// Panel k0 (w columns): block b is tile (ti, tj), ti >= tj, of the trailing
// triangle's T x T tiles.  Wave 0 factors; then the waves solve the panel rows of
// tile rows ti and tj (X = A L^-T on the matrix cores, 16 rows at a time, the
// operands loaded before the factorisation) and each updates a quarter of the tile.
template <int T>
__global__ __launch_bounds__(256) void k_chol_step(double* __restrict__ A, int n, long ld, int k0,
                                                   double shift, int32_t* __restrict__ bad,
                                                   double* __restrict__ Yinv,
                                                   double* __restrict__ rhs,
                                                   double* __restrict__ yout) {
    constexpr int NG = T / 32;  // row groups per wave, 16 x 16 tiles per quarter side
    __shared__ double Y[CH_NB][CH_XD];  // L_kk^-1
    __shared__ double yk[CH_NB];
    __shared__ double Xs[2 * T][CH_XD];  // solved rows of tile row ti, then tj
    const int w = n - k0 < CH_NB ? n - k0 : CH_NB, k1 = k0 + w;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lk = lane >> 4;
    const int b = blockIdx.x;
    int ti = (int)((sqrtf(8.0f * (float)b + 1.0f) - 1.0f) * 0.5f);
    while ((ti + 1) * (ti + 2) / 2 <= b) ++ti;
    while (ti * (ti + 1) / 2 > b) --ti;
    const int tj = b - ti * (ti + 1) / 2;
    const int ri = k1 + ti * T, cj = k1 + tj * T;
    const bool rest = k1 < n;  // (the last panel has no trailing rows: one block)
    double x[CH_NB];
    if (wave == 0) {
        const int c = lane & 31;
#pragma unroll
        for (int i = 0; i < CH_NB; ++i) {
            double v = i == c ? 1.0 : 0.0;  // (identity past w, and on the right)
            const int hi = i > c ? i : c, lo = i > c ? c : i;
            if (lane < 32 && hi < w)
                v = A[(long)(k0 + hi) * ld + k0 + lo] + (i == c ? shift : 0.0);
            x[i] = v;
        }
    }
    // panel rows in MFMA order (row lr of 16, columns 4 q + lk), the tile in
    // accumulator order, the right-hand side: all loaded before the barrier
    double pa[NG][CH_NB / 4];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const int gr = 16 * (wave + 4 * g);  // row of Xs
        const int r = (gr < T ? ri + gr : cj + gr - T) + lr;
#pragma unroll
        for (int q = 0; q < CH_NB / 4; ++q)
            pa[g][q] = r < n ? A[(long)r * ld + k0 + 4 * q + lk] : 0.0;
    }
    const int r0 = ri + (wave >> 1) * (T / 2), c0 = cj + (wave & 1) * (T / 2);
    double ct[NG][NG][4];
#pragma unroll
    for (int a = 0; a < NG; ++a)
#pragma unroll
        for (int c = 0; c < NG; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int row = r0 + a * 16 + acc_row<double>(lk, q), col = c0 + c * 16 + lr;
                ct[a][c][q] = row < n && col <= row ? A[(long)row * ld + col] : 0.0;
            }
    const double fk = tid < w ? rhs[k0 + tid] : 0.0;
    const double fr = tid < T && ri + tid < n ? rhs[ri + tid] : 0.0;
    __builtin_amdgcn_sched_barrier(0);
    if (wave == 0) {
        const bool ok = chol_block32(x);
        if (!ok && b == 0 && lane == 0) *bad = 1;
        if (lane >= 32) {
#pragma unroll
            for (int i = 0; i < CH_NB; ++i) Y[i][lane - 32] = x[i];
        }
        if (lane < CH_NB) yk[lane] = fk;  // f_k for now
    }
    __syncthreads();
    if (rest) {
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const int gr = 16 * (wave + 4 * g);
            if (gr >= T && ti == tj) continue;
            v4d xa[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) xa[c] = v4d{0, 0, 0, 0};
#pragma unroll
            for (int q = 0; q < CH_NB / 4; ++q)
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    xa[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(pa[g][q], Y[16 * c + lr][4 * q + lk],
                                                                 xa[c], 0, 0, 0);
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    Xs[gr + acc_row<double>(lk, q)][16 * c + lr] = xa[c][q];
        }
    }
    double y = 0.0;  // y_k = L_kk^-1 f_k, by the last wave's lanes
    const int yl = tid - 192;
    if (yl >= 0 && yl < CH_NB) {
#pragma unroll
        for (int m = 0; m < CH_NB; ++m) y = fma(Y[yl][m], yk[m], y);  // (Y lower)
    }
    __syncthreads();
    if (b == 0) {
        for (int e = tid; e < CH_NB * CH_NB; e += 256)
            Yinv[(size_t)(k0 / CH_NB) * CH_NB * CH_NB + e] = Y[e / CH_NB][e % CH_NB];
        if (yl >= 0 && yl < w) yout[k0 + yl] = y;
    }
    if (!rest) return;
    const double(*Xi)[CH_XD] = Xs;
    const double(*Xj)[CH_XD] = Xs + (ti == tj ? 0 : T);
    v4d acc[NG][NG];
#pragma unroll
    for (int a = 0; a < NG; ++a)
#pragma unroll
        for (int c = 0; c < NG; ++c) acc[a][c] = v4d{0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < CH_NB; k += 4) {
        double fa[NG], fb[NG];
#pragma unroll
        for (int a = 0; a < NG; ++a) {
            fa[a] = Xi[(wave >> 1) * (T / 2) + a * 16 + lr][k + lk];
            fb[a] = Xj[(wave & 1) * (T / 2) + a * 16 + lr][k + lk];
        }
#pragma unroll
        for (int a = 0; a < NG; ++a)
#pragma unroll
            for (int c = 0; c < NG; ++c)
                acc[a][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[a], fb[c], acc[a][c], 0, 0, 0);
    }
#pragma unroll
    for (int a = 0; a < NG; ++a)
#pragma unroll
        for (int c = 0; c < NG; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int row = r0 + a * 16 + acc_row<double>(lk, q), col = c0 + c * 16 + lr;
                if (row < n && col <= row) A[(long)row * ld + col] = ct[a][c][q] - acc[a][c][q];
            }
    if (ti != tj) return;  // (uniform over the block)
    // this tile row's solved panel rows to the upper triangle, and their part out of
    // the right-hand side
    if (yl >= 0 && yl < CH_NB) yk[yl] = y;
    __syncthreads();
    for (int e = tid; e < T * CH_NB; e += 256) {
        const int r = e % T, c = e / T;
        if (ri + r < n) A[(long)(k0 + c) * ld + ri + r] = Xs[r][c];
    }
    if (tid < T && ri + tid < n) {
        double a[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int c = 0; c < CH_NB; ++c) a[c & 3] = fma(Xs[tid][c], yk[c], a[c & 3]);
        rhs[ri + tid] = fr - ((a[0] + a[1]) + (a[2] + a[3]));
    }
}

// 32 x 32 tiles (bi, bj), bi > bj, of L from the mirrored place in the upper
// triangle (the diagonal blocks are used through their inverses only).
__global__ __launch_bounds__(256) void k_chol_mirror(double* __restrict__ A, int n, long ld) {
    __shared__ double T[CH_NB][CH_NB + 1];
    const int tid = threadIdx.x;
    const long b = blockIdx.x;
    long bi = (long)((sqrt(8.0 * (double)b + 1.0) + 1.0) * 0.5);
    while (bi * (bi + 1) / 2 <= b) ++bi;
    while (bi * (bi - 1) / 2 > b) --bi;
    const long bj = b - bi * (bi - 1) / 2;
    const int tx = tid & 31, ty = tid >> 5;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const long r = bi * CH_NB + tx;
        if (r < n) T[ty + 8 * m][tx] = A[(bj * CH_NB + ty + 8 * m) * ld + r];
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const long r = bi * CH_NB + ty + 8 * m;
        if (r < n) A[r * ld + bj * CH_NB + tx] = T[tx][ty + 8 * m];
    }
}

// x_k = Yinv_k^T s_k by the first 32 lanes (s in LDS), into xk.  The products with an
// inverse run in order, here and for y_k: in four partial sums a nearly singular block
// left a residual 1.3 times as large.
__device__ __forceinline__ void chol_back_block(const double (*Yk)[CH_NB + 1], const double* s,
                                                double* xk) {
    const int c = threadIdx.x;
    if (c >= CH_NB) return;
    double a = 0.0;
#pragma unroll
    for (int m = 0; m < CH_NB; ++m) a = fma(Yk[m][c], s[m], a);  // (Yinv lower)
    xk[c] = a;
}

// L^T x = y in one workgroup, a column per thread (n <= 1024), the columns' running
// right-hand side in registers: per diagonal block its 32 values meet in LDS, x_k,
// then every earlier column loses its part.  The block's rows of L are loaded ahead of
// that chain and stay in flight across its barriers.
__global__ __launch_bounds__(1024) void k_chol_back(const double* __restrict__ L, int n, long ld,
                                                    const double* __restrict__ Yinv,
                                                    const double* __restrict__ y,
                                                    double* __restrict__ x) {
    __shared__ double Yk[2][CH_NB][CH_NB + 1];
    __shared__ double sk[CH_NB], xk[CH_NB];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nblk = (n + CH_NB - 1) / CH_NB;
    double s = tid < n ? y[tid] : 0.0;
    double yn = Yinv[(size_t)(nblk - 1) * CH_NB * CH_NB + tid];
    for (int kb = nblk - 1; kb >= 0; --kb) {
        const int k0 = kb * CH_NB;
        Yk[kb & 1][tid >> 5][tid & 31] = yn;  // (waits for it before the loads below)
        double l[CH_NB];
        const double* Lk = L + (long)k0 * ld;
        const int last = n - 1 - k0;  // (rows past n repeat the last one; their x is 0)
        const unsigned i = (unsigned)min(tid, n - 1);
        if (64 * wave < k0) {  // (the wave has earlier columns)
#pragma unroll
            for (int m = 0; m < CH_NB; ++m) l[m] = (Lk + (long)min(m, last) * ld)[i];
        }
        yn = Yinv[(size_t)max(kb - 1, 0) * CH_NB * CH_NB + tid];
        if (tid >= k0 && tid < k0 + CH_NB) sk[tid - k0] = s;  // (zero past n)
        lds_barrier();
        chol_back_block(Yk[kb & 1], sk, xk);
        if (tid < CH_NB && k0 + tid < n) x[k0 + tid] = xk[tid];
        lds_barrier();
        if (tid < k0) {
            double a[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int m = 0; m < CH_NB; ++m) a[m & 3] = fma(l[m], xk[m], a[m & 3]);
            s -= (a[0] + a[1]) + (a[2] + a[3]);
        }
    }
}

// The same, one diagonal block per launch: every block forms x_k for itself, the
// first one stores it, and each takes its part out of its own 256 columns of y.
__global__ __launch_bounds__(256) void k_chol_back_step(const double* __restrict__ L, int n,
                                                        long ld, int k0,
                                                        const double* __restrict__ Yinv,
                                                        double* __restrict__ y,
                                                        double* __restrict__ x) {
    __shared__ double Yk[CH_NB][CH_NB + 1];
    __shared__ double sk[CH_NB], xk[CH_NB];
    const int tid = threadIdx.x;
    const int i = blockIdx.x * 256 + tid;
    double l[CH_NB];
    if (i < k0) {
#pragma unroll
        for (int m = 0; m < CH_NB; ++m) l[m] = L[(long)min(k0 + m, n - 1) * ld + i];
    }
    for (int e = tid; e < CH_NB * CH_NB; e += 256)
        Yk[e / CH_NB][e % CH_NB] = Yinv[(size_t)(k0 / CH_NB) * CH_NB * CH_NB + e];
    if (tid < CH_NB) sk[tid] = k0 + tid < n ? y[k0 + tid] : 0.0;
    __syncthreads();
    chol_back_block(Yk, sk, xk);
    if (blockIdx.x == 0 && tid < CH_NB && k0 + tid < n) x[k0 + tid] = xk[tid];
    __syncthreads();
    if (i < k0) {
        double a[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int m = 0; m < CH_NB; ++m) a[m & 3] = fma(l[m], xk[m], a[m & 3]);
        y[i] -= (a[0] + a[1]) + (a[2] + a[3]);
    }
}

// CG scalars of a direct solve: no iterations, converged, zero residual (the
// solve is exact up to rounding), bad when a pivot was not positive
__global__ void k_chol_status(const int32_t* __restrict__ bad, CgScalars* sc) {
    if (threadIdx.x) return;
    sc->iters = 0;
    sc->rr = 0.0;
    sc->rr0 = 1.0;
    sc->tol2 = 0.0;
    sc->done = 1;
    sc->bad = *bad ? 1 : 0;
}

// ---------------------------------------------------------------------------
size_t chol_side_bytes(int n) { return (size_t)((n + CH_NB - 1) / CH_NB) * CH_NB * CH_NB * 8; }
__global__ void k_copy_vec(const double* __restrict__ a, double* __restrict__ b, int n) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e < n) b[e] = a[e];
}

void launch_chol_solve(hipStream_t st, double* A, int n, long ld, double shift, const double* f,
                       double* x, int32_t* bad, double* Yinv, double* y, CgScalars* sc) {
    launch_zero(st, bad, sizeof(int32_t));
    // x holds the right-hand side as the panels eliminate it (L y = f), y gets y
    k_copy_vec<<<(n + 255) / 256, 256, 0, st>>>(f, x, n);
    // (tiles of 32: shorter steps, but every block factors the panel's block again:
    // up to 2,048 only)
    const int T = n <= 2048 ? 32 : 64;
    for (int k0 = 0; k0 < n; k0 += CH_NB) {
        const int below = n - k0 - CH_NB;
        const int mt = below > 0 ? (below + T - 1) / T : 1, nb = mt * (mt + 1) / 2;
        if (T == 32)
            k_chol_step<32><<<nb, 256, 0, st>>>(A, n, ld, k0, shift, bad, Yinv, x, y);
        else
            k_chol_step<64><<<nb, 256, 0, st>>>(A, n, ld, k0, shift, bad, Yinv, x, y);
    }
    const int nblk = (n + CH_NB - 1) / CH_NB;
    if (nblk > 1)
        k_chol_mirror<<<(unsigned)((long)nblk * (nblk - 1) / 2), 256, 0, st>>>(A, n, ld);
    // (n = 880: 72 us in one workgroup, 28 launches of 4.4 otherwise; past 1,024 the rows of
    // L no longer fit the workgroup's registers: whole SR solves at n = 1,056 841 us with
    // two columns a thread, 782 in launches; 1,456: 1,276, 1,118; 1,982: 2,133, 1,794)
    if (n <= 1024) {
        k_chol_back<<<1, 1024, 0, st>>>(A, n, ld, Yinv, y, x);
    } else {
        for (int k0 = (nblk - 1) * CH_NB; k0 >= 0; k0 -= CH_NB)
            k_chol_back_step<<<k0 > 0 ? (k0 + 255) / 256 : 1, 256, 0, st>>>(A, n, ld, k0, Yinv, y,
                                                                            x);
    }
    k_chol_status<<<1, 64, 0, st>>>(bad, sc);
}

}  // namespace nqs
