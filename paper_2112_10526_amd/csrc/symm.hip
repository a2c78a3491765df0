// Symmetric RBM (paper: table of models, RBMSymm; symmetric-RBM equation of the
// symmetric NQS section): alpha features over a permutation group G of sites,
//   ln psi(s) = a sum_k s_k + sum_{i < alpha, g in G} ln cosh f_g^(i)(s),
//   f_g^(i)(s) = b_i + sum_k W_i[k] s[perm_g[k]].
// The model is held as its symmetric parameters psym = [a | b (alpha) | W (alpha x N)]
// (biases as flagged) and expanded, whenever they change, into the equal plain
// RBM with M = alpha |G| hidden units: hidden unit j = i |G| + g has the weights
// W_i scattered by perm_g (W[j][perm_g[k]] = W_i[k]), the bias b_i, and every
// visible bias is a.  Its tables then drive the sampler, theta and the local
// energies unchanged, in every precision form.  Derivatives with respect to psym
// are sums over the group of the plain ones (chain rule through the expansion):
//   O_a = sum_k s_k,  O_{b_i} = sum_g t_{i|G|+g},
//   O_{W_i[k]} = sum_g t_{i|G|+g} s[perm_g[k]],   t = tanh theta.
#include "kernels.h"

namespace nqs {

// psym -> the plain RBM's packed parameters [a (N) | b (M) | W (M x N)]
__global__ void k_symm_expand(int N, int G, int alpha, int vb, int hb,
                              const int32_t* __restrict__ perms, const double* __restrict__ psym,
                              double* __restrict__ out) {
    const long M = (long)alpha * G;
    const long e = (long)blockIdx.x * 256 + threadIdx.x;
    const long ofs_b = vb ? N : 0, ofs_w = ofs_b + (hb ? M : 0);
    const double* b = psym + (vb ? 1 : 0);
    const double* W = b + (hb ? alpha : 0);
    if (e < M * N) {  // (j, k): every k of row j is hit once (perm_g is a bijection)
        const long j = e / N;
        const int k = (int)(e - j * N);
        const int i = (int)(j / G), g = (int)(j - (long)i * G);
        out[ofs_w + j * N + perms[(long)g * N + k]] = W[(long)i * N + k];
    }
    if (vb && e < N) out[e] = psym[0];
    if (hb && e < M) out[ofs_b + e] = b[e / G];
}

// the plain force (augmented layout [Ma][Na]: row j < M = (dW_j., db_j), row M =
// da) -> the symmetric one: one wave per parameter, the group's terms over its lanes
// (one thread per parameter walked the group serially: 66 us for 203 parameters
// over 100 translations, now 3)
__global__ __launch_bounds__(256) void k_symm_tie(int N, int G, int alpha, int vb, int hb, int Na,
                                                  const int32_t* __restrict__ perms,
                                                  const double* __restrict__ grad,
                                                  double* __restrict__ out) {
    const int M = alpha * G;
    const int nb = vb ? 1 : 0, nh = hb ? alpha : 0;
    const int P = nb + nh + alpha * N;
    const int lane = threadIdx.x & 63;
    const int e = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (e >= P) return;
    double v = 0.0;
    if (e < nb) {
        for (int k = lane; k < N; k += 64) v += grad[(size_t)M * Na + k];
    } else if (e < nb + nh) {
        const int i = e - nb;
        for (int g = lane; g < G; g += 64) v += grad[(size_t)(i * G + g) * Na + N];
    } else {
        const int q = e - nb - nh, i = q / N, k = q - i * N;
        for (int g = lane; g < G; g += 64)
            v += grad[(size_t)(i * G + g) * Na + perms[(size_t)g * N + k]];
    }
    v = wave_sum(v);
    if (lane == 0) out[e] = v;
}

// O[r][p] = d ln psi(s_r) / d psym_p (FP64; columns P .. ld - 1 zero).  A block takes
// SJ_R rows, their spins (a byte each in one word per site) and activations (FP64,
// the rows side by side) in LDS; a wave takes 128 sites, two per lane, and all
// features: per group element and site one index and one word of spins, converted
// once for all features, and each activation read once for both sites.
// Bound by vector issue and LDS reads: 16,384 rows of 203 columns over 100
// translations in 59 us, against 116 us for one thread per column and row.
constexpr int SJ_R = 4;   // rows per block
constexpr int SJ_A = 2;   // features at a time
template <typename T>
__global__ __launch_bounds__(256) void k_symm_jacobian(int N, int G, int alpha, int vb, int hb,
                                                       int Mw, const int32_t* __restrict__ perms,
                                                       const int8_t* __restrict__ s,
                                                       const T* __restrict__ t, long n, long ld,
                                                       double* __restrict__ O) {
    extern __shared__ __align__(16) char sj_lds[];
    const int M = alpha * G;
    double* ta = (double*)sj_lds;                 // [M][SJ_R]
    uint32_t* sj = (uint32_t*)(ta + SJ_R * M);    // [N]
    const long r0 = (long)blockIdx.x * SJ_R;
    const int lane = threadIdx.x & 63, nth = blockDim.x, nw = nth >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nr = (int)min((long)SJ_R, n - r0);
    for (int k = threadIdx.x; k < N; k += nth) {
        uint32_t v = 0;
#pragma unroll
        for (int r = 0; r < SJ_R; ++r)
            v |= (uint32_t)(uint8_t)s[(r0 + min(r, nr - 1)) * N + k] << (8 * r);
        sj[k] = v;
    }
    for (int j = threadIdx.x; j < M; j += nth) {
        double v[SJ_R];
#pragma unroll
        for (int r = 0; r < SJ_R; ++r) v[r] = (double)t[(r0 + min(r, nr - 1)) * Mw + j];
        *(double2*)(ta + SJ_R * j) = make_double2(v[0], v[1]);
        *(double2*)(ta + SJ_R * j + 2) = make_double2(v[2], v[3]);
    }
    __syncthreads();
    const int nb = vb ? 1 : 0, nh = hb ? alpha : 0;
    const int P = nb + nh + alpha * N;
    for (int c = wave; 128 * c < N; c += nw) {
        int k[2], kk[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            k[h] = 128 * c + 64 * h + lane;
            kk[h] = min(k[h], N - 1);
        }
        for (int i0 = 0; i0 < alpha; i0 += SJ_A) {
            const double* t0 = ta + SJ_R * i0 * G;
            const double* t1 = ta + SJ_R * min(i0 + 1, alpha - 1) * G;  // (repeats the last one)
            double acc[2][SJ_A][SJ_R];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int a = 0; a < SJ_A; ++a)
#pragma unroll
                    for (int r = 0; r < SJ_R; ++r) acc[h][a][r] = 0.0;
#pragma unroll 4
            for (int g = 0; g < G; ++g) {
                double tv[SJ_A][SJ_R];
#pragma unroll
                for (int r = 0; r < SJ_R; ++r) {
                    tv[0][r] = t0[SJ_R * g + r];
                    tv[1][r] = t1[SJ_R * g + r];
                }
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint32_t w = sj[perms[g * N + kk[h]]];
#pragma unroll
                    for (int r = 0; r < SJ_R; ++r) {
                        const double sv = (double)(int8_t)(w >> (8 * r));
#pragma unroll
                        for (int a = 0; a < SJ_A; ++a) acc[h][a][r] = fma(tv[a][r], sv, acc[h][a][r]);
                    }
                }
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int a = 0; a < SJ_A; ++a)
#pragma unroll
                    for (int r = 0; r < SJ_R; ++r)
                        if (k[h] < N && i0 + a < alpha && r < nr)
                            O[(r0 + r) * ld + nb + nh + (i0 + a) * N + k[h]] = acc[h][a][r];
        }
    }
    // the bias columns (wave w: row w, w + nw, ...) and the padding
    for (int r = wave; r < nr; r += nw) {
        double* row = O + (r0 + r) * ld;
        if (vb) {
            double v = 0.0;
            for (int k = lane; k < N; k += 64) v += (double)(int8_t)(sj[k] >> (8 * r));
            v = wave_sum(v);
            if (lane == 0) row[0] = v;
        }
        for (int i = 0; i < nh; ++i) {
            double v = 0.0;
            for (int g = lane; g < G; g += 64) v += ta[SJ_R * (i * G + g) + r];
            v = wave_sum(v);
            if (lane == 0) row[nb + i] = v;
        }
        for (long p = P + lane; p < ld; p += 64) row[p] = 0.0;
    }
}

// ---------------------------------------------------------------------------
static inline unsigned nbk(long n, int b) { return (unsigned)((n + b - 1) / b); }

int symm_num_params(int N, int alpha, int vb, int hb) {
    return (vb ? 1 : 0) + (hb ? alpha : 0) + alpha * N;
}
void launch_symm_expand(hipStream_t st, int N, int G, int alpha, int vb, int hb,
                        const int32_t* perms, const double* psym, double* out) {
    const long M = (long)alpha * G;
    const long n = M * N > M ? M * N : M;
    k_symm_expand<<<nbk(n > N ? n : N, 256), 256, 0, st>>>(N, G, alpha, vb, hb, perms, psym, out);
}
void launch_symm_tie(hipStream_t st, int N, int G, int alpha, int vb, int hb, int Na,
                     const int32_t* perms, const double* grad, double* out) {
    k_symm_tie<<<nbk(symm_num_params(N, alpha, vb, hb), 4), 256, 0, st>>>(N, G, alpha, vb, hb,
                                                                           Na, perms, grad, out);
}
void launch_symm_jacobian(hipStream_t st, int prec, int N, int G, int alpha, int vb, int hb,
                          int Mw, const int32_t* perms, const int8_t* s, const void* t, long n,
                          long ld, double* O) {
    if (n <= 0) return;
    // a wave per 128 sites, at most four
    const int nw = N > 384 ? 4 : (N + 127) / 128;
    const unsigned nb = nbk(n, SJ_R);
    const size_t lds = 8 * (size_t)SJ_R * alpha * G + 4 * (size_t)N;
    const void* k = prec == 0 ? (const void*)k_symm_jacobian<double>
                              : (const void*)k_symm_jacobian<float>;
    if (lds > 65536)
        (void)hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (prec == 0)
        k_symm_jacobian<double><<<nb, 64 * nw, lds, st>>>(N, G, alpha, vb, hb, Mw, perms, s,
                                                            (const double*)t, n, ld, O);
    else
        k_symm_jacobian<float><<<nb, 64 * nw, lds, st>>>(N, G, alpha, vb, hb, Mw, perms, s,
                                                           (const float*)t, n, ld, O);
}

}  // namespace nqs
