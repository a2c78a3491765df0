// Sums over a batch of the log-derivatives' outer products,
//   out = sum_k g_k t~_k (x) s~_k     (an [Ma][Na] matrix, common.h),
// straight from the caller's sample order: with the weights g of a backward
// pass it is the vector-Jacobian product of ln psi (paper, appendix on
// Jacobians and their products), without weights the column sums of the
// Jacobian that centre it.  Accumulated in A on the matrix cores (A = R for the
// vector-Jacobian product; FP64 for the column sums whatever R).
#include "kernels.h"

#include <algorithm>
#include <type_traits>

namespace nqs {

// Block (x, y, z): hidden tiles 4 x .. 4 x + 3 (one per wave), row slice y, site
// tiles PT z .. PT z + PT - 1.  The operand t~ g goes from global memory straight to
// the wave that multiplies it (each value is used by one wave; 16 neighbours per
// row), four 16-sample units ahead; the spins, which every wave of the block needs
// transposed, are staged in LDS for up to TS_K samples at a time ([site][sample]
// bytes).  Within a unit, k-step e of lane quad lk takes sample 4 e + lk.
// Column sums of 4,000 x (64 sites, 512 hidden units), FP32 rows: 22 us (360 blocks,
// 8 slices: what the slot buffer of that batch holds); 16,384 rows: 58 us, against
// 150 us for one thread per column and slice.  FP64 vector-Jacobian product of
// 16,384 x (100 sites, 200 hidden units): 29 us, against 92 us with t~ g staged in
// LDS and bytes read one at a time.
constexpr int TS_K = 256;             // samples per stage
constexpr int TS_LW = TS_K / 4 + 4;   // LDS words per site row (16-byte reads, spread banks)
constexpr int TS_NW = 4;              // waves (hidden tiles) per block

template <typename R, typename A, bool G, int PT>
__global__ __launch_bounds__(64 * TS_NW) void k_tts(Dims d, const int8_t* __restrict__ s,
                                                    int words, const R* __restrict__ tact, long n,
                                                    const R* __restrict__ g, long rps,
                                                    A* __restrict__ part) {
    constexpr int NT = 64 * TS_NW, SITES = 16 * PT;
    __shared__ __align__(16) uint32_t Ls[(SITES + 1) * TS_LW];  // (the last row takes what is not a site)
    typedef typename std::conditional<sizeof(A) == 8, v4d, v4f>::type acc_t;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lk = lane >> 4;
    const int t0 = blockIdx.z * PT, i0 = 16 * t0;
    const int nt = min(PT, d.Na / 16 - t0);  // tiles of this block
    const long r0 = (long)blockIdx.y * rps, r1 = min(n, r0 + rps);
    const int jt = blockIdx.x * TS_NW + wave;
    const bool live = jt * 16 < d.Ma;
    const R* tj = tact + (live ? jt * 16 : 0) + lr;
    const int sites = min(d.N - i0, SITES);  // lattice sites of these tiles (may be <= 0)
    // the constant row N (1) and the padding rows (0)
    for (int e = max(sites, 0) * TS_LW + tid; e < SITES * TS_LW; e += NT)
        Ls[e] = i0 + e / TS_LW == d.N ? 0x01010101u : 0u;
    struct Raw {
        R t[4], g[4];
    };
    // samples k0 + 4 e + lk, loads only: a uniform base plus a lane offset, except
    // at the batch's end (rows past it repeat the last one)
    unsigned off[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) off[e] = (unsigned)((4 * e + lk) * d.Mw);
    auto fetch = [&](long k0, Raw& x) {
        if (k0 + 16 <= n) {
            const R* b = tj + k0 * d.Mw;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                x.t[e] = b[off[e]];
                if constexpr (G) x.g[e] = (g + k0)[4 * e + lk];
            }
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const long k = min(k0 + 4 * e + lk, n - 1);
                x.t[e] = tj[k * d.Mw];
                if constexpr (G) x.g[e] = g[k];
            }
        }
    };
    acc_t acc[PT];
#pragma unroll
    for (int p = 0; p < PT; ++p) acc[p] = acc_t{0, 0, 0, 0};
    auto unit = [&](long k0, int kl, const Raw& x) {
        uint4 w[PT];
#pragma unroll
        for (int p = 0; p < PT; ++p) w[p] = *(const uint4*)&Ls[(16 * p + lr) * TS_LW + kl / 4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            R v = x.t[e];
            if constexpr (G) v *= x.g[e];
            A a = (A)v;
            if (k0 + 16 > r1 && k0 + 4 * e + lk >= r1) a = (A)0;  // (past the slice)
#pragma unroll
            for (int p = 0; p < PT; ++p) {
                const uint32_t x = e == 0 ? w[p].x : e == 1 ? w[p].y : e == 2 ? w[p].z : w[p].w;
                const A b = (A)(int)__builtin_amdgcn_sbfe((int)x, 8 * lk, 8);
                if constexpr (sizeof(A) == 8)
                    acc[p] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[p], 0, 0, 0);
                else
                    acc[p] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc[p], 0, 0, 0);
            }
        }
    };
    for (long ks = r0; ks < r1; ks += TS_K) {
        const int rows = (int)min((long)TS_K, r1 - ks);
        Raw x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) fetch(ks + 16 * u, x[u]);
        __syncthreads();  // the previous stage is no longer read
        if (sites > 0) {
            const int W = (sites + 3) / 4, items = rows * W;
            // four words per thread and step (items past the end repeat the last one)
            auto stage = [&](auto word) {
#pragma unroll 1
                for (int e0 = tid; e0 < items; e0 += 4 * NT) {
                    uint32_t v[4];
                    int row[4], i[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int e = min(e0 + u * NT, items - 1);
                        row[u] = e / W;
                        i[u] = 4 * (e - row[u] * W);
                        v[u] = word(s + (ks + row[u]) * d.N + i0 + i[u], sites - 1 - i[u]);
                    }
                    int8_t* b = (int8_t*)Ls;
#pragma unroll
                    for (int u = 0; u < 4; ++u)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const int il = i[u] + q < sites ? i[u] + q : SITES;
                            b[il * (4 * TS_LW) + row[u]] = (int8_t)(v[u] >> (8 * q));
                        }
                }
            };
            if (words)  // rows of whole aligned words
                stage([](const int8_t* p, int) { return *(const uint32_t*)p; });
            else  // (m: the last of the word's bytes that lies in the row)
                stage([](const int8_t* p, int m) {
                    const uint8_t* q = (const uint8_t*)p;
                    return (uint32_t)q[0] | (uint32_t)q[min(1, m)] << 8 |
                           (uint32_t)q[min(2, m)] << 16 | (uint32_t)q[min(3, m)] << 24;
                });
        }
        __syncthreads();
        if (!live) continue;
#pragma unroll 1
        for (int kl = 0; kl < rows; kl += 64) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                unit(ks + kl + 16 * u, kl + 16 * u, x[u]);
                fetch(ks + kl + 64 + 16 * u, x[u]);
                __builtin_amdgcn_sched_barrier(0);  // (loads ahead of the next unit's products)
            }
        }
    }
    if (!live) return;
    A* out = part + (size_t)blockIdx.y * d.Ma * d.Na;
#pragma unroll
    for (int p = 0; p < PT; ++p)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (p < nt) out[(size_t)(jt * 16 + acc_row<A>(lk, q)) * d.Na + i0 + 16 * p + lr] = acc[p][q];
}

// out[p] (packed parameter order) = sum of the slices in a fixed order, on top
// of acc (kept in the [Ma][Na] layout between the parts of a long batch).  A
// block covers 64 entries; wave w sums the slices [w S / 4, (w + 1) S / 4).
template <typename A, typename O>
__global__ __launch_bounds__(256) void k_tts_reduce(Dims d, const A* __restrict__ part, int S,
                                                    double* __restrict__ acc, int first, int last,
                                                    O* __restrict__ out) {
    __shared__ double ws[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int total = d.Ma * d.Na;
    const int e = blockIdx.x * 64 + lane;  // (total is a multiple of 256)
    const int b0 = wave * S / 4, b1 = (wave + 1) * S / 4;
    double v = 0.0;
    for (int b = b0; b < b1; b += 8) {
        A x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = part[(size_t)min(b + u, S - 1) * total + e];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (b + u < b1) v += (double)x[u];
    }
    ws[wave][lane] = v;
    __syncthreads();
    if (wave != 0) return;
    v = (ws[0][lane] + ws[1][lane]) + (ws[2][lane] + ws[3][lane]);
    if (!first) v += acc[e];
    if (!last) {
        acc[e] = v;
        return;
    }
    const int j = e / d.Na, i = e - j * d.Na;
    const long ob = d.vb ? d.N : 0, ow = ob + (d.hb ? d.M : 0);
    long p = -1;
    if (j < d.M && i < d.N) p = ow + (long)j * d.N + i;
    else if (d.hb && j < d.M && i == d.N) p = ob + j;
    else if (d.vb && j == d.M && i < d.N) p = i;
    if (p >= 0) out[p] = (O)v;
}

template <typename R, typename A, bool G>
static int tts(hipStream_t st, const Dims& d, const int8_t* s, const void* tact, long n,
               const void* g, void* part, size_t part_bytes, int ncu) {
    // row slices: FP32 sums of 256 rows (the slices are added in FP64); FP64 sums as
    // many as the scratch holds, at most two blocks per compute unit at one site
    // pass, at least 64 rows.  Then as many passes over the site tiles (each reads
    // its t~ again) as two blocks per compute unit take.
    const int nx = (d.Ma / 16 + TS_NW - 1) / TS_NW, ni = d.Na / 16;
    const long fit = (long)(part_bytes / (sizeof(A) * (size_t)d.Ma * d.Na));
    const long want = std::max(1L, std::min({2L * ncu / nx, fit, (n + 63) / 64}));
    const long rps = sizeof(A) == 4 ? 256 : ((n + want - 1) / want + 63) / 64 * 64;
    const int S = (int)((n + rps - 1) / rps);
    int np = (ni + 7) / 8;
    while (np < ni && (long)nx * S * np < 2L * ncu) ++np;
    const int pt = (ni + np - 1) / np;
    const int words = d.N % 4 == 0 && ((uintptr_t)s & 3) == 0;
    const dim3 grid((unsigned)nx, (unsigned)S, (unsigned)((ni + pt - 1) / pt));
#define TTS_CASE(PT)                                                                             \
    case PT:                                                                                     \
        k_tts<R, A, G, PT><<<grid, 64 * TS_NW, 0, st>>>(d, s, words, (const R*)tact, n,          \
                                                        (const R*)g, rps, (A*)part);             \
        break
    switch (pt) {
        TTS_CASE(1);
        TTS_CASE(2);
        TTS_CASE(3);
        TTS_CASE(4);
        TTS_CASE(5);
        TTS_CASE(6);
        TTS_CASE(7);
        TTS_CASE(8);
    }
#undef TTS_CASE
    return S;
}

void launch_colsum(hipStream_t st, const Dims& d, int prec, const int8_t* s, const void* tact,
                   long n, void* part, size_t part_bytes, int ncu, double* acc, bool first,
                   bool last, double* out) {
    const int S = prec == 0
                      ? tts<double, double, false>(st, d, s, tact, n, nullptr, part, part_bytes, ncu)
                      : tts<float, double, false>(st, d, s, tact, n, nullptr, part, part_bytes, ncu);
    k_tts_reduce<double, double><<<d.Ma * d.Na / 64, 256, 0, st>>>(d, (const double*)part, S, acc,
                                                                   first, last, out);
}

void launch_vjp(hipStream_t st, const Dims& d, int prec, const int8_t* s, const void* tact, long n,
                const void* g, void* part, size_t part_bytes, int ncu, double* acc, bool first,
                bool last, void* out) {
    const int nb = d.Ma * d.Na / 64;
    if (prec == 0) {
        const int S = tts<double, double, true>(st, d, s, tact, n, g, part, part_bytes, ncu);
        k_tts_reduce<double, double><<<nb, 256, 0, st>>>(d, (const double*)part, S, acc, first,
                                                         last, (double*)out);
    } else {
        const int S = tts<float, float, true>(st, d, s, tact, n, g, part, part_bytes, ncu);
        k_tts_reduce<float, float><<<nb, 256, 0, st>>>(d, (const float*)part, S, acc, first, last,
                                                       (float*)out);
    }
}

}  // namespace nqs
