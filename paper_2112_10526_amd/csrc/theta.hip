// Hidden pre-activations theta = W s + b on MFMA, with tanh in the epilogue,
// and ln psi(s).
//
// The contraction Theta[r][j] = sum_i s~[r][i] W~^T[i][j] (s~ augmented with a
// 1 at i = N so that row N of W~^T adds b) runs on CDNA4 matrix cores:
//   FP64 path: v_mfma_f64_16x16x4f64,
//   FP32 path: v_mfma_f32_16x16x4f32,
//   BF16 form: v_mfma_f32_16x16x32_bf16 twice (W = W_hi + W_lo, both BF16,
//              spins exact), FP32 accumulation.
// Operand lane layouts (16x16 tiles, 64 lanes): A[row = lane % 16][k = lane / 16]
// (BF16: k = 8 * (lane / 16) + e), B[k][col = lane % 16]; accumulator slot i
// of lane l holds D[acc_row(l / 16, i)][l % 16] (see common.h).
#include "kernels.h"

#include <type_traits>

namespace nqs {

// e^{-y} = 2^k e^r for y in [0, 44]: a two-term (Cody-Waite) reduction by ln 2, with what
// rounding takes off r as rl, and c of e^r - 1 = r + r^2 / 2 + r^3 c by its Taylor
// polynomial (|r| <= ln 2 / 2, degree 13: the remainder is below 2^-56 of the result).
struct ExpRed {
    double r, rl, c;
    int k;
};
__device__ __forceinline__ ExpRed exp_red(double y) {
    const double k = rint(-y * 1.4426950408889634074);
    const double r0 = fma(-k, 0.6931471805601177, -y);      // ln 2 to 40 bits (exact)
    const double r = fma(-k, -1.7239444525614835e-13, r0);  // the rest of ln 2
    double p = 1.0 / 6227020800.0;
    p = fma(p, r, 1.0 / 479001600.0);
    p = fma(p, r, 1.0 / 39916800.0);
    p = fma(p, r, 1.0 / 3628800.0);
    p = fma(p, r, 1.0 / 362880.0);
    p = fma(p, r, 1.0 / 40320.0);
    p = fma(p, r, 1.0 / 5040.0);
    p = fma(p, r, 1.0 / 720.0);
    p = fma(p, r, 1.0 / 120.0);
    p = fma(p, r, 1.0 / 24.0);
    p = fma(p, r, 1.0 / 6.0);
    return ExpRed{r, fma(-k, -1.7239444525614835e-13, r0 - r), p, (int)k};
}
// e^{-y} as its FP64 value `e` and as `m` = e^{-y} - 1, each with its own relative accuracy
struct ExpNeg {
    double e, m;
};
__device__ __forceinline__ ExpNeg exp_neg(double y) {
    const ExpRed x = exp_red(y);
    const double p = fma(fma(x.c, x.r, 0.5) * x.r, x.r, x.r);  // e^r - 1
    const double s = ldexp(1.0, x.k);
    return ExpNeg{fma(s, p, s), fma(s, p, s - 1.0)};
}
__device__ __forceinline__ double recip64(double x) {
    double y = __builtin_amdgcn_rcp(x);
    y = fma(fma(-x, y, 1.0), y, y);
    return fma(fma(-x, y, 1.0), y, y);
}
// tanh|x| = -m / (2 + m), m = e^{-2|x|} - 1 (1 past |x| = 22).  m and 2 + m are carried
// as sums of two numbers, so that the quotient's is the only full rounding: at most 0.7
// units in the last place, 0.29 rms (0.84 and 0.32 for the library's; m and 2 + m rounded
// to one number each: 2.5 and 0.93).
__device__ __forceinline__ double tanh64(double x) {
    const double a = fabs(x);
    const ExpRed g = exp_red(2.0 * (a > 22.0 ? 22.0 : a));
    const double h = 0.5 * g.r, q2 = h * g.r;  // e^r - 1 = hi + lo
    double hi = g.r + q2, lo = q2 - (hi - g.r);
    lo += fma(2.0 * q2 * g.r, g.c, fma(h, g.r, -q2) + g.rl);
    const double t = hi + lo;
    lo -= t - hi;
    hi = t;
    const double s = ldexp(1.0, g.k), u = s * hi, v = s - 1.0;
    const double m = v + u;  // (|v| >= |u|, or v = 0)
    const double ml = fma(s, lo, (u - (m - v)) + (s - (v + 1.0)));
    const double d = 2.0 + m, dl = (m - (d - 2.0)) + ml;
    double y = __builtin_amdgcn_rcp(d);
    y = fma(fma(-d, y, 1.0), y, y);
    const double q = -m * y;
    return copysign(fma(fma(-d, q, -m) - fma(dl, q, ml), y, q), x);
}
// cosh x - 1 = m^2 / (2 e^{-|x|}), m = e^{-|x|} - 1, for |x| <= 22 (larger: its value at 22)
__device__ __forceinline__ double coshm1(double a) {
    const ExpNeg x = exp_neg(a > 22.0 ? 22.0 : a);
    return x.m * x.m * (0.5 * recip64(x.e));
}
__device__ __forceinline__ double act(double th, int col, int M) {
    const double t = tanh64(th);  // (no branch around it)
    return col < M ? t : (col == M ? 1.0 : 0.0);
}
__device__ __forceinline__ float act(float th, int col, int M) {
    return col < M ? tanhf(th) : (col == M ? 1.0f : 0.0f);
}

// FP64 and FP32 paths.  A wave keeps the W~^T fragments of its 16 hidden columns
// in registers (G groups of 16 sites) and walks the block's rows, RT 16-row tiles
// at a time, so W is read once per block and wave and each MFMA takes one bit-field
// extract and one conversion of spins staged in LDS ([row][site] bytes, rows an odd
// number of 16-byte pieces apart: a fragment read hits distinct banks).  The
// accumulation over sites is one chain in site order.  EPI 0 (k_theta): a block
// covers 64 columns, tanh in the epilogue; EPI 1 (ln psi): a block covers all
// columns, its waves taking tiles w, w + nw, ..., and sums ln cosh over them: the
// factors cosh x are multiplied over 16 columns before one logarithm.  G is
// exact (no test inside the products: with one, the compiler moved every
// accumulator between register files around each MFMA), past 8 groups the next of 10,
// 12, 14 and 17 with zero weights; MULTI: wider lattices walk the sites in chunks of G
// groups for all rows of a block, W reloaded for each.
// 16,384 x (100 sites, 200 hidden units) FP64, 0.76 GFLOP (12 us at the FP64 matrix
// rate): theta 62 -> 37 us against staging W in LDS for every 64 x 64 tile with the
// library tanh, ln psi 289 -> 40 us against a vector dot product per hidden unit.
// 16,384 x (256 sites, 1,024 hidden units): theta FP64 492 -> 296, FP32 200 -> 150 us
// (409 and 314 in chunks of 8 groups), ln psi 2,886 -> 352 and 1,027 -> 248.
// What is left is vector issue: conversions, tanh and the drain of 512 blocks.  The
// FP64 ln psi forms of 14 and 17 groups keep 28 to 90 of their registers in scratch.
constexpr int TH_ST = 8;  // staging words per thread and step

// (1 + f) multiplied over the 16 lanes of a DPP row, less 1
__device__ __forceinline__ double row16_prod1(double f) {
    auto mul = [](double a, double b) { return fma(a, b, a + b); };
    f = mul(f, dpp<0xB1>(f));
    f = mul(f, dpp<0x4E>(f));
    f = mul(f, dpp<0x124>(f));
    return mul(f, dpp<0x128>(f));
}

// Spins i0 .. i0 + 4 W - 1 of the block's rows into LDS (row stride LD bytes),
// augmented (1 at site N, then 0); eight words per thread loaded together (items past
// the end repeat the last one).  Rows start at any byte: the words are loaded as they
// lie (the row's last one from its last four bytes, shifted).
template <int W>
__device__ __forceinline__ void stage_spins(int8_t* lds, int LD, const int8_t* __restrict__ s, int N,
                                            long r0, int nr, int RB, int i0, int tid, int nth) {
    const int items = RB * W;
    auto fill = [&](auto word, auto finish) {
#pragma unroll 1
        for (int e0 = tid; e0 < items; e0 += TH_ST * nth) {
            uint32_t v[TH_ST];
            int at[TH_ST], i[TH_ST];
#pragma unroll
            for (int u = 0; u < TH_ST; ++u) {
                const int e = min(e0 + u * nth, items - 1);
                const int row = e / W, q = 4 * (e - row * W);
                at[u] = row * LD + q;
                i[u] = i0 + q;
                v[u] = word(s + (r0 + min(row, nr - 1)) * N, i[u]);
            }
#pragma unroll
            for (int u = 0; u < TH_ST; ++u) *(uint32_t*)(lds + at[u]) = finish(v[u], i[u]);
        }
    };
    auto load = [&](const int8_t* p, int i) {
        uint32_t v;
        __builtin_memcpy(&v, p + min(i, N - 4), 4);
        return v;
    };
    auto augment = [&](uint32_t v, int i) {
        return i <= N && N < i + 4 ? v | 1u << (8 * (N - i)) : v;
    };
    if (N % 4 == 0)  // (a word is all spins or all constants)
        fill(load, [&](uint32_t v, int i) { return i < N ? v : (i == N ? 1u : 0u); });
    else if (N >= 4)
        fill(load, [&](uint32_t v, int i) {
            return augment(i < N ? v >> (8 * max(i - (N - 4), 0)) : 0u, i);
        });
    else
        fill([&](const int8_t* p, int i) {
                uint32_t v = 0;
                if (i == 0)
                    for (int q = 0; q < N; ++q) v |= (uint32_t)(uint8_t)p[q] << (8 * q);
                return v;
            }, augment);
}

template <typename R, int G, int RT, int EPI, bool MULTI>
__global__ __launch_bounds__(EPI ? 512 : 256) void k_theta(
    Dims d, const int8_t* __restrict__ s, long rows, int RB, const R* __restrict__ Wa,
    R* __restrict__ dst1, R* __restrict__ dst2, long dst2_stride, const double* __restrict__ av) {
    extern __shared__ __align__(16) int8_t th_lds[];
    typedef typename std::conditional<sizeof(R) == 8, v4d, v4f>::type acc_t;
    constexpr int LD = 16 * (G | 1);  // LDS row stride
    const int tid = threadIdx.x, lane = tid & 63, nth = blockDim.x, nw = nth >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lk = lane >> 4;
    const long r0 = (long)blockIdx.x * RB;
    const int nr = (int)min((long)RB, rows - r0);  // rows of this block
    const int ng = d.Na / 16;
    const int nch = MULTI ? (ng + G - 1) / G : 1;  // site chunks
    double* red = (double*)(th_lds + (size_t)RB * LD);  // EPI 1: [nw][RB]
    auto stage = [&](int c) {
        stage_spins<4 * G>(th_lds, LD, s, d.N, r0, nr, RB, 16 * G * c, tid, nth);
    };
    const int tiles = EPI ? (d.M + 15) / 16 : d.Mw / 16;
    R wf[4 * G];
    auto load_w = [&](int tile, int c) {  // (tiles past the last one repeat it)
        const R* w = Wa + 16 * min(tile, tiles - 1) + lr;
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = 16 * (c * G + g) + 4 * e + lk;
                if constexpr (MULTI || G > 8) {
                    const R v = w[(size_t)min(k, d.Na - 1) * d.Mw];
                    wf[4 * g + e] = k < d.Na ? v : (R)0;
                } else {
                    wf[4 * g + e] = w[(size_t)k * d.Mw];
                }
            }
    };
    const int tile0 = (EPI ? 0 : (int)blockIdx.y * nw) + wave;
    // ln psi of one row tile of up to 15 sites, the smallest calls: the visible part's
    // operands are loaded along with W's, 16 lanes per row (64 rows of 10 sites, 10 units:
    // kernel 4.6 -> 4.13 us; from two groups of sites on it does not pay)
    constexpr bool VIS = EPI == 1 && RT == 1 && G == 1 && !MULTI;
    double vis[4] = {0.0, 0.0, 0.0, 0.0};  // of rows 4 (wave + nw k) + lk
    if constexpr (!MULTI) {
        int8_t sv[4];
        double a = 0.0;
        if constexpr (VIS) {
            const int i = min(lr, d.N - 1);
            if (av) a = av[i];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                sv[k] = s[(r0 + min(4 * (wave + nw * k) + lk, nr - 1)) * d.N + i];
        }
        load_w(tile0, 0);
        stage(0);
        if constexpr (VIS) {
#pragma unroll
            for (int k = 0; k < 4; ++k) vis[k] = lr < d.N ? a * (double)sv[k] : 0.0;
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
    }
    const int trounds = EPI ? (tiles + nw - 1) / nw : 1;
    const int sh = 8 * lk;
    for (int q = 0; q < trounds; ++q) {
        const int tile = tile0 + q * nw;
        const bool work = tile < tiles && 16 * tile < d.M;  // (past M: constants only)
        if (!MULTI && q > 0) load_w(tile, 0);
        const int col = 16 * tile + lr;
#pragma unroll 1
        for (int rt = 0; rt < nr; rt += 16 * RT) {
            acc_t acc[RT];
#pragma unroll
            for (int u = 0; u < RT; ++u) acc[u] = acc_t{0, 0, 0, 0};
            const int8_t* row_lds = th_lds + (rt + lr) * LD;
            auto products = [&]() {
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    uint4 sp[RT];
#pragma unroll
                    for (int u = 0; u < RT; ++u)
                        sp[u] = *(const uint4*)(row_lds + 16 * u * LD + 16 * g);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int u = 0; u < RT; ++u) {
                            const uint32_t w = e == 0 ? sp[u].x : e == 1 ? sp[u].y : e == 2 ? sp[u].z : sp[u].w;
                            const R a = (R)(int)__builtin_amdgcn_sbfe((int)w, sh, 8);
                            if constexpr (sizeof(R) == 8)
                                acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, wf[4 * g + e], acc[u], 0, 0, 0);
                            else
                                acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, wf[4 * g + e], acc[u], 0, 0, 0);
                        }
                }
            };
            if constexpr (MULTI) {
                for (int c = 0; c < nch; ++c) {
                    __syncthreads();  // (the same trip counts in every wave)
                    stage(c);
                    load_w(tile, c);
                    __syncthreads();
                    products();
                }
            } else if (work) {
                products();
            }
            if constexpr (EPI == 0) {
                if (tile >= tiles) continue;
                const long b1 = (r0 + rt) * d.Mw, b2 = (r0 + rt) * dst2_stride;
#pragma unroll
                for (int u = 0; u < RT; ++u)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int row = 16 * u + acc_row<R>(lk, i);
                        const R t = work ? act(acc[u][i], col, d.M) : (R)(col == d.M ? 1 : 0);
                        if (rt + 16 * RT <= nr || rt + row < nr) {
                            (dst1 + b1)[(unsigned)(row * d.Mw + col)] = t;
                            if (dst2) (dst2 + b2)[row * dst2_stride + col] = t;
                        }
                    }
            } else if (work) {
                // each row's sum over the tile's 16 columns (lanes of a DPP row):
                // ln prod cosh with the product kept as its difference from 1, so
                // that small activations keep their relative accuracy; past |x| = 22,
                // ln cosh x = ln cosh 22 + |x| - 22
#pragma unroll
                for (int u = 0; u < RT; ++u) {
                    double f[4], big[4];
                    bool any = false;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const double x = col < d.M ? fabs((double)acc[u][i]) : 0.0;
                        f[i] = row16_prod1(coshm1(x));
                        big[i] = x > 22.0 ? x - 22.0 : 0.0;
                        any = any || !(x <= 22.0);
                    }
                    if (__any(any)) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) big[i] = row16_sum(big[i]);
                    }
                    // lane lr takes row slot lr % 4: one logarithm for the four rows
                    const int i = lr & 3;
                    const double p = i == 0 ? f[0] : i == 1 ? f[1] : i == 2 ? f[2] : f[3];
                    const double a = i == 0 ? big[0] : i == 1 ? big[1] : i == 2 ? big[2] : big[3];
                    const int row = rt + 16 * u + acc_row<R>(lk, i);
                    if (lr < 4 && row < RB) {
                        double* o = red + wave * RB + row;
                        *o = (q > 0 ? *o : 0.0) + (a + log1p(p));
                    }
                    __builtin_amdgcn_sched_barrier(0);  // one tile's values live at a time
                }
            }
        }
    }
    if constexpr (EPI == 1) {  // the waves' sums in order, and the visible part
        __syncthreads();
        // (16 lanes per row, nw <= 8; every lane stays in the loop for the row sums)
        auto row_out = [&](int rb, double v) {
            const int row = min(rb + lk, nr - 1);
            if (lr < nw) v += red[lr * RB + row];
            v = row16_sum(v);
            if (lr == 0 && rb + lk < nr) dst1[r0 + row] = (R)v;
        };
        if constexpr (VIS) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (4 * (wave + nw * k) < nr) row_out(4 * (wave + nw * k), vis[k]);
        } else {
            for (int rb = 4 * wave; rb < nr; rb += 4 * nw) {
                const int row = min(rb + lk, nr - 1);
                double v = 0.0;
                if (av)
                    for (int i = lr; i < d.N; i += 16) v += av[i] * (double)s[(r0 + row) * d.N + i];
                row_out(rb, v);
            }
        }
    }
}

typedef short v8s __attribute__((ext_vector_type(8)));

// BF16 form: eight spins (bytes, 0 past the bias site) as BF16, +1 = 0x3F80,
// -1 = 0xBF80 (0 comes out as +1: its weights are zero)
__device__ __forceinline__ v8bf spins_bf16(uint2 b) {
    uint4 v;
    v.x = (__builtin_amdgcn_perm(b.x, b.x, 0x010c000cu) & 0x80008000u) | 0x3F803F80u;
    v.y = (__builtin_amdgcn_perm(b.x, b.x, 0x030c020cu) & 0x80008000u) | 0x3F803F80u;
    v.z = (__builtin_amdgcn_perm(b.y, b.y, 0x010c000cu) & 0x80008000u) | 0x3F803F80u;
    v.w = (__builtin_amdgcn_perm(b.y, b.y, 0x030c020cu) & 0x80008000u) | 0x3F803F80u;
    return __builtin_bit_cast(v8bf, v);
}

// As k_theta, a wave keeps the weights of its 16 columns in registers (hi and lo
// planes, KS k-steps of 32 sites) and walks the block's rows, RT tiles of 16 at a time;
// the spins are staged as bytes, rows an odd number of 32-byte pieces apart.  Per
// element the accumulation order is that of one k-step at a time: + a W_hi, then
// + a W_lo.  MULTI: wider lattices in chunks of KS k-steps for all rows of the block.
// What bounds it is the vector ALU in the epilogue (tanh).  16,384 rows of 256 sites,
// 1,024 units: 61 us (157 with spins loaded byte by byte for every 64 columns); 4,096
// rows of 100 sites, 200 units: 7.0 (11).
template <int KS, int RT, bool MULTI>
__global__ __launch_bounds__(256) void k_theta_bf16(Dims d, const int8_t* __restrict__ s, long rows,
                                                    int RB,
                                                    const uint16_t* __restrict__ Whi,
                                                    const uint16_t* __restrict__ Wlo,
                                                    float* __restrict__ dst1,
                                                    float* __restrict__ dst2, long dst2_stride) {
    extern __shared__ __align__(16) int8_t th_lds[];
    constexpr int LD = 32 * (KS | 1);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lk = lane >> 4;
    const long r0 = (long)blockIdx.x * RB;
    const int nr = (int)min((long)RB, rows - r0);
    const int tiles = d.Mw / 16, tile = (int)blockIdx.y * 4 + wave;
    const int nks = d.Kb / 32, nch = MULTI ? (nks + KS - 1) / KS : 1;
    const bool work = tile < tiles && 16 * tile < d.M;  // (past M: constants only)
    const int col = 16 * tile + lr;
    v8bf wh[KS], wl[KS];
    auto load_w = [&](int c) {  // (tiles past the last one repeat it)
        const size_t o = (size_t)(16 * min(tile, tiles - 1) + lr) * d.Kb + 8 * lk;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if constexpr (MULTI) {
                const int k = c * KS + ks;
                const v8s z = {0, 0, 0, 0, 0, 0, 0, 0};
                const v8s h = *(const v8s*)(Whi + o + 32 * min(k, nks - 1));
                const v8s l = *(const v8s*)(Wlo + o + 32 * min(k, nks - 1));
                wh[ks] = __builtin_bit_cast(v8bf, k < nks ? h : z);
                wl[ks] = __builtin_bit_cast(v8bf, k < nks ? l : z);
            } else {
                wh[ks] = *(const v8bf*)(Whi + o + 32 * ks);
                wl[ks] = *(const v8bf*)(Wlo + o + 32 * ks);
            }
        }
    };
    auto stage = [&](int c) {
        stage_spins<8 * KS>(th_lds, LD, s, d.N, r0, nr, RB, 32 * KS * c, tid, 256);
    };
    if constexpr (!MULTI) {
        load_w(0);
        stage(0);
        __syncthreads();
    }
#pragma unroll 1
    for (int rt = 0; rt < nr; rt += 16 * RT) {
        v4f acc[RT];
#pragma unroll
        for (int u = 0; u < RT; ++u) acc[u] = v4f{0, 0, 0, 0};
        auto products = [&]() {
            const int8_t* row = th_lds + (rt + lr) * LD + 8 * lk;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                v8bf a[RT];
#pragma unroll
                for (int u = 0; u < RT; ++u)
                    a[u] = spins_bf16(*(const uint2*)(row + 16 * u * LD + 32 * ks));
#pragma unroll
                for (int u = 0; u < RT; ++u)
                    acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u], wh[ks], acc[u], 0, 0, 0);
#pragma unroll
                for (int u = 0; u < RT; ++u)
                    acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u], wl[ks], acc[u], 0, 0, 0);
            }
        };
        if constexpr (MULTI) {  // (one step of rows: RB = 16 RT)
            for (int c = 0; c < nch; ++c) {
                __syncthreads();
                stage(c);
                load_w(c);
                __syncthreads();
                products();
            }
        } else if (work) {
            products();
        }
        if (tile >= tiles) continue;
        const long b1 = (r0 + rt) * d.Mw, b2 = (r0 + rt) * dst2_stride;
#pragma unroll
        for (int u = 0; u < RT; ++u) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = 16 * u + acc_row<float>(lk, i);
                const float t = work ? act(acc[u][i], col, d.M) : (col == d.M ? 1.0f : 0.0f);
                if (rt + row < nr) {
                    (dst1 + b1)[(unsigned)(row * d.Mw + col)] = t;
                    if (dst2) (dst2 + b2)[row * dst2_stride + col] = t;
                }
            }
            __builtin_amdgcn_sched_barrier(0);  // one tile's values live at a time
        }
    }
}

// Rows per block: the most of 16, 32, 64, 128 that leave `target` blocks or more
// (16 rows where even those are fewer).
static int theta_rows(long rows, long nby, long target) {
    int RB = 128;
    while (RB > 16 && ((rows + RB - 1) / RB) * nby < target) RB /= 2;
    return RB;
}

template <typename R, int G, int EPI, bool MULTI>
static void theta_g(hipStream_t st, const Dims& d, const int8_t* s, long rows, const R* Wa, R* dst1,
                    R* dst2, long dst2_stride, const double* av) {
    const int tiles = EPI ? (d.M + 15) / 16 : d.Mw / 16;
    // waves of an EPI 1 block: all tiles in rounds of at most eight, as equal as they come
    const int rounds = (tiles + 7) / 8;
    const int nw = EPI ? (tiles + rounds - 1) / rounds : 4;
    const int nby = EPI ? 1 : (tiles + nw - 1) / nw;
    const int fit = theta_rows(rows, nby, 512);
    const int RB = !MULTI ? fit : (!EPI && fit >= 64) ? 64 : 32;
    const size_t lds = (size_t)RB * 16 * (G | 1) + (EPI ? 8 * (size_t)nw * RB : 0);
    const dim3 grid((unsigned)((rows + RB - 1) / RB), (unsigned)nby);
    auto go = [&](auto kernel) {
        kernel<<<grid, 64 * nw, lds, st>>>(d, s, rows, RB, Wa, dst1, dst2, dst2_stride, av);
    };
    if constexpr (MULTI && !EPI) {  // (all of a block's rows at once)
        if (RB == 64) return go(k_theta<R, G, 4, EPI, MULTI>);
    }
    if (MULTI || RB > 16) go(k_theta<R, G, 2, EPI, MULTI>);
    else if constexpr (!MULTI) go(k_theta<R, G, 1, EPI, MULTI>);
}
template <typename R, int EPI>
static void theta_r(hipStream_t st, const Dims& d, const int8_t* s, long rows, const void* Wa,
                    void* dst1, void* dst2, long dst2_stride, const double* av) {
#define THETA_G(G, MULTI)                                                                     \
    theta_g<R, G, EPI, MULTI>(st, d, s, rows, (const R*)Wa, (R*)dst1, (R*)dst2, dst2_stride, av)
    switch (d.Na / 16) {
        case 1: return THETA_G(1, false);
        case 2: return THETA_G(2, false);
        case 3: return THETA_G(3, false);
        case 4: return THETA_G(4, false);
        case 5: return THETA_G(5, false);
        case 6: return THETA_G(6, false);
        case 7: return THETA_G(7, false);
        case 8: return THETA_G(8, false);
        case 9: case 10: return THETA_G(10, false);
        case 11: case 12: return THETA_G(12, false);
        case 13: case 14: return THETA_G(14, false);
        case 15: case 16: case 17: return THETA_G(17, false);
        default: return THETA_G(8, true);
    }
#undef THETA_G
}

template <int KS, bool MULTI>
static void theta_bf16(hipStream_t st, const Dims& d, const int8_t* s, long rows, const Tables& t,
                       float* dst1, float* dst2, long dst2_stride) {
    const long nby = (d.Mw + 63) / 64;
    const int RB = theta_rows(rows, nby, 1024);
    auto go = [&](auto kernel, int rb) {
        kernel<<<dim3((unsigned)((rows + rb - 1) / rb), (unsigned)nby), 256,
                 (size_t)rb * 32 * (KS | 1), st>>>(d, s, rows, rb, t.Whi, t.Wlo, dst1, dst2,
                                                   dst2_stride);
    };
    if constexpr (MULTI) {  // (all of a block's rows at once)
        if (RB >= 64) go(k_theta_bf16<KS, 4, true>, 64);
        else go(k_theta_bf16<KS, 2, true>, 32);
    } else {
        if (RB > 16) go(k_theta_bf16<KS, 2, false>, RB);
        else go(k_theta_bf16<KS, 1, false>, 16);
    }
}

void launch_theta(hipStream_t st, const Dims& d, int prec, const Tables& t, const int8_t* s,
                  int rows, void* dst1, void* dst2, long dst2_stride) {
    if (rows <= 0) return;
    if (prec == 0) {
        theta_r<double, 0>(st, d, s, rows, t.Wa, dst1, dst2, dst2_stride, nullptr);
    } else if (prec == 1) {
        theta_r<float, 0>(st, d, s, rows, t.Wa, dst1, dst2, dst2_stride, nullptr);
    } else {
#define THETA_B(KS, MULTI) \
    theta_bf16<KS, MULTI>(st, d, s, rows, t, (float*)dst1, (float*)dst2, dst2_stride)
        switch (d.Kb / 32) {
            case 1: return THETA_B(1, false);
            case 2: return THETA_B(2, false);
            case 3: return THETA_B(3, false);
            case 4: return THETA_B(4, false);
            case 5: return THETA_B(5, false);
            case 6: return THETA_B(6, false);
            case 7: return THETA_B(7, false);
            case 8: return THETA_B(8, false);
            case 9: return THETA_B(9, false);
            default: return THETA_B(4, true);
        }
#undef THETA_B
    }
}

void launch_log_psi(hipStream_t st, const Dims& d, int prec, const double* Pm, const Tables& t,
                    const int8_t* s, long n, void* out) {
    if (n <= 0) return;
    const double* av = d.vb ? Pm + (size_t)d.M * d.Na : nullptr;
    if (prec == 0) theta_r<double, 1>(st, d, s, n, t.Wa, out, nullptr, 0, av);
    else theta_r<float, 1>(st, d, s, n, t.Wa, out, nullptr, 0, av);
}

}  // namespace nqs
