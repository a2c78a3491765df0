// Dense-Jacobian form of the QGT (paper, QGTJacobianDense and its appendix):
// the Jacobian O[k][p] = d ln psi(s_k) / d p_p is materialised in the packed
// parameter order, centred and scaled (dJ = (O - mean O) / sqrt(N_s)), the
// Gram matrix G = dJ^T dJ is formed on MFMA, and CG runs on G v + eps v.
#include "kernels.h"

#include <vector>

namespace nqs {

// Column sums of O in two fixed-order passes: slices of rows (one thread per column
// and slice, eight rows' loads together), then each column adds its slices: a block
// covers 64 columns, wave w the slices [w S / 4, (w + 1) S / 4).  Then O <- (O -
// colsum / n) / sqrt(n), four columns per thread where the rows are 16-byte aligned.
constexpr int CS_ROWS = 32;  // rows per slice, where the scratch holds that many
__global__ __launch_bounds__(256) void k_colsum_part(const double* __restrict__ O, long n, long ld,
                                                     int P, int splits, double* __restrict__ part) {
    const long p = (long)blockIdx.x * 256 + threadIdx.x;
    if (p >= P) return;
    const long k0 = n * blockIdx.y / splits, k1 = n * (blockIdx.y + 1) / splits;
    double acc = 0.0;
    for (long k = k0; k < k1; k += 8) {
        double x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = O[min(k + u, k1 - 1) * ld + p];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (k + u < k1) acc += x[u];
    }
    part[(size_t)blockIdx.y * P + p] = acc;
}
__global__ __launch_bounds__(256) void k_colsum_fin(const double* __restrict__ part, int P,
                                                    int splits, double* __restrict__ cs) {
    __shared__ double ws[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int p = blockIdx.x * 64 + lane, pc = p < P ? p : P - 1;
    const int b0 = wave * splits / 4, b1 = (wave + 1) * splits / 4;
    double acc = 0.0;
    for (int q = b0; q < b1; q += 8) {
        double x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = part[(size_t)min(q + u, splits - 1) * P + pc];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (q + u < b1) acc += x[u];
    }
    ws[wave][lane] = acc;
    __syncthreads();
    if (wave == 0 && p < P) cs[p] = (ws[0][lane] + ws[1][lane]) + (ws[2][lane] + ws[3][lane]);
}
__global__ __launch_bounds__(256) void k_center_scale(double* __restrict__ O, long n, long ld,
                                                      int P, const double* __restrict__ cs,
                                                      int vec) {
    const long k = blockIdx.y;
    const int W = vec ? 4 : 1;  // columns per thread
    const long p = W * ((long)blockIdx.x * 256 + threadIdx.x);
    if (p >= P || k >= n) return;
    const double inv = 1.0 / (double)n;
    const double rs = 1.0 / sqrt((double)n);
    double* e = O + k * ld + p;
    if (vec && p + 4 <= P) {  // (ld a multiple of 4, base 16-byte aligned, p a multiple of 4)
        double2 a = *(double2*)e, b = *(double2*)(e + 2);
        a.x = (a.x - cs[p] * inv) * rs;
        a.y = (a.y - cs[p + 1] * inv) * rs;
        b.x = (b.x - cs[p + 2] * inv) * rs;
        b.y = (b.y - cs[p + 3] * inv) * rs;
        *(double2*)e = a;
        *(double2*)(e + 2) = b;
    } else {
        for (long q = p; q < P && q < p + W; ++q) e[q - p] = (e[q - p] - cs[q] * inv) * rs;
    }
}

// The Jacobian's entries straight from a sample's spins and activations: the
// entry of column p is s_i (visible bias), t_j (hidden bias) or t_j s_i (W_ji),
// with the packed order [a | b | W] and W row-major (p = off + j N + i); t_j s_i
// with s_i = +-1 is exact in FP32, so it is the stored entry's value.
struct JacCol {
    int kind, j, i;  // kind 0: s_i, 1: t_j, 2: t_j s_i, 3: padding (zero)
};
__device__ __forceinline__ JacCol jac_col(const Dims& d, long p, int P) {
    JacCol c{3, 0, 0};
    if (p >= P) return c;
    long idx = p;
    if (d.vb) {
        if (idx < d.N) return JacCol{0, 0, (int)idx};
        idx -= d.N;
    }
    if (d.hb) {
        if (idx < d.M) return JacCol{1, (int)idx, 0};
        idx -= d.M;
    }
    const int j = (int)idx / d.N;  // (P fits 32 bits)
    return JacCol{2, j, (int)idx - j * d.N};
}
// The Jacobian's rows in one write pass: O[k][p] = t s (CENTER: dJ = (O - cs[p] / n)
// / sqrt(n), with the column sums cs), zero in the padding columns P <= p < ld.
// A block writes 1,024 columns of `rpb` rows; each thread finds its four columns'
// spin and activation once (pointers and row strides, a missing factor being the
// constant 1, or 0 for padding, with stride 0) and walks the rows, four rows'
// loads ahead of their arithmetic.  VEC: ld a multiple of 4 and O 16-byte aligned:
// four neighbouring columns per thread, one 16-byte store per FP32 row; else
// columns 256 apart, so that every store instruction still covers whole lines.
// In the VEC form four columns of one hidden unit (N a multiple of 4) read one
// activation and one word of spins.
// Bound by the write: 4,000 x 33,344 FP32 entries (534 MB) in 127 us, 4.2 TB/s (a
// copy moves 5.1 TB/s); with the column sums 150 us, against 1,980 us for the three
// passes (rows, column sums by one thread per column, centring) it replaces.
__device__ const int8_t k_one_s = 1, k_zero_s = 0;
template <typename R>
__device__ const R k_one_t = (R)1;
template <typename R, bool CENTER, bool VEC>
__global__ __launch_bounds__(256) void k_jac_rows(Dims d, const int8_t* __restrict__ s,
                                                  const R* __restrict__ tact, long rows, int rpb,
                                                  double inv, double rs, int P, long ld,
                                                  const double* __restrict__ cs,
                                                  R* __restrict__ O) {
    const long c0 = (long)blockIdx.x * 1024;
    const long p0 = VEC ? c0 + 4 * threadIdx.x : c0 + threadIdx.x;
    if (p0 >= ld) return;
    const int8_t* sp[4];
    const R* tp[4];
    int ss[4], ts[4];
    double mean[4];
    JacCol cc[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const long p = VEC ? p0 + e : p0 + 256 * e;
        const JacCol c = jac_col(d, p, P);
        const bool has_s = c.kind == 0 || c.kind == 2, has_t = c.kind == 1 || c.kind == 2;
        sp[e] = has_s ? s + c.i : (c.kind == 3 ? &k_zero_s : &k_one_s);
        ss[e] = has_s ? d.N : 0;
        tp[e] = has_t ? tact + c.j : &k_one_t<R>;
        ts[e] = has_t ? d.Mw : 0;
        mean[e] = CENTER && c.kind != 3 ? cs[p] * inv : 0.0;
        cc[e] = c;
    }
    const long k0 = (long)blockIdx.y * rpb, k1 = min(rows, k0 + rpb);
    auto entry = [&](R t, int sv, int e) -> R {
        if constexpr (CENTER)
            return (R)(((double)t * (double)sv - mean[e]) * rs);
        else
            return t * (R)sv;
    };
    auto put = [&](long k, const R (&v)[4]) {
        R* row = O + k * ld;
        if constexpr (VEC) {
            if constexpr (sizeof(R) == 4) {
                *(float4*)(row + p0) = make_float4(v[0], v[1], v[2], v[3]);
            } else {
                *(double2*)(row + p0) = make_double2(v[0], v[1]);
                *(double2*)(row + p0 + 2) = make_double2(v[2], v[3]);
            }
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (p0 + 256 * e < ld) row[p0 + 256 * e] = v[e];
        }
    };
    constexpr int U = 4;  // rows in flight
    if (VEC && d.N % 4 == 0 && ((uintptr_t)s & 3) == 0 && cc[0].kind == 2 && cc[3].kind == 2 &&
        cc[0].j == cc[3].j && cc[0].i % 4 == 0) {
        const R* t = tp[0];
        const int8_t* w = sp[0];
        for (long k = k0; k < k1; k += U) {
            R tv[U];
            uint32_t wv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const long kk = min(k + u, k1 - 1);
                tv[u] = t[kk * d.Mw];
                wv[u] = *(const uint32_t*)(w + kk * d.N);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                R v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = entry(tv[u], (int8_t)(wv[u] >> (8 * e)), e);
                if (k + u < k1) put(k + u, v);
            }
        }
        return;
    }
    for (long k = k0; k < k1; k += U) {
        R tv[U][4];
        int sv[U][4];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const long kk = min(k + u, k1 - 1);
                tv[u][e] = tp[e][kk * ts[e]];
                sv[u][e] = sp[e][kk * ss[e]];
            }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            R v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = entry(tv[u][e], sv[u][e], e);
            if (k + u < k1) put(k + u, v);
        }
    }
}

// G[p][q] = sum_k A[k][p] A[k][q] for the upper block triangle, mirrored where the
// products read the lower one too.  Block = 4 waves = a tile of G of 32 T rows and
// columns, SUB x SUB of them per listed 128 x 128 tile; each wave a quarter as T x T
// MFMA tiles of 16 x 16.  The operands of the next U steps of 4 samples are loaded,
// lanes over columns, while these U are multiplied; rows of A are whole tiles of
// columns long.  FP32, 4,096 samples: P = 860 (28 tiles, in quarters) 135 us, 653 with
// the loads of each step waited for; P = 3,320 (351 whole tiles) 680, 917; from some
// thousand tiles on the waves hide the loads either way (U = 1: 8,384 columns 3.3 ms).
template <typename R, int T, int U, int SUB>
__global__ __launch_bounds__(256, 2) void k_gram(const R* __restrict__ A, long n, long ld, int P,
                                                 R* __restrict__ G, const int* __restrict__ tiles,
                                                 bool mirror) {
    const int lt = blockIdx.x / (SUB * SUB), sub = blockIdx.x % (SUB * SUB);
    const int lp = tiles[2 * lt], lq = tiles[2 * lt + 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lr = lane & 15, lk = lane >> 4;
    const int p0 = 32 * T * (lp * SUB + sub / SUB) + (wave >> 1) * 16 * T;
    const int q0 = 32 * T * (lq * SUB + sub % SUB) + (wave & 1) * 16 * T;
    typedef typename std::conditional<sizeof(R) == 8, v4d, v4f>::type acc_t;
    acc_t acc[T][T];
#pragma unroll
    for (int a = 0; a < T; ++a)
#pragma unroll
        for (int b = 0; b < T; ++b) acc[a][b] = acc_t{0, 0, 0, 0};
    R na[U][T], nb[U][T];
    auto load = [&](long k0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const R* row = A + min(k0 + 4 * u + lk, n - 1) * ld + lr;
#pragma unroll
            for (int a = 0; a < T; ++a) {
                na[u][a] = row[p0 + 16 * a];
                nb[u][a] = row[q0 + 16 * a];
            }
        }
    };
    load(0);
    for (long k0 = 0; k0 < n; k0 += 4 * U) {
        R fa[U][T], fb[U][T];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int a = 0; a < T; ++a) {
                const bool in = k0 + 4 * u + lk < n;
                fa[u][a] = in ? na[u][a] : (R)0;
                fb[u][a] = nb[u][a];
            }
        load(k0 + 4 * U);  // (past n: the last row)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int a = 0; a < T; ++a)
#pragma unroll
                for (int b = 0; b < T; ++b) {
                    if constexpr (sizeof(R) == 8)
                        acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[u][a], fb[u][b], acc[a][b], 0, 0, 0);
                    else
                        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[u][a], fb[u][b], acc[a][b], 0, 0, 0);
                }
    }
#pragma unroll
    for (int a = 0; a < T; ++a)
#pragma unroll
        for (int b = 0; b < T; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const long p = p0 + a * 16 + acc_row<R>(lk, i), q = q0 + b * 16 + lr;
                if (p < P && q < P) {
                    G[p * ld + q] = acc[a][b][i];
                    if (mirror && lp != lq) G[q * ld + p] = acc[a][b][i];
                }
            }
}

// FP64 Gram over row slices, for matrices with few tiles (a small P leaves most
// compute units idle when each tile walks all n rows): block = (tile, slice of
// rows), the tile's partial written in tile order [128][128]; k_gram_fin sums
// the slices in order (deterministic) and writes G with the lower triangle
// mirrored (within a diagonal tile only entries on or above the diagonal are
// taken, so G is exactly symmetric).  The next step's operands are loaded while
// this one's are multiplied.
__global__ __launch_bounds__(256, 2) void k_gram_slices(const double* __restrict__ A, long n, long ld,
                                                     int ntiles, long rows_per_slice,
                                                     const int* __restrict__ tiles,
                                                     double* __restrict__ part) {
    const int t = (int)(blockIdx.x % (unsigned)ntiles), ks = (int)(blockIdx.x / (unsigned)ntiles);
    const int tp = tiles[2 * t], tq = tiles[2 * t + 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lr = lane & 15, lk = lane >> 4;
    const long p0 = (long)tp * 128 + (wave >> 1) * 64;
    const long q0 = (long)tq * 128 + (wave & 1) * 64;
    const long r0 = (long)ks * rows_per_slice;
    const long r1 = r0 + rows_per_slice < n ? r0 + rows_per_slice : n;
    v4d acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = v4d{0, 0, 0, 0};
    double na[4], nb[4];
    auto load = [&](long k0) {
        const double* row = A + min(k0 + lk, r1 - 1) * ld + lr;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            na[a] = row[p0 + a * 16];
            nb[a] = row[q0 + a * 16];
        }
    };
    if (r0 < r1) load(r0);  // (a slice past the rows is zero)
    for (long k0 = r0; k0 < r1; k0 += 4) {
        double fa[4], fb[4];
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            fa[a] = k0 + lk < r1 ? na[a] : 0.0;
            fb[a] = nb[a];
        }
        load(k0 + 4);  // (past r1: the last row)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[a], fb[b], acc[a][b], 0, 0, 0);
    }
    double* pt = part + (size_t)blockIdx.x * 128 * 128;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int pr = (wave >> 1) * 64 + a * 16 + acc_row<double>(lk, i);
                const int qc = (wave & 1) * 64 + b * 16 + lr;
                pt[pr * 128 + qc] = acc[a][b][i];
            }
}

// (a block covers 64 entries of a tile row, its waves a quarter of the slices each,
// eight loads together: three tiles of 128 slices, 50 MB, in 9 us against 150 us
// for 32 x 32 entries per block, each thread walking all slices)
__global__ __launch_bounds__(256) void k_gram_fin(const double* __restrict__ part, int ntiles,
                                                  int slices, const int* __restrict__ tiles, int P,
                                                  long ld, double* __restrict__ G) {
    __shared__ double ws[4][64];
    const int t = blockIdx.x >> 8, sub = blockIdx.x & 255;
    const int tp = tiles[2 * t], tq = tiles[2 * t + 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long p = (long)tp * 128 + (sub >> 1), q = (long)tq * 128 + 64 * (sub & 1) + lane;
    const double* src = part + (size_t)t * 128 * 128 + 64 * sub + lane;
    const size_t step = (size_t)ntiles * 128 * 128;
    const int b0 = wave * slices / 4, b1 = (wave + 1) * slices / 4;
    double a = 0.0;
    for (int b = b0; b < b1; b += 8) {
        double x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = src[(size_t)min(b + u, slices - 1) * step];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (b + u < b1) a += x[u];
    }
    ws[wave][lane] = a;
    __syncthreads();
    if (wave != 0 || p >= P || q >= P || (tp == tq && p > q)) return;
    a = (ws[0][lane] + ws[1][lane]) + (ws[2][lane] + ws[3][lane]);
    G[p * ld + q] = a;
    if (p != q) G[q * ld + p] = a;
}

// The BF16 form's Gram: each centred entry x as the pair hi = bf16(x), lo = bf16(x -
// hi), and G = sum over samples of hi.hi, then hi.lo, then lo.hi of every 32 samples on
// the 16x16x32 BF16 MFMA, in FP32.
//
// The Jacobian is written as that instruction's operands: fragment (kb, ct) holds
// samples 32 kb .. + 31 of columns 16 ct .. + 15, plane hi, then lo, each [lane][8
// samples], lane = column + 16 (sample / 8); samples past n and columns past P are zero.
// A wave takes one tile of columns through `kbs` k-blocks.  16,384 x 33,344 entries
// (2.19 GB) in 685 us.
typedef short v8s_g __attribute__((ext_vector_type(8)));
__global__ __launch_bounds__(256) void k_jac_frags(Dims d, const int8_t* __restrict__ s,
                                                   const float* __restrict__ tact, long n, int nkb,
                                                   int kbs, double inv, double rs, int P, int nct,
                                                   const double* __restrict__ cs,
                                                   uint4* __restrict__ F) {
    const int lane = threadIdx.x & 63, ct = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (ct >= nct) return;
    const long p = 16L * ct + (lane & 15);
    const JacCol c = jac_col(d, p, P);
    const bool has_s = c.kind == 0 || c.kind == 2, has_t = c.kind == 1 || c.kind == 2;
    const int8_t* sp = has_s ? s + c.i : (c.kind == 3 ? &k_zero_s : &k_one_s);
    const float* tp = has_t ? tact + c.j : &k_one_t<float>;
    const int ss = has_s ? d.N : 0, ts = has_t ? d.Mw : 0;
    const double mean = c.kind != 3 ? cs[p] * inv : 0.0;
    const int kb1 = min(nkb, (int)(blockIdx.y + 1) * kbs);
    for (int kb = blockIdx.y * kbs; kb < kb1; ++kb) {
        const long k0 = 32L * kb + 8 * (lane >> 4);
        float t[8];
        int sv[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const long k = min(k0 + e, n - 1);
            t[e] = tp[k * ts];
            sv[e] = sp[k * ss];
        }
        uint32_t hi[8], lo[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float x = k0 + e < n ? (float)(((double)t[e] * (double)sv[e] - mean) * rs) : 0.0f;
            hi[e] = f32_to_bf16_bits(x);
            lo[e] = f32_to_bf16_bits(x - bf16_bits_to_f32((uint16_t)hi[e]));
        }
        uint4* f = F + ((size_t)kb * nct + ct) * 128 + lane;
        f[0] = make_uint4(hi[0] | hi[1] << 16, hi[2] | hi[3] << 16, hi[4] | hi[5] << 16,
                          hi[6] | hi[7] << 16);
        f[64] = make_uint4(lo[0] | lo[1] << 16, lo[2] | lo[3] << 16, lo[4] | lo[5] << 16,
                           lo[6] | lo[7] << 16);
    }
}

// A block of WP x WQ waves takes a tile of G of 16 WP AT rows and 16 WQ BT columns,
// each wave AT x BT MFMA tiles; both panels' fragments of a k-block move through one of
// two LDS buffers, the next k-block's in registers while this one is multiplied.  The
// products of one kind run over a row of tiles before the next kind, so that none
// waits for the one before.
// A product reads (AT + BT) / (3 AT BT) fragment pairs from LDS: a wave's 64 x 64 part
// of a 128 x 128 tile keeps LDS as busy as the matrix cores, 128 x 64 of 256 x 256
// needs a quarter less, and half the writes.  D: k-blocks the loads run ahead.  16,384
// samples, P = 33,344: 48 ms, 1.14 PFLOP/s (the library's plain BF16 product reaches 1.2
// here), 68 ms with pairs regrouped on the way into LDS; 4,096 samples, P = 860: 43 us,
// 202.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
template <int WP, int WQ, int AT, int BT, int D, int SUB>
__global__ __launch_bounds__(64 * WP * WQ, 2) void k_gram_frags(const u32x4* __restrict__ F, int nkb,
                                                             int nct, long ld, int P,
                                                             float* __restrict__ G,
                                                             const int* __restrict__ tiles,
                                                             bool mirror) {
    constexpr int PA = WP * AT, PB = WQ * BT, T = 64 * WP * WQ, NP = (PA + PB) * 128 / T;
    extern __shared__ __align__(16) u32x4 Lf[];  // [2][PA + PB][128]
    // SUB x SUB blocks share a listed tile
    const int lt = blockIdx.x / (SUB * SUB), sub = blockIdx.x % (SUB * SUB);
    const int lp = tiles[2 * lt], lq = tiles[2 * lt + 1];
    const int tp = lp * SUB + sub / SUB, tq = lq * SUB + sub % SUB;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wp = wave / WQ, wq = wave % WQ;
    const u32x4* src[NP];
#pragma unroll
    for (int m = 0; m < NP; ++m) {  // (a ragged tile's missing columns: the last ones again)
        const int f = (tid + m * T) >> 7;
        const int ct = min(f < PA ? tp * PA + f : tq * PB + f - PA, nct - 1);
        src[m] = F + (size_t)ct * 128 + (tid & 127);
    }
    const size_t step = (size_t)nct * 128;
    v4f acc[AT][BT];
#pragma unroll
    for (int a = 0; a < AT; ++a)
#pragma unroll
        for (int b = 0; b < BT; ++b) acc[a][b] = v4f{0, 0, 0, 0};
    auto load = [&](u32x4 (&g)[NP], int kb) {
        const size_t o = (size_t)min(kb, nkb - 1) * step;
#pragma unroll
        for (int m = 0; m < NP; ++m) g[m] = src[m][o];
    };
    auto put = [&](const u32x4 (&g)[NP], int kb) {
        u32x4* L = Lf + (kb & 1) * (PA + PB) * 128;
#pragma unroll
        for (int m = 0; m < NP; ++m) L[tid + m * T] = g[m];
    };
    // k-block kb; `in` takes k-block kb + D, `next` holds kb + 1
    auto block = [&](int kb, u32x4 (&in)[NP], const u32x4 (&next)[NP]) {
        load(in, kb + D);
        __builtin_amdgcn_sched_barrier(0);  // (the loads stay ahead of the products)
        const u32x4* L = Lf + (kb & 1) * (PA + PB) * 128;
        const u32x4* La = L + wp * AT * 128 + lane;
        const u32x4* Lb = L + (PA + wq * BT) * 128 + lane;
        v8bf bh[BT], bl[BT];
#pragma unroll
        for (int b = 0; b < BT; ++b) {
            bh[b] = __builtin_bit_cast(v8bf, Lb[b * 128]);
            bl[b] = __builtin_bit_cast(v8bf, Lb[b * 128 + 64]);
        }
#pragma unroll
        for (int a = 0; a < AT; ++a) {
            const v8bf xh = __builtin_bit_cast(v8bf, La[a * 128]);
            const v8bf xl = __builtin_bit_cast(v8bf, La[a * 128 + 64]);
#pragma unroll
            for (int b = 0; b < BT; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xh, bh[b], acc[a][b], 0, 0, 0);
#pragma unroll
            for (int b = 0; b < BT; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xh, bl[b], acc[a][b], 0, 0, 0);
#pragma unroll
            for (int b = 0; b < BT; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xl, bh[b], acc[a][b], 0, 0, 0);
        }
        put(next, kb + 1);
        lds_barrier();
    };
    u32x4 g0[NP], g1[D > 1 ? NP : 1];
    load(g0, 0);
    put(g0, 0);
    if constexpr (D > 1) load(g1, 1);
    lds_barrier();
    if constexpr (D > 1) {
        for (int kb = 0; kb + 1 < nkb; kb += 2) {
            block(kb, g0, g1);
            block(kb + 1, g1, g0);
        }
        if (nkb & 1) block(nkb - 1, g0, g1);
    } else {
        for (int kb = 0; kb < nkb; ++kb) block(kb, g0, g0);
    }
    const int lr = lane & 15, lk = lane >> 4;
#pragma unroll
    for (int a = 0; a < AT; ++a)
#pragma unroll
        for (int b = 0; b < BT; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const long p = 16L * (tp * PA + wp * AT + a) + acc_row<float>(lk, i);
                const long q = 16L * (tq * PB + wq * BT + b) + lr;
                if (p < P && q < P) {
                    G[p * ld + q] = acc[a][b][i];
                    if (mirror && lp != lq) G[q * ld + p] = acc[a][b][i];
                }
            }
}

// out = G v + shift v (FP64 accumulation) and the block partials of v . out.
// Each wave handles DMV_RW rows at once, so every 4-element slice of v it loads
// serves DMV_RW rows of G (4 consecutive entries per lane per step).  No
// cross-block step: the CG update sums the partials.
constexpr int DMV_RW = 4;
template <typename R>
__global__ __launch_bounds__(256) void k_dense_matvec(const R* __restrict__ G, int P, long ld,
                                                      const double* __restrict__ v,
                                                      double* __restrict__ out,
                                                      double* __restrict__ dpart,
                                                      const CgScalars* __restrict__ sc) {
    if (sc->done) return;
    __shared__ double sh[4];
    const double shift = sc->shift;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long p0 = ((long)blockIdx.x * 4 + wave) * DMV_RW;
    double acc[DMV_RW];
#pragma unroll
    for (int r = 0; r < DMV_RW; ++r) acc[r] = 0.0;
    for (long q = 4 * lane; q < P; q += 256) {
        if (q + 4 <= P) {
            const double2 v01 = *(const double2*)(v + q), v23 = *(const double2*)(v + q + 2);
#pragma unroll
            for (int r = 0; r < DMV_RW; ++r) {
                if (p0 + r >= P) break;
                const R* g = G + (p0 + r) * ld + q;
                double g0, g1, g2, g3;
                if constexpr (sizeof(R) == 4) {
                    const float4 t = *(const float4*)g;
                    g0 = t.x; g1 = t.y; g2 = t.z; g3 = t.w;
                } else {
                    const double2 a = *(const double2*)g, b = *(const double2*)(g + 2);
                    g0 = a.x; g1 = a.y; g2 = b.x; g3 = b.y;
                }
                acc[r] += (g0 * v01.x + g1 * v01.y) + (g2 * v23.x + g3 * v23.y);
            }
        } else {  // ragged end of the row
            for (long qq = q; qq < P; ++qq)
#pragma unroll
                for (int r = 0; r < DMV_RW; ++r)
                    if (p0 + r < P) acc[r] += (double)G[(p0 + r) * ld + qq] * v[qq];
        }
    }
    double dot = 0.0;
#pragma unroll
    for (int r = 0; r < DMV_RW; ++r) {
        const double s = wave_sum(acc[r]);
        if (p0 + r < P) {
            const double o = s + shift * v[p0 + r];
            if (lane == 0) out[p0 + r] = o;
            dot += o * v[p0 + r];
        }
    }
    if (lane == 0) sh[wave] = dot;
    __syncthreads();
    if (threadIdx.x == 0) dpart[blockIdx.x] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// The same product from the upper triangle of a large G, which halves what an
// iteration reads: block (segment, panel) takes rows 128 panel .. + 127 against NC x
// 256 of the columns from 128 panel on.  A lane holds 4 columns of each 256 and a
// wave 8 rows at a time; every entry right of the panel's diagonal tile also gives
// its mirror's product, summed per column in registers over the wave's 32 rows and
// over the four waves through LDS.  The diagonal tile is used whole: its two halves
// are products of their own (the split BF16 products add lo.hi and hi.lo in the other
// order there).  Row sums go to rowp[segment][P], column sums to colp[panel][P];
// k_tri_sum adds them in that order, with the shift, and forms the partials of v . out.
// Memory bound, 5.1 TB/s of G's upper half at P = 25,024 (FP32): 253 us with the sum,
// 430 over the whole matrix.
constexpr int TRI_H = 128;
template <typename R, int NC>
__global__ __launch_bounds__(256) void k_tri_matvec(const R* __restrict__ G, int P, long ld,
                                                    const double* __restrict__ v,
                                                    double* __restrict__ rowp,
                                                    double* __restrict__ colp,
                                                    const CgScalars* __restrict__ sc) {
    constexpr int W = 256 * NC;
    if (sc->done) return;
    __shared__ __align__(16) double vs[W];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r0 = blockIdx.y * TRI_H, q0 = r0 + blockIdx.x * W;
    if (q0 >= P) return;
    for (int i = threadIdx.x; i < W; i += 256) vs[i] = q0 + i < P ? v[q0 + i] : 0.0;
    __syncthreads();
    double cs[NC][4];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) cs[c][e] = 0.0;
    for (int g = 0; g < 4; ++g) {
        const int p0 = r0 + 32 * wave + 8 * g;
        if (p0 >= P) break;
        double rs[8], x[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            rs[r] = 0.0;
            x[r] = p0 + r < P ? v[p0 + r] : 0.0;
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int qc = q0 + 256 * c;
            if (qc >= P) break;
            const bool ragged = qc + 256 > P;  // (entries past P are stored as anything)
            const long q = min((long)qc + 4 * lane, ld - 4);
            const double2 v01 = *(const double2*)&vs[256 * c + 4 * lane];
            const double2 v23 = *(const double2*)&vs[256 * c + 4 * lane + 2];
            R t[8][4];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const R* a = G + (long)min(p0 + r, P - 1) * ld + q;
                if constexpr (sizeof(R) == 4) {
                    const float4 f = *(const float4*)a;
                    t[r][0] = f.x; t[r][1] = f.y; t[r][2] = f.z; t[r][3] = f.w;
                } else {
                    const double2 f = *(const double2*)a, h = *(const double2*)(a + 2);
                    t[r][0] = f.x; t[r][1] = f.y; t[r][2] = h.x; t[r][3] = h.y;
                }
            }
            if (ragged) {
#pragma unroll
                for (int r = 0; r < 8; ++r)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (qc + 4 * lane + e >= P) t[r][e] = R(0);
            }
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const double g0 = t[r][0], g1 = t[r][1], g2 = t[r][2], g3 = t[r][3];
                rs[r] += (g0 * v01.x + g1 * v01.y) + (g2 * v23.x + g3 * v23.y);
                cs[c][0] += g0 * x[r];
                cs[c][1] += g1 * x[r];
                cs[c][2] += g2 * x[r];
                cs[c][3] += g3 * x[r];
            }
        }
        // row r's sum to the lanes with lane % 8 == r: halve the rows held by
        // exchanges over three lane bits, then add over the other three
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const bool up = (lane >> m) & 1;
#pragma unroll
            for (int i = 0; i < (4 >> m); ++i) {
                const double keep = up ? rs[2 * i + 1] : rs[2 * i];
                const double send = up ? rs[2 * i] : rs[2 * i + 1];
                rs[i] = keep + __shfl_xor(send, 1 << m);
            }
        }
        rs[0] += __shfl_xor(rs[0], 8);
        rs[0] += __shfl_xor(rs[0], 16);
        rs[0] += __shfl_xor(rs[0], 32);
        if (lane < 8 && p0 + lane < P) rowp[(size_t)blockIdx.x * P + p0 + lane] = rs[0];
    }
    __syncthreads();
    for (int w = 0; w < 4; ++w) {
        if (wave == w) {
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    double& o = vs[256 * c + 4 * lane + e];
                    o = w ? o + cs[c][e] : cs[c][e];
                }
        }
        __syncthreads();
    }
    for (int i = threadIdx.x; i < W; i += 256) {
        const int q = q0 + i;
        if (q >= r0 + TRI_H && q < P) colp[(size_t)blockIdx.y * P + q] = vs[i];
    }
}

__global__ __launch_bounds__(256) void k_tri_sum(const double* __restrict__ rowp,
                                                 const double* __restrict__ colp, int P, int W,
                                                 const double* __restrict__ v,
                                                 double* __restrict__ out,
                                                 double* __restrict__ dpart,
                                                 const CgScalars* __restrict__ sc) {
    if (sc->done) return;
    __shared__ double ws[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int p = blockIdx.x * 64 + lane, pc = min(p, P - 1);
    const int panel = blockIdx.x * 64 / TRI_H;  // (its segments and the panels above it)
    const int ns = (P - panel * TRI_H + W - 1) / W, n = ns + panel;
    const int b0 = wave * n / 4, b1 = (wave + 1) * n / 4;
    double a = 0.0;
    for (int q = b0; q < b1; q += 8) {
        double x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int e = min(q + u, n - 1);
            x[u] = e < ns ? rowp[(size_t)e * P + pc] : colp[(size_t)(e - ns) * P + pc];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (q + u < b1) a += x[u];
    }
    ws[wave][lane] = a;
    __syncthreads();
    if (wave == 0) {
        const double o = ((ws[0][lane] + ws[1][lane]) + (ws[2][lane] + ws[3][lane])) +
                         sc->shift * v[pc];
        if (p < P) out[p] = o;
        const double dot = wave_sum(p < P ? o * v[pc] : 0.0);
        if (lane == 0) dpart[blockIdx.x] = dot;
    }
}

// Columns per block of the triangle product in units of 256, or 0 for the product
// over all of G: the triangle form where G (entries of `elem` bytes) is more than the
// XCDs' L2s hold together, 32 MiB.  FP32, product and sum against the whole product:
// P = 2,143 (18 MB) 12.2 against 9.6 us, 3,320 (44 MB) 14.2 against 19.4, 16,704 118
// against 200, 25,024 253 against 430.  512 columns from 20,480 on, where that leaves
// enough blocks (25,024: 253 us, 258 with 256; 16,704: 122, 118).  `scratch` bytes must
// hold the row and column partials.
int dense_tri(int P, size_t elem, size_t scratch) {
    if (elem * P * P <= (size_t)32 << 20) return 0;
    const int nc = P < 20480 ? 1 : 2;
    const size_t rows = (size_t)(P + 256 * nc - 1) / (256 * nc) + (P + TRI_H - 1) / TRI_H;
    return 8 * rows * P <= scratch ? nc : 0;
}
int dense_matvec_blocks(int P, int tri) {
    return tri ? (P + 63) / 64 : (P + 4 * DMV_RW - 1) / (4 * DMV_RW);
}
template <typename R, int NC>
static void tri_matvec(hipStream_t st, const R* G, int P, long ld, const double* v, double* out,
                       double* dpart, const CgScalars* sc, double* scratch) {
    const int ns = (P + 256 * NC - 1) / (256 * NC), np = (P + TRI_H - 1) / TRI_H;
    double* colp = scratch + (size_t)ns * P;
    k_tri_matvec<R, NC><<<dim3(ns, np), 256, 0, st>>>(G, P, ld, v, scratch, colp, sc);
    k_tri_sum<<<(P + 63) / 64, 256, 0, st>>>(scratch, colp, P, 256 * NC, v, out, dpart, sc);
}
template <typename R>
static void dense_matvec(hipStream_t st, const R* G, int P, long ld, const double* v, double* out,
                         double* dpart, const CgScalars* sc, int tri, double* scratch) {
    if (tri == 1) tri_matvec<R, 1>(st, G, P, ld, v, out, dpart, sc, scratch);
    else if (tri == 2) tri_matvec<R, 2>(st, G, P, ld, v, out, dpart, sc, scratch);
    else
        k_dense_matvec<R><<<dense_matvec_blocks(P, 0), 256, 0, st>>>(G, P, ld, v, out, dpart, sc);
}

// ---------------------------------------------------------------------------
// rows per block: long enough to pay for finding the columns (64), shorter where
// that leaves fewer than about four blocks per compute unit
template <typename R, bool CENTER>
static void jac_rows(hipStream_t st, const Dims& d, const int8_t* s, const void* tact, long n,
                     long nmean, void* O, int P, long ld, const double* cs) {
    const long cb = (ld + 1023) / 1024;
    int rpb = 64;
    while (rpb > 4 && cb * ((n + rpb - 1) / rpb) < 1024) rpb /= 2;
    const double inv = 1.0 / (double)nmean, rs = 1.0 / sqrt((double)nmean);
    const bool vec = ld % 4 == 0 && ((uintptr_t)O & 15) == 0;
    const long chunk = 65535L * rpb;  // rows per launch (grid y limit)
    for (long r0 = 0; r0 < n; r0 += chunk) {
        const long m = n - r0 < chunk ? n - r0 : chunk;
        const dim3 g((unsigned)cb, (unsigned)((m + rpb - 1) / rpb));
        const int8_t* sr = s + r0 * d.N;
        const R* tr = (const R*)tact + r0 * d.Mw;
        R* orow = (R*)O + r0 * ld;
        if (vec)
            k_jac_rows<R, CENTER, true><<<g, 256, 0, st>>>(d, sr, tr, m, rpb, inv, rs, P, ld,
                                                                  cs, orow);
        else
            k_jac_rows<R, CENTER, false><<<g, 256, 0, st>>>(d, sr, tr, m, rpb, inv, rs, P,
                                                                   ld, cs, orow);
    }
}
void launch_jacobian(hipStream_t st, const Dims& d, int prec, const int8_t* s, const void* tact,
                     long n, void* O, int P, long ld) {
    if (n <= 0) return;
    if (prec == 0) jac_rows<double, false>(st, d, s, tact, n, n, O, P, ld, nullptr);
    else jac_rows<float, false>(st, d, s, tact, n, n, O, P, ld, nullptr);
}
// `n` rows of a centred, scaled Jacobian over nmean samples with column sums cs
void launch_jacobian_centred(hipStream_t st, const Dims& d, int prec, const int8_t* s,
                             const void* tact, long n, long nmean, void* O, int P, long ld,
                             const double* cs) {
    if (n <= 0) return;
    if (prec == 0) jac_rows<double, true>(st, d, s, tact, n, nmean, O, P, ld, cs);
    else jac_rows<float, true>(st, d, s, tact, n, nmean, O, P, ld, cs);
}
// all n rows as operand fragments of the BF16 Gram, (n + 31) / 32 * 32 rows
void launch_jacobian_frags(hipStream_t st, const Dims& d, const int8_t* s, const float* tact, long n,
                           void* F, int P, long ld, const double* cs) {
    const int nct = (int)(ld / 16), nkb = (int)((n + 31) / 32);
    int kbs = 16;  // k-blocks per wave: enough blocks first
    while (kbs > 1 && (long)((nct + 3) / 4) * ((nkb + kbs - 1) / kbs) < 2048) kbs /= 2;
    k_jac_frags<<<dim3((nct + 3) / 4, (nkb + kbs - 1) / kbs), 256, 0, st>>>(
        d, s, tact, n, nkb, kbs, 1.0 / (double)n, 1.0 / sqrt((double)n), P, nct, cs, (uint4*)F);
}

void launch_center_cols(hipStream_t st, double* O, long n, long ld, int P, double* cs,
                        double* scratch, size_t scratch_bytes) {
    const int nb = (P + 255) / 256;
    const long fit = (long)(scratch_bytes / (8 * (size_t)P)), want = (n + CS_ROWS - 1) / CS_ROWS;
    const int splits = (int)(want < fit ? want : (fit < 1 ? 1 : fit));
    k_colsum_part<<<dim3(nb, splits), 256, 0, st>>>(O, n, ld, P, splits, scratch);
    k_colsum_fin<<<(P + 63) / 64, 256, 0, st>>>(scratch, P, splits, cs);
    const int vec = (ld % 4 == 0 && ((uintptr_t)O & 15) == 0) ? 1 : 0;
    const dim3 g2(vec ? (P + 1023) / 1024 : nb, (unsigned)n);
    k_center_scale<<<g2, 256, 0, st>>>(O, n, ld, P, cs, vec);
}

// Edge of the BF16 Gram's tiles: 256 where nothing reads the mirrored half (a tile on
// the diagonal holds two of G's 128 x 128 tiles of one triangle) and they are enough
// for half the compute units (4,096 samples: P = 4,224, 153 tiles of 256, 271 us, 326
// with 128; 3,320, 91 tiles, 254, 180 with 128).
int gram_edge(int P, bool mirror) {
    const int nt = (P + 255) / 256;
    return !mirror && nt * (nt + 1) / 2 >= 128 ? 256 : 128;
}
int gram_tiles(int P, int edge) {
    const int nt = (P + edge - 1) / edge;
    return nt * (nt + 1) / 2;
}
// Tile order, XCD-aware.  The hardware deals consecutive blocks to the 8 XCDs
// in turn, so block 8 i + e runs on XCD e.  The upper block triangle is cut into
// GT_SUPER x GT_SUPER supertiles, dealt to the XCDs in turn; each XCD runs its
// supertiles one after the other, so the blocks resident on one XCD at a time
// (about 64) share GT_SUPER row panels and GT_SUPER column panels in its L2
// instead of each streaming a panel of its own.  Every tile appears once; the
// ragged end (XCDs with fewer tiles) is filled in order.
constexpr int GT_XCD = 8, GT_SUPER = 8;
void fill_gram_tiles(int P, int edge, int* host_tiles) {
    const int nt = (P + edge - 1) / edge, ns = (nt + GT_SUPER - 1) / GT_SUPER;
    std::vector<std::vector<int>> seq(GT_XCD);
    int sid = 0;
    for (int A = 0; A < ns; ++A)
        for (int B = A; B < ns; ++B, ++sid) {
            std::vector<int>& q = seq[sid % GT_XCD];
            for (int a = A * GT_SUPER; a < (A + 1) * GT_SUPER && a < nt; ++a)
                for (int b = B * GT_SUPER; b < (B + 1) * GT_SUPER && b < nt; ++b)
                    if (b >= a) {
                        q.push_back(a);
                        q.push_back(b);
                    }
        }
    size_t pos[GT_XCD] = {0};
    const long total = (long)nt * (nt + 1) / 2;
    long e = 0;
    while (e < total) {  // slot e goes to XCD e % 8 while that XCD has tiles left
        int src = (int)(e % GT_XCD);
        for (int tries = 0; tries < GT_XCD && pos[src] >= seq[src].size(); ++tries)
            src = (src + 1) % GT_XCD;
        host_tiles[2 * e] = seq[src][pos[src]];
        host_tiles[2 * e + 1] = seq[src][pos[src] + 1];
        pos[src] += 2;
        ++e;
    }
}
// Row slices for the FP64 Gram: enough (tile, slice) blocks for two per compute
// unit, each slice at least 128 rows; 1 = the unsliced kernel.
int gram_slices(int ntiles, long n) {
    int S = 1;
    while (S < 256 && (long)ntiles * S < 512 && n / (2 * S) >= 128) S *= 2;
    return S;
}
size_t gram_part_bytes(int ntiles, int slices) {
    return slices > 1 ? (size_t)ntiles * slices * 128 * 128 * 8 : 0;
}
void launch_gram_sliced(hipStream_t st, const double* A, long n, long ld, int P, double* G,
                        const int* tiles, int ntiles, int slices, double* part) {
    if (slices <= 1 || !part) {
        k_gram<double, 4, 1, 1><<<ntiles, 256, 0, st>>>(A, n, ld, P, G, tiles, true);
        return;
    }
    long rps = (n + slices - 1) / slices;
    rps = (rps + 3) / 4 * 4;
    k_gram_slices<<<(unsigned)(ntiles * slices), 256, 0, st>>>(A, n, ld, ntiles, rps, tiles, part);
    k_gram_fin<<<(unsigned)(ntiles * 256), 256, 0, st>>>(part, ntiles, slices, tiles, P, ld, G);
}
// Up to one tile of 128 per compute unit, four blocks of 64 x 64 share it: they wait for
// the same loads with a quarter of the products each.  4,096 samples, BF16 form: 860
// columns (28 tiles) 43 us, 106 with whole tiles; 2,143 (153) 99, 115; 3,320 (351) 205,
// 179; FP32: 135; 360; 694, 680.
constexpr int GRAM_SMALL = 256;
void launch_gram(hipStream_t st, const float* A, long n, long ld, int P, float* G, const int* tiles,
                 int ntiles, bool mirror) {
    if (ntiles > GRAM_SMALL)
        k_gram<float, 4, 1, 1><<<ntiles, 256, 0, st>>>(A, n, ld, P, G, tiles, mirror);
    else
        k_gram<float, 2, 8, 2><<<4 * ntiles, 256, 0, st>>>(A, n, ld, P, G, tiles, mirror);
}
void launch_gram_frags(hipStream_t st, const void* F, long n, long ld, int P, float* G,
                       const int* tiles, int ntiles, int edge, bool mirror) {
    const int nkb = (int)((n + 31) / 32), nct = (int)(ld / 16);
    const u32x4* f = (const u32x4*)F;
    if (edge == 256) {
        const size_t lds = 2 * 32 * 2048;
        (void)hipFuncSetAttribute((const void*)k_gram_frags<2, 4, 8, 4, 1, 1>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        k_gram_frags<2, 4, 8, 4, 1, 1><<<ntiles, 512, lds, st>>>(f, nkb, nct, ld, P, G, tiles, mirror);
    } else if (ntiles > GRAM_SMALL) {
        k_gram_frags<2, 2, 4, 4, 2, 1><<<ntiles, 256, 2 * 16 * 2048, st>>>(f, nkb, nct, ld, P, G,
                                                                          tiles, mirror);
    } else {
        k_gram_frags<2, 2, 2, 2, 2, 2><<<4 * ntiles, 256, 2 * 8 * 2048, st>>>(f, nkb, nct, ld, P, G,
                                                                             tiles, mirror);
    }
}
void launch_dense_matvec(hipStream_t st, int prec, const void* G, int P, long ld, const double* v,
                         double* out, double* dpart, const CgScalars* sc, int tri, void* scratch) {
    if (prec == 0)
        dense_matvec(st, (const double*)G, P, ld, v, out, dpart, sc, tri, (double*)scratch);
    else
        dense_matvec(st, (const float*)G, P, ld, v, out, dpart, sc, tri, (double*)scratch);
}

}  // namespace nqs
