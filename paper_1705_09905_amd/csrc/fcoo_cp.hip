// CP-ALS dense steps (Algorithm 1): Gram products on the matrix cores, the
// R x R float64 solve, the row solve with column normalisation, the fit, and
// the sweep driver fcoo_cp_als_iter.
//
// Per mode n of a sweep: M = SpMTTKRP_n (segmented-scan kernels);
// V = Hadamard product of the Grams G_m, m != n (float64);
// W = V^-1 by Gauss-Jordan elimination (its pivots are the squared pivots of
// the Cholesky factorisation V = L L^T), or the pseudo-inverse from a
// symmetric eigendecomposition (cyclic Jacobi) when V is not numerically
// positive definite; A_n = M W with column 2-norms lambda,
// A_n / lambda stored as float32 or bfloat16 (round to nearest even);
// G_n = A_n^T A_n from the stored values.  After the last mode:
// fit = 1 - sqrt(max(0, |X|^2 + |Xhat|^2 - 2 <X, Xhat>)) / |X|, with
// |Xhat|^2 = lambda^T (Hadamard of all Grams) lambda and
// <X, Xhat> = sum_r lambda_r sum_i M_{N-1}(i, r) A_{N-1}(i, r).
// Every reduction runs in a fixed order: results are bitwise repeatable.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "fcoo_device.h"
#include "fcoo_internal.h"

namespace fcoo {
namespace dev {

// rows that the row solve sums in float32 before they go to float64 with bfloat16
// factors: the order of sums that CP-ALS keeps there, see TileProblem::keep_order
constexpr int kGramChain = 256;
constexpr int kMaxCpR = 64;            // R bound of the in-LDS solve

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef short shortx4 __attribute__((ext_vector_type(4)));

// Partial Gram of `rows` rows (float32: 256 or 1024; bfloat16: 1024) for the 32 x 32
// tile pair (tr, tc): each wave accumulates its quarter of the rows on the matrix
// cores (float32 inputs: 32x32x2; bfloat16: 32x32x8), the four waves are summed in
// float64 and written to partial[blk][R x R].  The operands of the next GU matrix
// steps are loaded while the current ones run.  (Shorter chains in float32, added
// up every 64 rows, cost 10-20%: 1.1M rows, R = 12, 58 us.)
template <typename FT>
__global__ __launch_bounds__(256) void gram_partial_kernel(const FT *__restrict__ A, int64_t I, int R, int rows,
                                                           double *__restrict__ partial)
{
    __shared__ float red[4][32][33];
    const int ntile = (R + 31) / 32;
    const int tr = blockIdx.y / ntile, tc = blockIdx.y % ntile;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t r0 = (int64_t)blockIdx.x * rows + (int64_t)w * (rows / 4);
    int64_t r1 = r0 + rows / 4;
    if (r1 > I) r1 = I;
    const int ca = tr * 32 + (lane & 31), cb = tc * 32 + (lane & 31);
    const bool va = ca < R, vb = cb < R;
    const int kk = lane >> 5;
    floatx16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    constexpr int GU = 8;                                    // matrix steps per operand batch
    if constexpr (sizeof(FT) == 4) {
        const float *Af = reinterpret_cast<const float *>(A);
        constexpr int STEP = 2 * GU;                         // rows per batch
        auto ld = [&](int64_t i, float (&a)[GU], float (&b)[GU]) {
#pragma unroll
            for (int u = 0; u < GU; ++u) {
                const int64_t row = i + 2 * u + kk;
                a[u] = (row < r1 && va) ? Af[row * R + ca] : 0.f;
                b[u] = (row < r1 && vb) ? Af[row * R + cb] : 0.f;
            }
        };
        float a0[GU], b0v[GU];
        ld(r0, a0, b0v);
        for (int64_t i = r0; i < r1; i += STEP) {
            float a1[GU], b1[GU];
            ld(i + STEP, a1, b1);
#pragma unroll
            for (int u = 0; u < GU; ++u) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a0[u], b0v[u], acc, 0, 0, 0);
#pragma unroll
            for (int u = 0; u < GU; ++u) { a0[u] = a1[u]; b0v[u] = b1[u]; }
        }
    } else {
        const uint16_t *Ab = reinterpret_cast<const uint16_t *>(A);
        constexpr int GB = GU / 2;
        constexpr int STEP = 8 * GB;
        auto ld = [&](int64_t i, shortx4 (&a)[GB], shortx4 (&b)[GB]) {
#pragma unroll
            for (int u = 0; u < GB; ++u) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int64_t row = i + 8 * u + 4 * kk + t;
                    a[u][t] = (short)((row < r1 && va) ? Ab[row * R + ca] : 0);
                    b[u][t] = (short)((row < r1 && vb) ? Ab[row * R + cb] : 0);
                }
            }
        };
        shortx4 a0[GB], b0v[GB];
        ld(r0, a0, b0v);
        for (int64_t i = r0; i < r1; i += STEP) {
            shortx4 a1[GB], b1[GB];
            ld(i + STEP, a1, b1);
#pragma unroll
            for (int u = 0; u < GB; ++u) acc = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(a0[u], b0v[u], acc, 0, 0, 0);
#pragma unroll
            for (int u = 0; u < GB; ++u) { a0[u] = a1[u]; b0v[u] = b1[u]; }
        }
    }
    // accumulator v of lane l holds tile element (8 (v/4) + 4 (l/32) + v%4, l%32)
#pragma unroll
    for (int v = 0; v < 16; ++v) red[w][8 * (v >> 2) + 4 * kk + (v & 3)][lane & 31] = acc[v];
    __syncthreads();
    for (int e = threadIdx.x; e < 32 * 32; e += 256) {
        const int i = e >> 5, jj = e & 31;
        const int gi = tr * 32 + i, gj = tc * 32 + jj;
        if (gi < R && gj < R) {
            const double s = ((double)red[0][i][jj] + (double)red[1][i][jj]) + ((double)red[2][i][jj] + (double)red[3][i][jj]);
            partial[(int64_t)blockIdx.x * R * R + (int64_t)gi * R + gj] = s;
        }
    }
}

// out[e] = sum_b partial[b][e] (b < nblk): X elements x Y strided shares of the
// blocks per workgroup, the shares added in a fixed order, so repeatable.
template <int X, int Y>
__global__ __launch_bounds__(X * Y) void sum_blocks_kernel(const double *__restrict__ partial, int64_t nblk,
                                                           int64_t n_per, double *__restrict__ out)
{
    __shared__ double red[Y][X];
    const int x = threadIdx.x % X, y = threadIdx.x / X;
    const int64_t e = (int64_t)blockIdx.x * X + x;
    double s = 0.0;
    if (e < n_per) {
        for (int64_t b = y; b < nblk; b += 8 * Y) {
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = b + Y * u < nblk ? partial[(b + Y * u) * n_per + e] : 0.0;
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
    }
    red[y][x] = s;
    __syncthreads();
    for (int o = Y / 2; o >= 8; o >>= 1) {
        if (y < o) red[y][x] += red[y + o][x];
        __syncthreads();
    }
    if (y == 0 && e < n_per) {
        s = red[0][x];
        for (int k = 1; k < 8; ++k) s += red[k][x];
        out[e] = s;
    }
}

// One workgroup: V = Hadamard of the Grams but mode n; W = V^-1 by
// Gauss-Jordan elimination without row exchanges (the pivots are the
// Schur-complement diagonal, i.e. the squared Cholesky pivots of V = L L^T), or
// V^+ from a cyclic Jacobi eigendecomposition when a pivot is <= 0 or below
// 1e-13 * max(diag V).  flags[n] = 1 when the pseudo-inverse was used.
// R <= 4 RPL <= kMaxCpR.  Wave q holds rows q, q + 4, ... in registers, lane k
// column k: a step passes the pivot row through LDS (one barrier; the buffers
// alternate) and takes the pivot column by lane reads.  (With the matrix in LDS
// and three barriers a step it took 61 us at R = 32; 21 now.)  The Jacobi fallback works in LDS, its eigenvectors in tmp (R x R).
__device__ void form_hadamard(const double *__restrict__ grams, int N, int n, int R,
                              double (*V)[kMaxCpR + 1])
{
    for (int e = threadIdx.x; e < R * R; e += blockDim.x) {
        double h = 1.0;
        for (int m = 0; m < N; ++m)
            if (m != n) h *= grams[(int64_t)m * R * R + e];
        V[e / R][e % R] = h;
    }
}

__device__ __forceinline__ double lane_value(double x, int lane)
{
    const uint64_t u = __double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
    return __longlong_as_double(((uint64_t)hi << 32) | lo);
}

template <int RPL>
__global__ __launch_bounds__(256) void als_solve_kernel(const double *__restrict__ grams, int N, int n,
                                                        int R, double *__restrict__ W,
                                                        double *__restrict__ tmp, int *__restrict__ flags)
{
    __shared__ double V[kMaxCpR][kMaxCpR + 1];
    __shared__ double prow[2][kMaxCpR];
    __shared__ double cs_s[4];
    const int tid = threadIdx.x;
    const int k = tid & 63;                         // column of this lane
    const int q = tid >> 6;                         // rows q, q + 4, q + 8, ... of that column
    double a[RPL];
    double dmax = 0.0;
#pragma unroll
    for (int u = 0; u < RPL; ++u) {
        const int i = q + 4 * u;
        double h = 0.0;
        if (i < R && k < R) {
            h = 1.0;
            for (int m = 0; m < N; ++m)
                if (m != n) h *= grams[(int64_t)m * R * R + i * R + k];
        }
        a[u] = h;
        if (i < R) {
            const double d = lane_value(h, i);
            dmax = d > dmax ? d : dmax;
        }
    }
    if (k == 0) cs_s[q] = dmax;
    __syncthreads();
    for (int i = 0; i < 4; ++i) dmax = cs_s[i] > dmax ? cs_s[i] : dmax;
    bool fail = false;
#pragma unroll
    for (int u0 = 0; u0 < RPL; ++u0) {
        for (int qq = 0; qq < 4 && !fail; ++qq) {
            const int j = 4 * u0 + qq;
            if (j >= R) break;
            double *pr = prow[j & 1];
            if (q == qq) pr[k] = a[u0];
            __syncthreads();
            const double p = pr[j];                  // Schur-complement pivot (same on every lane)
            if (!(p > 0.0) || p <= 1e-13 * dmax) { fail = true; break; }
            const double ip = 1.0 / p;
            const double rjk = pr[k] * ip;
            // rows i != j: a - c_i rjk (column j: -c_i / p); row j: rjk (1 / p)
#pragma unroll
            for (int u = 0; u < RPL; ++u) {
                const double c = lane_value(a[u], j);
                const double t = a[u] - c * rjk;
                const double tc = -c * ip;
                const bool own = u == u0 && q == qq;
                a[u] = own ? (k == j ? ip : rjk) : (k == j ? tc : t);
            }
        }
    }
    if (!fail) {
#pragma unroll
        for (int u = 0; u < RPL; ++u) {
            const int i = q + 4 * u;
            if (i < R && k < R) W[i * R + k] = a[u];
        }
        if (tid == 0) flags[n] = 0;
        return;
    }
    // ---- pseudo-inverse: cyclic Jacobi on V (symmetric), eigenvectors in tmp
    __syncthreads();
    form_hadamard(grams, N, n, R, V);
    for (int e = tid; e < R * R; e += 256) tmp[e] = (e / R == e % R) ? 1.0 : 0.0;
    __syncthreads();
    for (int sweep = 0; sweep < 30; ++sweep) {
        for (int p = 0; p < R - 1; ++p) {
            for (int q = p + 1; q < R; ++q) {
                if (tid == 0) {
                    const double apq = V[p][q];
                    double c = 1.0, sn = 0.0;
                    if (fabs(apq) > 1e-300) {
                        const double theta = (V[q][q] - V[p][p]) / (2.0 * apq);
                        const double t = (theta >= 0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
                        c = 1.0 / sqrt(t * t + 1.0);
                        sn = t * c;
                    }
                    cs_s[0] = c;
                    cs_s[1] = sn;
                }
                __syncthreads();
                const double c = cs_s[0], sn = cs_s[1];
                if (sn != 0.0) {
                    // V <- J^T V J, J the rotation in the (p, q) plane; eigenvectors <- Q J
                    for (int k = tid; k < R; k += 256) {
                        const double vkp = V[k][p], vkq = V[k][q];
                        V[k][p] = c * vkp - sn * vkq;
                        V[k][q] = sn * vkp + c * vkq;
                    }
                    __syncthreads();
                    for (int k = tid; k < R; k += 256) {
                        const double vpk = V[p][k], vqk = V[q][k];
                        V[p][k] = c * vpk - sn * vqk;
                        V[q][k] = sn * vpk + c * vqk;
                        const double qkp = tmp[k * R + p], qkq = tmp[k * R + q];
                        tmp[k * R + p] = c * qkp - sn * qkq;
                        tmp[k * R + q] = sn * qkp + c * qkq;
                    }
                }
                __syncthreads();
            }
        }
        // stop once the off-diagonal mass is negligible
        if (tid == 0) {
            double off = 0.0, dia = 0.0;
            for (int i = 0; i < R; ++i)
                for (int j = 0; j < R; ++j) {
                    if (i == j) dia += V[i][j] * V[i][j];
                    else off += V[i][j] * V[i][j];
                }
            cs_s[0] = (off <= 1e-30 * (dia > 0 ? dia : 1.0)) ? 1.0 : 0.0;
        }
        __syncthreads();
        const bool done = cs_s[0] != 0.0;
        __syncthreads();
        if (done) break;
    }
    double dm = 0.0;
    for (int i = 0; i < R; ++i) dm = V[i][i] > dm ? V[i][i] : dm;
    const double cut = (double)R * 2.220446049250313e-16 * dm;
    __syncthreads();
    for (int e = tid; e < R * R; e += 256) {
        const int i = e / R, j = e % R;
        double se = 0.0;
        for (int k = 0; k < R; ++k) {
            const double d = V[k][k];
            if (d > cut) se += tmp[i * R + k] * tmp[j * R + k] / d;
        }
        W[e] = se;
    }
    if (tid == 0) flags[n] = 1;
}


// Row solve, Y = M W (I x R, float64 accumulation), in row tiles of M staged in
// LDS, RC = R rounded up to a power of two (R <= kMaxCpR).  A thread has NY
// elements of a tile's Y, all of one column.  From RC = 16 on they come from the
// matrix cores (16x16x4 float64; a wave has one 16 x 16 block of the tile, and its
// columns of W in registers), below from a loop over W in LDS.  A workgroup takes
// tiles_per_block tiles, the next one's rows of M in flight meanwhile, so that what
// is summed over workgroups is short enough for the next pass to sum in each of
// its own:
//   rownorm_kernel:  per block, the column sums of Y^2 -> partial[blk][R];
//   rowstore_kernel: lambda_c = sqrt(sum_b partial[b][c]); A(i, c) = Y(i, c) /
//                    lambda_c (0 when lambda_c = 0) stored as FT (bfloat16: round
//                    to nearest even); the block's share of A^T A from the
//                    stored values on the matrix cores -> gpart[blk][R x R], if
//                    given; and (ipart) of the fit's sum_i sum_r lambda_r M(i, r)
//                    A(i, r).
// (As five kernels -- norms, lambda, store, partial Gram, inner product -- they
// took 11 + 5 + 10 + 13 us a mode, 14 the last, over the modes of 50k to 1k rows
// at R = 32, now 6 + 14; for 200 rows at R = 8 21 us, now 8.  Products by a loop
// over W and M in LDS, 4 rows a thread, waited on those reads: R = 48, modes of
// 108k, 41k, 24k and 4k rows, 37 + 45 us a mode, now 18 + 26.)
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

typedef double doublex4 __attribute__((ext_vector_type(4)));

// TH threads: 1024; 256 for few short rows, whose tiles would be few (RC <= 8)
template <int RC, int TH> struct RowTile {
    static constexpr bool MAT = RC >= 16;
    static constexpr int SLOTS = TH / RC;                     // threads of a column
    static constexpr int NY = MAT ? 4 : SLOTS < 64 ? 64 / SLOTS : 1;
    static constexpr int ROWS = SLOTS * NY;                   // rows per tile (64 .. 1024)
    static constexpr int LD = RC >= 4 ? RC + 4 : RC;          // row stride of M's tile in LDS
    int slot, c;                                              // this thread's
    int lane, rt;
    __device__ RowTile()
    {
        lane = threadIdx.x & 63;
        const int w = threadIdx.x >> 6;
        if constexpr (MAT) {
            // block (rt, ct) of the wave: register v of lane (g, m) is element (4 v + g, m)
            rt = w / (RC / 16);
            c = w % (RC / 16) * 16 + (lane & 15);
            slot = rt * 4 + (lane >> 4);
        } else {
            rt = 0;
            slot = threadIdx.x / RC;
            c = threadIdx.x % RC;
        }
    }
    // tile row of element u
    __device__ int row(int u) const { return MAT ? rt * 16 + 4 * u + (lane >> 4) : u * SLOTS + slot; }
};

// W for a thread's products: its column's elements (MAT), or all of it in LDS
template <int RC, int TH> struct RowW {
    static constexpr bool MAT = RC >= 16;
    double w[MAT ? RC / 4 : 1];
    const double *sW;
    __device__ RowW(const RowTile<RC, TH> &t, const double *__restrict__ W, int R, double *lds) : sW(lds)
    {
        if constexpr (MAT) {
#pragma unroll
            for (int q = 0; q < RC / 4; ++q) {
                const int k = 4 * q + (t.lane >> 4);
                w[q] = (k < R && t.c < R) ? W[k * R + t.c] : 0.0;
            }
        } else {
            for (int e = threadIdx.x; e < RC * RC; e += TH) {
                const int k = e / RC, cc = e % RC;
                lds[e] = (k < R && cc < R) ? W[k * R + cc] : 0.0;
            }
        }
    }
    // y[u] = (row t.row(u) of the tile) . (column t.c of W)
    __device__ void products(const RowTile<RC, TH> &t, const float *sM, double (&y)[RowTile<RC, TH>::NY]) const
    {
        using RT = RowTile<RC, TH>;
        if constexpr (MAT) {
            doublex4 d = {0.0, 0.0, 0.0, 0.0};
            const float *m = sM + (t.rt * 16 + (t.lane & 15)) * RT::LD + (t.lane >> 4);
#pragma unroll
            for (int q = 0; q < RC / 4; ++q)
                d = __builtin_amdgcn_mfma_f64_16x16x4f64((double)m[4 * q], w[q], d, 0, 0, 0);
#pragma unroll
            for (int u = 0; u < 4; ++u) y[u] = d[u];
        } else {
#pragma unroll
            for (int u = 0; u < RT::NY; ++u) y[u] = 0.0;
#pragma unroll
            for (int k = 0; k < RC; ++k) {
                const double wk = sW[k * RC + t.c];
#pragma unroll
                for (int u = 0; u < RT::NY; ++u) y[u] += (double)sM[t.row(u) * RT::LD + k] * wk;
            }
        }
    }
};

// rows [i0, i0 + ROWS) of M into registers, zeros past row I and column R, and from
// there to LDS
template <int RC, int TH>
__device__ __forceinline__ void fetch_m(const float *__restrict__ M, int64_t i0, int64_t I, int R,
                                        float (&m)[RowTile<RC, TH>::NY])
{
#pragma unroll
    for (int u = 0; u < RowTile<RC, TH>::NY; ++u) {
        const int e = threadIdx.x + u * TH, r = e / RC, cc = e % RC;
        m[u] = (i0 + r < I && cc < R) ? M[(i0 + r) * R + cc] : 0.f;
    }
}

template <int RC, int TH>
__device__ __forceinline__ void stage_m(const float (&m)[RowTile<RC, TH>::NY], float *sM)
{
#pragma unroll
    for (int u = 0; u < RowTile<RC, TH>::NY; ++u) {
        const int e = threadIdx.x + u * TH;
        sM[e / RC * RowTile<RC, TH>::LD + e % RC] = m[u];
    }
}

template <int RC, int TH>
__global__ __launch_bounds__(TH) void rownorm_kernel(const float *__restrict__ M, const double *__restrict__ W,
                                                     int64_t I, int R, int tiles_per_block,
                                                     double *__restrict__ partial)
{
    using RT = RowTile<RC, TH>;
    __shared__ double sW[RT::MAT ? 1 : RC * RC];
    __shared__ float sM[RT::ROWS * RT::LD];
    __shared__ double red[TH];
    const RT t;
    const int64_t first = (int64_t)blockIdx.x * tiles_per_block * RT::ROWS;
    const int64_t last = first + (int64_t)tiles_per_block * RT::ROWS < I ? first + (int64_t)tiles_per_block * RT::ROWS : I;
    float m[RT::NY];
    fetch_m<RC, TH>(M, first, I, R, m);
    const RowW<RC, TH> w(t, W, R, sW);
    double ss = 0.0;
    for (int64_t i0 = first; i0 < last; i0 += RT::ROWS) {
        __syncthreads();                                   // sW written / previous tile consumed
        stage_m<RC, TH>(m, sM);
        __syncthreads();
        if (i0 + RT::ROWS < last) fetch_m<RC, TH>(M, i0 + RT::ROWS, I, R, m);
        double y[RT::NY];
        w.products(t, sM, y);
#pragma unroll
        for (int u = 0; u < RT::NY; ++u) ss += y[u] * y[u];   // rows and columns past the end are 0
    }
    red[t.slot * RC + t.c] = ss;
    __syncthreads();
    if ((int)threadIdx.x < R) {
        double s = 0.0;
        for (int k = 0; k < RT::SLOTS; ++k) s += red[k * RC + threadIdx.x];
        partial[(int64_t)blockIdx.x * R + threadIdx.x] = s;
    }
}

template <typename FT, int RC, int TH>
__global__ __launch_bounds__(TH) void rowstore_kernel(const float *__restrict__ M, const double *__restrict__ W,
                                                      const double *__restrict__ partial, int64_t I, int R,
                                                      int tiles_per_block, double *__restrict__ lambda,
                                                      FT *__restrict__ A, double *__restrict__ gpart,
                                                      double *__restrict__ ipart)
{
    using RT = RowTile<RC, TH>;
    __shared__ double sW[RT::MAT ? 1 : RC * RC];
    __shared__ float sM[RT::ROWS * RT::LD];                    // M's tile, then the stored rows
    __shared__ double red[TH];
    __shared__ double sLam[RC];
    __shared__ double gbuf[RC <= 32 ? 1024 : 4096];
    const RT t;
    const int tid = threadIdx.x;
    const int64_t first = (int64_t)blockIdx.x * tiles_per_block * RT::ROWS;
    const int64_t last = first + (int64_t)tiles_per_block * RT::ROWS < I ? first + (int64_t)tiles_per_block * RT::ROWS : I;
    float m[RT::NY];
    fetch_m<RC, TH>(M, first, I, R, m);
    const RowW<RC, TH> wgt(t, W, R, sW);
    {   // lambda, in the same order in every workgroup
        double s = 0.0;
        const int nblk = gridDim.x;
        if (t.c < R)
            for (int b = t.slot; b < nblk; b += 8 * RT::SLOTS) {
                double v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = b + u * RT::SLOTS < nblk ? partial[(int64_t)(b + u * RT::SLOTS) * R + t.c] : 0.0;
#pragma unroll
                for (int u = 0; u < 8; ++u) s += v[u];
            }
        red[t.slot * RC + t.c] = s;
        __syncthreads();
        if (tid < RC) {
            double l = 0.0;
            for (int k = 0; k < RT::SLOTS; ++k) l += red[k * RC + tid];
            l = tid < R ? sqrt(l) : 0.0;
            sLam[tid] = l;
            if (blockIdx.x == 0 && tid < R) lambda[tid] = l;
        }
        __syncthreads();
    }
    const double lam = sLam[t.c];
    double inner = 0.0;
    // this wave's part of the block's Gram: a share of the rows of the one 32 x 32
    // tile, or with RC = 64 of tile (w / 2 % 2, w % 2).  bfloat16 keeps the order of
    // sums of gram_partial_kernel (wave 0, or with RC = 64 waves 0 .. 3, 8 rows a step,
    // in float32 over each 256 rows: a block's rows are whole numbers of them)
    const int lane = tid & 63, w = tid >> 6, kk = lane >> 5;
    const int ca = (RC <= 32 ? 0 : (w >> 1 & 1) * 32) + (lane & 31), cb = (RC <= 32 ? 0 : (w & 1) * 32) + (lane & 31);
    constexpr int NW = TH / 64, GP = RC <= 32 ? NW : NW / 4;   // waves, waves per tile
    constexpr int GR = RT::ROWS / GP;
    const int g0 = (RC <= 32 ? w : w >> 2) * GR;
    double gsum[16];
    floatx16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) { gsum[v] = 0.0; acc[v] = 0.f; }
    auto flush = [&]() {
#pragma unroll
        for (int v = 0; v < 16; ++v) { gsum[v] += (double)acc[v]; acc[v] = 0.f; }
    };
    for (int64_t i0 = first; i0 < last; i0 += RT::ROWS) {
        const int nrow = I - i0 < RT::ROWS ? (int)(I - i0) : RT::ROWS;
        __syncthreads();                                   // previous tile consumed
        stage_m<RC, TH>(m, sM);
        __syncthreads();
        if (i0 + RT::ROWS < last) fetch_m<RC, TH>(M, i0 + RT::ROWS, I, R, m);
        double y[RT::NY];
        wgt.products(t, sM, y);
        __syncthreads();                                   // from here each element is its own thread's
#pragma unroll
        for (int u = 0; u < RT::NY; ++u) {
            const int r = t.row(u);
            float f = lam > 0.0 ? (float)(y[u] / lam) : 0.f;
            const int64_t o = (i0 + r) * R + t.c;
            const bool in = r < nrow && t.c < R;
            if constexpr (sizeof(FT) == 4) {
                if (in) reinterpret_cast<float *>(A)[o] = f;
            } else {
                const uint16_t h = f32_to_bf16_rne(f);
                if (in) reinterpret_cast<uint16_t *>(A)[o] = h;
                f = bf16_to_f32(h);
            }
            if (ipart && in) inner += lam * (double)sM[r * RT::LD + t.c] * (double)f;
            sM[r * RT::LD + t.c] = in ? f : 0.f;
        }
        if (!gpart) continue;
        __syncthreads();
        if constexpr (sizeof(FT) == 2) {
            if (w >= (RC <= 32 ? 1 : 4)) continue;
#pragma unroll 4
            for (int i = 0; i < RT::ROWS; i += 8) {
                shortx4 av, bv;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float *row = sM + (i + 4 * kk + k) * RT::LD;
                    av[k] = (short)(ca < RC ? __float_as_uint(row[ca]) >> 16 : 0u);
                    bv[k] = (short)(cb < RC ? __float_as_uint(row[cb]) >> 16 : 0u);
                }
                acc = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(av, bv, acc, 0, 0, 0);
                if ((i0 + i + 8) % kGramChain == 0) flush();
            }
            if (i0 + RT::ROWS >= I) flush();
            continue;
        }
#pragma unroll 8
        for (int i = 0; i < GR; i += 2) {
            const int row = (g0 + i + kk) * RT::LD;
            const float av = ca < RC ? sM[row + ca] : 0.f, bv = cb < RC ? sM[row + cb] : 0.f;
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av, bv, acc, 0, 0, 0);
        }
        flush();
    }
    if (gpart) {
        double *gp = gpart + (int64_t)blockIdx.x * R * R;
        // the waves' shares of a tile added in turn
        constexpr bool ONE = sizeof(FT) == 2;
        for (int k = 0; k < (ONE ? 1 : GP); ++k) {
            if ((RC <= 32 ? w : w >> 2) == k) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    double &x = gbuf[(RC <= 32 ? 0 : w & 3) * 1024 + (8 * (v >> 2) + 4 * kk + (v & 3)) * 32 + (lane & 31)];
                    x = k ? x + gsum[v] : gsum[v];
                }
            }
            __syncthreads();
        }
        for (int e = tid; e < R * R; e += TH) {
            const int gi = e / R, gj = e % R;
            gp[e] = gbuf[(RC <= 32 ? 0 : (gi >> 5) * 2 + (gj >> 5)) * 1024 + (gi & 31) * 32 + (gj & 31)];
        }
    }
    if (ipart) {
        __syncthreads();                                       // red has been read
        red[tid] = inner;
        __syncthreads();
        for (int o = TH / 2; o >= 1; o >>= 1) {
            if (tid < o) red[tid] += red[tid + o];
            __syncthreads();
        }
        if (tid == 0) ipart[blockIdx.x] = red[0];
    }
}

// Fit (one workgroup), from the blocks' inner products.
__global__ __launch_bounds__(256) void fit_kernel(const double *__restrict__ partial, int64_t nblk,
                                                  const double *__restrict__ grams, int N, int R,
                                                  const double *__restrict__ lambda, double normX2,
                                                  double *__restrict__ fit)
{
    __shared__ double red[256];
    double s = 0.0;
    for (int64_t b = threadIdx.x; b < nblk; b += 256) s += partial[b];
    double x2 = 0.0;
    for (int e = threadIdx.x; e < R * R; e += 256) {
        double h = 1.0;
        for (int m = 0; m < N; ++m) h *= grams[(int64_t)m * R * R + e];
        x2 += lambda[e / R] * h * lambda[e % R];
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o >= 1; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    const double inner = red[0];
    __syncthreads();
    red[threadIdx.x] = x2;
    __syncthreads();
    for (int o = 128; o >= 1; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double xhat2 = red[0];
        double res2 = normX2 + xhat2 - 2.0 * inner;
        if (res2 < 0.0) res2 = 0.0;
        fit[0] = normX2 > 0.0 ? 1.0 - sqrt(res2) / sqrt(normX2) : 0.0;
    }
}

}  // namespace dev

static int ceil_div(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

static int pow2_ceil(int x)
{
    int p = 1;
    while (p < x) p <<= 1;
    return p;
}

// The row solve of an I x R mode: its threads, rows per tile, tiles per workgroup and
// workgroups.  bfloat16 past 262,144 rows leaves the Gram to gram_partial_kernel:
// one wave's chains of 256 rows, one after the other in each workgroup, take
// longer there (R = 7, modes of 1.7M, 93k and few rows: rowstore_kernel 430 us a sweep,
// without 107 and gram_partial_kernel 40).
struct RowPlan {
    int RC, TH, rows, tpb, nblk;
    bool gram;
};

static int cp_blocks(int RC) { return RC <= 16 ? 512 : 256; }   // (each sums the others' norms: R doubles each)

static RowPlan row_plan(int64_t I, int R, int dtype)
{
    RowPlan p;
    p.RC = pow2_ceil(R);
    p.TH = p.RC >= 16 || I > 65536 ? 1024 : 256;
    const int slots = p.TH / p.RC;
    p.rows = p.RC >= 16 ? 4 * slots : std::max(slots, 64);
    p.gram = dtype == FCOO_F32 || I <= 262144;
    const int ntiles = ceil_div(I, p.rows);
    // (bfloat16: whole chains of 256 rows a workgroup, see rowstore_kernel)
    const int chain = dtype == FCOO_F32 || !p.gram ? 1 : std::max(1, 256 / p.rows);
    p.tpb = chain * ceil_div(ceil_div(ntiles, cp_blocks(p.RC)), chain);
    p.nblk = ceil_div(ntiles, p.tpb);
    return p;
}

template <int RC, int TH>
static hipError_t rowsolve_th(const RowPlan &p, hipStream_t s, const float *M, const double *W, int64_t I, int R,
                              double *norms, double *lambda, void *A, int dtype, double *gpart, double *ipart)
{
    const dim3 g((unsigned)p.nblk), b(TH);
    hipLaunchKernelGGL((dev::rownorm_kernel<RC, TH>), g, b, 0, s, M, W, I, R, p.tpb, norms);
    if (dtype == FCOO_F32)
        hipLaunchKernelGGL((dev::rowstore_kernel<float, RC, TH>), g, b, 0, s, M, W, norms, I, R, p.tpb, lambda,
                           (float *)A, gpart, ipart);
    else
        hipLaunchKernelGGL((dev::rowstore_kernel<dev::bf16raw, RC, TH>), g, b, 0, s, M, W, norms, I, R, p.tpb, lambda,
                           (dev::bf16raw *)A, gpart, ipart);
    return hipGetLastError();
}

template <int RC>
static hipError_t rowsolve_rc(const RowPlan &p, hipStream_t s, const float *M, const double *W, int64_t I, int R,
                              double *norms, double *lambda, void *A, int dtype, double *gpart, double *ipart)
{
    if constexpr (RC < 16)
        if (p.TH == 256) return rowsolve_th<RC, 256>(p, s, M, W, I, R, norms, lambda, A, dtype, gpart, ipart);
    return rowsolve_th<RC, 1024>(p, s, M, W, I, R, norms, lambda, A, dtype, gpart, ipart);
}

// out = sum over nblk blocks of R x R partials: 32 elements a workgroup (whole
// 256-byte pieces per load), with few elements and many blocks 8
static hipError_t sum_blocks(const double *partial, int nblk, int R, double *out, hipStream_t s)
{
    const int n = R * R;
    const dim3 g((unsigned)((n + 31) / 32)), g8((unsigned)((n + 7) / 8));
    if (nblk <= 256)
        hipLaunchKernelGGL((dev::sum_blocks_kernel<32, 8>), g, dim3(256), 0, s, partial, (int64_t)nblk, (int64_t)n, out);
    else if (n > 1024)
        hipLaunchKernelGGL((dev::sum_blocks_kernel<32, 32>), g, dim3(1024), 0, s, partial, (int64_t)nblk, (int64_t)n, out);
    else
        hipLaunchKernelGGL((dev::sum_blocks_kernel<8, 128>), g8, dim3(1024), 0, s, partial, (int64_t)nblk, (int64_t)n, out);
    return hipGetLastError();
}

// Rows per Gram workgroup: 1024, or 256 where there are few (float32; bfloat16 has
// whole chains of its order of sums).
static int gram_rows(int64_t I, int dtype) { return dtype == FCOO_F32 && I <= 16384 ? 256 : 1024; }

// ... and its workgroups, of which a smaller I can have more
static int gram_blocks(int64_t I, int dtype) { return ceil_div(I, gram_rows(I, dtype)); }

// G = A^T A (float64) of an I x R factor; partials (gram_blocks x R x R) in gpart.
static int gram_launch(const void *A, int dtype, int64_t I, int R, double *gpart, double *G, hipStream_t s)
{
    const int rows = gram_rows(I, dtype), nblk = gram_blocks(I, dtype);
    const int ntile = (R + 31) / 32;
    if (dtype == FCOO_F32)
        hipLaunchKernelGGL(dev::gram_partial_kernel<float>, dim3(nblk, ntile * ntile), dim3(256), 0, s,
                           (const float *)A, I, R, rows, gpart);
    else
        hipLaunchKernelGGL(dev::gram_partial_kernel<dev::bf16raw>, dim3(nblk, ntile * ntile), dim3(256), 0, s,
                           (const dev::bf16raw *)A, I, R, rows, gpart);
    FCOO_HIP(hipGetLastError());
    FCOO_HIP(sum_blocks(gpart, nblk, R, G, s));
    return FCOO_OK;
}

// Whether mode n's solve runs beside its SpMTTKRP (it needs only the other modes'
// Grams), on a stream of its own.  The two waits between the streams cost as much
// as the solve takes at R = 32 (20 us) and four times that at R = 8, so only where it
// is longer and the SpMTTKRP is too: R > 32 with bfloat16 (R = 48, five modes, 2.3M
// nonzeros, a sweep: 1256 us in turn, beside it 1112), and where V is singular for sure,
// having at most as many dimensions as the other modes' extents have products, so
// that the solve is the eigendecomposition (R = 17, 253 x 5: 1426, 1313).
static bool solve_aside(const fcoo_tensor *t, int n, int R, int dtype)
{
    int64_t dim = 1;
    for (int m = 0; m < t->order && dim < R; ++m)
        if (m != n) dim *= t->dims[m];
    return dim < R || (dtype == FCOO_BF16 && R > 32);
}

static int aux_stream(fcoo_tensor *t)
{
    if (!t->aux) FCOO_HIP(hipStreamCreateWithFlags(&t->aux, hipStreamNonBlocking));
    if (!t->ev_dep) FCOO_HIP(hipEventCreateWithFlags(&t->ev_dep, hipEventDisableTiming));
    if (!t->ev_solved) FCOO_HIP(hipEventCreateWithFlags(&t->ev_solved, hipEventDisableTiming));
    return FCOO_OK;
}

}  // namespace fcoo

using namespace fcoo;

extern "C" {

int fcoo_gram(fcoo_tensor *t, int mode, const void *A, int dtype, int R, double *G, void *stream)
{
    clear_error();
    if (!t || !A || !G) return fail(FCOO_EINVAL, "null argument");
    if (mode < 0 || mode >= t->order) return fail(FCOO_EINVAL, "mode %d out of range", mode);
    if (dtype != FCOO_F32 && dtype != FCOO_BF16) return fail(FCOO_EUNSUPPORTED, "unknown dtype %d", dtype);
    if (R < 1 || R > kMaxR) return fail(FCOO_EUNSUPPORTED, "R = %d outside [1, %d]", R, kMaxR);
    hipStream_t s = (hipStream_t)stream;
    const int64_t I = t->dims[mode];
    const int rc = ensure_device_doubles(&t->ws.dbl, &t->ws.dbl_cap, (int64_t)gram_blocks(I, dtype) * R * R + 16, s);
    return rc ? rc : gram_launch(A, dtype, I, R, t->ws.dbl, G, s);
}

int fcoo_cp_als_iter(fcoo_tensor *t, void *const *factors, int dtype, int R, double *lambda,
                     double *grams, int grams_valid, double *fit, int *used_pinv, void *stream)
{
    clear_error();
    if (!t) return fail(FCOO_EINVAL, "null handle");
    int rc = check_factors(t, -1, (const void *const *)factors, dtype, R);
    if (rc) return rc;
    if (!lambda || !grams || !fit) return fail(FCOO_EINVAL, "lambda, grams or fit is NULL");
    if (R > dev::kMaxCpR) return fail(FCOO_EUNSUPPORTED, "cp_als_iter supports R <= %d (R = %d)", dev::kMaxCpR, R);
    const int N = t->order;
    for (int n = 0; n < N; ++n)
        if (!t->b[FCOO_OP_MTTKRP][n].built || !t->b[FCOO_OP_MTTKRP][n].on_device)
            return fail(FCOO_ENOTBUILT, "cp_als_iter needs the MTTKRP build of every mode (mode %d missing)", n);
    hipStream_t s = (hipStream_t)stream;
    int64_t maxI = 0;
    for (int n = 0; n < N; ++n) maxI = t->dims[n] > maxI ? t->dims[n] : maxI;
    if ((rc = ensure_device_floats(&t->ws.M, &t->ws.M_cap, maxI * R, s))) return rc;
    // scratch doubles: gram partials | W | tmp | column norms | inner products | fit, flags
    int most_blocks = cp_blocks(pow2_ceil(R));
    const int64_t norm_blocks = most_blocks;
    for (int n = 0; n < N; ++n) most_blocks = std::max(most_blocks, gram_blocks(t->dims[n], dtype));
    const int64_t gram_need = (int64_t)most_blocks * R * R + 16;
    const int64_t need = gram_need + 2 * (int64_t)R * R + norm_blocks * (R + 1) + 16;
    if ((rc = ensure_device_doubles(&t->ws.dbl, &t->ws.dbl_cap, need, s))) return rc;
    if (!t->ws.host_pinned) FCOO_HIP(hipHostMalloc((void **)&t->ws.host_pinned, 64, hipHostMallocDefault));
    double *gpart = t->ws.dbl;
    double *Wd = gpart + gram_need;
    double *tmpd = Wd + (int64_t)R * R;
    double *norms = tmpd + (int64_t)R * R;
    double *ipart = norms + norm_blocks * R;
    double *fitd = ipart + norm_blocks;
    int *flagd = reinterpret_cast<int *>(fitd + 1);

    if (!grams_valid)
        for (int m = 0; m < N; ++m)
            if ((rc = gram_launch(factors[m], dtype, t->dims[m], R, gpart, grams + (int64_t)m * R * R, s))) return rc;

    int nblk = 0;
    for (int n = 0; n < N; ++n) {
        const int64_t I = t->dims[n];
        const bool aside = solve_aside(t, n, R, dtype);
        hipStream_t ss = s;
        if (aside) {
            if ((rc = aux_stream(t))) return rc;
            ss = t->aux;
            FCOO_HIP(hipEventRecord(t->ev_dep, s));
            FCOO_HIP(hipStreamWaitEvent(ss, t->ev_dep, 0));
        } else if ((rc = spmttkrp(t, n, (const void *const *)factors, dtype, R, t->ws.M, dtype == FCOO_BF16, s))) {
            return rc;
        }
        if (R <= 16) hipLaunchKernelGGL(dev::als_solve_kernel<4>, dim3(1), dim3(256), 0, ss, grams, N, n, R, Wd, tmpd, flagd);
        else if (R <= 32) hipLaunchKernelGGL(dev::als_solve_kernel<8>, dim3(1), dim3(256), 0, ss, grams, N, n, R, Wd, tmpd, flagd);
        else hipLaunchKernelGGL(dev::als_solve_kernel<16>, dim3(1), dim3(256), 0, ss, grams, N, n, R, Wd, tmpd, flagd);
        FCOO_HIP(hipGetLastError());
        if (aside) {
            FCOO_HIP(hipEventRecord(t->ev_solved, ss));
            rc = spmttkrp(t, n, (const void *const *)factors, dtype, R, t->ws.M, dtype == FCOO_BF16, s);
            FCOO_HIP(hipStreamWaitEvent(s, t->ev_solved, 0));
            if (rc) return rc;
        }
        const RowPlan p = row_plan(I, R, dtype);
        nblk = p.nblk;
        double *ip = n == N - 1 ? ipart : nullptr, *gp = p.gram ? gpart : nullptr, *G = grams + (int64_t)n * R * R;
        hipError_t e;
        switch (p.RC) {
            case 1: e = rowsolve_rc<1>(p, s, t->ws.M, Wd, I, R, norms, lambda, factors[n], dtype, gp, ip); break;
            case 2: e = rowsolve_rc<2>(p, s, t->ws.M, Wd, I, R, norms, lambda, factors[n], dtype, gp, ip); break;
            case 4: e = rowsolve_rc<4>(p, s, t->ws.M, Wd, I, R, norms, lambda, factors[n], dtype, gp, ip); break;
            case 8: e = rowsolve_rc<8>(p, s, t->ws.M, Wd, I, R, norms, lambda, factors[n], dtype, gp, ip); break;
            case 16: e = rowsolve_rc<16>(p, s, t->ws.M, Wd, I, R, norms, lambda, factors[n], dtype, gp, ip); break;
            case 32: e = rowsolve_rc<32>(p, s, t->ws.M, Wd, I, R, norms, lambda, factors[n], dtype, gp, ip); break;
            default: e = rowsolve_rc<64>(p, s, t->ws.M, Wd, I, R, norms, lambda, factors[n], dtype, gp, ip); break;
        }
        if (e != hipSuccess) return hip_fail(e, "row solve");
        if (p.gram) FCOO_HIP(sum_blocks(gpart, nblk, R, G, s));
        else if ((rc = gram_launch(factors[n], dtype, I, R, gpart, G, s))) return rc;
    }
    hipLaunchKernelGGL(dev::fit_kernel, dim3(1), dim3(256), 0, s, ipart, (int64_t)nblk, grams, N, R, lambda,
                       t->normX2, fitd);
    FCOO_HIP(hipGetLastError());
    // the fit and, next to it, the modes' flags
    int *hflags = reinterpret_cast<int *>(t->ws.host_pinned + 1);
    FCOO_HIP(hipMemcpyAsync(t->ws.host_pinned, fitd, sizeof(double) + (size_t)N * sizeof(int), hipMemcpyDeviceToHost, s));
    FCOO_HIP(hipStreamSynchronize(s));
    *fit = t->ws.host_pinned[0];
    if (used_pinv) {
        int bits = 0;
        for (int n = 0; n < N; ++n) bits |= (hflags[n] ? 1 : 0) << n;
        *used_pinv = bits;
    }
    return FCOO_OK;
}

}  // extern "C"
