// hyper.hip -- FP64 Normal-Wishart hyperparameter draw of one side on the GPU.
//
// Algorithm 1 samples the movie hyperparameters from V before the movie loop
// and the user hyperparameters from U before the user loop.  With the
// Normal-Wishart hyperprior of BPMF (mu0, beta0, W0, nu0) and the n rows x_i
// of the side's factor, the conjugate posterior is
//   beta* = beta0 + n,  nu* = nu0 + n,  mu* = (beta0 mu0 + n xbar) / beta*,
//   W*^-1 = W0^-1 + S + beta0 n / beta* (xbar - mu0)(xbar - mu0)^T,
//   S = sum_i (x_i - xbar)(x_i - xbar)^T,
// and the draw is Lambda ~ Wishart(W*, nu*) by the Bartlett decomposition
// (Lambda = (L_W A)(L_W A)^T, L_W = chol(W*), A lower triangular with
// A_kk = sqrt(chi2(nu* - k)), k = 0..K-1, and N(0,1) below the diagonal in
// row-major order), then mu = mu* + chol(beta* Lambda)^-T z.
//
// Three launches: per-block FP64 moment sums over row chunks on the FP64 matrix
// cores (S is formed as sum x x^T - n xbar xbar^T); a fixed-order reduction of
// the block sums, whose spare workgroups draw the noise of the step (it
// depends on the counters alone); and one workgroup for the K x K algebra.
// The algebra avoids forming W* and two of the three factorisations:
//   * L_W is obtained from one Cholesky of the index-reversed W*^-1:
//     J W*^-1 J = C C^T gives W*^-1 = (J C J)(J C J)^T with J C J upper
//     triangular, hence W* = (J C J)^-T (J C J)^-1 and, by uniqueness of the
//     Cholesky factor, L_W = J C^-T J, i.e. L_W[i][j] = (C^-1)[n-1-j][n-1-i];
//   * B = L_W A is lower triangular with a positive diagonal, so it is the
//     Cholesky factor of Lambda, and chol(beta* Lambda) = sqrt(beta*) B:
//     mu = mu* + B^-T z / sqrt(beta*).
// The order is padded to n = 16 ceil(K / 16) with the identity, which every
// step carries through (reversed, the padding leads), so that all matrices are
// whole 16 x 16 blocks in LDS and every product runs on the matrix cores.
#include <algorithm>
#include <type_traits>

#include "internal.h"
#include "rng_device.h"
#include "row_common.h"

namespace bpmf {
namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void tri_index(int e, int &i, int &j)
{
    int ii = (int)((sqrtf(8.0f * (float)e + 1.0f) - 1.0f) * 0.5f);
    while ((ii + 1) * (ii + 2) / 2 <= e) ++ii;
    while (ii * (ii + 1) / 2 > e) --ii;
    i = ii;
    j = e - ii * (ii + 1) / 2;
}

__device__ __forceinline__ double as_f64(float v) { return (double)v; }
__device__ __forceinline__ double as_f64(double v) { return v; }

// The block sums on the FP64 matrix cores: four wavefronts per block of rows,
// four rows per v_mfma_f64_16x16x4f64 step -- lane l holds component
// 16*bi + (l % 16) of row 4g + l / 16 as an FP64 value (FP32 factors convert
// exactly), which is both the A operand of block row bi and the B operand of
// block column bj, so only the nb(nb+1)/2 lower 16x16 blocks of X^T X are
// accumulated; sum x on the VALU from the same registers.  (The FP64
// instruction returns D[4 v + l / 16][l % 16] in value v of lane l, unlike the
// FP32 one.)  Products of FP32 values are exact in FP64, and every sum is in
// FP64 in a fixed order.  The rows of the next four steps are in flight during
// a step's products.  Up to K = 64 each wave takes a quarter of the rows and
// the four sums are added in LDS; above, where one wave's accumulators would
// fill the register file, each wave takes a quarter of the 16x16 blocks of
// every row (the rows come from the L1 three times in four).  Either way a
// block's sums leave the GPU's registers once for four waves: writing and
// reading them back (41 KB at K = 100) costs more than the rows themselves
// (120,047 rows, K = 100, 1024 one-wave blocks: 46 us, and 14 us more in the
// reduction).
constexpr int kMomentsAhead = 4;
constexpr int kMomentsWaves = 4;

// Rows of one wave's range of the factor, read through its range check: rows
// past the range are 0, components >= K whatever follows (their sums are
// ignored).
template <int NB, typename XT>
struct MomentRows {
    __amdgpu_buffer_rsrc_t src;
    uint32_t off, step;  // of this lane's row of the next step, bytes of four rows
    __device__ __forceinline__ MomentRows(const XT *X, int ld, int64_t r0, int64_t r1)
    {
        const int lane = threadIdx.x & 63;
        src = make_rsrc(X + (size_t)r0 * ld, (uint32_t)((r1 - r0) * ld * sizeof(XT)));
        off = (uint32_t)(((lane >> 4) * ld + (lane & 15)) * sizeof(XT));
        step = (uint32_t)(4 * ld * sizeof(XT));
    }
    __device__ __forceinline__ void load(XT (&y)[NB])
    {
#pragma unroll
        for (int bi = 0; bi < NB; ++bi) {
            if constexpr (sizeof(XT) == 4)
                y[bi] = buf_f32(src, off + 64u * bi);
            else
                y[bi] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(src, (int)(off + 128u * bi), 0, 0));
        }
        off += step;
    }
};

template <int NB, typename XT>
__global__ __launch_bounds__(64 * kMomentsWaves) void hyper_moments_mfma(int K, const XT *__restrict__ X, int ld,
                                                                         int64_t rows, int64_t chunk,
                                                                         double *__restrict__ part)
{
    constexpr int NBLK = NB * (NB + 1) / 2;
    constexpr int A = kMomentsAhead;
    __shared__ double sums[NBLK * 256 + 16 * NB];  // value v of lane l of block q at 256 q + 64 v + l, then sum x
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, kq = lane >> 4;
    const int64_t r0 = min<int64_t>(rows, ((int64_t)blockIdx.x * kMomentsWaves + wave) * chunk);
    const int64_t r1 = min<int64_t>(rows, r0 + chunk);
    const int E = K + K * (K + 1) / 2;
    doublex4 acc[NBLK];
#pragma unroll
    for (int q = 0; q < NBLK; ++q) acc[q] = doublex4{0.0, 0.0, 0.0, 0.0};
    double sx[NB];
#pragma unroll
    for (int bi = 0; bi < NB; ++bi) sx[bi] = 0.0;
    MomentRows<NB, XT> in(X, ld, r0, r1);
    XT ring[A][NB];
#pragma unroll
    for (int a = 0; a < A; ++a) in.load(ring[a]);
    for (int64_t base = r0; base < r1; base += 4 * A) {
#pragma unroll
        for (int a = 0; a < A; ++a) {  // steps past r1 multiply zeros
            double y[NB];
#pragma unroll
            for (int bi = 0; bi < NB; ++bi) {
                y[bi] = as_f64(ring[a][bi]);
                sx[bi] += y[bi];
            }
            in.load(ring[a]);
            int q = 0;
#pragma unroll
            for (int bi = 0; bi < NB; ++bi)
#pragma unroll
                for (int bj = 0; bj <= bi; ++bj) {
                    acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(y[bi], y[bj], acc[q], 0, 0, 0);
                    ++q;
                }
        }
    }
#pragma unroll
    for (int bi = 0; bi < NB; ++bi) {
        sx[bi] += __shfl_xor(sx[bi], 16);
        sx[bi] += __shfl_xor(sx[bi], 32);
    }
    for (int w = 0; w < kMomentsWaves; ++w) {  // in wave order
        if (w == wave) {
#pragma unroll
            for (int q = 0; q < NBLK; ++q)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    double *d = sums + 256 * q + 64 * v + lane;
                    *d = w == 0 ? acc[q][v] : *d + acc[q][v];
                }
            if (kq == 0)
#pragma unroll
                for (int bi = 0; bi < NB; ++bi) {
                    double *d = sums + NBLK * 256 + 16 * bi + col;
                    *d = w == 0 ? sx[bi] : *d + sx[bi];
                }
        }
        __syncthreads();
    }
    double *dst = part + (size_t)blockIdx.x * E;
    for (int k = threadIdx.x; k < K; k += 64 * kMomentsWaves) dst[k] = sums[NBLK * 256 + k];
#pragma unroll
    for (int bi = 0; bi < NB; ++bi)
#pragma unroll
        for (int bj = 0; bj <= bi; ++bj) {
            // FP64 result layout: lane l, value v holds D[4 v + l / 16][l % 16]
            const int i = 16 * bi + 4 * wave + kq, j = 16 * bj + col;
            if (i < K && j <= i) dst[K + pk(i, j)] = sums[256 * pk(bi, bj) + 64 * wave + lane];
        }
}

// Wave W's blocks q = W, W + 4, ... of rows [r0, r1), and sum x of its
// components' blocks.
template <int NB, int W, typename XT>
__device__ __forceinline__ void moments_quarter(int K, const XT *__restrict__ X, int ld, int64_t r0, int64_t r1,
                                                double *__restrict__ dst)
{
    constexpr int NBLK = NB * (NB + 1) / 2;
    constexpr int MINE = (NBLK - W + kMomentsWaves - 1) / kMomentsWaves;
    constexpr int A = kMomentsAhead;
    const int lane = threadIdx.x & 63;
    const int col = lane & 15, kq = lane >> 4;
    doublex4 acc[MINE];
#pragma unroll
    for (int m = 0; m < MINE; ++m) acc[m] = doublex4{0.0, 0.0, 0.0, 0.0};
    double sx[(NB + kMomentsWaves - 1) / kMomentsWaves] = {};
    XT ring[A][NB];
    MomentRows<NB, XT> in(X, ld, r0, r1);
#pragma unroll
    for (int a = 0; a < A; ++a) in.load(ring[a]);
    for (int64_t base = r0; base < r1; base += 4 * A) {
#pragma unroll
        for (int a = 0; a < A; ++a) {  // steps past r1 multiply zeros
            double y[NB];
#pragma unroll
            for (int bi = 0; bi < NB; ++bi) y[bi] = as_f64(ring[a][bi]);
#pragma unroll
            for (int bi = W; bi < NB; bi += kMomentsWaves) sx[bi / kMomentsWaves] += y[bi];
            in.load(ring[a]);
            static_for<0, NB>([&](auto ic) {
                static_for<0, decltype(ic)::value + 1>([&](auto jc) {
                    constexpr int i = decltype(ic)::value, j = decltype(jc)::value, q = i * (i + 1) / 2 + j;
                    if constexpr (q % kMomentsWaves == W)
                        acc[q / kMomentsWaves] =
                            __builtin_amdgcn_mfma_f64_16x16x4f64(y[i], y[j], acc[q / kMomentsWaves], 0, 0, 0);
                });
            });
        }
    }
#pragma unroll
    for (int bi = W; bi < NB; bi += kMomentsWaves) {
        double t = sx[bi / kMomentsWaves];
        t += __shfl_xor(t, 16);
        t += __shfl_xor(t, 32);
        const int c = 16 * bi + col;
        if (kq == 0 && c < K) dst[c] = t;
    }
    static_for<0, NB>([&](auto ic) {
        static_for<0, decltype(ic)::value + 1>([&](auto jc) {
            constexpr int bi = decltype(ic)::value, bj = decltype(jc)::value, q = bi * (bi + 1) / 2 + bj;
            if constexpr (q % kMomentsWaves == W)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = 16 * bi + 4 * v + kq, j = 16 * bj + col;
                    if (i < K && j <= i) dst[K + pk(i, j)] = acc[q / kMomentsWaves][v];
                }
        });
    });
}

template <int NB, typename XT>
__global__ __launch_bounds__(64 * kMomentsWaves, 2) void hyper_moments_wide(int K, const XT *__restrict__ X, int ld,
                                                                            int64_t rows, int64_t chunk,
                                                                            double *__restrict__ part)
{
    const int64_t r0 = min<int64_t>(rows, (int64_t)blockIdx.x * chunk * kMomentsWaves);
    const int64_t r1 = min<int64_t>(rows, r0 + chunk * kMomentsWaves);
    double *dst = part + (size_t)blockIdx.x * (K + K * (K + 1) / 2);
    switch (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) {
    case 0: moments_quarter<NB, 0>(K, X, ld, r0, r1, dst); break;
    case 1: moments_quarter<NB, 1>(K, X, ld, r0, r1, dst); break;
    case 2: moments_quarter<NB, 2>(K, X, ld, r0, r1, dst); break;
    default: moments_quarter<NB, 3>(K, X, ld, r0, r1, dst); break;
    }
}

// stats[e] = sum over blocks of part[b][e], in a fixed order: a workgroup takes
// 16 entries (128 contiguous bytes of each block's sums), thread (sub, e) adds
// blocks sub, sub + 32, sub + 64, ..., then the 32 sums are added across lanes
// and wavefronts.  The workgroups past the entries draw the step's noise:
// noise[0, K(K-1)/2) the normals below the Bartlett factor's diagonal in
// row-major order, the next K the mean's normals, the last K the diagonal
// sqrt(chi2(nu* - k)).  Replaces two passes of one-wave workgroups (9.6 and
// 3.4 us at K = 32 with 2048 blocks) and takes the transcendentals off the
// draw's one workgroup.
constexpr int kRedThreads = 512;

__global__ __launch_bounds__(kRedThreads) void hyper_reduce(int K, int nblk, const double *__restrict__ part,
                                                            double *__restrict__ stats, int entry_groups,
                                                            double nu_s, uint64_t seed, uint32_t stream,
                                                            SweepT sweep,
                                                            double *__restrict__ noise, int *__restrict__ status)
{
    __shared__ double ws[kRedThreads / 64][16];
    const int tid = threadIdx.x;
    const int E = K + K * (K + 1) / 2;
    if ((int)blockIdx.x >= entry_groups) {
        const uint32_t t = sweep.t();
        const int n_low = K * (K - 1) / 2, b_low = (n_low + 3) / 4, b_mu = (K + 3) / 4;
        const int job = ((int)blockIdx.x - entry_groups) * kRedThreads + tid;
        if (job < b_low + b_mu) {
            const bool low = job < b_low;
            const int blk = low ? job : job - b_low;
            double z[4];
            normals_block(seed, (uint32_t)blk, t, stream, low ? 1u : 2u, 0u, z);
            for (int l = 0; l < 4; ++l)
                if (4 * blk + l < (low ? n_low : K)) noise[(low ? 0 : n_low) + 4 * blk + l] = z[l];
        } else if (job - b_low - b_mu < K) {
            const int k = job - b_low - b_mu;
            int ok = 1;
            noise[n_low + K + k] = sqrt(chi_square(seed, stream, t, (uint32_t)k, nu_s - (double)k, &ok));
            if (!ok) *status = 0;
        }
        return;
    }
    const int e = (int)blockIdx.x * 16 + (tid & 15);
    double s = 0.0;
    if (e < E) {
#pragma unroll 8
        for (int b = tid >> 4; b < nblk; b += kRedThreads / 16) s += part[(size_t)b * E + e];
    }
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    if ((tid & 63) < 16) ws[tid >> 6][tid & 15] = s;
    __syncthreads();
    if (tid < 16 && e < E) {
        double r = 0.0;
#pragma unroll
        for (int w = 0; w < kRedThreads / 64; ++w) r += ws[w][tid];
        stats[e] = r;
    }
}

// ---- block algebra in LDS ----
// A matrix of nb x nb lower 16 x 16 blocks: block (i, j), i >= j, is row-major
// at bo(i, j) with rows 17 doubles apart (so that the 16 lanes of an operand
// read, one row each, fall into different banks).  Lane (g, c) = (l / 16, l %
// 16) of a wave feeds X[c][4 s + g] (A operand) and Y[4 s + g][c] (B operand)
// in step s of a block product and receives D[4 v + g][c] in value v.
constexpr int kBS = 17;
constexpr int kBlk = 16 * kBS;

__device__ __forceinline__ int bo(int i, int j) { return pk(i, j) * kBlk; }
__device__ __forceinline__ int el(int i, int j) { return bo(i >> 4, j >> 4) + (i & 15) * kBS + (j & 15); }

__device__ __forceinline__ void lds_wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// acc += sgn X Y^T (both blocks row-major): the A operand of each.
__device__ __forceinline__ doublex4 mul_abt(const double *X, const double *Y, double sgn, doublex4 acc, int g, int c)
{
    double a[4], b[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        a[s] = X[c * kBS + 4 * s + g];
        b[s] = Y[c * kBS + 4 * s + g];
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(sgn * a[s], b[s], acc, 0, 0, 0);
    return acc;
}

// acc += X Y.
__device__ __forceinline__ doublex4 mul_ab(const double *X, const double *Y, doublex4 acc, int g, int c)
{
    double a[4], b[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        a[s] = X[c * kBS + 4 * s + g];
        b[s] = Y[(4 * s + g) * kBS + c];
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[s], acc, 0, 0, 0);
    return acc;
}

__device__ __forceinline__ doublex4 load_blk(const double *X, int g, int c)
{
    doublex4 r;
#pragma unroll
    for (int v = 0; v < 4; ++v) r[v] = X[(4 * v + g) * kBS + c];
    return r;
}

__device__ __forceinline__ void store_blk(double *X, doublex4 r, int g, int c)
{
#pragma unroll
    for (int v = 0; v < 4; ++v) X[(4 * v + g) * kBS + c] = r[v];
}

// One wave: the whole symmetric block D = L L^T replaced by X = L^-1.  Lane
// (g, c) holds rows 4 v + g of column c; column c > k takes -(d_kc / d_kk)
// times column k on the stacked [G; d] (row k leaves d for G = L_unit^-T once
// it has served as pivot row), the pivot row coming from the lane row that
// holds it.  X = D^-1/2 G^T.  Clears *ok on a non-positive pivot (taken as 1).
__device__ __forceinline__ void factor_block(double *D, int g, int c, int *ok)
{
    double u[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) u[v] = D[(4 * v + g) * kBS + c];
    double mydiag = 1.0;
    static_for<0, 16>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        constexpr int gk = k & 3, vk = k >> 2;
        const double pr = row_of_wave<gk>(u[vk]);  // row k of column c
        const double d = lane_of_row<k>(pr);
        const double dk = d > 0.0 ? d : 1.0;
        if (c == k) mydiag = d;
        const double nf = c > k ? -pr * rcp_f64(dk) : 0.0;
        if (g == gk) u[vk] = c == k ? 1.0 : 0.0;
#pragma unroll
        for (int v = 0; v < 4; ++v) u[v] = fma(nf, lane_of_row<k>(u[v]), u[v]);
    });
    if (!(mydiag > 0.0)) *ok = 0;
    const double inv_s = 1.0 / sqrt(mydiag > 0.0 ? mydiag : 1.0);
#pragma unroll
    for (int v = 0; v < 4; ++v) D[c * kBS + 4 * v + g] = u[v] * inv_s;
}

// Workgroup: in-place blocked Cholesky of the lower blocks T (diagonal blocks
// whole); the diagonal blocks end as the inverses of the factor's.  The first
// wave updates and factors the next diagonal block while the others update
// the remaining trailing blocks: two barriers per block column.  (K = 64: 36 us
// and 32 barriers when it went by pairs of columns.)
template <int NW>
__device__ void chol_blocks(int nb, double *T, int *ok)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, c = lane & 15;
    for (int kb = 0; kb < nb; ++kb) {
        auto trail = [&](int i, int j) {
            double *D = T + bo(i, j);
            store_blk(D, mul_abt(T + bo(i, kb - 1), T + bo(j, kb - 1), -1.0, load_blk(D, g, c), g, c), g, c);
        };
        if (wave == 0) {
            if (kb > 0) {
                trail(kb, kb);
                lds_wave_sync();
            }
            factor_block(T + bo(kb, kb), g, c, ok);
        } else if (kb > 0) {
            const int m = nb - kb;
            for (int q = wave; q < m * (m + 1) / 2; q += NW - 1) {
                int i, j;
                tri_index(q, i, j);
                trail(kb + i, kb + j);
            }
        }
        __syncthreads();
        for (int i = kb + 1 + wave; i < nb; i += NW) {
            double *D = T + bo(i, kb);
            store_blk(D, mul_abt(D, T + bo(kb, kb), 1.0, doublex4{0.0, 0.0, 0.0, 0.0}, g, c), g, c);
        }
        __syncthreads();
    }
}

// Workgroup: the off-diagonal blocks of I = C^-1, whose diagonal blocks hold
// the inverses of C's already; C's off-diagonal blocks are read.  A wave takes
// a block column: X_ij = -X_ii sum_{j <= k < i} C_ik X_kj, the sum staying in
// registers as the second product's operand.
template <int NW>
__device__ void inverse_blocks(int nb, const double *C, double *I)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, c = lane & 15;
    for (int j = wave; j < nb; j += NW)
        for (int i = j + 1; i < nb; ++i) {
            // the sum in two chains of products, which wait for each other
            // less than one would
            doublex4 s0 = {0.0, 0.0, 0.0, 0.0}, s1 = s0;
            int k = j;
            for (; k + 2 <= i; k += 2) {
                s0 = mul_ab(C + bo(i, k), I + bo(k, j), s0, g, c);
                s1 = mul_ab(C + bo(i, k + 1), I + bo(k + 1, j), s1, g, c);
            }
            if (k < i) s0 = mul_ab(C + bo(i, k), I + bo(k, j), s0, g, c);
            const double *X = I + bo(i, i);
            doublex4 r = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int v = 0; v < 4; ++v)
                r = __builtin_amdgcn_mfma_f64_16x16x4f64(-X[c * kBS + 4 * v + g], s0[v] + s1[v], r, 0, 0, 0);
            store_blk(I + bo(i, j), r, g, c);
            lds_wave_sync();
        }
}

// One wave: X = D^-1 of a lower triangular block, lane c the column c.
__device__ __forceinline__ void tri_inverse_block(const double *D, double *X, int g, int c)
{
    double x[16];
    static_for<0, 16>([&](auto rc) {
        constexpr int r = decltype(rc)::value;
        double s = c == r ? 1.0 : 0.0;
#pragma unroll
        for (int k = 0; k < r; ++k) s = fma(-D[r * kBS + k], x[k], s);
        x[r] = s * rcp_f64(D[r * kBS + r]);
    });
    if (g == 0)
#pragma unroll
        for (int r = 0; r < 16; ++r) X[r * kBS + c] = x[r];
}

// y[i] = sum_j M[j][i] x[j] (TRANS) or sum_j M[i][j] x[j], M lower with zeros
// above the diagonal and x 0 past K, four lanes per entry; out(i, y_i) is
// called by one of them.
template <bool TRANS, typename OUT>
__device__ __forceinline__ void tri_matvec(int K, int nb, const double *M, const double *x, OUT out)
{
    const int i = threadIdx.x >> 2, p = threadIdx.x & 3;
    double s = 0.0;
    if (i < K) {
        const int bi = i >> 4, r = i & 15;
        for (int bj = TRANS ? bi : 0; bj < (TRANS ? nb : bi + 1); ++bj) {
            const double *m = M + (TRANS ? bo(bj, bi) + r : bo(bi, bj) + r * kBS);
#pragma unroll
            for (int q = 0; q < 4; ++q) s = fma(m[(4 * q + p) * (TRANS ? kBS : 1)], x[16 * bj + 4 * q + p], s);
        }
    }
    s += __shfl_xor(s, 1);
    s += __shfl_xor(s, 2);
    if (i < K && p == 0) out(i, s);
}

// L^-1 (lower, zeros above) to a K x K array, a wave per row.
template <int NW, typename T>
__device__ __forceinline__ void store_lower(int K, const double *M, T *out)
{
    const int lane = threadIdx.x & 63;
    for (int r = threadIdx.x >> 6; r < K; r += NW)
        for (int cc = lane; cc < K; cc += 64) out[r * K + cc] = cc <= r ? (T)M[el(r, cc)] : (T)0;
}

// Elements (i, j) of the stored blocks of an n x n matrix, dealt to the threads
// (16 x 16 of them to every NT / 256-th block, consecutive threads along a row
// of the block, or with ALONG_I along a column, as f's loads are consecutive):
// all of a thread's values f(i, j) first, so that their loads are in flight
// together, then stored.
template <int NT, bool ALONG_I, int U, typename F>
__device__ __forceinline__ void load_blocks(int nb, double (&x)[U], F f)
{
    constexpr int STEP = NT / 256;
    const int hi = (threadIdx.x >> 4) & 15, lo = threadIdx.x & 15;
    const int r = ALONG_I ? lo : hi, c = ALONG_I ? hi : lo;
    int bi = 0, bj = threadIdx.x >> 8;  // block q is (bi, bj)
#pragma unroll
    for (int u = 0; u < U; ++u) {
        while (bj > bi) bj -= ++bi;
        if (bi < nb) x[u] = f(16 * bi + r, 16 * bj + c);
        bj += STEP;
    }
}

template <int NT, bool ALONG_I, int U>
__device__ __forceinline__ void store_blocks(int nb, double *T, const double (&x)[U])
{
    constexpr int STEP = NT / 256;
    const int hi = (threadIdx.x >> 4) & 15, lo = threadIdx.x & 15;
    const int at = ALONG_I ? lo * kBS + hi : hi * kBS + lo;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int q = (threadIdx.x >> 8) + u * STEP;
        if (q < pk(nb, 0)) T[q * kBlk + at] = x[u];
    }
}

constexpr int kMaxBlocks = 8;  // ceil(128 / 16)

// LDS: two block matrices and four vectors.
size_t draw_lds(int K)
{
    const size_t nb = (K + 15) / 16;
    return sizeof(double) * (nb * (nb + 1) * kBlk + 4 * 16 * nb);
}

// The K x K algebra in one workgroup.  Bound by its chain: at K = 100 about a
// third is the seven diagonal factorisations, a quarter the two inversions,
// the rest loads of fresh sums, products and barriers.  In whole 16 x 16 blocks
// on the matrix cores, with the noise drawn elsewhere: 10.5 us at K = 10, 16 at
// 32, 32 at 64, 55 at 100 (packed triangles eliminated two columns a barrier:
// 20, 46, 115 and 238 us).
template <int NT, typename T>
__global__ __launch_bounds__(NT) void hyper_draw(
    int K, int64_t n, const double *__restrict__ stats, const double *__restrict__ noise,
    const double *__restrict__ mu0, const double *__restrict__ W0inv, double beta0,
    double *__restrict__ mu_out, double *__restrict__ Lam_out, T *__restrict__ Lam_w, T *__restrict__ Lmu_w,
    T *__restrict__ Linv_w, T *__restrict__ Ltmu_w, int *__restrict__ status)
{
    constexpr int NW = NT / 64;
    extern __shared__ __align__(16) char smem_raw[];
    const int nb = (K + 15) / 16, np = 16 * nb;
    double *M1 = (double *)smem_raw;  // reversed W*^-1, its factor, A, then B
    double *M2 = M1 + pk(nb, 0) * kBlk;  // C^-1, then B^-1
    double *xbar = M2 + pk(nb, 0) * kBlk, *mus = xbar + np, *zv = mus + np, *mu = zv + np;
    __shared__ int ok;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, c = lane & 15;
    const double dn = (double)n;
    const double beta_s = beta0 + dn;
    const double shrink = beta0 * dn / beta_s;
    const int n_low = K * (K - 1) / 2;
    if (tid == 0) ok = 1;
    for (int k = tid; k < np; k += NT) {
        const int kk = min(k, K - 1);
        const double xb = stats[kk] / dn, m0 = mu0[kk];
        xbar[k] = k < K ? xb : 0.0;
        mu[k] = k < K ? xb - m0 : 0.0;
        mus[k] = k < K ? (beta0 * m0 + dn * xb) / beta_s : 0.0;
        zv[k] = k < K ? noise[n_low + kk] : 0.0;
    }
    // the Bartlett factor A (the identity on the padding), read ahead of its use
    constexpr int kFill = NT == 256 ? 10 : kMaxBlocks * (kMaxBlocks + 1) / 4;
    double areg[kFill];
    load_blocks<NT, false>(nb, areg, [&](int i, int j) {
        const int ii = min(i, K - 1);
        const double z = noise[i == j ? n_low + K + ii : (j < ii ? pk(ii - 1, j) : 0)];  // a load without a branch
        return i < K ? (j <= i ? z : 0.0) : (i == j ? 1.0 : 0.0);
    });
    __syncthreads();
    // J W*^-1 J over the padded order: entry (i, j) is W*^-1[np-1-j][np-1-i]
    {
        double w[kFill];
        load_blocks<NT, true>(nb, w, [&](int i, int j) {
            const int a = np - 1 - min(i, j), b = np - 1 - max(i, j);  // a >= b
            const int aa = min(a, K - 1), bb = min(b, K - 1);          // loads without a branch
            const double S = stats[K + pk(aa, bb)] - dn * xbar[aa] * xbar[bb];
            const double x = W0inv[aa * K + bb] + S + shrink * mu[aa] * mu[bb];  // mu: xbar - mu0
            return a < K ? x : (i == j ? 1.0 : 0.0);
        });
        store_blocks<NT, true>(nb, M1, w);
    }
    __syncthreads();
    chol_blocks<NW>(nb, M1, &ok);
    for (int b = wave; b < nb; b += NW) store_blk(M2 + bo(b, b), load_blk(M1 + bo(b, b), g, c), g, c);
    __syncthreads();
    inverse_blocks<NW>(nb, M1, M2);
    __syncthreads();
    store_blocks<NT, false>(nb, M1, areg);
    __syncthreads();
    // B = L_W A, L_W[r][m] = C^-1[np-1-m][np-1-r]; kept in registers until every
    // wave has read A
    {
        constexpr int kMine = (NT == 256 ? 10 : kMaxBlocks * (kMaxBlocks + 1) / 2) / NW + 1;
        doublex4 acc[kMine];
#pragma unroll
        for (int m = 0; m < kMine; ++m) {
            const int q = wave + m * NW;
            if (q >= pk(nb, 0)) break;
            int bi, bj;
            tri_index(q, bi, bj);
            acc[m] = doublex4{0.0, 0.0, 0.0, 0.0};
            for (int bm = bj; bm <= bi; ++bm) {
                const double *Cb = M2 + bo(nb - 1 - bm, nb - 1 - bi), *Ab = M1 + bo(bm, bj);
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    acc[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(Cb[(15 - 4 * s - g) * kBS + 15 - c],
                                                                  Ab[(4 * s + g) * kBS + c], acc[m], 0, 0, 0);
            }
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < kMine; ++m) {
            const int q = wave + m * NW;
            if (q < pk(nb, 0)) store_blk(M1 + q * kBlk, acc[m], g, c);
        }
    }
    __syncthreads();
    // B^-1 into M2 (block columns by wave), then Lambda = B B^T
    for (int b = wave; b < nb; b += NW) tri_inverse_block(M1 + bo(b, b), M2 + bo(b, b), g, c);
    __syncthreads();
    inverse_blocks<NW>(nb, M1, M2);
    for (int q = NW - 1 - wave; q < pk(nb, 0); q += NW) {  // the last waves have the shortest columns above
        int bi, bj;
        tri_index(q, bi, bj);
        doublex4 acc = {0.0, 0.0, 0.0, 0.0};
        for (int bm = 0; bm <= bj; ++bm) acc = mul_abt(M1 + bo(bi, bm), M1 + bo(bj, bm), 1.0, acc, g, c);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = 16 * bi + 4 * v + g, j = 16 * bj + c;
            if (i < K && j <= i) {
                Lam_out[i * K + j] = acc[v];
                Lam_out[j * K + i] = acc[v];
                Lam_w[i * K + j] = (T)acc[v];
                Lam_w[j * K + i] = (T)acc[v];
            }
        }
    }
    __syncthreads();
    const double rs = 1.0 / sqrt(beta_s);
    tri_matvec<true>(K, nb, M2, zv, [&](int i, double x) {
        mu[i] = mus[i] + x * rs;
        mu_out[i] = mu[i];
    });
    __syncthreads();
    // Lambda mu = B (B^T mu)
    tri_matvec<true>(K, nb, M1, mu, [&](int i, double x) { xbar[i] = x; });  // xbar and mu stay 0 past K
    __syncthreads();
    tri_matvec<false>(K, nb, M1, xbar, [&](int i, double x) { Lmu_w[i] = (T)x; });
    if (Linv_w) {
        // for the rank-one row path: chol(Lambda)^-1 = B^-1 and B^T mu
        for (int i = tid; i < K; i += NT) Ltmu_w[i] = (T)xbar[i];
        store_lower<NW>(K, M2, Linv_w);
    }
    if (tid == 0 && !ok) *status = 0;
}

// For the rank-one row path after (mu, Lambda) were set by the host:
// L^-1 and L^T mu = L^-1 (Lambda mu), L = chol(Lambda), FP64 in one workgroup.
template <int NT, typename T>
__global__ __launch_bounds__(NT) void prior_factor(int K, const double *__restrict__ mu,
                                                    const double *__restrict__ Lam, T *__restrict__ Linv_w,
                                                    T *__restrict__ Ltmu_w, int *__restrict__ status)
{
    extern __shared__ __align__(16) char smem_raw[];
    const int nb = (K + 15) / 16;
    double *M1 = (double *)smem_raw, *M2 = M1 + pk(nb, 0) * kBlk, *lm = M2 + pk(nb, 0) * kBlk;
    __shared__ int ok;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, c = lane & 15;
    if (tid == 0) ok = 1;
    constexpr int kFill = NT == 256 ? 10 : kMaxBlocks * (kMaxBlocks + 1) / 4;
    double w[kFill];
    load_blocks<NT, false>(nb, w, [&](int i, int j) {
        const int a = max(i, j), b = min(i, j);  // the lower triangle
        return a < K ? Lam[a * K + b] : (i == j ? 1.0 : 0.0);
    });
    store_blocks<NT, false>(nb, M1, w);
    for (int i = tid; i < 16 * nb; i += NT) {
        double s = 0.0;
        const int ii = min(i, K - 1);
#pragma unroll 16
        for (int j = 0; j < K; ++j) s += Lam[ii >= j ? ii * K + j : j * K + ii] * mu[j];  // loads in flight together
        lm[i] = i < K ? s : 0.0;
    }
    __syncthreads();
    chol_blocks<NT / 64>(nb, M1, &ok);
    for (int b = wave; b < nb; b += NT / 64) store_blk(M2 + bo(b, b), load_blk(M1 + bo(b, b), g, c), g, c);
    __syncthreads();
    inverse_blocks<NT / 64>(nb, M1, M2);
    __syncthreads();
    store_lower<NT / 64>(K, M2, Linv_w);
    tri_matvec<false>(K, nb, M2, lm, [&](int i, double x) { Ltmu_w[i] = (T)x; });
    if (tid == 0 && !ok) *status = 0;
}

// Working-precision prior from FP64 (mu, Lambda) set by the host: workgroup 0
// Lambda mu, the others Lambda.
template <typename T>
__global__ __launch_bounds__(256) void prior_to_working(int K, const double *__restrict__ mu,
                                                        const double *__restrict__ Lam, T *__restrict__ Lam_w,
                                                        T *__restrict__ Lmu_w)
{
    const int tid = threadIdx.x;
    if (blockIdx.x > 0) {
        const int q = ((int)blockIdx.x - 1) * 256 + tid;
        if (q < K * K) Lam_w[q] = (T)Lam[q];
    } else if (tid < K) {
        double s = 0.0;
#pragma unroll 16
        for (int j = 0; j < K; ++j) s += Lam[tid * K + j] * mu[j];  // loads in flight together
        Lmu_w[tid] = (T)s;
    }
}

}  // namespace

hipError_t launch_hyper(bpmf_ctx *c, int side_id, hipStream_t s, uint32_t t_off)
{
    double *part = c->hyp_part[side_id], *stats = c->hyp_stats[side_id];
    double *noise = c->hyp_noise[side_id];
    Side &sd = c->side[side_id];
    const int K = c->K;
    const int E = K + K * (K + 1) / 2;
    const int64_t rows = sd.rows;
    // rows a wave: at least 16, with fewer the reduction reads more than the
    // moments did
    const int64_t waves = (int64_t)c->hyp_blocks * kMomentsWaves;
    const int64_t chunk = std::max<int64_t>(16, (rows + waves - 1) / waves);
    const int used = (int)((rows + chunk * kMomentsWaves - 1) / (chunk * kMomentsWaves));
    auto moments = [&](auto nbc) {
        constexpr int NB = decltype(nbc)::value;
        auto go = [&](auto kern, auto *X) {
            hipLaunchKernelGGL(kern, dim3(used), dim3(64 * kMomentsWaves), 0, s, K, X, c->ld, rows, chunk, part);
        };
        if constexpr (NB <= 4) {
            if (c->prec == 0)
                go(hyper_moments_mfma<NB, double>, (const double *)sd.X);
            else
                go(hyper_moments_mfma<NB, float>, (const float *)sd.X);
        } else {  // FP64 factors stop at K = 64
            go(hyper_moments_wide<NB, float>, (const float *)sd.X);
        }
    };
    switch ((K + 15) / 16) {
    case 1: moments(std::integral_constant<int, 1>{}); break;
    case 2: moments(std::integral_constant<int, 2>{}); break;
    case 3: moments(std::integral_constant<int, 3>{}); break;
    case 4: moments(std::integral_constant<int, 4>{}); break;
    case 5: moments(std::integral_constant<int, 5>{}); break;
    case 6: moments(std::integral_constant<int, 6>{}); break;
    case 7: moments(std::integral_constant<int, 7>{}); break;
    default: moments(std::integral_constant<int, 8>{}); break;
    }
    const int groups = (E + 15) / 16;
    const int jobs = (K * (K - 1) / 2 + 3) / 4 + (K + 3) / 4 + K;
    hipLaunchKernelGGL(hyper_reduce, dim3(groups + (jobs + kRedThreads - 1) / kRedThreads), dim3(kRedThreads), 0, s,
                       K, used, (const double *)part, stats, groups, c->nu0 + (double)rows, c->seed, sd.stream_hyp,
                       c->sweep_t(t_off), noise, c->hyp_status);
    const size_t lds = draw_lds(K);
    // K <= 64: four waves (at most four block columns), which find room beside
    // the other side's row kernels; above, eight
    auto draw = [&](auto ntc) {
        constexpr int NT = decltype(ntc)::value;
        if constexpr (NT == 256)  // FP64 factors stop at K = 64
            if (c->prec == 0) {
                hipLaunchKernelGGL((hyper_draw<NT, double>), dim3(1), dim3(NT), lds, s, K, rows, stats, noise, c->d_mu0,
                                   c->d_W0inv, c->beta0, sd.mu, sd.Lam, (double *)sd.Lam_w, (double *)sd.Lmu_w,
                                   (double *)nullptr, (double *)nullptr, c->hyp_status);
                return;
            }
        hipLaunchKernelGGL((hyper_draw<NT, float>), dim3(1), dim3(NT), lds, s, K, rows, stats, noise, c->d_mu0,
                           c->d_W0inv, c->beta0, sd.mu, sd.Lam, (float *)sd.Lam_w, (float *)sd.Lmu_w,
                           sd.n_low ? (float *)sd.Linv_w : (float *)nullptr,
                           sd.n_low ? (float *)sd.Ltmu_w : (float *)nullptr, c->hyp_status);
    };
    if (K <= 64)
        draw(std::integral_constant<int, 256>{});
    else
        draw(std::integral_constant<int, 512>{});
    return hipGetLastError();
}

hipError_t prepare_hyper(bpmf_ctx *c)
{
    const int need = (int)draw_lds(c->K);
    if (need <= 65536) return hipSuccess;  // only above K = 64 (FP32 factors, 512 threads)
    const hipError_t e =
        hipFuncSetAttribute((const void *)hyper_draw<512, float>, hipFuncAttributeMaxDynamicSharedMemorySize, need);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute((const void *)prior_factor<512, float>, hipFuncAttributeMaxDynamicSharedMemorySize, need);
}

hipError_t launch_prior_to_working(bpmf_ctx *c, int side_id, hipStream_t s)
{
    Side &sd = c->side[side_id];
    if (sd.n_low && c->prec == 1) {
        auto factor = [&](auto ntc) {
            constexpr int NT = decltype(ntc)::value;
            hipLaunchKernelGGL((prior_factor<NT, float>), dim3(1), dim3(NT), draw_lds(c->K), s, c->K, sd.mu, sd.Lam,
                               (float *)sd.Linv_w, (float *)sd.Ltmu_w, c->hyp_status);
        };
        if (c->K <= 64)
            factor(std::integral_constant<int, 256>{});
        else
            factor(std::integral_constant<int, 512>{});
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const dim3 grid(1 + (unsigned)((c->K * c->K + 255) / 256));
    if (c->prec == 0)
        hipLaunchKernelGGL((prior_to_working<double>), grid, dim3(256), 0, s, c->K, sd.mu,
                           sd.Lam, (double *)sd.Lam_w, (double *)sd.Lmu_w);
    else
        hipLaunchKernelGGL((prior_to_working<float>), grid, dim3(256), 0, s, c->K, sd.mu,
                           sd.Lam, (float *)sd.Lam_w, (float *)sd.Lmu_w);
    return hipGetLastError();
}

}  // namespace bpmf
