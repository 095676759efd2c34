// row_f64.hip -- matrix-core row update in FP64 (K <= 64).
//
// Per row (Algorithm 1's item body with BPMF's conditional):
//   P = Lambda + alpha sum_j y_j y_j^T,  b = Lambda mu + alpha sum_j r'_j y_j,
//   P = L L^T,  y = L^-1 b,  x = L^-T (y + z).
//
// Gram: v_mfma_f64_16x16x4_f64 on the 16 x 16 blocks of P's upper half, lane
// l holding component 16 bi + l % 16 of the neighbour row of rating 4g + l / 16
// (A operand of block row bi and B operand of block column bj at once),
// gathered by buffer loads whose range check masks the ragged tail.  A
// wavefront then factorises its row's blocks where they are, on the matrix
// cores (row_f64_blocked); many light rows of K <= 16 go four to a wavefront
// through LDS instead (row_f64_packed).
//
// What bounds it: the FP64 vector instructions and the serial chain of the
// 16 x 16 diagonal blocks; on problems of a few thousand rows the latency of
// one row's chain.  Against a column-per-lane elimination (530 FP64 FMAs and
// twice as many lane reads a row at K = 32), us a call, users / movies:
//   6000 x 3500, 500 k ratings   K = 16  46.2 / 40.6 -> 34.9 / 36.6
//                                K = 32  59.0 / 75.5 -> 50.4 / 55.2
//                                K = 64   212 / 213  ->  137 / 139
//   48,424 x 1252, 436 k         K = 21   178 / 57   ->  176 / 50
//                                K = 49   972 / 153  ->  522 / 113
#include <type_traits>

#include "internal.h"
#include "rng_device.h"
#include "row_common.h"

namespace bpmf {
namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ double buf_f64(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0));
}

__device__ __forceinline__ double buf_f64_stream(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, kStreamPolicy));
}

template <int RPW, int k>
__device__ __forceinline__ double bcast_f64(double x)
{
    const u32x2 w = __builtin_bit_cast(u32x2, x);
    u32x2 o;
    o.x = __float_as_uint(bcast<RPW, k>(__uint_as_float(w.x)));
    o.y = __float_as_uint(bcast<RPW, k>(__uint_as_float(w.y)));
    return __builtin_bit_cast(double, o);
}

__device__ __forceinline__ void wave_sync_f64()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Standard normal `comp` of a row: value comp % 4 of Philox block comp / 4, from
// one Box-Muller pair.
__device__ __forceinline__ double normal_f64(uint32_t row, uint32_t t, uint32_t comp, uint64_t seed,
                                             uint32_t stream)
{
    const Block4 bl = philox4x32_10(row, t, (stream << 24) | (comp >> 2), 0u, seed);
    const bool hi = (comp & 2) != 0;
    const double rho = sqrt(-2.0 * log(open_unit(hi ? bl.w2 : bl.w0)));
    double sv, cv;
    sincospi(2.0 * open_unit(hi ? bl.w3 : bl.w1), &sv, &cv);
    return rho * ((comp & 1) ? sv : cv);
}

// Gram (upper block (bj, bi), bi >= bj, in acc[bi (bi + 1) / 2 + bj]; value v of
// lane l is D[4 v + l / 16][l % 16]) and rhs of one work item.  Two chunks of 4 kU ratings: the rows of the next one and the
// ids of the one after are in flight while a chunk is multiplied.  Ratings
// past the end and ids past the end read 0; components >= K read what follows
// in the factor, whose Gram entries the caller ignores.
template <int NB>
__device__ __forceinline__ void gram_item_f64(const RowItem &it, const int32_t *__restrict__ nbr,
                                              const double *__restrict__ rc, __amdgpu_buffer_rsrc_t ysrc,
                                              uint32_t ldy8, int kq, int col,
                                              doublex4 (&acc)[NB * (NB + 1) / 2], double (&bacc)[NB])
{
    constexpr int kU = NB == 1 ? 8 : (NB == 2 ? 4 : 2);
    constexpr uint32_t kChunk = 4 * kU;
    const uint32_t cnt = (uint32_t)(it.end - it.beg);
    const __amdgpu_buffer_rsrc_t jsrc = make_rsrc(nbr + it.beg, cnt * 4u);
    const __amdgpu_buffer_rsrc_t rsrc = make_rsrc(rc + it.beg, cnt * 8u);
    const uint32_t nchunk = (cnt + kChunk - 1) / kChunk;
    const uint32_t coff = 8u * col;
    uint32_t jb[2][kU];
    double yb[2][kU][NB], rb[2][kU];
    auto load_ids = [&](int buf, uint32_t ch) {
#pragma unroll
        for (int g = 0; g < kU; ++g) jb[buf][g] = buf_u32_stream(jsrc, (ch * kChunk + 4 * g + kq) * 4u);
    };
    auto load_rows = [&](int buf, uint32_t ch) {
#pragma unroll
        for (int g = 0; g < kU; ++g) {
            const uint32_t t = ch * kChunk + 4 * g + kq;
            rb[buf][g] = buf_f64_stream(rsrc, t * 8u);  // 0 past the end
            const uint32_t base = t < cnt ? __umul24(jb[buf][g], ldy8) + coff : kOOB;  // fewer than 2^24 rows
#pragma unroll
            for (int bi = 0; bi < NB; ++bi) yb[buf][g][bi] = buf_f64(ysrc, base + 128u * bi);
        }
    };
    auto compute = [&](int buf) {
#pragma unroll
        for (int g = 0; g < kU; ++g) {
            int q = 0;
#pragma unroll
            for (int bi = 0; bi < NB; ++bi) {
#pragma unroll
                for (int bj = 0; bj <= bi; ++bj, ++q)
                    acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(yb[buf][g][bj], yb[buf][g][bi], acc[q], 0, 0, 0);
                bacc[bi] += rb[buf][g] * yb[buf][g][bi];
            }
        }
    };
    if (nchunk == 0) return;
    load_ids(0, 0);
    load_ids(1, 1);
    load_rows(0, 0);
    for (uint32_t ch = 0; ch < nchunk; ch += 2) {
        load_ids(0, ch + 2);
        load_rows(1, ch + 1);
        compute(0);
        if (ch + 1 >= nchunk) break;
        load_ids(1, ch + 3);
        load_rows(0, ch + 2);
        compute(1);
    }
}

constexpr int kWaves = 4;    // wavefronts per workgroup
constexpr int kPackRows = 4;  // rows per wavefront of the packed kernel

// Factor and sample four rows of K <= 16, column-per-lane in 16 lanes each:
// lane c of a group has v[r] = P[r][c] for r < 16 (identity outside the
// leading K x K block) and v[16] = b_c; elimination without square roots, b
// carried as an extra row.  Returns x_c (meaningful for c < K).  A live lane
// whose pivot is not positive clears *status.
__device__ __forceinline__ double packed_sample_f64(double (&v)[17], int K, int c, uint32_t row, uint32_t t,
                                                    uint64_t seed, uint32_t stream, bool live,
                                                    int *__restrict__ status)
{
    double mydiag = 1.0;
    static_for<0, 16>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        if (k >= K) return;  // uniform: the padding is the identity
        const double dk = bcast_f64<kPackRows, k>(v[k]);
        if (c == k) mydiag = dk;
        // lanes c <= k hold finished columns: multiplier 0 leaves them unchanged
        const double f = c > k ? v[k] * rcp_f64(dk) : 0.0;
        static_for<k + 1, 17>([&](auto rcc) {
            constexpr int r = decltype(rcc)::value;
            v[r] -= f * bcast_f64<kPackRows, k>(v[r]);
        });
    });
    if (live && !(mydiag > 0.0)) *status = 0;
    const double inv_s = rcp_f64(sqrt(mydiag));
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] *= inv_s;  // column c of L (rows > c)

    const double w = v[16] * inv_s + (c < K ? normal_f64(row, t, (uint32_t)c, seed, stream) : 0.0);
    // x = L^-T w, rows from the last (padded rows carry w = 0, x = 0)
    double accx = 0.0, myx = 0.0;
    static_for<0, 16>([&](auto qc) {
        constexpr int r = 15 - decltype(qc)::value;
        if (r >= K) return;  // uniform
        const double xr = bcast_f64<kPackRows, r>((w - accx) * inv_s);
        if (c == r) myx = xr;
        if (c < r) accx += v[r] * xr;
    });
    return myx;
}

// The Gram of a whole work item of K <= 16 by one wavefront, raw, into a
// packed lower triangle P with b behind it at `boff`.
__device__ __forceinline__ void gram_to_lds(const RowItem &it, int K, const int32_t *__restrict__ nbr,
                                            const double *__restrict__ rc, __amdgpu_buffer_rsrc_t ysrc, int kq,
                                            int col, double *P, int boff)
{
    doublex4 acc[1] = {{0.0, 0.0, 0.0, 0.0}};
    double bacc[1] = {0.0};
    gram_item_f64<1>(it, nbr, rc, ysrc, (uint32_t)K * 8u, kq, col, acc, bacc);
    bacc[0] += __shfl_xor(bacc[0], 16);
    bacc[0] += __shfl_xor(bacc[0], 32);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int r = 4 * v + kq;
        if (r < K && col <= r) P[pk(r, col)] = acc[0][v];
    }
    if (kq == 0 && col < K) P[boff + col] = bacc[0];
}

// K <= 16, many light rows.  Workgroups [0, n_heavy) take one heavy item each,
// its ratings dealt to the four wavefronts and their Grams summed in wave
// order; the others give each wavefront four light rows.
__global__ __launch_bounds__(64 * kWaves) void row_f64_packed(
    int K, double alpha, const RowItem *__restrict__ items, int64_t n_heavy, int64_t n_items,
    const int32_t *__restrict__ nbr, const double *__restrict__ rc, const double *__restrict__ Y,
    uint32_t y_bytes, const double *__restrict__ Lam, const double *__restrict__ Lmu, double *__restrict__ X,
    double *__restrict__ part, uint64_t seed, uint32_t stream, SweepT sweep, int *__restrict__ status)
{
    constexpr int PE = 16 * 17 / 2;
    constexpr int REGION = PE + 16;  // packed lower triangle, then b
    __shared__ double Ps[kWaves * kPackRows * REGION];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, kq = lane >> 4;
    const __amdgpu_buffer_rsrc_t ysrc = make_rsrc(Y, y_bytes);
    const int KK2 = K * (K + 1) / 2;
    double *Pw = Ps + wave * kPackRows * REGION;  // this wave's rows
    int row_of[kPackRows];
#pragma unroll
    for (int h = 0; h < kPackRows; ++h) row_of[h] = -1;
    if ((int64_t)blockIdx.x < n_heavy) {
        const RowItem it = items[blockIdx.x];
        const int64_t per = (it.end - it.beg + kWaves - 1) / kWaves;
        RowItem mine = it;
        mine.beg = min<int64_t>(it.end, it.beg + wave * per);
        mine.end = min<int64_t>(it.end, mine.beg + per);
        gram_to_lds(mine, K, nbr, rc, ysrc, kq, col, Ps + wave * REGION, PE);
        __syncthreads();
        double *dst = it.slot >= 0 ? part + (size_t)it.slot * (KK2 + K) : nullptr;
        for (int e = threadIdx.x; e < KK2 + K; e += 64 * kWaves) {
            const int q = e < KK2 ? e : PE + e - KK2;
            double g = Ps[q];
#pragma unroll
            for (int w = 1; w < kWaves; ++w) g += Ps[w * REGION + q];
            if (dst)
                dst[e] = g;  // segment of a split row: raw partial sums
            else
                Ps[q] = g;
        }
        __syncthreads();
        if (dst || wave > 0) return;
        row_of[0] = it.row;
    } else {
        const int64_t first = n_heavy + (((int64_t)blockIdx.x - n_heavy) * kWaves + wave) * kPackRows;
        if (first >= n_items) return;
        static_for<0, kPackRows>([&](auto hc) {
            constexpr int h = decltype(hc)::value;
            if (first + h >= n_items) return;
            const RowItem it = items[first + h];
            gram_to_lds(it, K, nbr, rc, ysrc, kq, col, Pw + h * REGION, PE);
            row_of[h] = it.row;
        });
        wave_sync_f64();
    }

    const int grp = lane >> 4, c = lane & 15;
    int my_row = row_of[0];
#pragma unroll
    for (int h = 1; h < kPackRows; ++h)
        if (grp == h) my_row = row_of[h];
    const bool live = my_row >= 0 && c < K;
    const double *P = Pw + grp * REGION;
    double v[17];
#pragma unroll
    for (int r = 0; r < 16; ++r)
        v[r] = (live && r < K) ? Lam[r * K + c] + alpha * P[r >= c ? pk(r, c) : pk(c, r)] : (r == c ? 1.0 : 0.0);
    v[16] = live ? Lmu[c] + alpha * P[PE + c] : 0.0;
    const double x = packed_sample_f64(v, K, c, (uint32_t)my_row, sweep.t(), seed, stream, live, status);
    if (live) X[(size_t)my_row * K + c] = x;
}

// Sum over the 16 lanes of each 16-lane row, left in lane 15 of the row.
__device__ __forceinline__ double row_sum16_f64(double x)
{
    auto shr = [](double y, auto nc) {
        constexpr int N = decltype(nc)::value;
        const u32x2 w = __builtin_bit_cast(u32x2, y);
        u32x2 o;
        o.x = __builtin_amdgcn_update_dpp(0, (int)w.x, 0x110 + N, 0xf, 0xf, true);
        o.y = __builtin_amdgcn_update_dpp(0, (int)w.y, 0x110 + N, 0xf, 0xf, true);
        return __builtin_bit_cast(double, o);
    };
    x += shr(x, std::integral_constant<int, 1>{});
    x += shr(x, std::integral_constant<int, 2>{});
    x += shr(x, std::integral_constant<int, 4>{});
    x += shr(x, std::integral_constant<int, 8>{});
    return x;
}

// Blocked factorisation and draw of one row by one wave, the FP32 blocked
// kernel's algorithm in doubles.  acc: the negated matrix -(Lambda + alpha G),
// identity on the padding, as upper 16 x 16 blocks: block (i, j), i >= j, keeps
// T[16 j + 4 v + g][16 i + c] in value v of lane (g, c), which is what every
// product takes as operand and returns.  vec: b (n = 16 NB values), then room
// for n more.  Only the diagonal blocks are eliminated on the vector units, all
// 64 lanes busy; the rest are 16 x 16 products.
template <int NB>
__device__ __forceinline__ void blocked_sample_f64(doublex4 (&acc)[NB * (NB + 1) / 2], double *vec, int K,
                                                   uint32_t row, uint32_t t, uint64_t seed, uint32_t stream,
                                                   double *__restrict__ xrow, int *__restrict__ status)
{
    const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
    double *bv = vec, *xv = vec + 16 * NB;
    double xa[NB][4];  // X_kb = L_kk^-1: X[c][4 v + g]
    static_for<0, NB>([&](auto kbc) {
        constexpr int kb = decltype(kbc)::value;
        constexpr int qd = kb * (kb + 1) / 2 + kb;
        // the diagonal block: column k' > k takes -(d_kk' / d_kk) times column k
        // on [G; d], b's segment rides along
        double u[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) u[v] = -acc[qd][v];
        double bc = bv[16 * kb + c], mydiag = 1.0;
        static_for<0, 16>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            if (kb + 1 < NB || 16 * kb + k < K) {  // uniform: the padding is the identity
                constexpr int gk = k & 3, vk = k >> 2;
                const double pr = row_of_wave<gk>(u[vk]);
                const double dk = lane_of_row<k>(pr);
                if (c == k) mydiag = dk;
                const double nf = c > k ? -pr * rcp_f64(dk) : 0.0;
                if (g == gk) u[vk] = c == k ? 1.0 : 0.0;
#pragma unroll
                for (int v = 0; v < 4; ++v) u[v] = fma(nf, lane_of_row<k>(u[v]), u[v]);
                bc = fma(nf, lane_of_row<k>(bc), bc);
            }
        });
        if (kb + 1 == NB)  // rows of the padding: G is the identity there
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (16 * kb + 4 * v + g >= K) u[v] = c == 4 * v + g ? 1.0 : 0.0;
        if (g == 0 && 16 * kb + c < K && !(mydiag > 0.0)) *status = 0;
        const double inv_s = rcp_f64(sqrt(mydiag));
#pragma unroll
        for (int v = 0; v < 4; ++v) xa[kb][v] = u[v] * inv_s;
        if (g == 0) bv[16 * kb + c] = bc * inv_s;  // y_kb
        wave_sync_f64();
        if constexpr (kb + 1 < NB) {
            // R_kb,i = X T_kb,i, then b_i -= R_kb,i^T y_kb
            double y[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) y[v] = bv[16 * kb + 4 * v + g];
            static_for<kb + 1, NB>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                constexpr int q = i * (i + 1) / 2 + kb;
                doublex4 r = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    r = __builtin_amdgcn_mfma_f64_16x16x4f64(-xa[kb][v], acc[q][v], r, 0, 0, 0);
                acc[q] = r;
                double p = r[0] * y[0] + r[1] * y[1] + r[2] * y[2] + r[3] * y[3];
                p += __shfl_xor(p, 16);
                p += __shfl_xor(p, 32);
                if (g == 0) bv[16 * i + c] -= p;
            });
            // T_j,i -= R_kb,j^T R_kb,i (the negated T takes the product)
            static_for<kb + 1, NB>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                static_for<kb + 1, i + 1>([&](auto jc) {
                    constexpr int j = decltype(jc)::value;
                    constexpr int qi = i * (i + 1) / 2 + kb, qj = j * (j + 1) / 2 + kb, q = i * (i + 1) / 2 + j;
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(acc[qj][v], acc[qi][v], acc[q], 0, 0, 0);
                });
            });
            wave_sync_f64();
        }
    });
    // w = y + z: lane l takes component l
    if (lane < K) bv[lane] += normal_f64(row, t, (uint32_t)lane, seed, stream);
    wave_sync_f64();
    // x_kb = X^T (w_kb - sum_{i > kb} R_kb,i x_i), from the last block row
    static_for<0, NB>([&](auto qc) {
        constexpr int kb = NB - 1 - decltype(qc)::value;
        if constexpr (kb + 1 < NB) {
            double s[4] = {0.0, 0.0, 0.0, 0.0};
            static_for<kb + 1, NB>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                const double xc = xv[16 * i + c];
#pragma unroll
                for (int v = 0; v < 4; ++v) s[v] += acc[i * (i + 1) / 2 + kb][v] * xc;
            });
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                s[v] = row_sum16_f64(s[v]);
                if (c == 15) bv[16 * kb + 4 * v + g] -= s[v];
            }
            wave_sync_f64();
        }
        const double wc = bv[16 * kb + c];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const double o = row_sum16_f64(xa[kb][v] * wc);
            if (c == 15) xv[16 * kb + 4 * v + g] = o;
        }
        wave_sync_f64();
    });
    if (lane < K) xrow[lane] = xv[lane];
}

// A light item for each wavefront; workgroups [0, n_heavy) take one heavy item
// each, its ratings dealt to the four wavefronts and their Grams summed in wave
// order.  Register budget: as many waves a SIMD as hold the blocks unspilled.
template <int NB>
__global__ __launch_bounds__(64 * kWaves, (NB <= 2 ? 4 : (NB == 3 ? 3 : 2))) void row_f64_blocked(
    int K, double alpha, const RowItem *__restrict__ items, int64_t n_heavy, int64_t n_items,
    const int32_t *__restrict__ nbr, const double *__restrict__ rc, const double *__restrict__ Y,
    uint32_t y_bytes, const double *__restrict__ Lam, const double *__restrict__ Lmu, double *__restrict__ X,
    double *__restrict__ part, uint64_t seed, uint32_t stream, SweepT sweep, int *__restrict__ status)
{
    constexpr int NBLK = NB * (NB + 1) / 2;
    __shared__ double sums[NBLK * 256 + 64 * NB];
    __shared__ double vecs[kWaves][32 * NB];
    const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool heavy = (int64_t)blockIdx.x < n_heavy;
    const int64_t id = heavy ? (int64_t)blockIdx.x : n_heavy + ((int64_t)blockIdx.x - n_heavy) * kWaves + wave;
    if (id >= n_items) return;
    const RowItem it = items[id];
    RowItem mine = it;
    if (heavy) {
        const int64_t per = (it.end - it.beg + kWaves - 1) / kWaves;
        mine.beg = min<int64_t>(it.end, it.beg + wave * per);
        mine.end = min<int64_t>(it.end, mine.beg + per);
    }
    doublex4 acc[NBLK];
    double bacc[NB];
#pragma unroll
    for (int q = 0; q < NBLK; ++q) acc[q] = doublex4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int bi = 0; bi < NB; ++bi) bacc[bi] = 0.0;
    gram_item_f64<NB>(mine, nbr, rc, make_rsrc(Y, y_bytes), (uint32_t)K * 8u, g, c, acc, bacc);
    if (heavy) {
        for (int w = kWaves - 1; w > 0; --w) {
            if (wave == w) {
#pragma unroll
                for (int q = 0; q < NBLK; ++q)
#pragma unroll
                    for (int v = 0; v < 4; ++v) sums[256 * q + 64 * v + lane] = acc[q][v];
#pragma unroll
                for (int bi = 0; bi < NB; ++bi) sums[256 * NBLK + 64 * bi + lane] = bacc[bi];
            }
            __syncthreads();
            if (wave == w - 1) {
#pragma unroll
                for (int q = 0; q < NBLK; ++q)
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[q][v] += sums[256 * q + 64 * v + lane];
#pragma unroll
                for (int bi = 0; bi < NB; ++bi) bacc[bi] += sums[256 * NBLK + 64 * bi + lane];
            }
        }
        if (wave > 0) return;
    }
#pragma unroll
    for (int bi = 0; bi < NB; ++bi) {
        bacc[bi] += __shfl_xor(bacc[bi], 16);
        bacc[bi] += __shfl_xor(bacc[bi], 32);
    }
    if (it.slot >= 0) {  // segment of a split row: raw partial sums, packed lower
        const int KK2 = K * (K + 1) / 2;
        double *dst = part + (size_t)it.slot * (KK2 + K);
#pragma unroll
        for (int i = 0; i < NB; ++i) {
#pragma unroll
            for (int j = 0; j <= i; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int r = 16 * j + 4 * v + g, cc = 16 * i + c;
                    if (cc < K && r <= cc) dst[pk(cc, r)] = acc[i * (i + 1) / 2 + j][v];
                }
            if (g == 0 && 16 * i + c < K) dst[KK2 + 16 * i + c] = bacc[i];
        }
        return;
    }
    double *vec = vecs[wave];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
#pragma unroll
        for (int j = 0; j <= i; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = 16 * j + 4 * v + g, cc = 16 * i + c;
                const int q = i * (i + 1) / 2 + j;
                acc[q][v] = (r < K && cc < K) ? -alpha * acc[q][v] - Lam[r * K + cc] : (r == cc ? -1.0 : 0.0);
            }
        const int cc = 16 * i + c;
        if (g == 0) vec[cc] = cc < K ? Lmu[cc] + alpha * bacc[i] : 0.0;
    }
    wave_sync_f64();
    blocked_sample_f64<NB>(acc, vec, K, (uint32_t)it.row, sweep.t(), seed, stream, X + (size_t)it.row * K, status);
}

// Sum the partial slots of every split row into its first slot, in slot order
// (one thread per row and entry, eight slots' loads in flight).
__global__ __launch_bounds__(256) void part_reduce_f64(const FinishItem *__restrict__ fin, int E,
                                                       double *__restrict__ part)
{
    const FinishItem f = fin[blockIdx.x];
    const int e = blockIdx.y * 256 + threadIdx.x;
    if (e >= E || f.count <= 1) return;
    double *base = part + (size_t)f.first * E + e;
    double s = 0.0;
    int q = 0;
    for (; q + 8 <= f.count; q += 8) {
        double x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = base[(size_t)(q + u) * E];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += x[u];
    }
    for (; q < f.count; ++q) s += base[(size_t)q * E];
    base[0] = s;
}

// Split rows from their summed partials, one wavefront each.
template <int NB>
__global__ __launch_bounds__(64) void row_finish_f64(int K, double alpha,
                                                             const FinishItem *__restrict__ fin,
                                                             const double *__restrict__ part,
                                                             const double *__restrict__ Lam,
                                                             const double *__restrict__ Lmu,
                                                             double *__restrict__ X, uint64_t seed,
                                                             uint32_t stream, SweepT sweep,
                                                             int *__restrict__ status)
{
    __shared__ double vec[32 * NB];
    const int g = threadIdx.x >> 4, c = threadIdx.x & 15;
    const FinishItem f = fin[blockIdx.x];
    const int KK2 = K * (K + 1) / 2;
    const double *src = part + (size_t)f.first * (KK2 + K);
    doublex4 acc[NB * (NB + 1) / 2];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int cc = 16 * i + c;
#pragma unroll
        for (int j = 0; j <= i; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = 16 * j + 4 * v + g;
                acc[i * (i + 1) / 2 + j][v] =
                    (r < K && cc < K) ? -alpha * src[r >= cc ? pk(r, cc) : pk(cc, r)] - Lam[r * K + cc]
                                      : (r == cc ? -1.0 : 0.0);
            }
        if (g == 0) vec[cc] = cc < K ? Lmu[cc] + alpha * src[KK2 + cc] : 0.0;
    }
    wave_sync_f64();
    blocked_sample_f64<NB>(acc, vec, K, (uint32_t)f.row, sweep.t(), seed, stream, X + (size_t)f.row * K, status);
}

// K <= 16: light rows above which four share a wavefront.  Packed, a wave walks
// its rows' ratings one after the other but the chip needs a quarter of the
// waves; 300 k ratings, us, a row a wave against packed, K = 10 / K = 16:
//    8,000 users  27.8, 35.2 / 32.2, 36.1
//   12,000        34.4, 35.9 / 40.8, 38.6
//   16,000        41.2, 37.6 / 49.4, 40.3
//   24,000        54.9, 38.4 / 67.1, 42.9
// Above K = 16 a row a wave is at worst equal (48,424 rows: K = 21 176 against
// 178 two a wave, K = 32 215 against 214) and up to 27% faster.
constexpr int64_t kPackedAbove = 10240;

template <int NB>
hipError_t launch_f64(bpmf_ctx *c, Side &sd, Side &ot, hipStream_t s, int stage)
{
    const int K = c->K;
    if (stage == kStageFinish) {
        if (sd.n_fin == 0) return hipSuccess;
        const int E = K * (K + 1) / 2 + K;
        hipLaunchKernelGGL(part_reduce_f64, dim3((unsigned)sd.n_fin, (unsigned)((E + 255) / 256)), dim3(256), 0, s,
                           sd.fin, E, (double *)c->part);
        hipLaunchKernelGGL((row_finish_f64<NB>), dim3((unsigned)sd.n_fin), dim3(64), 0, s, K, c->alpha, sd.fin,
                           (const double *)c->part, (const double *)sd.Lam_w, (const double *)sd.Lmu_w,
                           (double *)sd.X, c->seed, sd.stream_row, c->sweep_t(), c->hyp_status + 1);
        return hipGetLastError();
    }
    if (stage != kStageSegments || sd.n_items == 0) return hipSuccess;
    // the segments come first, then the whole rows in descending degree order.
    // Waves a SIMD for the limit: the six that run at one block (movies of 60,000 x
    // 17,770, K = 16: 170 us with three, 152 with six); above it one less than
    // the four and three that run (movies of 12,000 x 500, K = 24: 45.5 us with three,
    // 47.6 with four; K = 48 the same either way)
    const int64_t n_heavy =
        sd.n_slots + whole_rows_above(sd, heavy_limit(sd, c->nnz, K, 1024 * (NB == 1 ? 6 : (NB == 2 ? 3 : 2))));
    const int64_t n_light = sd.n_items - n_heavy;
    auto go = [&](auto kernel, int rows_per_wave) {
        const int64_t per = (int64_t)rows_per_wave * kWaves, blocks = n_heavy + (n_light + per - 1) / per;
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(64 * kWaves), 0, s, K, c->alpha, sd.items, n_heavy,
                           sd.n_items, sd.nbr, (const double *)sd.rc, (const double *)ot.X,
                           (uint32_t)(ot.rows * K * sizeof(double)), (const double *)sd.Lam_w,
                           (const double *)sd.Lmu_w, (double *)sd.X, (double *)c->part, c->seed, sd.stream_row,
                           c->sweep_t(), c->hyp_status + 1);
    };
    if (NB == 1 && n_light > kPackedAbove)
        go(row_f64_packed, kPackRows);
    else
        go(row_f64_blocked<NB>, 1);
    return hipGetLastError();
}

}  // namespace

// FP64 factors (K <= 64) whose buffers fit 32-bit offsets and whose row ids
// fit 24 bits; beyond that the generic kernel.
bool f64_path_available(const bpmf_ctx *c)
{
    if (c->prec != 0 || c->K > 64) return false;
    for (int s = 0; s < 2; ++s)
        if ((uint64_t)c->side[s].rows * c->K * sizeof(double) >= kOOB || c->side[s].rows >= (1 << 24)) return false;
    return (uint64_t)c->split_threshold * 8u < kOOB;
}

// Every work item in the segments stage, the split rows in the finishing one.
hipError_t launch_row_f64(bpmf_ctx *c, int side_id, hipStream_t s, int stage, bool *handled)
{
    *handled = false;
    if (!f64_path_available(c)) return hipSuccess;
    *handled = true;
    Side &sd = c->side[side_id];
    Side &ot = c->side[1 - side_id];
    switch ((c->K + 15) / 16) {
    case 1: return launch_f64<1>(c, sd, ot, s, stage);
    case 2: return launch_f64<2>(c, sd, ot, s, stage);
    case 3: return launch_f64<3>(c, sd, ot, s, stage);
    default: return launch_f64<4>(c, sd, ot, s, stage);
    }
}

}  // namespace bpmf
