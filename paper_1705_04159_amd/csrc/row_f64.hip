// row_f64.hip -- matrix-core row update in FP64 (K <= 64).
//
// Per row (Algorithm 1's item body with BPMF's conditional):
//   P = Lambda + alpha sum_j y_j y_j^T,  b = Lambda mu + alpha sum_j r'_j y_j,
//   P = L L^T,  y = L^-1 b,  x = L^-T (y + z).
//
// The layout of the FP32 kernel for K <= 64 in doubles.  Gram: v_mfma_f64_16x16x4_f64 on the lower 16 x 16
// blocks of P, lane l holding component 16 bi + l % 16 of the neighbour row of
// rating 4g + l / 16 (A operand of block row bi and B operand of block column
// bj at once), gathered by buffer loads whose range check masks the ragged
// tail.  Factorisation: the accumulators go through LDS into a
// column-per-lane layout and are eliminated without square roots, b carried
// as an extra row; pivot columns are broadcast by v_readlane (one row a wave)
// or ds_swizzle (rows packed into lane groups).
//
// What bounds it: at K = 32 the vector instructions of the factorisation
// (about 530 FP64 FMAs and twice as many broadcasts a row) and, on problems
// of a few thousand rows, the latency of one row's chain.
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

// 1 / d to an ulp or so for normal d: the hardware's estimate and two Newton
// steps (half the dependent instructions of a division, which sits in the
// chain of every elimination step).
__device__ __forceinline__ double rcp_f64(double d)
{
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    return fma(fma(-d, r, 1.0), r, r);
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

// Gram (lower blocks; value v of lane l is D[4 v + l / 16][l % 16]) and rhs of
// one work item.  Two chunks of 4 kU ratings: the rows of the next one and the
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
                    acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(yb[buf][g][bi], yb[buf][g][bj], acc[q], 0, 0, 0);
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

// Factor and sample one row held column-per-lane: lane c of the group has
// v[r] = P[r][c] for r < KP (identity outside the leading K x K block) and
// v[KP] = b_c.  Returns x_c (meaningful for c < K).  A live lane whose pivot
// is not positive clears *status.
template <int KP, int RPW>
__device__ __forceinline__ double chol_sample_f64(double (&v)[KP + 1], int K, int c, uint32_t row, uint32_t t,
                                                  uint64_t seed, uint32_t stream, bool live,
                                                  int *__restrict__ status)
{
    double mydiag = 1.0;
    static_for<0, KP>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        if (k >= K) return;  // uniform: the padding is the identity
        const double dk = bcast_f64<RPW, k>(v[k]);
        if (c == k) mydiag = dk;
        // lanes c <= k hold finished columns: multiplier 0 leaves them unchanged
        const double f = c > k ? v[k] * rcp_f64(dk) : 0.0;
        static_for<k + 1, KP + 1>([&](auto rcc) {
            constexpr int r = decltype(rcc)::value;
            v[r] -= f * bcast_f64<RPW, k>(v[r]);
        });
    });
    if (live && !(mydiag > 0.0)) *status = 0;
    const double inv_s = rcp_f64(sqrt(mydiag));
#pragma unroll
    for (int r = 0; r < KP; ++r) v[r] *= inv_s;  // column c of L (rows > c)

    // w = L^-1 b + z: normal c is value c % 4 of block c / 4, from one
    // Box-Muller pair
    double w = v[KP] * inv_s;
    if (c < K) {
        const Block4 bl = philox4x32_10(row, t, (stream << 24) | (uint32_t)(c >> 2), 0u, seed);
        const bool hi = (c & 2) != 0;
        const double rho = sqrt(-2.0 * log(open_unit(hi ? bl.w2 : bl.w0)));
        double sv, cv;
        sincospi(2.0 * open_unit(hi ? bl.w3 : bl.w1), &sv, &cv);
        w += rho * ((c & 1) ? sv : cv);
    }
    // x = L^-T w, rows from the last (padded rows carry w = 0, x = 0)
    double accx = 0.0, myx = 0.0;
    static_for<0, KP>([&](auto qc) {
        constexpr int r = KP - 1 - decltype(qc)::value;
        if (r >= K) return;  // uniform
        const double xr = bcast_f64<RPW, r>((w - accx) * inv_s);
        if (c == r) myx = xr;
        if (c < r) accx += v[r] * xr;
    });
    return myx;
}

// The Gram of a whole work item by one wavefront, raw, into a packed lower
// triangle P with b behind it at `boff`.
template <int NB>
__device__ __forceinline__ void gram_to_lds(const RowItem &it, int K, const int32_t *__restrict__ nbr,
                                            const double *__restrict__ rc, __amdgpu_buffer_rsrc_t ysrc, int kq,
                                            int col, double *P, int boff)
{
    doublex4 acc[NB * (NB + 1) / 2];
    double bacc[NB];
#pragma unroll
    for (int q = 0; q < NB * (NB + 1) / 2; ++q) acc[q] = doublex4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int bi = 0; bi < NB; ++bi) bacc[bi] = 0.0;
    gram_item_f64<NB>(it, nbr, rc, ysrc, (uint32_t)K * 8u, kq, col, acc, bacc);
    int q = 0;
#pragma unroll
    for (int bi = 0; bi < NB; ++bi) {
        bacc[bi] += __shfl_xor(bacc[bi], 16);
        bacc[bi] += __shfl_xor(bacc[bi], 32);
#pragma unroll
        for (int bj = 0; bj <= bi; ++bj, ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = 16 * bi + 4 * v + kq, c = 16 * bj + col;
                if (r < K && c <= r) P[pk(r, c)] = acc[q][v];
            }
        const int c = 16 * bi + col;
        if (kq == 0 && c < K) P[boff + c] = bacc[bi];
    }
}

constexpr int kWaves = 4;  // wavefronts per workgroup

// Workgroups [0, n_heavy) take one heavy item each, its ratings dealt to the
// four wavefronts and their Grams summed in wave order; the others give each
// wavefront RPW light rows.  With a wavefront to every item the launch lasted
// as long as the longest rows: K = 32, 6000 x 3500 with 450 k ratings 171 us
// (users, two a wave) and 99 us (movies).
template <int NB, int RPW>
__global__ __launch_bounds__(64 * kWaves) void row_f64(
    int K, double alpha, const RowItem *__restrict__ items, int64_t n_heavy, int64_t n_items,
    const int32_t *__restrict__ nbr, const double *__restrict__ rc, const double *__restrict__ Y,
    uint32_t y_bytes, const double *__restrict__ Lam, const double *__restrict__ Lmu, double *__restrict__ X,
    double *__restrict__ part, uint64_t seed, uint32_t stream, SweepT sweep,
    int *__restrict__ status)
{
    constexpr int KP = 16 * NB;
    constexpr int LPR = 64 / RPW;
    constexpr int PE = KP * (KP + 1) / 2;
    constexpr int REGION = PE + KP;  // packed lower triangle, then b
    __shared__ double Ps[kWaves * RPW * REGION];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, kq = lane >> 4;
    const __amdgpu_buffer_rsrc_t ysrc = make_rsrc(Y, y_bytes);
    const int KK2 = K * (K + 1) / 2;
    double *Pw = Ps + wave * RPW * REGION;  // this wave's rows
    int row_of[RPW];
#pragma unroll
    for (int h = 0; h < RPW; ++h) row_of[h] = -1;
    if ((int64_t)blockIdx.x < n_heavy) {
        const RowItem it = items[blockIdx.x];
        const int64_t per = (it.end - it.beg + kWaves - 1) / kWaves;
        RowItem mine = it;
        mine.beg = min<int64_t>(it.end, it.beg + wave * per);
        mine.end = min<int64_t>(it.end, mine.beg + per);
        gram_to_lds<NB>(mine, K, nbr, rc, ysrc, kq, col, Ps + wave * REGION, PE);
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
        const int64_t first = n_heavy + (((int64_t)blockIdx.x - n_heavy) * kWaves + wave) * RPW;
        if (first >= n_items) return;
        static_for<0, RPW>([&](auto hc) {
            constexpr int h = decltype(hc)::value;
            if (first + h >= n_items) return;
            const RowItem it = items[first + h];
            gram_to_lds<NB>(it, K, nbr, rc, ysrc, kq, col, Pw + h * REGION, PE);
            row_of[h] = it.row;
        });
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }

    const int grp = lane / LPR, c = lane & (LPR - 1);
    int my_row = row_of[0];
#pragma unroll
    for (int h = 1; h < RPW; ++h)
        if (grp == h) my_row = row_of[h];
    const bool live = my_row >= 0 && c < K;
    const double *P = Pw + grp * REGION;
    const int cc = c < KP ? c : 0;
    double v[KP + 1];
#pragma unroll
    for (int r = 0; r < KP; ++r)
        v[r] = (live && r < K) ? Lam[r * K + c] + alpha * P[r >= cc ? pk(r, cc) : pk(cc, r)] : (r == c ? 1.0 : 0.0);
    v[KP] = live ? Lmu[c] + alpha * P[PE + cc] : 0.0;
    const double x = chol_sample_f64<KP, RPW>(v, K, c, (uint32_t)my_row, sweep.t(), seed, stream, live, status);
    if (live) X[(size_t)my_row * K + c] = x;
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
__global__ __launch_bounds__(64) void row_finish_f64(int K, double alpha, const FinishItem *__restrict__ fin,
                                                     const double *__restrict__ part,
                                                     const double *__restrict__ Lam,
                                                     const double *__restrict__ Lmu, double *__restrict__ X,
                                                     uint64_t seed, uint32_t stream,
                                                     SweepT sweep, int *__restrict__ status)
{
    constexpr int KP = 16 * NB;
    const int c = threadIdx.x;
    const FinishItem f = fin[blockIdx.x];
    const int KK2 = K * (K + 1) / 2;
    const bool live = c < K;
    const double *src = part + (size_t)f.first * (KK2 + K);
    double v[KP + 1];
#pragma unroll
    for (int r = 0; r < KP; ++r)
        v[r] = (live && r < K) ? Lam[r * K + c] + alpha * src[r >= c ? pk(r, c) : pk(c, r)] : (r == c ? 1.0 : 0.0);
    v[KP] = live ? Lmu[c] + alpha * src[KK2 + c] : 0.0;
    const double x = chol_sample_f64<KP, 1>(v, K, c, (uint32_t)f.row, sweep.t(), seed, stream, live, status);
    if (live) X[(size_t)f.row * K + c] = x;
}

// Light rows up to which each takes a wavefront of its own: below it the GPU's
// 1024 SIMDs have at most four waves each either way, and packing rows only
// makes a wave walk their ratings one after the other.
constexpr int64_t kUnpackedItems = 4096;

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
    // the segments come first, then the whole rows in descending degree order
    const int64_t n_heavy = sd.n_slots + whole_rows_above(sd, heavy_limit(sd, c->nnz, K, 1024 * (NB <= 2 ? 3 : 2)));
    const int64_t n_light = sd.n_items - n_heavy;
    auto go = [&](auto rpwc) {
        constexpr int RPW = decltype(rpwc)::value;
        const int64_t blocks = n_heavy + (n_light + RPW * kWaves - 1) / (RPW * kWaves);
        hipLaunchKernelGGL((row_f64<NB, RPW>), dim3((unsigned)blocks), dim3(64 * kWaves), 0, s, K, c->alpha,
                           sd.items, n_heavy, sd.n_items, sd.nbr, (const double *)sd.rc, (const double *)ot.X,
                           (uint32_t)(ot.rows * K * sizeof(double)), (const double *)sd.Lam_w,
                           (const double *)sd.Lmu_w, (double *)sd.X, (double *)c->part, c->seed, sd.stream_row,
                           c->sweep_t(), c->hyp_status + 1);
    };
    constexpr int kPacked = NB == 1 ? 4 : (NB == 2 ? 2 : 1);
    if (n_light > kUnpackedItems)
        go(std::integral_constant<int, kPacked>{});
    else
        go(std::integral_constant<int, 1>{});
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
