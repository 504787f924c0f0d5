// Dense contractions of the prefill and the DiT step: C[M][N] = A[M][K] . W[N][K]^T
// with fused epilogues (bias, q/k/v store + paged KV scatter, GELU, residual add).
// 16-bit modes run on the matrix cores (gemm_small.hip, gemm_large.hip; gemm_plan
// chooses); FTTS_F32 mode has the plain fp32 FMA tile kernel below (4x4 outputs per
// thread).
#include <algorithm>

#include "decode_entry.hpp"
#include "gemm_epilogue.hpp"

namespace ftts {

// Where row m of a packed prefill batch lands in the KV pool: its physical
// page (-1 if the page table does not cover it) and slot within the page.
struct RowSlot { int phys, slot; };
__device__ __forceinline__ RowSlot row_slot(const GemmArgs& a, int m) {
    const int s = a.kv.slots[m];
    return s < 0 ? RowSlot{-1, 0} : RowSlot{s / kPage, s % kPage};
}

// Store of one biased output element for the non-residual epilogues (rs: the
// row's KV destination, EPI_QKV only).
template <bool F32, int EPI>
__device__ __forceinline__ void gemm_store(const GemmArgs& a, int m, int n, float v, RowSlot rs) {
    if constexpr (EPI == EPI_GELU) {
        st_act<F32>(a.out, (size_t)m * a.N + n, gelu_tanh(v));
    } else {
        st_act<F32>(a.out, (size_t)m * a.N + n, v);
        if constexpr (EPI == EPI_QKV) {
            const int d = a.kv.d_model;
            if (n >= d && rs.phys >= 0) {
                const int kvsel = n >= 2 * d;
                const int r = n - d - kvsel * d;
                const size_t off = kv_offset(a.kv.layer, a.kv.n_pages, rs.phys, kvsel, a.kv.n_head, r / kHeadDim,
                                             rs.slot) + (r % kHeadDim);
                st_act<F32>(a.kv.base, off, v);
            }
        }
    }
}

// Epilogue of one output element.
template <bool F32, int EPI>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& a, int m, int n, float v, RowSlot rs) {
    v += ld_act<F32>(a.bias, n);
    if constexpr (EPI == EPI_RESID) {
        float* o = reinterpret_cast<float*>(a.out) + (size_t)m * a.N + n;
        *o += v;
    } else {
        gemm_store<F32, EPI>(a, m, n, v, rs);
    }
}

// fp32 tile GEMM: 64x64 outputs per 256-thread block, 4x4 per thread, k-tiles of 16.
template <int EPI>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const GemmArgs a) {
    __shared__ float sA[16][64 + 4];
    __shared__ float sB[16][64 + 4];
    const int tid = threadIdx.x, ty = tid >> 4, tx = tid & 15;
    const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
    const float* A = reinterpret_cast<const float*>(a.a);
    const float* W = reinterpret_cast<const float*>(a.w);
    float acc[4][4] = {};
    const int lr = tid >> 2, lk = (tid & 3) * 4;
    for (int k0 = 0; k0 < a.K; k0 += 16) {
        const int am = m0 + lr, bn = n0 + lr;
        float4 va = am < a.M ? *reinterpret_cast<const float4*>(A + (size_t)am * a.K + k0 + lk) : make_float4(0, 0, 0, 0);
        float4 vb = bn < a.N ? *reinterpret_cast<const float4*>(W + (size_t)bn * a.K + k0 + lk) : make_float4(0, 0, 0, 0);
        __syncthreads();
        sA[lk + 0][lr] = va.x; sA[lk + 1][lr] = va.y; sA[lk + 2][lr] = va.z; sA[lk + 3][lr] = va.w;
        sB[lk + 0][lr] = vb.x; sB[lk + 1][lr] = vb.y; sB[lk + 2][lr] = vb.z; sB[lk + 3][lr] = vb.w;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            float av[4], bv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) { av[i] = sA[k][ty * 4 + i]; bv[i] = sB[k][tx * 4 + i]; }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(av[i], bv[j], acc[i][j]);
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int m = m0 + ty * 4 + i, n = n0 + tx * 4 + j;
            if (m < a.M && n < a.N)
                gemm_epilogue<true, EPI>(a, m, n, acc[i][j], EPI == EPI_QKV ? row_slot(a, m) : RowSlot{-1, 0});
        }
}

// ---- launch shapes ------------------------------------------------------------------------
// Modelled times (us) of the two 16-bit kernels: least-squares fits to graph replays
// on 256 CUs, about 650 timings of 24 (N, K) x M shapes (66 to 10,800 rows, N and K
// 768-5120) over every tile shape and K split, with enough weight copies in turn that
// they come from where a model's weights do (500 MB for the GPT's widths, 190 MB for
// the DiT's); rms error 4-10% of those timings, which are of bare products: the model has
// no term for what an epilogue reads, computes and writes, which the launches compared for a
// shape share.  In the calls themselves launches take 13% longer than modelled on
// average (-7 to +39%): 256 x 5120 x 1280 + GELU 11.0 modelled and 15.1 traced, 10,827 x
// 1280 x 1280 residual 37.1 and 51.6, 10,827 x 3840 x 1280 99.4 and 107.8, 697 x 1280 x
// 5120 int8 22.6 and 24.9, 1000 x 3072 x 768 + GELU 11.8 and 12.9.  Choosing by the model costs 0.5%
// on average over the best timed choice of a shape (14% at worst).  No rule on one dimension does: 1000 x
// 5120 x 1280 takes 20.6 us in 128 x 256 tiles against 25.5 / 28.3 in 64 x 128 / 64 x
// 64, 1000 x 1280 x 1280 20.0 against 12.1 / 11.4, 10,800 x 5120 x 1280 138 in 256 x
// 256, 7,000 x 5120 x 1280 88 in 192 x 256 against 100.
//
// large, tile (mt, nt): a + rounds (b + steps f) + steps x tiles / 256 x g, a round
// being up to 256 tiles (32 an XCD) and a step 64 columns.  small, width bn: a + steps /
// splits x max(lat, per x load), + r for a split's round trip; load is the workgroups
// per CU, weighted between the fullest CU's (w) and the mean.
static double large_us(int mt, int nt, int M, int N, int K) {
    static const double c[2][3][4] = {{{4.05, 0.09, 0.514, 0.166}, {3.32, 1.68, 0.606, 0.199}, {4.23, 1.32, 0.734, 0.285}},
                                      {{4.96, 0.00, 0.640, 0.374}, {4.93, 1.67, 0.816, 0.447}, {5.99, 2.17, 0.983, 0.554}}};
    const double* p = c[nt - 1][mt - 2];
    const long tiles = (long)((M + 64 * mt - 1) / (64 * mt)) * ((N + 128 * nt - 1) / (128 * nt));
    const long rounds = ((tiles + 7) / 8 + 31) / 32, steps = K / 64;
    return p[0] + rounds * (p[1] + steps * p[2]) + p[3] * steps * tiles / 256.0;
}

static double small_us(int wdtype, int bn, int splits, int M, int N, int K) {
    static const double c[3][2][5] = {{{3.40, 0.256, 0.240, 2.88, 0.89}, {4.16, 0.342, 0.372, 5.03, 0.72}},
                                      {{4.49, 0.227, 0.227, 2.53, 0.48}, {4.81, 0.365, 0.351, 4.46, 0.78}},
                                      {{4.49, 0.353, 0.307, 2.53, 0.84}, {4.91, 0.611, 0.540, 4.63, 0.99}}};
    const double* p = c[wdtype - FTTS_BF16][bn / 64 - 1];
    const long groups = (long)((M + 63) / 64) * ((N + bn - 1) / bn) * splits;
    const double load = p[4] * (double)((groups + 255) / 256) + (1.0 - p[4]) * (double)groups / 256.0;
    return p[0] + (K / 64) / (double)splits * std::max(p[1], p[2] * load) + (splits > 1 ? p[3] : 0.0);
}

// A plan that splits K has at most this many tiles, and workgroups (tiles x slices), of
// at least 6 steps of 64 columns each, as far as was timed.
constexpr int kSplitTiles = 256, kSplitGroups = 512, kMaxSplits = 8, kSplitSteps = 6;

// The best small plan for M rows (its modelled time in *us).
static void plan_small(int wdtype, int M, int N, int K, GemmPlan* p, double* us) {
    *us = 1e30;
    for (int bn = 64; bn <= 128; bn += 64) {
        const long tiles = (long)((M + 63) / 64) * ((N + bn - 1) / bn);
        for (int s = 1; s <= kMaxSplits; ++s) {
            if (s > 1 && (tiles > kSplitTiles || tiles * s > kSplitGroups || K / 64 / s < kSplitSteps)) break;
            const double t = small_us(wdtype, bn, s, M, N, K);
            if (t < *us) *us = t, p->bn = bn, p->splits = s;
        }
    }
}

// The fastest modelled way: all rows on one kernel, or (bf16 weights) as many rows
// as fill whole rounds of the large kernel and the rest, which would leave its last
// round mostly idle, on the small one.
GemmPlan gemm_plan(int wdtype, int M, int N, int K) {
    GemmPlan best{};
    if (wdtype == FTTS_F32) return best;
    double best_us;
    plan_small(wdtype, M, N, K, &best, &best_us);
    if (wdtype != FTTS_BF16) return best;
    for (int nt = 1; nt <= 2; ++nt)
        for (int mt = 2; mt <= 4; ++mt) {
            GemmPlan p{};
            p.mt = mt, p.nt = nt;
            double us = large_us(mt, nt, M, N, K);
            if (us < best_us) best_us = us, best = p, best.rows_large = M;
            const int tn = (N + 128 * nt - 1) / (128 * nt), bm = 64 * mt;
            const int rounds = ((M + bm - 1) / bm * tn + 255) / 256;
            const int rows = (rounds - 1) * 256 / tn * bm;  // full rounds
            if (rows <= 0 || rows >= M) continue;
            double rest;
            plan_small(wdtype, M - rows, N, K, &p, &rest);
            us = large_us(mt, nt, rows, N, K) + rest;
            if (us < best_us) best_us = us, best = p, best.rows_large = rows;
        }
    return best;
}

// (A call of fewer rows may split where one of M rows does not, and the rows past the
// large kernel's are planned by themselves: the most that the small plan of any row
// count up to M writes.  A plan depends on the count of 64-row blocks only, and splits
// while there are at most kSplitTiles tiles.)
GemmScratch gemm_scratch(int wdtype, int M, int N, int K) {
    GemmScratch r{0, 0};
    if (wdtype == FTTS_F32 || K / 64 / kSplitSteps < 2) return r;
    const int blocks = std::min((M + 63) / 64, kSplitTiles / ((N + 127) / 128));
    for (int b = 1; b <= blocks; ++b) {
        GemmPlan p{};
        double us;
        plan_small(wdtype, 64 * b, N, K, &p, &us);
        if (p.splits < 2) continue;
        const int tiles = b * ((N + p.bn - 1) / p.bn);
        r.part_floats = std::max(r.part_floats, (size_t)tiles * p.splits * 64 * p.bn);
        r.n_count = std::max(r.n_count, tiles);
    }
    return r;
}

hipError_t launch_gemm(int wdtype, int epi, const GemmArgs& a, const GemmPlan& p, hipStream_t st) {
    if (wdtype == FTTS_F32) {
        const dim3 g((a.N + 63) / 64, (a.M + 63) / 64);
        switch (epi) {
            case EPI_STORE: hipLaunchKernelGGL(gemm_f32_kernel<EPI_STORE>, g, dim3(256), 0, st, a); break;
            case EPI_QKV: hipLaunchKernelGGL(gemm_f32_kernel<EPI_QKV>, g, dim3(256), 0, st, a); break;
            case EPI_GELU: hipLaunchKernelGGL(gemm_f32_kernel<EPI_GELU>, g, dim3(256), 0, st, a); break;
            case EPI_RESID: hipLaunchKernelGGL(gemm_f32_kernel<EPI_RESID>, g, dim3(256), 0, st, a); break;
            default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    if (p.rows_large > 0) {
        GemmArgs b = a;
        b.M = p.rows_large;
        const hipError_t e = launch_gemm_large(epi, b, p.mt, p.nt, st);
        if (e != hipSuccess || p.rows_large == a.M) return e;
    }
    GemmArgs b = a;
    b.M = a.M - p.rows_large;
    b.a = reinterpret_cast<const uint16_t*>(a.a) + (size_t)p.rows_large * a.K;
    b.out = reinterpret_cast<char*>(a.out) + (size_t)p.rows_large * a.N * (epi == EPI_RESID ? 4 : 2);
    if (epi == EPI_QKV) b.kv.slots = a.kv.slots + p.rows_large;
    return launch_gemm_small(wdtype, epi, b, p.bn, p.splits, st);
}

}  // namespace ftts

extern "C" int ftts_linear_plan(int32_t wdtype, int32_t M, int32_t N, int32_t K, ftts_linear_shape* out) {
    if (!out) return ftts::set_error(FTTS_E_INVALID_ARG, "out is NULL");
    if (wdtype < FTTS_BF16 || wdtype > FTTS_W4A16)
        return ftts::set_error(FTTS_E_DTYPE, "no matrix-core linears in wdtype %d", wdtype);
    if (M < 1 || M > (1 << 24) || N < 8 || N % 8 || K < 64 || K % (wdtype == FTTS_BF16 ? 64 : 128))
        return ftts::set_error(FTTS_E_SHAPE, "no matrix-core linear of %d x %d x %d", M, N, K);
    const ftts::GemmPlan p = ftts::gemm_plan(wdtype, M, N, K);
    const ftts::GemmScratch s = ftts::gemm_scratch(wdtype, M, N, K);
    *out = ftts_linear_shape{p.rows_large, p.rows_large ? 64 * p.mt : 0, p.rows_large ? 128 * p.nt : 0,
                             p.rows_large < M ? p.bn : 0, p.rows_large < M ? p.splits : 0, s.n_count,
                             (int64_t)s.part_floats};
    return FTTS_OK;
}
