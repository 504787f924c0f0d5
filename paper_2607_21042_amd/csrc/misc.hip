// Small kernels around the hot path: token+position embedding (with the
// per-row activity flag every later kernel reads), LayerNorm over packed rows
// (prefill), row gathers, the next-token sampler and the weight quantiser.
#include <algorithm>
#include <cfloat>
#include <climits>

#include "ftts_internal.hpp"

namespace ftts {

// ---- embedding ------------------------------------------------------------------------
// x[b] = tok_emb[tokens[b]] + pos_emb[positions[b]] (fp32).  A row is active when
// its token, position, KV slot and page are all in range; inactive rows get x = 0.
template <bool F32>
__global__ __launch_bounds__(256) void embed_kernel(const void* tok_emb, const void* pos_emb, int vocab,
                                                    int n_pos, int d, const int32_t* tokens,
                                                    const int32_t* positions, const int32_t* seq_lens,
                                                    const int32_t* block_table, int max_pages, int n_pages,
                                                    float* x, int32_t* active, float2* stats, uint32_t* zero,
                                                    int n_zero) {
    const int b = blockIdx.x, B = gridDim.x;
    const int t = tokens[b], p = positions[b], s = seq_lens[b];
    bool ok = t >= 0 && t < vocab && p >= 0 && p < n_pos && s >= 0 && s < max_pages * kPage;
    if (ok) {
        const int phys = block_table[(size_t)b * max_pages + s / kPage];
        ok = phys >= 0 && phys < n_pages;
    }
    if (threadIdx.x == 0) active[b] = ok ? 1 : 0;
    for (int i = b * 256 + threadIdx.x; i < n_zero; i += B * 256) zero[i] = 0u;
    float* xr = x + (size_t)b * d;
    // the embedding rows are read at clamped indices without waiting for the page
    // check (the value of an inactive row is dropped)
    const int tc = min(max(t, 0), vocab - 1), pc = min(max(p, 0), n_pos - 1);
    // d is a multiple of 64, so every pass of this loop keeps whole waves active
    for (int k = threadIdx.x; k < d; k += blockDim.x) {
        float v = ld_act<F32>(tok_emb, (size_t)tc * d + k) + ld_act<F32>(pos_emb, (size_t)pc * d + k);
        v = ok ? v : 0.f;
        xr[k] = v;
        if (stats) {
            const float2 ts = tile_stats32(v);
            if ((k & (kStatTile - 1)) == 0) stats[(size_t)(k / kStatTile) * B + b] = ts;
        }
    }
}

hipError_t launch_embed(int wdtype, const void* tok_emb, const void* pos_emb, int vocab, int n_pos, int d,
                        const int32_t* tokens, const int32_t* positions, const int32_t* seq_lens,
                        const int32_t* block_table, int max_pages, int n_pages, int B, float* x,
                        int32_t* active, float2* stats, uint32_t* zero, int n_zero, hipStream_t st) {
    if (stats && d % 64 != 0) return hipErrorInvalidValue;
    if (wdtype == FTTS_F32)
        hipLaunchKernelGGL(embed_kernel<true>, dim3(B), dim3(256), 0, st, tok_emb, pos_emb, vocab, n_pos, d,
                           tokens, positions, seq_lens, block_table, max_pages, n_pages, x, active, stats, zero,
                           n_zero);
    else
        hipLaunchKernelGGL(embed_kernel<false>, dim3(B), dim3(256), 0, st, tok_emb, pos_emb, vocab, n_pos, d,
                           tokens, positions, seq_lens, block_table, max_pages, n_pages, x, active, stats, zero,
                           n_zero);
    return hipGetLastError();
}

// ---- block reductions -------------------------------------------------------------------
__device__ __forceinline__ float block_sum256(float v, float* red) {
    v = wave_sum(v);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    return red[0] + red[1] + red[2] + red[3];
}

// ---- LayerNorm over packed rows (prefill): fp32 x -> activation dtype ----------------------
template <bool F32>
__global__ __launch_bounds__(256) void ln_rows_kernel(const float* x, const void* g, const void* bb, float eps,
                                                      int d, void* out) {
    __shared__ float red[4];
    const size_t r = blockIdx.x;
    const float* xr = x + r * d;
    float s = 0.f;
    for (int k = threadIdx.x; k < d; k += 256) s += xr[k];
    const float mean = block_sum256(s, red) / (float)d;
    float v = 0.f;
    for (int k = threadIdx.x; k < d; k += 256) {
        const float t = xr[k] - mean;
        v = fmaf(t, t, v);
    }
    const float var = block_sum256(v, red) / (float)d;
    const float rstd = 1.0f / sqrtf(var + eps);
    for (int k = threadIdx.x; k < d; k += 256)
        st_act<F32>(out, r * d + k, (xr[k] - mean) * rstd * ld_act<F32>(g, k) + ld_act<F32>(bb, k));
}

// One wave per row for rows of up to 2048 columns that split into float4 lanes (N per
// lane): the row stays in registers, both reductions are cross-lane, no barriers.  Short
// launches are bound by their dependent loads, so the gains and biases are requested
// with the row (bf16; asked for after the reductions they cost another trip to memory).
// Traced in a call, before (gains last, width a runtime value) and now: 256 x 1280 5.0 and
// 3.9 us, 10,827 x 1280 15.6 and 13.8, 1000 x 768 4.4 and 4.4, 11,154 x 768 11.0 and 9.0.
template <bool F32, int N>
__global__ __launch_bounds__(256) void ln_rows_wave_kernel(const float* x, const void* g, const void* bb, float eps,
                                                           int M, int d, void* out) {
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (r >= M) return;
    const float4* xr = reinterpret_cast<const float4*>(x + (size_t)r * d);
    const int n4 = d / 4;
    float4 v[N];
    uint2 gw[F32 ? 1 : N], bw[F32 ? 1 : N];
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = xr[min(lane + 64 * i, n4 - 1)];
    if constexpr (!F32) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            gw[i] = reinterpret_cast<const uint2*>(g)[min(lane + 64 * i, n4 - 1)];
            bw[i] = reinterpret_cast<const uint2*>(bb)[min(lane + 64 * i, n4 - 1)];
        }
    }
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if (lane + 64 * i >= n4) v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        s += (v[i].x + v[i].y) + (v[i].z + v[i].w);
    }
    const float mean = wave_sum(s) / (float)d;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if (lane + 64 * i < n4) {
            const float a = v[i].x - mean, b = v[i].y - mean, c = v[i].z - mean, e = v[i].w - mean;
            q = fmaf(a, a, fmaf(b, b, fmaf(c, c, fmaf(e, e, q))));
        }
    }
    const float rstd = 1.0f / sqrtf(wave_sum(q) / (float)d + eps);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int j = lane + 64 * i;
        if (j < n4) {
            const float xs[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
            if constexpr (F32) {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    st_act<F32>(out, (size_t)r * d + 4 * j + k,
                                (xs[k] - mean) * rstd * ld_act<F32>(g, 4 * j + k) + ld_act<F32>(bb, 4 * j + k));
            } else {
                // four bf16 gains, biases and outputs per 8-byte access (rows of d % 4 == 0)
                const uint32_t gs[2] = {gw[i].x, gw[i].y}, bs[2] = {bw[i].x, bw[i].y};
                uint32_t o[2];
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const float y0 = (xs[2 * k] - mean) * rstd * __uint_as_float(gs[k] << 16) +
                                     __uint_as_float(bs[k] << 16);
                    const float y1 = (xs[2 * k + 1] - mean) * rstd * __uint_as_float(gs[k] & 0xFFFF0000u) +
                                     __uint_as_float(bs[k] & 0xFFFF0000u);
                    o[k] = (uint32_t)f32_to_bf16(y0) | ((uint32_t)f32_to_bf16(y1) << 16);
                }
                reinterpret_cast<uint2*>(out)[((size_t)r * d) / 4 + j] = make_uint2(o[0], o[1]);
            }
        }
    }
}

template <bool F32, int N>
static void ln_rows_wave(const float* x, const void* g, const void* b, float eps, int M, int d, void* out, hipStream_t st) {
    if constexpr (N < 8) {
        if (d > 256 * N) return ln_rows_wave<F32, N + 1>(x, g, b, eps, M, d, out, st);
    }
    hipLaunchKernelGGL((ln_rows_wave_kernel<F32, N>), dim3((M + 3) / 4), dim3(256), 0, st, x, g, b, eps, M, d, out);
}

hipError_t launch_ln_rows(int wdtype, const float* x, const void* g, const void* b, float eps, int M, int d,
                          void* out, hipStream_t st) {
    if (d % 4 == 0 && d <= 2048) {
        if (wdtype == FTTS_F32) ln_rows_wave<true, 1>(x, g, b, eps, M, d, out, st);
        else ln_rows_wave<false, 1>(x, g, b, eps, M, d, out, st);
        return hipGetLastError();
    }
    if (wdtype == FTTS_F32) hipLaunchKernelGGL(ln_rows_kernel<true>, dim3(M), dim3(256), 0, st, x, g, b, eps, d, out);
    else hipLaunchKernelGGL(ln_rows_kernel<false>, dim3(M), dim3(256), 0, st, x, g, b, eps, d, out);
    return hipGetLastError();
}

// ---- fill (graph-safe replacement for a memset) -------------------------------------------------
__global__ void fill_u32_kernel(uint32_t* p, size_t n, uint32_t v) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}

hipError_t launch_fill_u32(uint32_t* p, size_t n, uint32_t v, hipStream_t st) {
    const int blocks = (int)((n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024);
    hipLaunchKernelGGL(fill_u32_kernel, dim3(blocks > 0 ? blocks : 1), dim3(256), 0, st, p, n, v);
    return hipGetLastError();
}

// ---- prefill bookkeeping: KV slot of every packed row, split-K counters ---------------------------
// A row's slot is physical page * 64 + slot in the page (pages stay below 2^25:
// a page of one layer is at least 32 KB), or -1.
__global__ __launch_bounds__(256) void prefill_setup_kernel(SeqTable seqs, const int32_t* block_table, int max_pages,
                                                            int n_pages, int M, int32_t* slots, uint32_t* count,
                                                            size_t n_count) {
    const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x, step = (size_t)gridDim.x * blockDim.x;
    for (size_t i = i0; i < n_count; i += step) count[i] = 0u;
    for (size_t i = i0; i < (size_t)M; i += step) {
        const int m = (int)i;
        int lo = 0, hi = seqs.n - 1;  // the sequence holding row m: cu[sq] <= m < cu[sq + 1]
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (seqs.cu[mid] <= m) lo = mid;
            else hi = mid - 1;
        }
        const int t = m - seqs.cu[lo], page = t / kPage;
        int phys = -1;
        if (page < max_pages) {
            phys = block_table[(size_t)lo * max_pages + page];
            if (phys < 0 || phys >= n_pages) phys = -1;
        }
        slots[m] = phys < 0 ? -1 : phys * kPage + t % kPage;
    }
}

hipError_t launch_prefill_setup(const SeqTable& seqs, const int32_t* block_table, int max_pages, int n_pages, int M,
                                int32_t* slots, uint32_t* count, size_t n_count, hipStream_t st) {
    const size_t n = std::max((size_t)M, n_count);
    const int blocks = (int)std::min<size_t>((n + 255) / 256, 1024);
    hipLaunchKernelGGL(prefill_setup_kernel, dim3(std::max(blocks, 1)), dim3(256), 0, st, seqs, block_table, max_pages,
                       n_pages, M, slots, count, n_count);
    return hipGetLastError();
}

// ---- row copies ----------------------------------------------------------------------------
__global__ void gather_last_kernel(const float* x, int d, SeqTable seqs, float* out) {
    const int b = blockIdx.x;
    const float* src = x + (size_t)(seqs.cu[b + 1] - 1) * d;
    for (int k = threadIdx.x; k < d; k += blockDim.x) out[(size_t)b * d + k] = src[k];
}

hipError_t launch_gather_rows(const float* x, int d, const SeqTable& seqs, float* out, hipStream_t st) {
    hipLaunchKernelGGL(gather_last_kernel, dim3(seqs.n), dim3(256), 0, st, x, d, seqs, out);
    return hipGetLastError();
}

template <bool F32>
__global__ void act_to_f32_kernel(const void* src, size_t n, float* dst) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        dst[i] = ld_act<F32>(src, i);
}

hipError_t launch_act_to_f32(int wdtype, const void* src, int rows, int d, float* dst, hipStream_t st) {
    const size_t n = (size_t)rows * d;
    const int blocks = (int)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096);
    if (wdtype == FTTS_F32) hipLaunchKernelGGL(act_to_f32_kernel<true>, dim3(blocks), dim3(256), 0, st, src, n, dst);
    else hipLaunchKernelGGL(act_to_f32_kernel<false>, dim3(blocks), dim3(256), 0, st, src, n, dst);
    return hipGetLastError();
}

// ---- prefill input assembly -----------------------------------------------------------------
// One workgroup per assembled row.  Text ids outside [0, text_vocab) read as a
// zero token row (only the position embedding remains); no access leaves the tables.
template <bool F32>
__global__ __launch_bounds__(256) void assemble_prefix_kernel(const AssembleArgs a) {
    const int r = blockIdx.x;
    int lo = 0, hi = a.seqs.n - 1;  // the sequence holding row r
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (a.seqs.cu[mid] <= r) lo = mid;
        else hi = mid - 1;
    }
    const int j = r - a.seqs.cu[lo], nc = a.cond_cu[lo + 1] - a.cond_cu[lo];
    float* xr = a.x + (size_t)r * a.d;
    if (j < nc) {
        const size_t src = (size_t)(a.cond_cu[lo] + j) * a.d;
        for (int k = threadIdx.x; k < a.d; k += blockDim.x) xr[k] = ld_act<F32>(a.cond, src + k);
        return;
    }
    const int i = j - nc;                                 // text position within the sequence
    const int id = a.text_ids[a.seqs.cu[lo] - a.cond_cu[lo] + i];
    const bool ok = id >= 0 && id < a.text_vocab;
    const size_t tr = (size_t)(a.vocab + (ok ? id : 0)) * a.d, pr = (size_t)(a.text_pos0 + i) * a.d;
    for (int k = threadIdx.x; k < a.d; k += blockDim.x)
        xr[k] = (ok ? ld_act<F32>(a.tok_emb, tr + k) : 0.f) + ld_act<F32>(a.pos_emb, pr + k);
}

hipError_t launch_assemble_prefix(int wdtype, const AssembleArgs& a, int rows, hipStream_t st) {
    if (wdtype == FTTS_F32) hipLaunchKernelGGL(assemble_prefix_kernel<true>, dim3(rows), dim3(256), 0, st, a);
    else hipLaunchKernelGGL(assemble_prefix_kernel<false>, dim3(rows), dim3(256), 0, st, a);
    return hipGetLastError();
}

// ---- sampler ------------------------------------------------------------------------------
// One 1024-thread workgroup per sequence; thread t holds the tempered logits of
// indices t, t + 1024, ... in registers.  Order is by (value, index): the larger
// value first, the lower index on ties.  NaN logits count as -inf.
//
// Top-k without k sequential block reductions.  If t is the k-th largest of the maxima
// over disjoint groups of entries, at least k entries are >= t, so every one of the k
// best is, and few others are.  The fewer the groups, the shorter the count that finds
// t, and the more candidates it lets through; so, where the row reaches k of them, the 16
// waves serve k <= 16 and 64 groups of 16 lanes k <= 32 (every wave finds t by itself
// after one barrier), else 256 groups of four lanes (one thread each and a second
// barrier; about 32 candidates for k = 30 and spread-out logits).  The entries >= t and
// above -inf are collected in LDS as 64-bit keys that sort by (value, index), each is
// ranked by counting the keys above it, and ranks below k fill the ordered top-k list.
// t = -inf, all entries above -inf, serves rows of up to kSampShort entries and rows masked
// so that few threads hold one; if there are fewer than k, the lowest-index -inf
// entries take the ranks after them.  Where the candidates exceed kSampShort (a crowd of
// equal entries, as in a row masked with a finite value), the best of the waves' own k-th
// largest lane maxima is tried; rows that still have more than kSampCand take k rounds of
// block argmax.
//
// A row is 33 KB, so the kernel is bound by its chain of short steps.  Measured, us a call:
// 32 rows of 8194 at k = 30: 8.2 (10.2 with 256 groups for every k; 24 with 256 threads, a threshold per
// wave that let about 180 candidates through, ranked one LDS read at a time); at k = 10
// 8.9 (9.9 with 256 groups), k = 64 12.0; at k = 30 100 entries 7.8, 8194 masked to a run of 90
// by -inf 8.6, by a finite value 11.4 (50-57 by rounds of argmax); 1024 rows of 16384, bound by reading them, 14.0
// greedy and 17.0 at k = 2 (25.1 with 256 groups).
constexpr int kSampThreads = 1024, kSampWaves = kSampThreads / kWave, kSampPer = 16;  // vocab <= 16384
constexpr int kSampCand = 1024;
constexpr int kSampFew = 128;    // masked rows: so few threads hold an entry above -inf that all of them are candidates
constexpr int kSampShort = 256;  // rows of up to this many entries are ranked whole

__device__ __forceinline__ bool beats(float v, int i, float bv, int bi) {
    return v > bv || (v == bv && i < bi);
}

template <int CTRL>
__device__ __forceinline__ int dpp_mov_int(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}
__device__ __forceinline__ int wave_min_int(int v) {
    v = min(v, dpp_mov_int<kDppQuadSwap1>(v));
    v = min(v, dpp_mov_int<kDppQuadSwap2>(v));
    v = min(v, dpp_mov_int<kDppHalfMirror>(v));
    v = min(v, dpp_mov_int<kDppMirror>(v));
    {
        const auto r = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
        v = min((int)r[0], (int)r[1]);
    }
    {
        const auto r = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
        v = min((int)r[0], (int)r[1]);
    }
    return v;
}

// Best (value, index) of the wave, in every lane: the largest value, then the
// lowest index holding it.  Lanes with nothing to offer pass (-inf, INT_MAX).
__device__ __forceinline__ void wave_best(float& v, int& i) {
    const float m = wave_max(v);
    i = wave_min_int(v == m ? i : INT_MAX);
    v = m;
}

// Best untaken entry of this lane (indices increase with the slot, so the
// first of equal values wins).
__device__ __forceinline__ void lane_best(const float (&z)[kSampPer], uint32_t taken, float& bv, int& bi) {
    bv = -INFINITY;
    bi = INT_MAX;
#pragma unroll
    for (int j = 0; j < kSampPer; ++j)
        if (!((taken >> j) & 1u) && (z[j] > bv || bi == INT_MAX)) {
            bv = z[j];
            bi = (int)threadIdx.x + kSampThreads * j;
        }
}

// Block-wide best; every thread receives it.
__device__ __forceinline__ void block_best(float& v, int& i, float* rv, int* ri) {
    wave_best(v, i);
    const int w = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0) {
        rv[w] = v;
        ri[w] = i;
    }
    __syncthreads();
    v = rv[0];
    i = ri[0];
    for (int j = 1; j < kSampWaves; ++j)
        if (beats(rv[j], ri[j], v, i)) {
            v = rv[j];
            i = ri[j];
        }
    __syncthreads();
}

// How many of the n values v (16-byte aligned) are above, and at or above, own.
template <int n>
__device__ __forceinline__ void count_above(const float* v, float own, int& gt, int& ge) {
    const float4* v4 = reinterpret_cast<const float4*>(v);
#pragma unroll 8
    for (int c = 0; c < n / 4; ++c) {
        const float4 o = v4[c];
        gt += (o.x > own) + (o.y > own) + (o.z > own) + (o.w > own);
        ge += (o.x >= own) + (o.y >= own) + (o.z >= own) + (o.w >= own);
    }
}
// The k-th largest of n values, in every lane (lane i looks at value `at` = i % n).
template <int n>
__device__ __forceinline__ float kth_largest(const float* v, int at, int k) {
    const float own = v[at];
    int gt = 0, ge = 0;
    count_above<n>(v, own, gt, ge);
    const uint64_t hit = __ballot(gt < k && k <= ge);
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(own), (int)__builtin_ctzll(hit)));
}

// This thread's entries of a row: tempered logits (GREEDY: as they are), NaN as -inf,
// -inf past the row.  The row, the draw and the activity flag are requested together;
// false if the sequence is not active.
template <bool GREEDY>
__device__ __forceinline__ bool sample_load(const float* row, int V, float temperature, const float* uniform,
                                            const int32_t* active, float (&z)[kSampPer], float& u) {
#pragma unroll
    for (int j = 0; j < kSampPer; ++j) {
        const int i = (int)threadIdx.x + kSampThreads * j;
        z[j] = i < V ? row[i] : -INFINITY;
    }
    u = GREEDY ? 0.f : *uniform;
    if (active && !*active) return false;
#pragma unroll
    for (int j = 0; j < kSampPer; ++j) {
        if (kSampThreads * j >= V) continue;  // uniform: slots past the row stay -inf
        const float v = GREEDY ? z[j] : z[j] / temperature;
        z[j] = v != v ? -INFINITY : v;
    }
    return true;
}

__global__ __launch_bounds__(kSampThreads) void greedy_kernel(const float* logits, int V, const int32_t* active,
                                                              int32_t* out) {
    __shared__ float rv[kSampWaves];
    __shared__ int ri[kSampWaves];
    const int b = blockIdx.x, tid = threadIdx.x;
    float z[kSampPer], u, bv;
    int bi;
    if (!sample_load<true>(logits + (size_t)b * V, V, 1.f, nullptr, active ? active + b : nullptr, z, u)) {
        if (tid == 0) out[b] = -1;
        return;
    }
    lane_best(z, 0, bv, bi);
    block_best(bv, bi, rv, ri);
    if (tid == 0) out[b] = bi < V ? bi : 0;
}

// G: the groups whose maxima are tried first.
template <int G>
__global__ __launch_bounds__(kSampThreads) void sample_kernel(const float* logits, int V, float temperature,
                                                              int top_k, float top_p, const float* uniforms,
                                                              const int32_t* active, int32_t* out) {
    __shared__ __attribute__((aligned(16))) float s_gm[kSampThreads / 4];  // group maxima
    __shared__ __attribute__((aligned(16))) float s_lane[kSampThreads];    // lane maxima
    __shared__ __attribute__((aligned(16))) uint64_t s_key[kSampCand + 8];
    __shared__ float selv[FTTS_MAX_TOP_K];
    __shared__ int seli[FTTS_MAX_TOP_K];
    __shared__ float rv[kSampWaves];
    __shared__ int ri[kSampWaves];
    __shared__ int s_cnt;
    __shared__ float s_t;
    const int b = blockIdx.x, tid = threadIdx.x, wave = tid / kWave, lane = tid & (kWave - 1);
    float z[kSampPer], u;
    if (tid == 0) s_cnt = 0;
    if (!sample_load<false>(logits + (size_t)b * V, V, temperature, uniforms + b, active ? active + b : nullptr, z, u)) {
        if (tid == 0) out[b] = -1;
        return;
    }
    float lm = -INFINITY;
#pragma unroll
    for (int j = 0; j < kSampPer; ++j) lm = fmaxf(lm, z[j]);
    float t = -INFINITY;
    if (V <= kSampShort) {
        __syncthreads();
    } else {
        int holders = kSampThreads;  // threads with an entry above -inf, where that is known
        if constexpr (G < kSampThreads / 4) {
            const float gm = group_max<kSampThreads / G>(lm);
            if ((lane & (kSampThreads / G - 1)) == 0) s_gm[tid / (kSampThreads / G)] = gm;
            __syncthreads();
            t = kth_largest<G>(s_gm, lane & (G - 1), top_k);
            if (t == -INFINITY) holders = __syncthreads_count(lm > -INFINITY);
        }
        if (t == -INFINITY && holders > kSampFew) {  // (uniform over the workgroup)
            const float gm = group_max<4>(lm);
            if ((lane & 3) == 0) s_gm[tid >> 2] = gm;
            __syncthreads();
            if (tid < kSampThreads / 4) {
                const float own = s_gm[tid];
                int gt = 0, ge = 0;
                count_above<kSampThreads / 4>(s_gm, own, gt, ge);
                if (gt < top_k && top_k <= ge) s_t = own;  // (every thread that writes holds the same value)
            }
            __syncthreads();
            t = s_t;
        }
    }
    t = fmaxf(t, -FLT_MAX);  // (neither the slots past the row nor masked entries compete)
    auto collect = [&] {
        if (lm >= t) {
#pragma unroll
            for (int j = 0; j < kSampPer; ++j)
                if (z[j] >= t) {
                    const int c = atomicAdd(&s_cnt, 1);
                    // larger value first, then lower index (+ 0.f: -0 ties with +0)
                    const uint32_t u = __float_as_uint(z[j] + 0.f), k = (u >> 31) ? ~u : u | 0x80000000u;
                    if (c < kSampCand) s_key[c] = ((uint64_t)k << 32) | (uint32_t)(0x7FFFFFFF - (tid + kSampThreads * j));
                }
        }
        __syncthreads();
        return s_cnt;
    };
    int total = collect();
    if (total > kSampShort) {
        // A crowd of equal entries at t, as a mask with a finite value leaves: the k-th largest
        // lane maximum of any one wave bounds the k best as well, and may lie above it.
        s_lane[tid] = lm;
        __syncthreads();
        const float tw = kth_largest<kWave>(s_lane + wave * kWave, lane, top_k);
        if (lane == 0) rv[wave] = tw;
        __syncthreads();
        float t2 = rv[0];
        for (int w = 1; w < kSampWaves; ++w) t2 = fmaxf(t2, rv[w]);
        if (t2 > t) {  // (uniform over the workgroup)
            t = t2;
            if (tid == 0) s_cnt = 0;
            __syncthreads();
            total = collect();
        }
    }
    if (total <= kSampCand) {
        if (tid < 8) s_key[total + tid] = 0;  // below every key, so that the ranking reads whole groups of 8
        if (total < top_k && wave == 0) {  // at least k - total of the first k <= 64 entries are -inf
            const uint64_t none = __ballot(lane < top_k && z[0] == -INFINITY);
            const int r = total + __popcll(none & ((1ull << lane) - 1));
            if (((none >> lane) & 1) && r < top_k) {
                selv[r] = -INFINITY;
                seli[r] = lane;
            }
        }
        __syncthreads();
        for (int c = tid; c < total; c += kSampThreads) {
            const uint64_t own = s_key[c];
            int r = 0;
            for (int c2 = 0; c2 < total; c2 += 8) {
                uint64_t o[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = s_key[c2 + e];
#pragma unroll
                for (int e = 0; e < 8; ++e) r += o[e] > own ? 1 : 0;
            }
            if (r < top_k) {
                const uint32_t k = (uint32_t)(own >> 32);
                selv[r] = __uint_as_float((k >> 31) ? k & 0x7FFFFFFFu : ~k);
                seli[r] = 0x7FFFFFFF - (int)(uint32_t)own;
            }
        }
        __syncthreads();
    } else {
        uint32_t taken = 0;
        float bv;
        int bi;
        __syncthreads();  // every thread has read the waves' thresholds in rv
        lane_best(z, taken, bv, bi);
        for (int r = 0; r < top_k; ++r) {
            float wv = bv;
            int wi = bi;
            block_best(wv, wi, rv, ri);
            if (tid == 0) {
                selv[r] = wv;
                seli[r] = wi;
            }
            if (wi == bi && (wi - tid) % kSampThreads == 0) {  // this thread held the winner
                taken |= 1u << ((wi - tid) / kSampThreads);
                lane_best(z, taken, bv, bi);
            }
        }
        __syncthreads();
    }
    if (wave != 0) return;
    // fp32 tail in wave 0, lane i holding rank i: the weights exp(z_i - z_1) side
    // by side, then the running sums in rank order (the same additions as a
    // sequential loop), the nucleus cut and the inverse-CDF draw by ballot.
    const bool in = lane < top_k;
    const float e = in ? expf(selv[lane] - selv[0]) : 0.f;
    float acc = 0.f, cum = 0.f;
    for (int i = 0; i < top_k; ++i) {
        acc = acc + __int_as_float(__builtin_amdgcn_readlane(__float_as_int(e), i));
        cum = lane == i ? acc : cum;
    }
    const float thresh = top_p * acc;
    const uint64_t ge = __ballot(in && cum >= thresh);
    const int n = ge ? (int)__builtin_ctzll(ge) + 1 : top_k;
    const float rr = u * __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cum), n - 1));
    const uint64_t gt = __ballot(lane < n && cum > rr);
    const int j = gt ? (int)__builtin_ctzll(gt) : n - 1;
    if (lane == 0) out[b] = seli[j] < V ? seli[j] : 0;
}

hipError_t launch_sample(const float* logits, int B, int V, const ftts_sampling& s, const float* uniforms,
                         const int32_t* active, int32_t* out, hipStream_t st) {
    if (V > kSampThreads * kSampPer || s.top_k < 1 || s.top_k > FTTS_MAX_TOP_K) return hipErrorInvalidValue;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(B), dim3(kSampThreads), 0, st, logits, V, s.temperature, s.top_k, s.top_p, uniforms,
                           active, out);
    };
    // as few groups as give a threshold near the k-th best, where the row reaches k of them
    if (s.top_k == 1) hipLaunchKernelGGL(greedy_kernel, dim3(B), dim3(kSampThreads), 0, st, logits, V, active, out);
    else if (s.top_k <= std::min(16, V / 64)) launch(sample_kernel<16>);
    else if (s.top_k <= std::min(32, V / 16)) launch(sample_kernel<64>);
    else launch(sample_kernel<256>);
    return hipGetLastError();
}

// ---- generation-loop bookkeeping -----------------------------------------------------------
__global__ __launch_bounds__(1024) void advance_kernel(int32_t* tokens, int32_t* positions, int32_t* seq_lens,
                                                       int32_t* sampled, int32_t* remaining, int32_t stop_token,
                                                       bool retire_on_stop, int32_t* history, int32_t* step_counter,
                                                       int max_steps, int B) {
    const int step = step_counter ? *step_counter : 0;
    // this thread's first row, requested with the counter (a row is read and
    // written by its own thread only)
    const int b0 = threadIdx.x;
    const int tok0 = b0 < B ? tokens[b0] : -1, smp0 = b0 < B ? sampled[b0] : -1;
    __syncthreads();  // every thread has read the counter before it moves
    for (int b = threadIdx.x; b < B; b += blockDim.x) {
        int h = -1;
        if ((b == b0 ? tok0 : tokens[b]) >= 0) {
            seq_lens[b] += 1;
            positions[b] += 1;
            int next = b == b0 ? smp0 : sampled[b];
            bool retire = retire_on_stop && next == stop_token;  // the model's own stop code
            if (remaining) {
                const int r = remaining[b] - 1;
                remaining[b] = r;
                if (r <= 0) {  // the budget's last step: forced stop code
                    next = stop_token;
                    sampled[b] = stop_token;
                    retire = true;
                }
            }
            tokens[b] = retire ? -1 : next;
            h = next;
        }
        if (history && step < max_steps) history[(size_t)step * B + b] = h;
    }
    if (step_counter && threadIdx.x == 0) *step_counter = step + 1;
}

hipError_t launch_advance(int32_t* tokens, int32_t* positions, int32_t* seq_lens, int32_t* sampled,
                          int32_t* remaining, int32_t stop_token, bool retire_on_stop, int32_t* history,
                          int32_t* step_counter, int max_steps, int B, hipStream_t st) {
    hipLaunchKernelGGL(advance_kernel, dim3(1), dim3(B < 64 ? 64 : (B + 63) / 64 * 64), 0, st, tokens, positions,
                       seq_lens, sampled, remaining, stop_token, retire_on_stop, history, step_counter, max_steps,
                       B);
    return hipGetLastError();
}

// ---- weight quantiser ----------------------------------------------------------------------
// W8A16: one block per row.  s = bf16(amax / 127) (1 if 0); code = clamp(rint(w / s), -127, 127).
__global__ __launch_bounds__(256) void quant_w8_kernel(const float* w, int64_t K, int8_t* codes,
                                                       uint16_t* scales) {
    __shared__ float red[4];
    const int64_t n = blockIdx.x;
    const float* wr = w + n * K;
    float m = 0.f;
    for (int64_t k = threadIdx.x; k < K; k += 256) m = fmaxf(m, fabsf(wr[k]));
    m = wave_max(m);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    const float amax = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    uint16_t sb = f32_to_bf16(amax / 127.0f);
    if ((sb & 0x7FFF) == 0) sb = 0x3F80;  // zero scale -> 1
    const float s = bf16_to_f32(sb);
    if (threadIdx.x == 0) scales[n] = sb;
    for (int64_t k = threadIdx.x; k < K; k += 256) {
        const float q = fminf(fmaxf(rintf(wr[k] / s), -127.f), 127.f);
        codes[n * K + k] = (int8_t)q;
    }
}

// W4A16: one block of `group` threads per (row, group).  The range [min(0, mn), max(0, mx)]
// sets s = bf16((mx - mn) / 15) (1 if 0) and z = clamp(rint(-mn / s), 0, 15);
// code = clamp(rint(w / s) + z, 0, 15), packed eight to an int32, low nibble first.
__global__ __launch_bounds__(128) void quant_w4_kernel(const float* w, int64_t K, int group, int32_t* codes,
                                                       uint16_t* scales, uint16_t* zeros) {
    __shared__ float rmin[2], rmax[2];
    __shared__ uint8_t q8[128];
    const int g = blockIdx.x;
    const int64_t n = blockIdx.y;
    const int t = threadIdx.x;
    const float v = w[n * K + (int64_t)g * group + t];
    float mn = v, mx = v;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        mn = fminf(mn, __shfl_xor(mn, o, kWave));
        mx = fmaxf(mx, __shfl_xor(mx, o, kWave));
    }
    if ((t & 63) == 0) {
        rmin[t >> 6] = mn;
        rmax[t >> 6] = mx;
    }
    __syncthreads();
    mn = fminf(fminf(rmin[0], rmin[1]), 0.f);
    mx = fmaxf(fmaxf(rmax[0], rmax[1]), 0.f);
    uint16_t sb = f32_to_bf16((mx - mn) / 15.0f);
    if ((sb & 0x7FFF) == 0) sb = 0x3F80;
    const float s = bf16_to_f32(sb);
    const float z = fminf(fmaxf(rintf(-mn / s), 0.f), 15.f);
    const float q = fminf(fmaxf(rintf(v / s) + z, 0.f), 15.f);
    q8[t] = (uint8_t)q;
    __syncthreads();
    const int n_groups = (int)(K / group);
    if (t == 0) {
        scales[n * n_groups + g] = sb;
        zeros[n * n_groups + g] = f32_to_bf16(z);
    }
    if (t < group / 8) {
        uint32_t word = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) word |= (uint32_t)q8[t * 8 + j] << (4 * j);
        codes[n * (K / 8) + (int64_t)g * (group / 8) + t] = (int32_t)word;
    }
}

hipError_t launch_quantize(int wdtype, const float* w, int64_t N, int64_t K, int group, void* codes,
                           uint16_t* scales, uint16_t* zeros, hipStream_t st) {
    if (wdtype == FTTS_W8A16) {
        hipLaunchKernelGGL(quant_w8_kernel, dim3((unsigned)N), dim3(256), 0, st, w, K, (int8_t*)codes, scales);
    } else {
        hipLaunchKernelGGL(quant_w4_kernel, dim3((unsigned)(K / group), (unsigned)N), dim3(group), 0, st, w, K,
                           group, (int32_t*)codes, scales, zeros);
    }
    return hipGetLastError();
}

}  // namespace ftts
