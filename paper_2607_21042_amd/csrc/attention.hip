// Attention kernels.
//
// Decode (one query row per sequence and head, over its paged KV cache):
//   o_h = softmax(q_h K_h^T / sqrt(64)) V_h over cached slots 0 .. seq_len
// One workgroup per (head, sequence) whose 8 waves stride over the logical
// pages (split-K inside the workgroup).  A 64x64 K or V page is read as 8 fully
// coalesced 1 KB wave loads, lane l holding dims (l%8)*8 .. +7 of tokens
// i*8 + l/8 (with 16-bit pages the next page's K and V would be loaded while
// the current one is used; only the fp32 instantiation is launched).
// Scores are reduced over the 8 lanes of a token, each page's softmax is
// folded into a running (max, sum, output) triple, and the 8 wave partials
// are merged in LDS with the log-sum-exp rule.  The walk follows logical
// pages, so the result does not depend on where pages live in the pool.  This
// is the fp32-KV kernel; the 16-bit KV kernel (attn_decode_bf16_kernel, below)
// keeps one page per wave in registers so that two groups share a CU.
//
// Prefill (causal attention over each prefix) and full attention (no mask: the
// flow-matching DiT's frames all see each other).  16-bit activations run on the
// matrix cores: attn_tile.hip, whose waves share each key tile on wide grids and split the
// keys of a 32-query tile on short ones.  A wave forms
// S^T = K Q^T (keys as rows, so every lane ends up holding 32 scores of its own query),
// applies the online softmax per lane, and accumulates O^T = V^T P^T with the
// probabilities taken straight from its score registers: the MFMA k order is a
// permutation shared by both operands, so P needs no reshuffle.  fp32 activations keep
// a VALU kernel: one thread per query row streams 64-key tiles of K and V through LDS.
#include <algorithm>

#include "kv_page.hpp"

namespace ftts {

template <bool F32>
__device__ __forceinline__ void load8(const void* base, size_t elem, float (&v)[8]) {
    if constexpr (F32) {
        const float4* p = reinterpret_cast<const float4*>(reinterpret_cast<const float*>(base) + elem);
        const float4 a = p[0], b = p[1];
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    } else {
        const uint4 w = *reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(base) + elem);
        v[0] = bf16lo(w.x); v[1] = bf16hi(w.x); v[2] = bf16lo(w.y); v[3] = bf16hi(w.y);
        v[4] = bf16lo(w.z); v[5] = bf16hi(w.z); v[6] = bf16lo(w.w); v[7] = bf16hi(w.w);
    }
}

constexpr int kAttnWaves = 8;

// One workgroup per (head, sequence); wave w walks logical pages w, w + 8, ...
template <bool F32>
__global__ __launch_bounds__(kAttnWaves * 64) void attn_decode_kernel(const AttnDecodeArgs a) {
    __shared__ float s_m[kAttnWaves], s_l[kAttnWaves];
    __shared__ float s_o[kAttnWaves][kHeadDim];
    const int h = blockIdx.x, b = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    float* out = a.o + (size_t)b * a.o_stride + h * kHeadDim;
    uint16_t* out16 = a.o_bf16 ? a.o_bf16 + (size_t)b * a.o_stride + h * kHeadDim : nullptr;
    if (!a.active[b]) {
        if (tid < kHeadDim) {
            if (out16) out16[tid] = 0;
            else out[tid] = 0.f;
        }
        return;
    }
    const int ctx = a.seq_lens[b] + 1;                 // cached slots incl. the new token
    const int npg = (ctx + kPage - 1) / kPage;
    const int grp = lane >> 3, sub = lane & 7;

    // This wave's page ids: lane j holds the id of its j-th page (logical page w + 8 j).
    const int lp = w + kAttnWaves * lane;
    int my_phys = lp < npg ? a.block_table[(size_t)b * a.max_pages + lp] : -1;
    float q[8];
    {
        const float* qp = a.qkv + (size_t)b * a.qkv_stride + h * kHeadDim + sub * 8;
#pragma unroll
        for (int j = 0; j < 8; ++j) q[j] = qp[j] * 0.125f;  // 1/sqrt(64), exact
    }
    float m = -INFINITY, l = 0.f, o[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) o[j] = 0.f;

    auto page_base = [&](int j, size_t& kb, size_t& vb) {
        int phys = __shfl(my_phys, j, kWave);
        const bool ok = phys >= 0 && phys < a.n_pages;
        phys = ok ? phys : 0;
        kb = kv_offset(a.layer, a.n_pages, phys, 0, a.n_head, h, 0);
        vb = kv_offset(a.layer, a.n_pages, phys, 1, a.n_head, h, 0);
        return ok;
    };

    const int my_pages = npg > w ? (npg - w + kAttnWaves - 1) / kAttnWaves : 0;
    PageRegs<F32> cur, nxt;
    size_t kb, vb;
    bool ok_cur = false, ok_nxt = false;
    if (my_pages > 0) {
        ok_cur = page_base(0, kb, vb);
        load_page<F32>(a.kv_base, kb, vb, lane, cur);
    }
    for (int j = 0; j < my_pages; ++j) {
        const int p = w + kAttnWaves * j;
        if (!F32 && j + 1 < my_pages) {                 // prefetch the next page (bf16 only)
            ok_nxt = page_base(j + 1, kb, vb);
            load_page<F32>(a.kv_base, kb, vb, lane, nxt);
        }
        float sc[8];
        float pm = -INFINITY;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            float kv[8];
            unpack8<F32>(cur, false, i, kv);
            float t = 0.f;
#pragma unroll
            for (int d = 0; d < 8; ++d) t = fmaf(q[d], kv[d], t);
            t = group_sum<8>(t);
            const int tok = p * kPage + i * 8 + grp;
            sc[i] = (ok_cur && tok < ctx) ? t : -INFINITY;
            pm = fmaxf(pm, sc[i]);
        }
        pm = stride8_max(pm);
        if (pm > -INFINITY) {
            const float mn = fmaxf(m, pm);
            const float alpha = expf(m - mn);          // 0 on this wave's first valid page
            m = mn;
            l *= alpha;
#pragma unroll
            for (int d = 0; d < 8; ++d) o[d] *= alpha;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                // Slots past the context (or of an invalid page) hold whatever the pool
                // held: keep them out of the sum (0 * NaN would poison it).
                if (sc[i] > -INFINITY) {
                    const float pr = expf(sc[i] - m);
                    float vv[8];
                    unpack8<F32>(cur, true, i, vv);
                    l += pr;
#pragma unroll
                    for (int d = 0; d < 8; ++d) o[d] = fmaf(pr, vv[d], o[d]);
                }
            }
        }
        if (j + 1 < my_pages) {
            if constexpr (F32) {
                ok_cur = page_base(j + 1, kb, vb);
                load_page<F32>(a.kv_base, kb, vb, lane, cur);
            } else {
                cur = nxt;
                ok_cur = ok_nxt;
            }
        }
    }
    // Sum over the 8 token groups (lanes with equal l % 8 hold the same dims).
#pragma unroll
    for (int d = 0; d < 8; ++d) o[d] = stride8_sum(o[d]);
    l = stride8_sum(l);
    if (lane < 8) {
#pragma unroll
        for (int d = 0; d < 8; ++d) s_o[w][lane * 8 + d] = o[d];
    }
    if (lane == 0) {
        s_m[w] = m;
        s_l[w] = l;
    }
    __syncthreads();
    if (tid < kHeadDim) {                               // log-sum-exp merge of the wave partials
        float M = -INFINITY;
#pragma unroll
        for (int i = 0; i < kAttnWaves; ++i) M = fmaxf(M, s_m[i]);
        float L = 0.f, acc = 0.f;
#pragma unroll
        for (int i = 0; i < kAttnWaves; ++i) {
            if (s_m[i] > -INFINITY) {
                const float wgt = expf(s_m[i] - M);
                L = fmaf(s_l[i], wgt, L);
                acc = fmaf(s_o[i][tid], wgt, acc);
            }
        }
        const float r = L > 0.f ? acc / L : 0.f;
        if (out16) out16[tid] = f32_to_bf16(r);
        else out[tid] = r;
    }
}

// 16-bit KV cache.  Same walk and merge as above with a register budget that lets
// two workgroups share a CU (at most 128 VGPRs): a page's K and V live in one set
// of registers each, and the next page's K is requested as soon as the scores are
// formed, its V as soon as the products are accumulated.  The activity flag, the
// length, this wave's page ids and the query are requested together at the start
// (nothing waits for the flag).  Scores use bf16 pair dot products against the
// query split into hi + lo bf16 halves (about 16 significant bits), in the exp2
// domain (query prescaled by 1/sqrt(64) * log2 e).
__device__ __forceinline__ float dot8_bf16(const uint4 k, const uint32_t (&hi)[4], const uint32_t (&lo)[4], float t) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const uint32_t kw[4] = {k.x, k.y, k.z, k.w};
#pragma unroll
    for (int e = 0; e < 4; ++e)
        t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, kw[e]), __builtin_bit_cast(bf16x2, lo[e]), t,
                                            false);
#pragma unroll
    for (int e = 0; e < 4; ++e)
        t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, kw[e]), __builtin_bit_cast(bf16x2, hi[e]), t,
                                            false);
    return t;
}

__device__ __forceinline__ void load_half_page(const uint16_t* base, size_t off, int lane, uint4 (&r)[8]) {
    const uint4* p = reinterpret_cast<const uint4*>(base + off);
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = p[i * 64 + lane];
}

__global__ __launch_bounds__(kAttnWaves * 64, 4) void attn_decode_bf16_kernel(const AttnDecodeArgs a) {
    __shared__ float s_m[kAttnWaves], s_l[kAttnWaves];
    __shared__ float s_o[kAttnWaves][kHeadDim];
    const int h = blockIdx.x, b = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int grp = lane >> 3, sub = lane & 7;
    const uint16_t* kvb = reinterpret_cast<const uint16_t*>(a.kv_base);
    // independent loads, all in flight together
    const int act = a.active[b];
    const int len = a.seq_lens[b];
    const int lp = w + kAttnWaves * lane;  // lane j: logical page w + 8 j
    const int phys_l = a.block_table[(size_t)b * a.max_pages + min(lp, a.max_pages - 1)];
    const float4* qp = reinterpret_cast<const float4*>(a.qkv + (size_t)b * a.qkv_stride + h * kHeadDim + sub * 8);
    const float4 qa = qp[0], qb = qp[1];

    const int ctx = act ? len + 1 : 0;      // cached slots incl. the new token
    const int npg = (ctx + kPage - 1) / kPage;
    const int my_pages = npg > w ? (npg - w + kAttnWaves - 1) / kAttnWaves : 0;
    uint32_t qh[4], ql[4];
    {
        const float kScale = 0.125f * 1.44269504088896340736f;
        const float qv[8] = {qa.x, qa.y, qa.z, qa.w, qb.x, qb.y, qb.z, qb.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float x0 = qv[2 * e] * kScale, x1 = qv[2 * e + 1] * kScale;
            const uint16_t h0 = f32_to_bf16(x0), h1 = f32_to_bf16(x1);
            qh[e] = (uint32_t)h0 | ((uint32_t)h1 << 16);
            ql[e] = (uint32_t)f32_to_bf16(x0 - bf16_to_f32(h0)) | ((uint32_t)f32_to_bf16(x1 - bf16_to_f32(h1)) << 16);
        }
    }
    auto page_off = [&](int j, int kv, bool& ok) {
        int phys = __shfl(phys_l, j, kWave);
        ok = phys >= 0 && phys < a.n_pages;
        phys = ok ? phys : 0;
        return kv_offset(a.layer, a.n_pages, phys, kv, a.n_head, h, 0);
    };
    float m = -INFINITY, l = 0.f, o[8];
#pragma unroll
    for (int d = 0; d < 8; ++d) o[d] = 0.f;
    uint4 K[8], V[8];
    bool ok_k = false, ok_v = false;
    if (my_pages > 0) {
        load_half_page(kvb, page_off(0, 0, ok_k), lane, K);
        load_half_page(kvb, page_off(0, 1, ok_v), lane, V);
    }
    for (int j = 0; j < my_pages; ++j) {
        const int p = w + kAttnWaves * j;
        const bool ok = ok_k;
        float sc[8];
        float pm = -INFINITY;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float t = group_sum<8>(dot8_bf16(K[i], qh, ql, 0.f));
            const int tok = p * kPage + i * 8 + grp;
            sc[i] = (ok && tok < ctx) ? t : -INFINITY;
            pm = fmaxf(pm, sc[i]);
        }
        if (j + 1 < my_pages) load_half_page(kvb, page_off(j + 1, 0, ok_k), lane, K);
        pm = stride8_max(pm);
        if (pm > -INFINITY) {
            const float mn = fmaxf(m, pm);
            const float alpha = exp2f(m - mn);  // 0 on this wave's first valid page
            m = mn;
            l *= alpha;
#pragma unroll
            for (int d = 0; d < 8; ++d) o[d] *= alpha;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                // slots past the context (or of an invalid page) may hold anything:
                // keep them out of the sum (0 * NaN would poison it)
                if (sc[i] > -INFINITY) {
                    const float pr = exp2f(sc[i] - m);
                    float vv[8];
                    vv[0] = bf16lo(V[i].x); vv[1] = bf16hi(V[i].x); vv[2] = bf16lo(V[i].y); vv[3] = bf16hi(V[i].y);
                    vv[4] = bf16lo(V[i].z); vv[5] = bf16hi(V[i].z); vv[6] = bf16lo(V[i].w); vv[7] = bf16hi(V[i].w);
                    l += pr;
#pragma unroll
                    for (int d = 0; d < 8; ++d) o[d] = fmaf(pr, vv[d], o[d]);
                }
            }
        }
        if (j + 1 < my_pages) load_half_page(kvb, page_off(j + 1, 1, ok_v), lane, V);
    }
#pragma unroll
    for (int d = 0; d < 8; ++d) o[d] = stride8_sum(o[d]);
    l = stride8_sum(l);
    if (lane < 8) {
#pragma unroll
        for (int d = 0; d < 8; ++d) s_o[w][lane * 8 + d] = o[d];
    }
    if (lane == 0) {
        s_m[w] = m;
        s_l[w] = l;
    }
    __syncthreads();
    if (tid < kHeadDim) {                   // log-sum-exp merge of the wave partials (exp2 domain)
        float M = -INFINITY;
#pragma unroll
        for (int i = 0; i < kAttnWaves; ++i) M = fmaxf(M, s_m[i]);
        float L = 0.f, acc = 0.f;
#pragma unroll
        for (int i = 0; i < kAttnWaves; ++i) {
            if (s_m[i] > -INFINITY) {
                const float wgt = exp2f(s_m[i] - M);
                L = fmaf(s_l[i], wgt, L);
                acc = fmaf(s_o[i][tid], wgt, acc);
            }
        }
        const float r = L > 0.f ? acc / L : 0.f;
        const size_t oi = (size_t)b * a.o_stride + h * kHeadDim + tid;
        if (a.o_bf16) a.o_bf16[oi] = f32_to_bf16(r);
        else a.o[oi] = r;
    }
}

hipError_t launch_attn_decode(int wdtype, const AttnDecodeArgs& a, int B, hipStream_t st) {
    const dim3 g(a.n_head, B);
    if (wdtype == FTTS_F32) hipLaunchKernelGGL(attn_decode_kernel<true>, g, dim3(kAttnWaves * 64), 0, st, a);
    else hipLaunchKernelGGL(attn_decode_bf16_kernel, g, dim3(kAttnWaves * 64), 0, st, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Causal prefill attention.  Block = one (sequence, 64-query tile, head); thread t owns
// query row tile*64 + t of that sequence.
template <bool F32>
__global__ __launch_bounds__(64) void attn_prefill_kernel(const AttnPrefillArgs a) {
    __shared__ float sk[64][kHeadDim + 1];
    __shared__ float sv[64][kHeadDim + 1];
    const int h = blockIdx.y, t = threadIdx.x;
    int gt = blockIdx.x, sq = 0;
    while (sq + 1 < a.seqs.n && a.tiles_cu[sq + 1] <= gt) ++sq;
    const int tile = gt - a.tiles_cu[sq];
    const int row0 = a.seqs.cu[sq];
    const int len = a.seqs.cu[sq + 1] - row0;
    const int qi = tile * 64 + t;                        // query position in the sequence
    const bool qok = qi < len;
    const int ld = 3 * a.d_model;

    float q[kHeadDim], o[kHeadDim];
#pragma unroll
    for (int j = 0; j < kHeadDim; ++j) {
        q[j] = qok ? ld_act<F32>(a.qkv, (size_t)(row0 + qi) * ld + h * kHeadDim + j) * 0.125f : 0.f;
        o[j] = 0.f;
    }
    float m = -INFINITY, l = 0.f;
    const int kend = min(len, tile * 64 + 64);            // keys needed by this tile
    for (int k0 = 0; k0 < kend; k0 += 64) {
        __syncthreads();
        for (int i = t; i < 64 * kHeadDim; i += 64) {
            const int r = i / kHeadDim, c = i % kHeadDim;
            const int kr = k0 + r;
            float kv = 0.f, vv = 0.f;
            if (kr < len) {
                const size_t base = (size_t)(row0 + kr) * ld + h * kHeadDim + c;
                kv = ld_act<F32>(a.qkv, base + a.d_model);
                vv = ld_act<F32>(a.qkv, base + 2 * a.d_model);
            }
            sk[r][c] = kv;
            sv[r][c] = vv;
        }
        __syncthreads();
        if (!qok) continue;
        const int nk = min(64, qi - k0 + 1);               // keys k0 .. qi are visible
        if (nk <= 0) continue;
        float sc[64];
        float tm = -INFINITY;
#pragma unroll
        for (int r = 0; r < 64; ++r) {
            float s = 0.f;
#pragma unroll
            for (int j = 0; j < kHeadDim; ++j) s = fmaf(q[j], sk[r][j], s);
            sc[r] = r < nk ? s : -INFINITY;
            tm = fmaxf(tm, sc[r]);
        }
        const float mn = fmaxf(m, tm);
        const float alpha = expf(m - mn);
        m = mn;
        l *= alpha;
#pragma unroll
        for (int j = 0; j < kHeadDim; ++j) o[j] *= alpha;
#pragma unroll
        for (int r = 0; r < 64; ++r) {
            const float p = expf(sc[r] - m);
            l += p;
#pragma unroll
            for (int j = 0; j < kHeadDim; ++j) o[j] = fmaf(p, sv[r][j], o[j]);
        }
    }
    if (!qok) return;
    const float inv = 1.0f / l;
#pragma unroll
    for (int j = 0; j < kHeadDim; ++j)
        st_act<F32>(a.o, (size_t)(row0 + qi) * a.d_model + h * kHeadDim + j, o[j] * inv);
}

// Query tiles of q rows per sequence; returns their number.
static int set_tiles(AttnPrefillArgs& a, int q) {
    a.tiles_cu[0] = 0;
    for (int i = 0; i < a.seqs.n; ++i)
        a.tiles_cu[i + 1] = a.tiles_cu[i] + (a.seqs.cu[i + 1] - a.seqs.cu[i] + q - 1) / q;
    return a.tiles_cu[a.seqs.n];
}

// Workgroups of 128 queries whose waves share each key tile (attn_tile.hip), or of 32
// whose waves split the keys.  The first reads a key tile a quarter as often, but walks
// the c = ceil(length / 64) tiles of a sequence in one chain, four times as long; so it
// needs enough workgroups g that the chip is busy while the longest chain runs.  Fitted to 214
// calls of both kernels (causal with 20, 8 and 4 heads, unmasked with 12 and 4; 1 to
// 28 sequences of 60 to 24,000 rows): they cross at about 24 workgroups per tile of the
// longest chain, for short sequences not before half a workgroup per compute unit, and at
// the latest where the workgroups fill the chip (768, three a unit).  Tile minus split kernel,
// us a layer: 20 heads, 3 / 4 x 300 rows (g 180 / 240, c 5) -2.8 / -3.3, 2 x 500 (160, c 8)
// +0.2, 3 x 500 (240) -2.3, one of 1500 (240, c 24) +6.2, 3000 (480, c 47) +1.7, 16,000
// (2500, c 250) -15; 12 heads unmasked, both branches, 500 frames (96, c 8) +2.7, 2 x 500
// (192) -1.1, 8 x 120 (192, c 2) -3.4, 1500 (288, c 24) +4.1.  Taking the worse of the two
// costs 0.3% of a call on average by this rule, 1.1% by a line at 256 workgroups.
static hipError_t launch_attn_bf16(bool causal, const AttnPrefillArgs& a, hipStream_t st) {
    constexpr int kPerTile = 24, kLeast = 128, kFull = 768;
    AttnPrefillArgs b = a;
    const int wide = set_tiles(b, attn_tile_queries());
    if (wide == 0) return hipSuccess;
    int longest = 0;
    for (int i = 0; i < a.seqs.n; ++i) longest = std::max(longest, a.seqs.cu[i + 1] - a.seqs.cu[i]);
    const int chain = (longest + 63) / 64;
    if ((long)wide * a.n_head >= std::min(std::max(kPerTile * chain, kLeast), kFull))
        return launch_attn_tile(causal, b, wide, st);
    const int split = set_tiles(b, attn_split_queries());
    return launch_attn_split(causal, b, split, st);
}

hipError_t launch_attn_prefill(int wdtype, const AttnPrefillArgs& a, hipStream_t st) {
    if (wdtype != FTTS_F32) return launch_attn_bf16(true, a, st);
    AttnPrefillArgs b = a;
    const int tiles = set_tiles(b, 64);
    hipLaunchKernelGGL(attn_prefill_kernel<true>, dim3(tiles, a.n_head), dim3(64), 0, st, b);
    return hipGetLastError();
}

hipError_t launch_attn_full_bf16(const AttnPrefillArgs& a, hipStream_t st) { return launch_attn_bf16(false, a, st); }

}  // namespace ftts
