// 16-bit GEMMs of short and middle row counts, bf16 / W8A16 / W4A16 weights:
// C[M][N] = A[M][K] . W[N][K]^T with the prefill and DiT epilogues.
//
// A 256-thread workgroup computes a 64 x BN tile (BN 64 or 128) as 2 x 2 waves,
// each wave one or two 32 x 32 accumulators.  At these sizes a GEMM is bound by how
// soon its operands arrive: A and W come through 1 KB direct-to-LDS loads of whole
// cache lines into a ring of LDS stages (64 bf16 columns a stage, 128 for quantised
// weights, whose raw codes are staged), all but one of which are in flight, and two
// workgroups share a CU, so one's epilogue overlaps the other's loads.  Quantised
// codes are expanded to bf16 exactly in registers as the operands are read (an int8
// code, or a 4-bit code minus its zero-point, is an integer below 2^8) and their
// scales applied to the fp32 accumulators: once per row for W8A16, once per
// 128-column group (a stage) for W4A16.
//
// Against the kernel it replaces (register staging, one 64-column step ahead, K
// split up to 8 ways to fill the chip; us per GEMM traced in the calls): 256 x 3840 x
// 1280 16.4 -> 10.6, 256 x 1280 x 1280 13.2 -> 8.7, 256 x 5120 x 1280 + GELU 20.2 ->
// 15.1, 256 x 1280 x 5120 23.2 -> 15.9, 1000 x 768 x 768 11.0 -> 6.7, 1000 x 768 x 3072
// 17.3 -> 16.1; int8 weights, 697 rows: 23.9 -> 19.0, 16.0 -> 9.5, 24.7 -> 19.4, 33.9 -> 24.9.
//
// Splitting K pays only where whole tiles would leave most of the chip idle over a
// long K (the plan's model decides): every slice stores its fp32 partial tile and the last of a
// tile's workgroups to arrive (a per-tile counter) adds the partials in slice order
// -- reproducible whatever the arrival order -- and runs the epilogue.
//
// FTTS_F32 mode has a plain fp32 kernel (gemm.hip).
#include <algorithm>
#include <atomic>

#include "gemm_epilogue.hpp"

namespace ftts {

typedef __bf16 sg_bf16x8 __attribute__((ext_vector_type(8)));
typedef float sg_f32x16 __attribute__((ext_vector_type(16)));

constexpr int kSgM = 64, kSgThreads = 256;

template <int WT, int BN> struct SgShape {
    static constexpr int KS = WT == FTTS_BF16 ? 64 : 128;                                  // columns of a stage
    static constexpr int AB = KS * 2;                                                      // bytes of an A row
    static constexpr int WB = WT == FTTS_BF16 ? KS * 2 : WT == FTTS_W8A16 ? KS : KS / 2;  // bytes of a W row
    static constexpr int NA = kSgM * AB / 1024, NW = BN * WB / 1024, NI = (NA + NW) / 4;    // loads: A, W, per wave
    static constexpr int STAGE = (NA + NW) * 1024;
    // as many stages as leave room for two workgroups on a CU
    static constexpr int S = WT == FTTS_BF16 ? (BN == 64 ? 4 : 3) : WT == FTTS_W8A16 ? (BN == 64 ? 3 : 2)
                                                                                     : (BN == 64 ? 3 : 2);
    static_assert((NA + NW) % 4 == 0, "every wave issues the same number of loads");
};

// Which 16-byte slot of a staged row holds piece p, rows of RB bytes: the 16 lanes
// whose 16-byte reads share a cycle (256 bytes) fall into different banks.
template <int RB>
__device__ __forceinline__ int sg_slot(int row, int p) {
    return RB == 256 ? p ^ (row & 15) : RB == 128 ? p ^ ((row >> 1) & 7) : p ^ ((row >> 2) & 3);
}

// Reads of staged operands, in inline assembly because the compiler cannot tell
// which stage a direct-to-LDS load writes; used only after sg_wait_lds and sg_tie.
template <int OFF>
__device__ __forceinline__ uint4 sg_read(uint32_t addr) {
    sg_bf16x8 r;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF) : "memory");
    return __builtin_bit_cast(uint4, r);
}
__device__ __forceinline__ void sg_wait_lds() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}
template <int N>
__device__ __forceinline__ void sg_tie(uint4 (&o)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
        sg_bf16x8 v = __builtin_bit_cast(sg_bf16x8, o[i]);
        asm volatile("" : "+v"(v)::"memory");
        o[i] = __builtin_bit_cast(uint4, v);
    }
}
template <int NI>
__device__ __forceinline__ void sg_wait_stage(int later) {  // `later` younger stages may be in flight
    if (later == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else if (later == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NI) : "memory");
    else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NI) : "memory");
}

// Four int8 codes to two words of bf16 pairs (integers below 2^8 are exact, so the
// upper halves of their fp32 values are).
__device__ __forceinline__ uint2 sg_expand4(uint32_t w) {
    const float f0 = (float)(int8_t)(w & 0xFF), f1 = (float)(int8_t)((w >> 8) & 0xFF);
    const float f2 = (float)(int8_t)((w >> 16) & 0xFF), f3 = (float)(int8_t)(w >> 24);
    return make_uint2(__builtin_amdgcn_perm(__float_as_uint(f1), __float_as_uint(f0), 0x07060302u),
                      __builtin_amdgcn_perm(__float_as_uint(f3), __float_as_uint(f2), 0x07060302u));
}
// Eight 4-bit codes minus the zero-point, rounded to bf16 (exact for integer zero-points).
__device__ __forceinline__ uint4 sg_expand_w4(uint32_t w, float z) {
    const uint32_t e = w & 0x0F0F0F0Fu, o = (w >> 4) & 0x0F0F0F0Fu;  // bytes: even codes, odd codes
    uint32_t r[4];
#pragma unroll
    for (int b = 0; b < 4; ++b)
        r[b] = bf16x2_rne((float)((e >> (8 * b)) & 0xFFu) - z, (float)((o >> (8 * b)) & 0xFFu) - z);
    return make_uint4(r[0], r[1], r[2], r[3]);
}

__device__ __forceinline__ void sg_store_pair(float* p, float x, float y) {  // device-coherent
    const uint64_t v = (uint64_t)__float_as_uint(x) | ((uint64_t)__float_as_uint(y) << 32);
    __hip_atomic_store(reinterpret_cast<uint64_t*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t sg_load_pair(const float* p) {
    return __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int WT, int EPI, int BN>
__global__ __launch_bounds__(kSgThreads, 2) void gemm_small_kernel(const GemmArgs a) {
    using SH = SgShape<WT, BN>;
    constexpr int NT = BN / 64, KS = SH::KS, S = SH::S, NI = SH::NI;
    // W4A16's scales differ by column and group: its product is formed with A rows as
    // the MFMA rows, so that a lane has one column; otherwise W rows are (TR), so that
    // a lane has four consecutive columns.
    constexpr bool TR = WT != FTTS_W4A16;
    extern __shared__ __attribute__((aligned(1024))) char smem[];  // stages, then W4A16's scale | zero words
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1, fr = lane & 31, fh = lane >> 5;
    const int tn = (a.N + BN - 1) / BN, tm = (a.M + kSgM - 1) / kSgM, T = tm * tn, SP = gridDim.y, sl = blockIdx.y;
    // Each XCD (workgroups are dealt to the 8 round-robin) takes a contiguous run of
    // tiles that walks 8 row blocks per column: a weight tile's row blocks share an L2.
    int m0, n0;
    {
        const int b = blockIdx.x, x = b & 7, l = b >> 3, q = T >> 3, r = T & 7;
        const int t = (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + l;
        constexpr int GM = 8;
        const int g = t / (GM * tn), gm = min(GM, tm - g * GM), w = t - g * GM * tn;
        m0 = (g * GM + w % gm) * kSgM;
        n0 = (w / gm) * BN;
    }
    const int steps = a.K / KS, k0 = sl * steps / SP, nk = (sl + 1) * steps / SP - k0;
    const int w_pitch = WT == FTTS_BF16 ? a.K * 2 : WT == FTTS_W8A16 ? a.K : a.K / 2;
    const char* ab = reinterpret_cast<const char*>(a.a) + (size_t)m0 * a.K * 2 + (size_t)k0 * SH::AB;
    const char* wb = reinterpret_cast<const char*>(a.w) + (size_t)n0 * w_pitch + (size_t)k0 * SH::WB;
    const int a_bytes = min(a.M - m0, kSgM) * a.K * 2 - k0 * SH::AB;
    const int w_bytes = min(a.N - n0, BN) * w_pitch - k0 * SH::WB;
    uint32_t* sz = reinterpret_cast<uint32_t*>(smem + S * SH::STAGE);  // [nk][BN], W4A16
    if constexpr (WT == FTTS_W4A16) {
        const int ng = a.K / 128;
        for (int i = tid; i < BN * nk; i += kSgThreads) {
            const int n = i % BN, g = i / BN;
            const size_t at = (size_t)min(n0 + n, a.N - 1) * ng + k0 + g;
            sz[i] = (uint32_t)a.scale[at] | ((uint32_t)a.zero[at] << 16);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // seen by every wave after the loop's first barrier
    }
    uint32_t vo[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {  // loads 0 .. NA - 1 bring A rows, the rest W rows
        const int j = wave * NI + i;
        constexpr int RA = 1024 / SH::AB, RW = 1024 / SH::WB, PA = SH::AB / 16, PW = SH::WB / 16;
        const int row = j < SH::NA ? j * RA + lane / PA : (j - SH::NA) * RW + lane / PW;
        vo[i] = j < SH::NA ? (uint32_t)row * a.K * 2 + sg_slot<SH::AB>(row, lane % PA) * 16
                           : (uint32_t)row * w_pitch + sg_slot<SH::WB>(row, lane % PW) * 16;
    }
    auto load = [&](int s, int kt) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int j = wave * NI + i;
            const bool isA = j < SH::NA;
            buffer_to_lds16(isA ? ab : wb, isA ? a_bytes : w_bytes, smem + s * SH::STAGE + j * 1024, vo[i],
                            kt * (isA ? SH::AB : SH::WB));
        }
    };
    // A operands of MFMA step i of a stage are the 16 bytes at piece: bf16 2 i + fh;
    // W8A16 4 (i / 2) + 2 fh + i % 2 (a lane's 16-byte read of codes covers two steps);
    // W4A16 8 (i / 4) + 4 fh + i % 4 (four steps) -- the K order of a step is the same
    // permutation for both operands.
    constexpr int NSTEP = KS / 16, NRW = NSTEP / (WT == FTTS_BF16 ? 1 : WT == FTTS_W8A16 ? 2 : 4);
    const uint32_t s0 = lds_address(smem);
    uint32_t ar[NSTEP], wr[NRW];
#pragma unroll
    for (int i = 0; i < NSTEP; ++i) {
        const int p = WT == FTTS_BF16 ? 2 * i + fh : WT == FTTS_W8A16 ? 4 * (i / 2) + 2 * fh + i % 2 : 8 * (i / 4) + 4 * fh + i % 4;
        ar[i] = s0 + (wm * 32 + fr) * SH::AB + sg_slot<SH::AB>(fr, p) * 16;
    }
#pragma unroll
    for (int i = 0; i < NRW; ++i)
        wr[i] = s0 + SH::NA * 1024 + (wn * 32 * NT + fr) * SH::WB + sg_slot<SH::WB>(fr, 2 * i + fh) * 16;

    sg_f32x16 acc[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[n][i] = 0.f;
#pragma unroll
    for (int s = 0; s < S - 1; ++s) {  // (the counted waits rely on this order)
        if (s < nk) load(s, s);
        __builtin_amdgcn_sched_barrier(0);
    }
    int st = 0;
    for (int kt = 0; kt < nk; ++kt) {
        sg_wait_stage<NI>(min(S - 2, nk - 1 - kt));
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();  // stage kt is in; every wave has read stage kt - 1
        __builtin_amdgcn_sched_barrier(0);
        uint4 av[NSTEP], wv[NT][NRW];
        const uint32_t so = st * SH::STAGE;
#pragma unroll
        for (int i = 0; i < NSTEP; ++i) av[i] = sg_read<0>(ar[i] + so);
#pragma unroll
        for (int i = 0; i < NRW; ++i) {
            wv[0][i] = sg_read<0>(wr[i] + so);
            if constexpr (NT > 1) wv[NT - 1][i] = sg_read<32 * SH::WB>(wr[i] + so);
        }
        uint32_t q[NT];  // this column's scale | zero-point of the group
        if constexpr (WT == FTTS_W4A16) {
            const uint32_t at = s0 + S * SH::STAGE + (kt * BN + wn * 32 * NT + fr) * 4;
#pragma unroll
            for (int n = 0; n < NT; ++n) asm volatile("ds_read_b32 %0, %1" : "=v"(q[n]) : "v"(at + n * 128) : "memory");
        }
        if (kt + S - 1 < nk) load(st == 0 ? S - 1 : st - 1, kt + S - 1);
        __builtin_amdgcn_sched_barrier(0);
        sg_wait_lds();
        sg_tie(av);
#pragma unroll
        for (int n = 0; n < NT; ++n) sg_tie(wv[n]);
        auto mfma = [&](uint4 w, uint4 x, sg_f32x16 c) {
            const sg_bf16x8 wo = __builtin_bit_cast(sg_bf16x8, w), xo = __builtin_bit_cast(sg_bf16x8, x);
            return TR ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(wo, xo, c, 0, 0, 0)
                      : __builtin_amdgcn_mfma_f32_32x32x16_bf16(xo, wo, c, 0, 0, 0);
        };
        if constexpr (WT == FTTS_BF16) {
#pragma unroll
            for (int i = 0; i < NSTEP; ++i)
#pragma unroll
                for (int n = 0; n < NT; ++n) acc[n] = mfma(wv[n][i], av[i], acc[n]);
        } else if constexpr (WT == FTTS_W8A16) {
#pragma unroll
            for (int i = 0; i < NSTEP; ++i)
#pragma unroll
                for (int n = 0; n < NT; ++n) {
                    const uint4 r = wv[n][i / 2];
                    const uint2 lo = sg_expand4(i % 2 ? r.z : r.x), hi = sg_expand4(i % 2 ? r.w : r.y);
                    acc[n] = mfma(make_uint4(lo.x, lo.y, hi.x, hi.y), av[i], acc[n]);
                }
        } else {
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                asm volatile("" : "+v"(q[n])::"memory");
                const float z = bf16hi(q[n]), sc = bf16lo(q[n]);
                sg_f32x16 g;
#pragma unroll
                for (int i = 0; i < 16; ++i) g[i] = 0.f;
#pragma unroll
                for (int i = 0; i < NSTEP; ++i) {
                    const uint4 r = wv[n][i / 4];
                    g = mfma(sg_expand_w4(i % 4 == 0 ? r.x : i % 4 == 1 ? r.y : i % 4 == 2 ? r.z : r.w, z), av[i], g);
                }
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[n][i] = fmaf(sc, g[i], acc[n][i]);
            }
        }
        st = st + 1 == S ? 0 : st + 1;
    }
    __syncthreads();  // the stages are free
    int& s_last = *reinterpret_cast<int*>(smem);
    if (SP > 1) {
        // Partials go out in fragment order -- pair e of thread t at (e * 256 + t) * 2,
        // 512 contiguous bytes per store -- with device-coherent stores waited for
        // before the arrival count, so the last workgroup reads them without a cache flush.
        constexpr int NV = NT * 16, RJ = 4;
        const int tile = blockIdx.x;
        auto slot = [&](int ss) { return a.part + ((size_t)ss * T + tile) * kSgThreads * NV + 2 * tid; };
        float* pp = slot(sl);
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int i = 0; i < 16; i += 2) sg_store_pair(pp + (n * 8 + i / 2) * 512, acc[n][i], acc[n][i + 1]);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0)
            s_last = __hip_atomic_fetch_add(a.count + tile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                     (unsigned)(SP - 1);
        __syncthreads();
        if (!s_last) return;
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[n][i] = 0.f;
        for (int q0 = 0; q0 < SP; q0 += RJ) {  // RJ slices' loads in flight at a time, added in slice order
            uint64_t pv[RJ][NV / 2];
#pragma unroll
            for (int j = 0; j < RJ; ++j) {
                const float* p = slot(min(q0 + j, SP - 1));
#pragma unroll
                for (int e = 0; e < NV / 2; ++e) pv[j][e] = sg_load_pair(p + e * 512);
            }
#pragma unroll
            for (int j = 0; j < RJ; ++j)
                if (q0 + j < SP) {
#pragma unroll
                    for (int n = 0; n < NT; ++n)
#pragma unroll
                        for (int i = 0; i < 16; i += 2) {
                            const uint64_t v = pv[j][(n * 16 + i) / 2];
                            acc[n][i] += __uint_as_float((uint32_t)v);
                            acc[n][i + 1] += __uint_as_float((uint32_t)(v >> 32));
                        }
                }
        }
        if (tid == 0) __hip_atomic_store(a.count + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();  // s_last has been read before the staging below overwrites it
    }
    // Epilogue through 4 KB of LDS per wave (16-byte row pieces out).
    char* eb = smem + wave * 4096;
    const int rw0 = m0 + wm * 32, cw0 = n0 + wn * 32 * NT;
    // element i of block n: column of the 32 x 32 block (TR: 8 (i / 4) + 4 fh + i % 4 in row fr; else fr)
    float y[NT][16];
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        if constexpr (TR) {
            float b[16], rs[16];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int c = min(cw0 + n * 32 + g * 8 + fh * 4, a.N - 4);
                load_bias4(a.bias, c, b + 4 * g);
                if constexpr (WT == FTTS_W8A16) load_bias4(a.scale, c, rs + 4 * g);
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) y[n][i] = (WT == FTTS_W8A16 ? acc[n][i] * rs[i] : acc[n][i]) + b[i];
        } else {
            const float b = ld_act<false>(a.bias, min(cw0 + n * 32 + fr, a.N - 1));
#pragma unroll
            for (int i = 0; i < 16; ++i) y[n][i] = acc[n][i] + b;
        }
    }
    if constexpr (EPI == EPI_RESID) {
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            float old[4][4];
            load_block_f32(a, rw0, cw0 + n * 32, lane, old);
            add_block_f32<TR>(a, y[n], old, eb, rw0, cw0 + n * 32, lane);
        }
    } else {
        int slots[2 * NT];
        load_slots<EPI, NT>(a, rw0, cw0, lane, slots);
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            if constexpr (EPI == EPI_GELU) {
#pragma unroll
                for (int i = 0; i < 16; ++i) y[n][i] = gelu_one_exp(y[n][i]);
            }
            if constexpr (!TR) {  // to the transposed order: a lane's four columns of one row, through the wave's LDS
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int rl = (i >> 2) * 8 + fh * 4 + (i & 3);
                    *reinterpret_cast<float*>(eb + rl * 128 + (((fr >> 2) ^ (rl & 7)) << 4) + (fr & 3) * 4) = y[n][i];
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float4 v = *reinterpret_cast<const float4*>(eb + fr * 128 + (((2 * g + fh) ^ (fr & 7)) << 4));
                    y[n][4 * g] = v.x, y[n][4 * g + 1] = v.y, y[n][4 * g + 2] = v.z, y[n][4 * g + 3] = v.w;
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
        }
        uint2 pk[NT][4];
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                pk[n][g] = make_uint2(bf16x2_rne(y[n][4 * g], y[n][4 * g + 1]), bf16x2_rne(y[n][4 * g + 2], y[n][4 * g + 3]));
        store_block_bf16<EPI, NT>(a, pk, slots, eb, rw0, cw0, lane);
    }
}

template <int WT, int EPI, int BN>
static hipError_t small_launch(const GemmArgs& a, int splits, hipStream_t st) {
    using SH = SgShape<WT, BN>;
    const int tiles = ((a.M + kSgM - 1) / kSgM) * ((a.N + BN - 1) / BN);
    const int steps = a.K / SH::KS, nk = (steps + splits - 1) / splits;
    const size_t lds = std::max<size_t>((size_t)SH::S * SH::STAGE + (WT == FTTS_W4A16 ? (size_t)BN * nk * 4 : 0), 4 * 4096);
    if (lds > 65536) {  // the limit is raised once per instantiation and device
        static std::atomic<uint64_t> raised{0};
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        const uint64_t bit = 1ull << (dev & 63);
        if (dev >= 64 || !(raised.load(std::memory_order_relaxed) & bit)) {
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_small_kernel<WT, EPI, BN>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
            if (e != hipSuccess) return e;
            raised.fetch_or(bit, std::memory_order_relaxed);
        }
    }
    hipLaunchKernelGGL((gemm_small_kernel<WT, EPI, BN>), dim3(tiles, splits), dim3(kSgThreads), lds, st, a);
    return hipGetLastError();
}

template <int WT, int EPI>
static hipError_t small_by_bn(const GemmArgs& a, int bn, int splits, hipStream_t st) {
    return bn == 64 ? small_launch<WT, EPI, 64>(a, splits, st) : small_launch<WT, EPI, 128>(a, splits, st);
}

template <int WT>
static hipError_t small_by_epi(int epi, const GemmArgs& a, int bn, int splits, hipStream_t st) {
    switch (epi) {
        case EPI_STORE: if constexpr (WT == FTTS_BF16) return small_by_bn<WT, EPI_STORE>(a, bn, splits, st); else break;
        case EPI_QKV: return small_by_bn<WT, EPI_QKV>(a, bn, splits, st);
        case EPI_GELU: return small_by_bn<WT, EPI_GELU>(a, bn, splits, st);
        case EPI_RESID: return small_by_bn<WT, EPI_RESID>(a, bn, splits, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_gemm_small(int wdtype, int epi, const GemmArgs& a, int bn, int splits, hipStream_t st) {
    if (a.K % (wdtype == FTTS_BF16 ? 64 : 128) || a.N % 8) return hipErrorInvalidValue;
    if (splits > 1) {
        const size_t tiles = (size_t)((a.M + kSgM - 1) / kSgM) * ((a.N + bn - 1) / bn);
        if (!a.part || !a.count || tiles > (size_t)a.n_count || tiles * splits * kSgM * bn > a.part_floats)
            return hipErrorInvalidValue;
    }
    switch (wdtype) {
        case FTTS_BF16: return small_by_epi<FTTS_BF16>(epi, a, bn, splits, st);
        case FTTS_W8A16: return small_by_epi<FTTS_W8A16>(epi, a, bn, splits, st);
        case FTTS_W4A16: return small_by_epi<FTTS_W4A16>(epi, a, bn, splits, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace ftts
