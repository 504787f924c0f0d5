// Large 16-bit GEMMs (bf16 weights): C[M][N] = A[M][K] . W[N][K]^T with the
// prefill and DiT epilogues (store, q/k/v store + paged KV scatter, GELU,
// residual add).
//
// A 512-thread workgroup computes a (64 MT) x (128 NT) tile as 2 x 4 waves, each
// wave MT x NT accumulators of 32 x 32, over 64-column K steps.  Three things
// bound the first form of this kernel (256 x 256 tiles, 32-column steps, one
// tile per workgroup): what a CU takes in from L2, the fixed cost of a tile,
// and the last round of tiles.
//  - Intake.  A 32-column step reads 64 bytes of a row, half a cache line, and
//    the other half is fetched again a step later: every tile height ran at the
//    same ~40 GB/s of operands per CU.  A 64-column step reads whole lines
//    (8 rows of 128 bytes per 1 KB direct-to-LDS load); 8192^3 with MT = 2 went
//    from 929 to 1231 TFLOP/s, with MT = 4 from 1314 to 1378 (a library GEMM
//    reaches 1365-1450 there; with all-zero operands 2250, so the rate on real
//    values is set by power more than by issue).
//  - Fixed cost (~9 us of a 36 us tile at K = 1280).  The grid is persistent (one
//    workgroup per CU walks its tiles) and requests the next tile's first two
//    steps before the epilogue, whose arithmetic covers their latency; epilogue
//    staging has LDS of its own.  The product is formed transposed (W rows as
//    the MFMA rows), so a lane holds 4 consecutive columns of one output row and
//    stages them in one 8- or 16-byte LDS write instead of four 2-byte ones.
//  - Last round.  The tile (128, 192 or 256 rows, 128 or 256 columns) is chosen per
//    shape, and rows past the last full round can go to the small kernel
//    (gemm_plan).  9,746 x 5120 x 1280 is 780 tiles of 256 x 256 -- four rounds on
//    256 CUs, the last with 12 tiles -- but four full rounds of 192 rows.
// Traced in the calls (us per GEMM, before -> now): 32 prefixes of 10,827 rows, QKV 129
// -> 108 (987 TFLOP/s), FC1 + GELU 171 -> 143 (its last rows on the small kernel), out-projection 53 -> 52,
// FC2 148 -> 126 (1,124 TFLOP/s); 11,154 rows of width 768, QKV 55 -> 43, FC1 + GELU 90 -> 67,
// out-projection 34 -> 27, FC2 91 -> 61.
//
// K loop: the 8 waves form two groups of 4 (one wave of each per SIMD) half a
// phase apart: while one group runs its matrix instructions the other reads its
// next operands from LDS and issues the loads of later steps, and a barrier swaps
// them.  A step has two such phases: the 64 W columns of the wave and the first
// MT/2 row blocks, then the rest of the row blocks.  Two LDS buffers hold a step
// each; a buffer's W part is refilled for step kt + 2 as soon as the first phase
// of step kt has read it, its A part when step kt is done.  A wave waits for its
// own loads of a step (vmcnt, in order) before the barrier that opens it.  Row r's
// 16-byte pieces are XOR-swizzled by (r / 2) % 8: a 16-byte operand read takes 256
// bytes (two rows) a cycle from 16 lanes that are not consecutive, and this swizzle
// gives none of them the same banks (counted: 0 conflicts; r % 8 counted a conflict
// cycle for every useful one, 823 against 798 us at 8192^3 with MT = 4 and 979
// against 894 with MT = 2).
//
// Rows past the matrix edge read as zero through the buffer descriptor's bound
// and are not stored.
#include <algorithm>

#include "ftts_internal.hpp"
#include "gemm_epilogue.hpp"

namespace ftts {

typedef __bf16 lg_bf16x8 __attribute__((ext_vector_type(8)));
typedef float lg_f32x16 __attribute__((ext_vector_type(16)));

constexpr int kLgK = 64;                        // K step
constexpr int kLgThreads = 512, kLgGroups = 256;  // threads per workgroup; workgroups (one per CU)
constexpr int kLgEpi = 4096;                    // epilogue staging bytes per wave
constexpr int lg_a_bytes(int mt) { return 64 * mt * kLgK * 2; }
constexpr int lg_w_bytes(int nt) { return 128 * nt * kLgK * 2; }

// An operand read from LDS.  In inline assembly because the compiler cannot tell
// which buffer a direct-to-LDS load writes and would wait for all of them before
// every read; the values are used only after lg_wait_lds and lg_tie.
template <int OFF>
__device__ __forceinline__ lg_bf16x8 lg_read(uint32_t addr) {
    lg_bf16x8 r;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF) : "memory");
    return r;
}
template <int OFF>
__device__ __forceinline__ void lg_read4(const uint32_t (&addr)[4], lg_bf16x8 (&o)[4]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) o[k] = lg_read<OFF>(addr[k]);
}
__device__ __forceinline__ void lg_wait_lds() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}
// Keeps the uses of o behind the wait that precedes this call.
template <int N>
__device__ __forceinline__ void lg_tie(lg_bf16x8 (&o)[N][4]) {
#pragma unroll
    for (int m = 0; m < N; ++m)
#pragma unroll
        for (int k = 0; k < 4; ++k) asm volatile("" : "+v"(o[m][k])::"memory");
}
__device__ __forceinline__ void lg_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
}

template <int MT, int NT>
struct LgCtx {
    const void *a, *w;       // the tile's first A row and first W row
    int a_bytes, w_bytes;    // their bounds
    uint32_t av[MT], wv[2 * NT];  // this lane's byte offsets of its A and W loads
    uint32_t ar[4], wr[4];   // this lane's LDS addresses of the four 16-column operands of a step
    int nk, wave;
};

// This wave's share of one step's A tile (8 MT loads over 8 waves) / W tile (16 NT loads).
template <int MT, int NT>
__device__ __forceinline__ void lg_load_a(const LgCtx<MT, NT>& c, char* smem, int s, int kt) {
#pragma unroll
    for (int i = 0; i < MT; ++i)
        buffer_to_lds16(c.a, c.a_bytes, smem + s * lg_a_bytes(MT) + (c.wave * MT + i) * 1024, c.av[i], kt * (kLgK * 2));
}
template <int MT, int NT>
__device__ __forceinline__ void lg_load_w(const LgCtx<MT, NT>& c, char* smem, int s, int kt) {
#pragma unroll
    for (int i = 0; i < 2 * NT; ++i)
        buffer_to_lds16(c.w, c.w_bytes, smem + 2 * lg_a_bytes(MT) + s * lg_w_bytes(NT) + (c.wave * 2 * NT + i) * 1024,
                        c.wv[i], kt * (kLgK * 2));
}

// Step kt + 1's loads of this wave have landed: only W of step kt + 2 (2 NT loads) may be out.
template <int NT>
__device__ __forceinline__ void lg_wait_next(bool w2_out) {
    if (w2_out) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NT) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

template <int M0, int NM, int MT, int NT>
__device__ __forceinline__ void lg_products(lg_f32x16 (&acc)[MT][NT], const lg_bf16x8 (&w)[NT][4],
                                            const lg_bf16x8 (&a)[NM][4]) {
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int n = 0; n < NT; ++n)
                acc[M0 + m][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[n][k], a[m][k], acc[M0 + m][n], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
}

// One K step on buffer S.  Group 1 runs one barrier behind group 0.
template <int MT, int NT, int S>
__device__ __forceinline__ void lg_step(const LgCtx<MT, NT>& c, char* smem, int kt, int grp, lg_f32x16 (&acc)[MT][NT]) {
    constexpr int M1 = MT / 2, M2 = MT - M1, AO = S * lg_a_bytes(MT), WO = S * lg_w_bytes(NT), BLK = 32 * kLgK * 2;
    lg_bf16x8 w[NT][4], a1[M1][4], a2[M2][4];
    lg_read4<WO>(c.wr, w[0]);
    lg_read4<AO>(c.ar, a1[0]);
    if constexpr (NT > 1) lg_read4<WO + BLK>(c.wr, w[NT - 1]);
    if constexpr (M1 > 1) lg_read4<AO + BLK>(c.ar, a1[M1 - 1]);
    // (steps 0 and 1 were requested before the loop)
    if (kt >= 1 && kt + 1 < c.nk) lg_load_a<MT, NT>(c, smem, S ^ 1, kt + 1);
    __builtin_amdgcn_sched_barrier(0);
    lg_wait_lds();
    lg_tie<NT>(w);
    lg_tie<M1>(a1);
    lg_barrier();
    lg_products<0, M1, MT, NT>(acc, w, a1);
    lg_barrier();
    lg_read4<AO + M1 * BLK>(c.ar, a2[0]);
    if constexpr (M2 > 1) lg_read4<AO + (M1 + 1) * BLK>(c.ar, a2[M2 - 1]);
    // both groups read this buffer's W before the last two barriers
    if (kt + 2 < c.nk) lg_load_w<MT, NT>(c, smem, S, kt + 2);
    __builtin_amdgcn_sched_barrier(0);
    lg_wait_lds();
    lg_tie<M2>(a2);
    if (grp == 1 && kt >= 1) lg_wait_next<NT>(kt + 2 < c.nk);
    lg_barrier();
    lg_products<M1, M2, MT, NT>(acc, w, a2);
    if (grp == 0 && kt >= 1) lg_wait_next<NT>(kt + 2 < c.nk);
    lg_barrier();
}

template <int MT, int NT, int EPI>
__global__ __launch_bounds__(kLgThreads) void gemm_large_kernel(const GemmArgs a) {
    constexpr int BM = 64 * MT, BN = 128 * NT, RING = 2 * (lg_a_bytes(MT) + lg_w_bytes(NT));
    __shared__ __attribute__((aligned(1024))) char smem[RING + 8 * kLgEpi];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave >> 2, wm = wave >> 2, wn = wave & 3, fr = lane & 31, fh = lane >> 5;
    // Workgroups are dealt to the 8 XCDs round-robin: XCD x gets a contiguous run
    // of tiles, its workgroups take them in turn, and the run walks 8 row blocks
    // per column, so the tiles an XCD runs at once share A and W rows in its L2.
    const int tn = (a.N + BN - 1) / BN, tm = (a.M + BM - 1) / BM, T = tm * tn;
    const int x = blockIdx.x & 7, q = T >> 3, r = T & 7;
    const int t_first = x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q;
    const int t_end = t_first + q + (x < r ? 1 : 0), t_step = ((int)gridDim.x - x + 7) >> 3;
    int t = t_first + ((int)blockIdx.x >> 3);
    if (t >= t_end) return;  // uniform over the workgroup

    LgCtx<MT, NT> c;
    c.nk = a.K / kLgK;
    c.wave = wave;
    {
        const uint32_t pitch = (uint32_t)a.K * 2;
        auto offset = [&](int row) { return row * pitch + (uint32_t)(((lane & 7) ^ ((row >> 1) & 7)) << 4); };
#pragma unroll
        for (int i = 0; i < MT; ++i) c.av[i] = offset((wave * MT + i) * 8 + (lane >> 3));
#pragma unroll
        for (int i = 0; i < 2 * NT; ++i) c.wv[i] = offset((wave * 2 * NT + i) * 8 + (lane >> 3));
        const uint32_t s0 = lds_address(smem);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t slot = (uint32_t)((2 * k + fh) ^ ((fr >> 1) & 7)) << 4;
            c.ar[k] = s0 + (wm * 32 * MT + fr) * (kLgK * 2) + slot;
            c.wr[k] = s0 + 2 * lg_a_bytes(MT) + (wn * 32 * NT + fr) * (kLgK * 2) + slot;
        }
    }
    int m0, n0;
    auto set_tile = [&](int tt) {
        constexpr int GM = 8;  // row blocks per column walk
        const int g = tt / (GM * tn), gm = min(GM, tm - g * GM), w = tt - g * GM * tn;
        m0 = (g * GM + w % gm) * BM;
        n0 = (w / gm) * BN;
        c.a = reinterpret_cast<const uint16_t*>(a.a) + (size_t)m0 * a.K;
        c.w = reinterpret_cast<const uint16_t*>(a.w) + (size_t)n0 * a.K;
        c.a_bytes = min(a.M - m0, BM) * a.K * 2;
        c.w_bytes = min(a.N - n0, BN) * a.K * 2;
    };
    auto prologue = [&]() {  // steps 0 and 1
        lg_load_w<MT, NT>(c, smem, 0, 0);
        lg_load_a<MT, NT>(c, smem, 0, 0);
        if (c.nk > 1) {
            lg_load_w<MT, NT>(c, smem, 1, 1);
            lg_load_a<MT, NT>(c, smem, 1, 1);
        }
    };
    set_tile(t);
    prologue();
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    char* eb = smem + RING + wave * kLgEpi;
    for (;;) {
        lg_f32x16 acc[MT][NT];
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int n = 0; n < NT; ++n)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[m][n][i] = 0.f;
        lg_barrier();  // every wave's loads of steps 0 and 1 have landed
        if (grp == 1) lg_barrier();
        for (int kt = 0; kt < c.nk; kt += 2) {
            lg_step<MT, NT, 0>(c, smem, kt, grp, acc);
            if (kt + 1 < c.nk) lg_step<MT, NT, 1>(c, smem, kt + 1, grp, acc);
        }
        // group 1's last operand reads ended before the barrier that group 0 passed
        // last: the buffers are free, and this barrier lets group 1 catch up
        if (grp == 0) lg_barrier();
        // acc[m][n][4 g + e]: row rw0 + 32 m + fr, column cw0 + 32 n + 8 g + 4 fh + e
        const int rw0 = m0 + wm * 32 * MT, cw0 = n0 + wn * 32 * NT;
        float bias[NT][16];
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                load_bias4(a.bias, min(cw0 + n * 32 + g * 8 + fh * 4, a.N - 4), &bias[n][4 * g]);
        int slots[MT][2 * NT];
#pragma unroll
        for (int m = 0; m < MT; ++m) load_slots<EPI, NT>(a, rw0 + m * 32, cw0, lane, slots[m]);
        t += t_step;
        const bool more = t < t_end;
        __builtin_amdgcn_sched_barrier(0);
        if (more) {
            set_tile(t);
            prologue();
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (EPI != EPI_RESID) {
            uint2 pk[MT][NT][4];
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int n = 0; n < NT; ++n)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        float y[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            y[e] = acc[m][n][4 * g + e] + bias[n][4 * g + e];
                            if constexpr (EPI == EPI_GELU) y[e] = gelu_one_exp(y[e]);
                        }
                        pk[m][n][g] = make_uint2(bf16x2_rne(y[0], y[1]), bf16x2_rne(y[2], y[3]));
                    }
            // The next tile's loads have landed (covered by the arithmetic above);
            // from here on only stores are out, and they have the first two K
            // steps to drain before a step waits for loads again.
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int m = 0; m < MT; ++m)
                store_block_bf16<EPI, NT>(a, pk[m], slots[m], eb, rw0 + m * 32, cw0, lane);
        } else {
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int n = 0; n < NT; ++n) {
                    float old[4][4];
                    load_block_f32(a, rw0 + m * 32, cw0 + n * 32, lane, old);
                    if (m == 0 && n == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // as above
                    float y[16];
#pragma unroll
                    for (int i = 0; i < 16; ++i) y[i] = acc[m][n][i] + bias[n][i];
                    add_block_f32(a, y, old, eb, rw0 + m * 32, cw0 + n * 32, lane);
                }
        }
        if (!more) break;
    }
}

template <int MT, int NT>
static hipError_t large_by_epi(int epi, const GemmArgs& a, hipStream_t st) {
    const long tiles = (long)((a.M + 64 * MT - 1) / (64 * MT)) * ((a.N + 128 * NT - 1) / (128 * NT));
    const dim3 g((unsigned)std::min<long>(tiles, kLgGroups)), t(kLgThreads);
    switch (epi) {
        case EPI_STORE: hipLaunchKernelGGL((gemm_large_kernel<MT, NT, EPI_STORE>), g, t, 0, st, a); break;
        case EPI_QKV: hipLaunchKernelGGL((gemm_large_kernel<MT, NT, EPI_QKV>), g, t, 0, st, a); break;
        case EPI_GELU: hipLaunchKernelGGL((gemm_large_kernel<MT, NT, EPI_GELU>), g, t, 0, st, a); break;
        case EPI_RESID: hipLaunchKernelGGL((gemm_large_kernel<MT, NT, EPI_RESID>), g, t, 0, st, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_gemm_large(int epi, const GemmArgs& a, int mt, int nt, hipStream_t st) {
    if (a.K % kLgK || a.N % 8 || (epi == EPI_QKV && !a.kv.slots)) return hipErrorInvalidValue;
    switch (mt * 10 + nt) {
        case 42: return large_by_epi<4, 2>(epi, a, st);
        case 32: return large_by_epi<3, 2>(epi, a, st);
        case 22: return large_by_epi<2, 2>(epi, a, st);
        case 41: return large_by_epi<4, 1>(epi, a, st);
        case 31: return large_by_epi<3, 1>(epi, a, st);
        case 21: return large_by_epi<2, 1>(epi, a, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace ftts
