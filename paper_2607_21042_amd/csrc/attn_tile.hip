// bf16 attention over packed sequences for wide grids, with or without the causal
// mask: o_h = softmax(q_h K_h^T / 8) V_h, one workgroup per 128 queries of a head.
//
// The 4 waves take 32 queries each and share 64-key tiles of K and V, which come in by
// 1 KB direct-to-LDS loads of whole rows (128 bytes of a head) into two stages, a tile
// ahead; one barrier a tile, three workgroups a CU.  A wave forms S^T = K Q^T (keys as matrix
// rows, so a lane holds 32 scores of its own query), applies the online softmax per
// lane, and accumulates O^T = V^T P^T with the probabilities taken straight from its
// score registers: the MFMA k order is a permutation shared by both operands.  V^T comes
// from the row-major V tile by transposing LDS reads (ds_read_b64_tr_b16: 16 lanes read a
// 4 x 16 block and get its columns), so nothing is transposed through registers.
//
// What bounds it is the softmax's vector work (one exponential and about three more
// operations a score) beside the matrix work, so: row sums are pair dot products with
// ones (of the rounded probabilities; the two halves meet once, at the end), the running maximum moves only when a tile exceeds it by more than 2^8
// (probabilities then stay below 256; nothing is lost in fp32), and masks are applied
// in a tile that needs one only.
//
// Traced (us per layer): 32 causal prefixes, 10,827 rows, 20 heads, 86 -> 41 (before: K
// rows read per wave from L2 with nothing in flight, V transposed through registers); 24
// sequences of 170-730 frames, 12 heads, 56 -> 42 (32-key tiles staged through
// registers).  Three stages measured 44 / 45, four workgroups a CU spill (causal: 101).
//
// Pieces of 16 bytes are XOR-swizzled by (row / 2) % 8 (two rows share the 256 bytes that
// a 16-byte read takes a cycle).
#include "gemm_epilogue.hpp"

namespace ftts {

typedef __bf16 at_bf16x8 __attribute__((ext_vector_type(8)));
typedef float at_f32x16 __attribute__((ext_vector_type(16)));

constexpr int kAtWaves = 4, kAtQ = 32 * kAtWaves, kAtK = 64, kAtStages = 2;
constexpr int kAtTile = kAtK * kHeadDim * 2;   // bytes of a K (or V) tile
constexpr int kAtStage = 2 * kAtTile;

// LDS reads in inline assembly (the compiler would wait for every direct-to-LDS load in
// flight before each); used only after at_wait and at_tie.
template <int OFF>
__device__ __forceinline__ uint4 at_read(uint32_t addr) {
    at_bf16x8 r;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF) : "memory");
    return __builtin_bit_cast(uint4, r);
}
template <int OFF>
__device__ __forceinline__ uint64_t at_read_tr(uint32_t addr) {
    uint64_t r;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF) : "memory");
    return r;
}
template <typename T, int N>
__device__ __forceinline__ void at_tie(T (&o)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(o[i])::"memory");
}
__device__ __forceinline__ void at_tie4(uint4 (&o)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        at_bf16x8 v = __builtin_bit_cast(at_bf16x8, o[i]);
        asm volatile("" : "+v"(v)::"memory");
        o[i] = __builtin_bit_cast(uint4, v);
    }
}
__device__ __forceinline__ at_bf16x8 at_op(uint4 v) { return __builtin_bit_cast(at_bf16x8, v); }

// One wave's running attention of 32 queries: O^T (dims 0..31 and 32..63: element i is
// dim (i/4)*8 + hh*4 + i%4 of the lane's query), the running maximum (exp2 domain) and
// the sum over the keys of this lane's half.
struct AtState {
    at_f32x16 o0, o1;
    float m, l;
};
__device__ __forceinline__ void at_init(AtState& a) {
#pragma unroll
    for (int i = 0; i < 16; ++i) a.o0[i] = a.o1[i] = 0.f;
    a.m = -INFINITY;
    a.l = 0.f;
}
// s[b][i] = raw score of key 32 b + (i/4)*8 + hh*4 + i%4 of the tile and the lane's query.
__device__ __forceinline__ void at_scores(const uint4 (&ka)[4], const uint4 (&kb)[4], const uint4 (&qr)[4], at_f32x16 (&s)[2]) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
#pragma unroll
        for (int i = 0; i < 16; ++i) s[b][i] = 0.f;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
            s[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(at_op(b ? kb[kk] : ka[kk]), at_op(qr[kk]), s[b], 0, 0, 0);
    }
}
// Masks the scores of keys k0 .. k0 + 63 (past len; CAUSAL: past the query) where some
// lane needs it, moves the running maximum and gives the probabilities in bf16 pairs.
// The first tile a state sees holds a key that every query of the wave sees.
template <bool CAUSAL>
__device__ __forceinline__ void at_softmax(AtState& a, at_f32x16 (&s)[2], int k0, int len, int qw, int qi, int hh,
                                           uint32_t (&pw)[16]) {
    const float kScale = 0.125f * 1.44269504088896340736f;  // 1/sqrt(64) * log2(e)
    if (k0 + kAtK > len || (CAUSAL && k0 + kAtK - 1 > qw)) {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int key = k0 + 32 * b + (i >> 2) * 8 + hh * 4 + (i & 3);
                if (key >= len || (CAUSAL && key > qi)) s[b][i] = -INFINITY;
            }
    }
    float tmax = fmaxf(s[0][0], s[1][0]);
#pragma unroll
    for (int i = 1; i < 16; ++i) tmax = fmaxf(tmax, fmaxf(s[0][i], s[1][i]));
    {
        const RowPair pr = swap32(tmax);
        tmax = fmaxf(pr.a, pr.b) * kScale;
    }
    if (__any(tmax > a.m + 8.f)) {
        const float mn = fmaxf(a.m, tmax), alpha = __builtin_amdgcn_exp2f(a.m - mn);  // m = -inf at first: 0
        a.m = mn;
        a.l *= alpha;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            a.o0[i] *= alpha;
            a.o1[i] *= alpha;
        }
    }
    // probabilities exp2(s * scale - m), rounded to bf16 once: the same values feed P V
    // and the row sums (the hardware exp2 flushes results below 2^-126 to 0)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < 16; i += 2)
            pw[b * 8 + i / 2] = bf16x2_rne(__builtin_amdgcn_exp2f(fmaf(s[b][i], kScale, -a.m)),
                                           __builtin_amdgcn_exp2f(fmaf(s[b][i + 1], kScale, -a.m)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const bf16x2 ones = __builtin_bit_cast(bf16x2, 0x3F803F80u);
#pragma unroll
    for (int j = 0; j < 16; ++j)
        a.l = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pw[j]), ones, a.l, false);
}
// O^T += V^T P^T over the tile's keys k0 .. k0 + 63.  v[d][e][st]: keys 16 st + 8 e +
// hh*4 + 0..3 of dim 32 d + lane % 32; k slots hh*8 .. +7 of step st carry the same keys
// on both operands.  CAUSAL: the second half is left out where no query qw .. qw + 31
// of the wave sees it, so that a later row that is not finite (0 x NaN is NaN) stays
// out of every earlier block of 32.
template <bool CAUSAL>
__device__ __forceinline__ void at_pv(AtState& a, const uint64_t (&v)[2][2][4], const uint32_t (&pw)[16], int k0, int qw) {
#pragma unroll
    for (int st = 0; st < 4; ++st) {
        if (CAUSAL && st == 2 && k0 >= qw) return;  // (uniform over the wave)
        const at_bf16x8 pb = at_op(make_uint4(pw[4 * st], pw[4 * st + 1], pw[4 * st + 2], pw[4 * st + 3]));
        auto vop = [&](int d) {
            return at_op(make_uint4((uint32_t)v[d][0][st], (uint32_t)(v[d][0][st] >> 32), (uint32_t)v[d][1][st],
                                    (uint32_t)(v[d][1][st] >> 32)));
        };
        a.o0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vop(0), pb, a.o0, 0, 0, 0);
        a.o1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vop(1), pb, a.o1, 0, 0, 0);
    }
}
// Lane addresses of a staged tile: K operands kr, V blocks vr by (second 8 keys, second 32 dims).
struct AtAddr {
    uint32_t kr[4], vr[2][2];
};
__device__ __forceinline__ AtAddr at_addresses(uint32_t s0, int lane) {
    const int ql = lane & 31, hh = lane >> 5, i16 = lane & 15, g16 = (lane >> 4) & 1;
    AtAddr r;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) r.kr[kk] = s0 + ql * 128 + (((2 * kk + hh) ^ ((ql >> 1) & 7)) << 4);
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const int row = e * 8 + hh * 4 + (i16 >> 2), piece = d * 4 + g16 * 2 + ((i16 & 3) >> 1);
            r.vr[e][d] = s0 + kAtTile + row * 128 + ((piece ^ ((row >> 1) & 7)) << 4) + (i16 & 1) * 8;
        }
    return r;
}
__device__ __forceinline__ void at_read_k(const AtAddr& r, uint32_t so, uint4 (&ka)[4], uint4 (&kb)[4]) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) ka[kk] = at_read<0>(r.kr[kk] + so);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) kb[kk] = at_read<4096>(r.kr[kk] + so);
}
__device__ __forceinline__ void at_read_v(const AtAddr& r, uint32_t so, uint64_t (&v)[2][2][4]) {
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            v[d][e][0] = at_read_tr<0>(r.vr[e][d] + so);
            v[d][e][1] = at_read_tr<2048>(r.vr[e][d] + so);
            v[d][e][2] = at_read_tr<4096>(r.vr[e][d] + so);
            v[d][e][3] = at_read_tr<6144>(r.vr[e][d] + so);
        }
}
__device__ __forceinline__ void at_tie_v(uint64_t (&v)[2][2][4]) {
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
        for (int e = 0; e < 2; ++e) at_tie(v[d][e]);
}
__device__ __forceinline__ void at_wait_lds() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}
// The wave's rows out (queries first <= qw + rl < len, to rows row0 + qw + rl), through
// 4 KB of its LDS.
__device__ __forceinline__ void at_store(const AttnPrefillArgs& a, const AtState& st, float inv, char* eb, int row0,
                                         int first, int len, int qw, int h, int lane) {
    const int ql = lane & 31, hh = lane >> 5;
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const at_f32x16& o = n ? st.o1 : st.o0;
            *reinterpret_cast<uint2*>(eb + ql * 128 + (((n * 4 + g) ^ (ql & 7)) << 4) + ((hh ^ ((ql >> 3) & 1)) << 3)) =
                make_uint2(bf16x2_rne(o[4 * g] * inv, o[4 * g + 1] * inv), bf16x2_rne(o[4 * g + 2] * inv, o[4 * g + 3] * inv));
        }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    uint16_t* out = reinterpret_cast<uint16_t*>(a.o) + h * kHeadDim;
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int rl = (lane >> 3) + 8 * it, q = lane & 7;
        uint4 v = *reinterpret_cast<const uint4*>(eb + rl * 128 + ((q ^ (rl & 7)) << 4));
        if (it & 1) v = make_uint4(v.z, v.w, v.x, v.y);
        if (qw + rl >= first && qw + rl < len)
            *reinterpret_cast<uint4*>(out + (size_t)(row0 + qw + rl) * a.d_model + q * 8) = v;
    }
}
// Q as the second operand of S^T = K Q^T: lane (q, hh) holds dims kk*16 + hh*8 .. +7.
__device__ __forceinline__ void at_load_q(const uint16_t* qrow, int hh, uint4 (&qr)[4]) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) qr[kk] = *reinterpret_cast<const uint4*>(qrow + kk * 16 + hh * 8);
}
// The sequence of query tile gt: how many end at or before it (at most 64, one per lane).
__device__ __forceinline__ int at_sequence(const AttnPrefillArgs& a, int gt, int lane) {
    static_assert(kMaxPrefillSeqs <= kWave, "one sequence per lane");
    return __popcll(__ballot(lane + 1 < a.seqs.n && a.tiles_cu[min(lane + 1, a.seqs.n)] <= gt));
}

template <bool CAUSAL>
__global__ __launch_bounds__(kAtWaves * 64, 3) void attn_tile_kernel(const AttnPrefillArgs a) {
    __shared__ __attribute__((aligned(1024))) char smem[kAtStages * kAtStage];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Workgroups are dealt to the 8 XCDs round-robin by linear id: each XCD gets a
    // contiguous run of (head, query tile) pairs, query tiles fastest, so the tiles of
    // one (sequence, head) read its K and V through one L2.
    int gt, h;
    {
        const int T = gridDim.x * gridDim.y, b = blockIdx.y * gridDim.x + blockIdx.x;
        const int x = b & 7, l = b >> 3, q = T >> 3, r = T & 7;
        const int t = (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + l;
        gt = t % gridDim.x;
        h = t / gridDim.x;
    }
    const int sq = at_sequence(a, gt, lane);
    const int row0 = a.seqs.cu[sq], len = a.seqs.cu[sq + 1] - row0;
    if (len <= 0) return;  // uniform over the workgroup
    // (causal: the longest tiles of a sequence first, so that a launch ends on short ones)
    const int tile = CAUSAL ? a.tiles_cu[sq + 1] - 1 - gt : gt - a.tiles_cu[sq];
    const size_t ld = 3 * (size_t)a.d_model;
    const uint16_t* qkv = reinterpret_cast<const uint16_t*>(a.qkv);
    const int ql = lane & 31, hh = lane >> 5;
    const int qw = tile * kAtQ + wave * 32, qi = qw + ql;
    uint4 qr[4];
    at_load_q(qkv + (size_t)(row0 + min(qi, len - 1)) * ld + h * kHeadDim, hh, qr);
    // loads: wave w brings rows 16 w .. 16 w + 15 of each tile, 8 rows an instruction
    uint32_t vo[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = wave * 16 + i * 8 + (lane >> 3);
        vo[i] = (uint32_t)(row * (int)ld * 2) + (((lane & 7) ^ ((row >> 1) & 7)) << 4);
    }
    const int kend = CAUSAL ? min(len, tile * kAtQ + kAtQ) : len;  // keys any query of the tile sees
    const int nt = (kend + kAtK - 1) / kAtK;
    auto load = [&](int t) {
        const int k0 = t * kAtK, bytes = (min(len - k0, kAtK) - 1) * (int)ld * 2 + kHeadDim * 2;  // rows past the end: zero
        const uint16_t* kb = qkv + (size_t)(row0 + k0) * ld + a.d_model + h * kHeadDim;
        char* dst = smem + (t % kAtStages) * kAtStage + wave * 2048;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            buffer_to_lds16(kb, bytes, dst + i * 1024, vo[i], 0);
            buffer_to_lds16(kb + a.d_model, bytes, dst + kAtTile + i * 1024, vo[i], 0);
        }
    };
    const AtAddr ad = at_addresses(lds_address(smem), lane);
    AtState st;
    at_init(st);
    load(0);
    for (int t = 0; t < nt; ++t) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's loads of tile t
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();  // tile t is in; every wave has read tile t - 1
        __builtin_amdgcn_sched_barrier(0);
        if (t + 1 < nt) load(t + 1);
        const int k0 = t * kAtK;
        if (qw >= len || (CAUSAL && k0 > qw + 31)) continue;  // no query of this wave sees the tile
        const uint32_t so = (uint32_t)(t % kAtStages) * kAtStage;
        uint4 ka[4], kb[4];
        at_read_k(ad, so, ka, kb);
        at_wait_lds();
        at_tie4(ka);
        at_tie4(kb);
        at_f32x16 s[2];
        at_scores(ka, kb, qr, s);
        __builtin_amdgcn_sched_barrier(0);
        uint64_t v[2][2][4];  // in flight during the softmax, in the registers K has left
        at_read_v(ad, so, v);
        uint32_t pw[16];
        at_softmax<CAUSAL>(st, s, k0, len, qw, qi, hh, pw);
        at_wait_lds();
        at_tie_v(v);
        at_pv<CAUSAL>(st, v, pw, k0, qw);
    }
    __syncthreads();  // the stages are free: rows go out through 4 KB per wave
    if (qw >= len) return;
    const RowPair ls = swap32(st.l);
    at_store(a, st, 1.0f / (ls.a + ls.b), smem + wave * 4096, row0, 0, len, qw, h, lane);
}

// The same for short grids: a workgroup takes 32 queries of one head and its 4 waves
// split the 64-key tiles round-robin (wave w takes tiles w, w + 4, ...), so a query
// tile's dependent chain is a quarter of its keys.  Each wave stages its own tiles: once
// a tile's K (V) operands are in registers the next tile's K (V) loads go out to the same
// place and land during the products; no barrier in the loop.  The four (max, sum, output) partials are merged by
// the log-sum-exp rule through LDS at the end.  Two workgroups a CU.  Bound by
// the chain load, product, softmax, product, merge.  Traced (us per layer), before
// (32-key tiles, V transposed through registers) and now: 2 x 500 frames, 12 heads, no
// mask, 12.5 and 10.4; 256 causal rows, 20 heads, 6.5 and 6.4.
//
// LAST: one workgroup per (sequence, head) that keeps only the last query, as row s of the
// output: all that the layer feeding the logits needs.
constexpr int kAsQ = 32;
template <bool CAUSAL, bool LAST>
__global__ __launch_bounds__(kAtWaves * 64, 2) void attn_split_kernel(const AttnPrefillArgs a) {
    __shared__ __attribute__((aligned(1024))) char smem[kAtWaves * kAtStage];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = blockIdx.y, gt = blockIdx.x, sq = LAST ? gt : at_sequence(a, gt, lane);
    const int row0 = a.seqs.cu[sq], len = a.seqs.cu[sq + 1] - row0;
    if (len <= 0) return;  // uniform over the workgroup
    const int tile = LAST ? (len - 1) / kAsQ : gt - a.tiles_cu[sq];
    const size_t ld = 3 * (size_t)a.d_model;
    const uint16_t* qkv = reinterpret_cast<const uint16_t*>(a.qkv);
    const int ql = lane & 31, hh = lane >> 5, qw = tile * kAsQ, qi = qw + ql;
    const int kend = CAUSAL ? min(len, qw + kAsQ) : len;  // keys any query of the tile sees
    const int nt = (kend + kAtK - 1) / kAtK;
    char* own = smem + wave * kAtStage;
    // K rows of tile t to the stage's first half (v = 0), V rows to its second (v = 1)
    auto load = [&](int t, int v) {
        const int k0 = t * kAtK, bytes = (min(len - k0, kAtK) - 1) * (int)ld * 2 + kHeadDim * 2;  // rows past the end: zero
        const uint16_t* src = qkv + (size_t)(row0 + k0) * ld + (1 + v) * a.d_model + h * kHeadDim;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int row = i * 8 + (lane >> 3);
            const uint32_t vo = (uint32_t)(row * (int)ld * 2) + (((lane & 7) ^ ((row >> 1) & 7)) << 4);
            buffer_to_lds16(src, bytes, own + v * kAtTile + i * 1024, vo, 0);
        }
    };
    uint4 qr[4];
    at_load_q(qkv + (size_t)(row0 + min(qi, len - 1)) * ld + h * kHeadDim, hh, qr);
    if (wave < nt) {  // (the counted wait for K relies on this order)
        load(wave, 0);
        __builtin_amdgcn_sched_barrier(0);
        load(wave, 1);
    }
    const AtAddr ad = at_addresses(lds_address(own), lane);
    AtState st;
    at_init(st);
    for (int t = wave; t < nt; t += kAtWaves) {
        const bool more = t + kAtWaves < nt;
        asm volatile("s_waitcnt vmcnt(8)" ::: "memory");  // K is in (this wave's own loads), V's 8 loads may be out
        __builtin_amdgcn_sched_barrier(0);
        uint4 ka[4], kb[4];
        at_read_k(ad, 0, ka, kb);
        at_wait_lds();
        at_tie4(ka);
        at_tie4(kb);
        __builtin_amdgcn_sched_barrier(0);
        if (more) load(t + kAtWaves, 0);
        __builtin_amdgcn_sched_barrier(0);
        at_f32x16 s[2];
        at_scores(ka, kb, qr, s);
        uint32_t pw[16];
        at_softmax<CAUSAL>(st, s, t * kAtK, len, qw, qi, hh, pw);
        __builtin_amdgcn_sched_barrier(0);
        if (more) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");  // V is in, the next K may be out
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        uint64_t v[2][2][4];
        at_read_v(ad, 0, v);
        at_wait_lds();
        at_tie_v(v);
        __builtin_amdgcn_sched_barrier(0);
        if (more) load(t + kAtWaves, 1);
        __builtin_amdgcn_sched_barrier(0);
        at_pv<CAUSAL>(st, v, pw, t * kAtK, qw);
    }
    __syncthreads();  // every wave has read its stage: the partials of waves 1 .. 3 go there, lane for lane
    float* mrg = reinterpret_cast<float*>(smem);  // [3][34][64]
    if (wave > 0) {
        float* mw = mrg + (wave - 1) * 34 * 64;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            mw[i * 64 + lane] = st.o0[i];
            mw[(16 + i) * 64 + lane] = st.o1[i];
        }
        mw[32 * 64 + lane] = st.m;
        mw[33 * 64 + lane] = st.l;
    }
    __syncthreads();
    if (wave > 0) return;
    // wave 0 always holds tile 0, so m is finite; a wave without tiles has m = -inf, l = 0, o = 0
    float mm = st.m;
#pragma unroll
    for (int w = 0; w < kAtWaves - 1; ++w) mm = fmaxf(mm, mrg[(w * 34 + 32) * 64 + lane]);
    const float f0 = exp2f(st.m - mm);
    st.l *= f0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        st.o0[i] *= f0;
        st.o1[i] *= f0;
    }
#pragma unroll
    for (int w = 0; w < kAtWaves - 1; ++w) {
        const float* mw = mrg + w * 34 * 64;
        const float f = exp2f(mw[32 * 64 + lane] - mm);
        st.l += mw[33 * 64 + lane] * f;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            st.o0[i] += mw[i * 64 + lane] * f;
            st.o1[i] += mw[(16 + i) * 64 + lane] * f;
        }
    }
    const RowPair ls = swap32(st.l);
    at_store(a, st, 1.0f / (ls.a + ls.b), smem + 3 * 34 * 64 * 4 + 1024, LAST ? sq - (len - 1) : row0,
             LAST ? len - 1 : 0, len, qw, h, lane);
}

int attn_tile_queries() { return kAtQ; }
int attn_split_queries() { return kAsQ; }

hipError_t launch_attn_tile(bool causal, const AttnPrefillArgs& a, int tiles, hipStream_t st) {
    const dim3 g(tiles, a.n_head), t(kAtWaves * 64);
    if (causal) hipLaunchKernelGGL(attn_tile_kernel<true>, g, t, 0, st, a);
    else hipLaunchKernelGGL(attn_tile_kernel<false>, g, t, 0, st, a);
    return hipGetLastError();
}

hipError_t launch_attn_split(bool causal, const AttnPrefillArgs& a, int tiles, hipStream_t st) {
    const dim3 g(tiles, a.n_head), t(kAtWaves * 64);
    if (causal) hipLaunchKernelGGL((attn_split_kernel<true, false>), g, t, 0, st, a);
    else hipLaunchKernelGGL((attn_split_kernel<false, false>), g, t, 0, st, a);
    return hipGetLastError();
}

hipError_t launch_attn_last(const AttnPrefillArgs& a, hipStream_t st) {
    hipLaunchKernelGGL((attn_split_kernel<true, true>), dim3(a.seqs.n, a.n_head), dim3(kAtWaves * 64), 0, st, a);
    return hipGetLastError();
}

}  // namespace ftts
