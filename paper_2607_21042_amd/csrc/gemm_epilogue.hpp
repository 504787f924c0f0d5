// Epilogue pieces of the 16-bit GEMMs whose accumulators are transposed (weight
// rows as the MFMA rows): a lane of a 32 x 32 block holds, for output row
// lane % 32, the columns 8 g + 4 (lane / 32) + e (g, e < 4) in acc[4 g + e].
#pragma once
#include "ftts_internal.hpp"

namespace ftts {

typedef __attribute__((address_space(3))) char lds_char;

__device__ __forceinline__ uint32_t lds_address(char* p) { return (uint32_t)(uintptr_t)(lds_char*)p; }

// One 1 KB direct-to-LDS load: lane i's 16 bytes at base + voff + soff go to
// dst + 16 i (dst uniform); offsets at or past `bytes` read as zero.
__device__ __forceinline__ void buffer_to_lds16(const void* base, int bytes, char* dst, uint32_t voff, uint32_t soff) {
#ifdef __HIP_DEVICE_COMPILE__
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000), (lds_char*)dst, 16, voff, soff,
        0, 0);
#endif
}

// Two fp32 values to packed bf16 (round to nearest even) in one gfx950 instruction.
__device__ __forceinline__ uint32_t bf16x2_rne(float lo, float hi) {
    typedef __bf16 bf16x2_v __attribute__((ext_vector_type(2)));
    typedef float f32x2_v __attribute__((ext_vector_type(2)));
    const f32x2_v v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_v));
}

// The tanh GELU written as u * sigmoid(2 c (u + 0.044715 u^3)) -- the same
// function, since 0.5 (1 + tanh z) = 1 / (1 + exp(-2 z)) -- on one exponential
// and one hardware reciprocal (the result is rounded to bf16).
__device__ __forceinline__ float gelu_one_exp(float u) {
    const float c2 = 2.0f * 0.7978845608028654f;
    return u * __builtin_amdgcn_rcpf(1.0f + __expf(-c2 * (u + 0.044715f * u * u * u)));
}

// Four consecutive bf16 biases (n a multiple of 4, bias 16-byte aligned).
__device__ __forceinline__ void load_bias4(const void* bias, int n, float* out) {
    const uint2 w = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint16_t*>(bias) + n);
    out[0] = bf16lo(w.x);
    out[1] = bf16hi(w.x);
    out[2] = bf16lo(w.y);
    out[3] = bf16hi(w.y);
}

// KV slots (page * 64 + slot, or -1) of the rows that store_block_bf16 writes for this lane.
template <int EPI, int NT>
__device__ __forceinline__ void load_slots(const GemmArgs& a, int m0, int n0, int lane, int (&slots)[2 * NT]) {
    if (EPI != EPI_QKV || n0 < a.kv.d_model) return;
#pragma unroll
    for (int it = 0; it < 2 * NT; ++it) slots[it] = a.kv.slots[min(m0 + (lane + 64 * it) / (4 * NT), a.M - 1)];
}

// A wave's 32 x (32 NT) block of bf16 outputs (pk[n][g]: the lane's four columns
// 32 n + 8 g + 4 fh ..) to rows m0.. and columns n0.. of a.out, through 4 KB of
// the wave's LDS (rows of 128 bytes) so that a row's bytes go out in 16-byte pieces
// of consecutive lanes; for q/k/v the keys and values (a block's columns belong to
// one head) also go into their KV pages.  Pieces are XOR-swizzled by row, and the
// halves of a piece by bit 3 of the row, so that neither the 8-byte writes nor the
// 16-byte reads collide in banks.  The KV slots of the rows come in registers
// (load_slots), read before the first store: a load issued among the stores would
// wait for all of them.
template <int EPI, int NT>
__device__ __forceinline__ void store_block_bf16(const GemmArgs& a, const uint2 (&pk)[NT][4], const int (&slots)[2 * NT],
                                                 char* eb, int m0, int n0, int lane) {
    const int fr = lane & 31, fh = lane >> 5;
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<uint2*>(eb + fr * 128 + (((n * 4 + g) ^ (fr & 7)) << 4) + ((fh ^ ((fr >> 3) & 1)) << 3)) =
                pk[n][g];
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    uint16_t* out = reinterpret_cast<uint16_t*>(a.out);
    constexpr int PR = 4 * NT;  // 16-byte pieces of a row
    const int d = a.kv.d_model;
    const bool is_kv = EPI == EPI_QKV && n0 >= d;  // uniform over the wave
#pragma unroll
    for (int it = 0; it < 2 * NT; ++it) {
        const int j = lane + 64 * it, rl = j / PR, q = j % PR, m = m0 + rl, n = n0 + q * 8;
        uint4 v = *reinterpret_cast<const uint4*>(eb + rl * 128 + ((q ^ (rl & 7)) << 4));
        if ((rl >> 3) & 1) v = make_uint4(v.z, v.w, v.x, v.y);
        if (m < a.M && n < a.N) {
            *reinterpret_cast<uint4*>(out + (size_t)m * a.N + n) = v;
            if (is_kv && slots[it] >= 0) {
                const int kvsel = n >= 2 * d, r = n - d - kvsel * d, s = slots[it];
                const size_t off = kv_offset(a.kv.layer, a.kv.n_pages, s / kPage, kvsel, a.kv.n_head, r / kHeadDim,
                                             s % kPage) + r % kHeadDim;
                *reinterpret_cast<uint4*>(reinterpret_cast<uint16_t*>(a.kv.base) + off) = v;
            }
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the block's reads end before the next block's writes
}

// The old values of a wave's 32 x 32 fp32 block, in the order add_block_f32 adds them.
__device__ __forceinline__ void load_block_f32(const GemmArgs& a, int m0, int n0, int lane, float (&old)[4][4]) {
    const float* x = reinterpret_cast<const float*>(a.out);
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int m = min(m0 + (lane >> 3) + 8 * it, a.M - 1), n = min(n0 + (lane & 7) * 4, a.N - 4);
        const float4 v = *reinterpret_cast<const float4*>(x + (size_t)m * a.N + n);
        old[it][0] = v.x, old[it][1] = v.y, old[it][2] = v.z, old[it][3] = v.w;
    }
}

// x += y for a wave's 32 x 32 block (y in accumulator order), through 4 KB of the
// wave's LDS as above (a row of the block is 128 bytes of fp32).  TR false: the
// accumulators are not transposed (element i is row 8 (i / 4) + 4 fh + i % 4, column fr).
template <bool TR = true>
__device__ __forceinline__ void add_block_f32(const GemmArgs& a, const float (&y)[16], const float (&old)[4][4], char* eb,
                                              int m0, int n0, int lane) {
    const int fr = lane & 31, fh = lane >> 5;
    if constexpr (TR) {
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<float4*>(eb + fr * 128 + (((g * 2 + fh) ^ (fr & 7)) << 4)) =
                make_float4(y[4 * g], y[4 * g + 1], y[4 * g + 2], y[4 * g + 3]);
    } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int rl = (i >> 2) * 8 + fh * 4 + (i & 3);
            *reinterpret_cast<float*>(eb + rl * 128 + (((fr >> 2) ^ (rl & 7)) << 4) + (fr & 3) * 4) = y[i];
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    float* x = reinterpret_cast<float*>(a.out);
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int rl = (lane >> 3) + 8 * it, q = lane & 7, m = m0 + rl, n = n0 + q * 4;
        const float4 v = *reinterpret_cast<const float4*>(eb + rl * 128 + ((q ^ (rl & 7)) << 4));
        if (m < a.M && n < a.N)
            *reinterpret_cast<float4*>(x + (size_t)m * a.N + n) =
                make_float4(old[it][0] + v.x, old[it][1] + v.y, old[it][2] + v.z, old[it][3] + v.w);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

}  // namespace ftts
