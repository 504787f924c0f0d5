// Which bytes the batched decode linears (bgemm.hip) stage through LDS: tile shapes and
// the addresses of their buffer loads.  Plain C++, so that the bounds of every load of
// a launch can be walked on the host as the kernel forms them.
#pragma once
#include <stdint.h>

#include "ftts.h"

#ifdef __HIPCC__
#define FTTS_HD __host__ __device__ inline __attribute__((always_inline))
#else
#define FTTS_HD inline
#endif

namespace ftts {

constexpr int kBgemmRows = 32;  // sequences per launch
constexpr int kBgemmFeat = 32;  // features per MFMA tile (a workgroup owns FT tiles)
constexpr int kBgemmWaves = 4, kBgemmThreads = kBgemmWaves * 64;

template <int WT> struct BChunkShape;  // a chunk: KC columns in STEPS matrix instructions, CB bytes of one weight row
template <> struct BChunkShape<FTTS_BF16> { static constexpr int KC = 32, STEPS = 2, CB = 64; };
template <> struct BChunkShape<FTTS_W8A16> { static constexpr int KC = 32, STEPS = 2, CB = 32; };
template <> struct BChunkShape<FTTS_W4A16> { static constexpr int KC = 128, STEPS = 8, CB = 64; };

// Chunks per wave (its whole share of a K slice).  A LayerNorm input is staged as
// fp32 rows in LDS (32 rows x 64 columns per wave, 128 for W4A16), which keeps
// three workgroups per CU.
template <int WT, bool LN> struct ChunksPerWave { static constexpr int value = LN ? 2 : 4; };
template <> struct ChunksPerWave<FTTS_W4A16, false> { static constexpr int value = 2; };
template <> struct ChunksPerWave<FTTS_W4A16, true> { static constexpr int value = 1; };

// Slice s of S over nchunks chunks, and the first chunk of a wave's share of it.
FTTS_HD int bgemm_slice(int s, int S, int nchunks) { return s * nchunks / S; }
template <int WT, bool LN> FTTS_HD int bgemm_wave_chunk(int c0, int wave) { return c0 + wave * ChunksPerWave<WT, LN>::value; }

// A wave's chunks are consecutive, so each staged row is one run of RB bytes;
// direct-to-LDS loads bring the runs in with 16 lanes (or fewer) per run and several
// whole runs per 1 KB instruction, and the products read their operands from LDS.
// The 16-byte pieces of row r are stored XOR-swizzled by the row (row_swizzle) so that
// the 32 rows of one operand read fall into different banks: the 16 lanes whose
// 16-byte reads share a cycle take 256 bytes, and rows of 64 and 128 bytes share that
// window four and two at a time.
template <int PIECES>
FTTS_HD int row_swizzle(int r) {
    return PIECES == 4 ? (r >> 2) & 3 : PIECES == 8 ? (r >> 1) & 7 : r & (PIECES - 1);
}
template <int ROWS, int RUN> struct StageShape {
    static constexpr int RB = RUN, PIECES = RB / 16, BYTES = ROWS * RB, OPS = BYTES / 1024;
    static_assert(BYTES % 1024 == 0 && (PIECES & (PIECES - 1)) == 0, "staging shape");
};
template <int WT, bool LN, int FT>  // weight rows
using WStage = StageShape<FT * kBgemmFeat, ChunksPerWave<WT, LN>::value * BChunkShape<WT>::CB>;
template <int WT>                   // fp32 rows of a LayerNorm input
using XStage = StageShape<kBgemmRows, ChunksPerWave<WT, true>::value * BChunkShape<WT>::KC * 4>;
template <int WT>                   // bf16 input rows
using AStage = StageShape<kBgemmRows, ChunksPerWave<WT, false>::value * BChunkShape<WT>::KC * 2>;

// Load i of a wave's run starting col bytes into rows of row_bytes: the lane's byte
// offset from the operand's first row.  Row, column and piece all go into the lane's
// offset, which the buffer descriptor's size bounds by itself: a run past the end of a
// row reads the next row, past the operand zero, and neither is used.  (A scalar offset
// must not carry the column: whether the range check subtracts it is the hardware's
// affair, and a share that starts past the end of the operand would make that wrap.)
template <class SH>
FTTS_HD uint32_t stage_offset(int lane, int i, int row_bytes, int col) {
    const int r = i * (1024 / SH::RB) + lane / SH::PIECES;
    const int pc = (lane % SH::PIECES) ^ row_swizzle<SH::PIECES>(r);  // the piece that lands in this lane's slot
    return (uint32_t)(r * row_bytes + col + pc * 16);
}
// Descriptor sizes (bytes from the operand's first row).
template <int WT> FTTS_HD int weight_row_bytes(int K) { return WT == FTTS_W4A16 ? K / 2 : WT == FTTS_W8A16 ? K : K * 2; }
template <int WT, int FT> FTTS_HD int weight_tile_bytes(int N, int K, int n0) {
    return (N - n0 < FT * kBgemmFeat ? N - n0 : FT * kBgemmFeat) * weight_row_bytes<WT>(K);
}

}  // namespace ftts
