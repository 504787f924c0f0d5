"""Bounds of the batched decode linears' staging loads (CPU): every load of every wave
of a launch, with the addresses the kernel forms (csrc/bgemm_stage.hpp, compiled here
as plain C++), lies inside its operand or starts at or past the descriptor's size,
where the hardware returns zero.  Among the shapes are waves with no chunk of their
slice (d_model 128, and W4A16's last slice at 1280), one-row batch tails and one-row
feature tails.  Also: each needed 16-byte piece is loaded, to the place it is read from.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

WALK = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "bgemm_stage.hpp"
using namespace ftts;

static long loads = 0, outside = 0;

// One operand of one wave: rows x row_bytes valid bytes, its run [col, col + RB) of every row;
// the chunks it uses end at byte `used` of a row.
template <class SH>
void walk(const char* what, int rows, int row_bytes, int bytes, int col, int used) {
    std::vector<int> got(SH::BYTES / 16, -1);
    for (int i = 0; i < SH::OPS; ++i)
        for (int lane = 0; lane < 64; ++lane) {
            const uint32_t off = stage_offset<SH>(lane, i, row_bytes, col);
            ++loads;
            if (off < (uint32_t)bytes && off + 16 > (uint32_t)bytes) {
                printf("%s: rows %d row_bytes %d col %d: bytes %u..%u of %d\n", what, rows, row_bytes, col, off, off + 16, bytes);
                exit(1);
            }
            if (off >= (uint32_t)bytes) ++outside;
            got[i * 64 + lane] = (int)off;
        }
    for (int r = 0; r < rows; ++r)
        for (int pc = 0; pc < SH::PIECES; ++pc)
            if (col + pc * 16 < used && got[r * SH::PIECES + (pc ^ row_swizzle<SH::PIECES>(r))] != r * row_bytes + col + pc * 16) {
                printf("%s: piece %d of row %d at column byte %d is not where it is read from\n", what, pc, r, col);
                exit(1);
            }
}

template <int WT, bool LN, int FT>
void launch(int N, int K, int B) {
    using C = BChunkShape<WT>;
    const int nchunks = K / C::KC, per = kBgemmWaves * ChunksPerWave<WT, LN>::value, S = (nchunks + per - 1) / per;
    for (int n0 = 0; n0 < N; n0 += FT * kBgemmFeat) {
        if (n0 > 0 && n0 + 2 * FT * kBgemmFeat < N) continue;  // the first tile and the last two
        for (int s = 0; s < S; ++s)
            for (int wave = 0; wave < kBgemmWaves; ++wave) {
                const int c1 = bgemm_slice(s + 1, S, nchunks), cw0 = bgemm_wave_chunk<WT, LN>(bgemm_slice(s, S, nchunks), wave);
                const int feats = N - n0 < FT * kBgemmFeat ? N - n0 : FT * kBgemmFeat;
                walk<WStage<WT, LN, FT>>("weights", feats, weight_row_bytes<WT>(K), weight_tile_bytes<WT, FT>(N, K, n0),
                                         cw0 * C::CB, c1 * C::CB);
                if (LN) walk<XStage<WT>>("fp32 input", B, K * 4, B * K * 4, cw0 * C::KC * 4, c1 * C::KC * 4);
                else walk<AStage<WT>>("bf16 input", B, K * 2, B * K * 2, cw0 * C::KC * 2, c1 * C::KC * 2);
            }
    }
}

template <int WT>
void shapes() {
    for (int B : {1, 3, 31, 32})
        for (int N : {1, 31, 33, 64, 65, 97, 640}) {
            for (int K : {128, 256, 384, 1280, 2048}) {
                launch<WT, true, 1>(N, K, B);
                if (WT != FTTS_W4A16) launch<WT, true, 2>(N, K, B);
            }
            for (int K : {128, 640, 1280, 5120, 6144}) launch<WT, false, 1>(N, K, B);
        }
}

int main() {
    shapes<FTTS_BF16>();
    shapes<FTTS_W8A16>();
    shapes<FTTS_W4A16>();
    printf("%ld loads, %ld of them past their operand\n", loads, outside);
    return outside > 0 ? 0 : 2;
}
"""


def test_staging_loads_stay_in_their_operands(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if not cxx:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(WALK)
    csrc, inc = os.path.join(ROOT, "paper_2607_21042_amd", "csrc"), os.path.join(ROOT, "include")
    r = subprocess.run([cxx, "-O2", "-std=c++17", "-I", csrc, "-I", inc, str(src), "-o", str(exe)], capture_output=True,
                       text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout


def test_staging_loads_use_no_scalar_offset():
    """The walk above bounds the lane offset alone, so the scalar offset of every
    staging load of the batched linears has to be zero."""
    with open(os.path.join(ROOT, "paper_2607_21042_amd", "csrc", "bgemm.hip")) as fh:
        text = " ".join(fh.read().split())
    calls = text.split("buffer_to_lds16(")[1:]
    assert len(calls) == 3
    for c in calls:
        assert c[:c.index(");")].rstrip().endswith(", 0"), c[:160]
