"""Launch shapes of the prefill and DiT linears (CPU, ftts_linear_plan): the split-K
scratch that a workspace holds covers the plan of every row count up to the one it was
sized for, and a model whose linears never split has none of it.  And the cases of
tests/test_gpu_gemm.py reach every launch shape that the widths they use give, by
epilogue, so that a change of the plan that leaves one untested fails here.
"""
import pytest

from paper_2607_21042_amd import ftts, workload
from tests import test_gpu_gemm as cases

SHAPES = [workload.INDEXTTS2, workload.TINY,
          workload.ModelShape(n_layer=1, d_model=4096, n_head=64, d_head=64, d_ff=16384, vocab=640)]
DITS = [workload.DIT_96M, workload.DIT_TINY]


def rows_up_to(most):
    """Every row count to 700 and the edges of the 64-row tiles beyond."""
    m = list(range(1, min(most, 700) + 1))
    return m + [r for e in range(704, most + 1, 64) for r in (e - 1, e, e + 1) if r <= most]


def linears(s):
    extra = [("in", s.d_model, s.n_mel + s.d_cond), ("mel", s.n_mel, s.d_model)] if hasattr(s, "n_mel") else []
    return list(s.matrices()) + extra


def used(p, rows, N):
    """(partial floats, counters) that the plan of so many rows writes."""
    if p.splits <= 1:
        return 0, 0
    tiles = -(-(rows - p.rows_large) // 64) * -(-N // p.small_cols)
    return p.splits * tiles * 64 * p.small_cols, tiles


@pytest.mark.parametrize("shape,wdtype", [(s, w) for s in SHAPES for w in (ftts.BF16, ftts.W8A16, ftts.W4A16)] +
                         [(s, ftts.BF16) for s in DITS])
def test_split_scratch_covers_every_plan(shape, wdtype):
    for name, N, K in linears(shape):
        floats = counters = 0
        for rows in rows_up_to(3000):
            p = ftts.linear_plan(wdtype, rows, N, K)
            assert 0 <= p.rows_large <= rows and (p.rows_large == rows) == (p.small_cols == 0)
            f, c = used(p, rows, N)
            floats, counters = max(floats, f), max(counters, c)
            # what a workspace sized for these rows holds covers this and every smaller call
            assert p.scratch_floats >= floats and p.scratch_counters >= counters, (name, rows)


def test_workspaces_hold_no_scratch_that_no_plan_uses():
    """A model whose K is too short to split needs none: 64 rows of a two-layer model
    of width 256 and d_ff 512 are 0.4 MB; and the full-size model's scratch at few rows
    is that of few tiles, not of the largest split."""
    small = workload.ModelShape(n_layer=2, d_model=256, n_head=4, d_head=64, d_ff=512, vocab=640)
    for wdtype in (ftts.BF16, ftts.W8A16, ftts.W4A16):
        for _, N, K in small.matrices():
            assert ftts.linear_plan(wdtype, 64, N, K).scratch_floats == 0
        assert ftts.workspace_bytes(ftts.make_config(small, wdtype), 1, 64) < 1 << 20
        full = ftts.make_config(workload.INDEXTTS2, wdtype)
        assert ftts.workspace_bytes(full, 1, 64) < 8 << 20
    assert ftts.dit_workspace_bytes(ftts.make_dit_config(workload.DIT_TINY), 16) < 1 << 20


def test_linear_plan_argument_errors():
    for args, code in [((ftts.F32, 64, 128, 128), -3), ((9, 64, 128, 128), -3), ((ftts.BF16, 0, 128, 128), -2),
                       ((ftts.BF16, 64, 12, 128), -2), ((ftts.BF16, 64, 128, 96), -2),
                       ((ftts.W8A16, 64, 128, 64), -2)]:
        with pytest.raises(ftts.FTTSError) as e:
            ftts.linear_plan(*args)
        assert e.value.code == code, args


def launches(shape, wdtype, rows):
    """(mode, epilogue, kernel, its tile or columns, K split) of every launch of the linears at so many rows."""
    dit = hasattr(shape, "n_mel")
    epilogue = {"qkv": "store" if dit else "qkv", "fc1": "gelu"}
    out = set()
    for name, N, K in linears(shape):
        e, p = epilogue.get(name, "residual"), ftts.linear_plan(wdtype, rows, N, K)
        if p.rows_large:
            out.add((wdtype, e, "large", p.large_rows, p.large_cols))
        if p.small_cols:
            out.add((wdtype, e, "small", p.small_cols, p.splits > 1))
        if p.rows_large and p.small_cols:
            out.add((wdtype, e, "large, rest small"))
    return out


def test_gemm_cases_reach_every_launch_shape():
    wd = {"bf16": ftts.BF16, "w8a16": ftts.W8A16, "w4a16": ftts.W4A16}
    reached, reachable = set(), set()
    for shape, prefills in ((cases.SHAPE, cases.PREFILLS), (cases.SHAPE_640, cases.PREFILLS_640)):
        assert shape.n_layer >= 2  # all rows of a prefill pass every linear of a layer before the last
        for mode, lens in prefills:
            reached |= launches(shape, wd[mode], sum(lens)) | launches(shape, wd[mode], len(lens))
        for mode in {m for m, _ in prefills}:
            for rows in range(8, 12001, 32):
                reachable |= launches(shape, wd[mode], rows)
    for shape, steps in ((cases.DIT, cases.DITS), (cases.DIT_640, cases.DITS_640)):
        for lens in steps:
            reached |= launches(shape, ftts.BF16, 2 * sum(lens))
        for rows in range(16, 12001, 32):
            reachable |= launches(shape, ftts.BF16, rows)
    assert len(reachable) > 40
    assert not reachable - reached, sorted(reachable - reached, key=str)
