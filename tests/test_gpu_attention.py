"""GPU parity of the 16-bit attention at the edges of its tiles: sequence lengths
on both sides of the 64-key tile, the 32-query and 128-query tiles and one and
two rounds of the key split, with and without the mask, packed into a short grid
(the keys of a query tile split over waves) and a wide one (key tiles shared by 128
queries; `wide` below is the launcher's rule), and at the edges of the rule between
them.  Through the public calls; bars as in tests/helpers.py (bf16 storage: 3e-2
absolute on logits; DiT: its own).
"""
import numpy as np
import pytest

from oracle import dit as odit
from oracle import gpt as ogpt
from paper_2607_21042_amd import workload
from tests import helpers

pytestmark = pytest.mark.gpu

EDGES = [1, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 191, 193, 255, 256, 257, 320, 321]
# (heads, lengths): the causal calls take the short grid at 4 heads and the wide one at 8
SHORT, WIDE = (4, EDGES), (8, EDGES + EDGES[::-1])


def wide(lens, n_head):
    """Whether so many sequences (a DiT step: both branches) take 128-query workgroups."""
    groups = sum(-(-n // 128) for n in lens) * n_head
    return groups >= min(max(24 * -(-max(lens) // 64), 128), 768)


@pytest.mark.parametrize("n_head,lens", [SHORT, WIDE])
def test_causal_attention_edges(n_head, lens):
    """Two layers: the first attends with every row, the last with each prefix's
    last row; the decode steps read both layers' cached keys and values."""
    from paper_2607_21042_amd import ftts
    lens = lens[:32]
    shape = workload.ModelShape(n_layer=2, d_model=64 * n_head, n_head=n_head, d_head=64, d_ff=512, vocab=640)
    assert wide(lens, n_head) == (n_head == 8)
    inputs = workload.bf16_weights(workload.master_weights(shape, seed=3))
    dm = ftts.DeviceModel(inputs, shape, ftts.BF16)
    rows = workload.prefix_embeddings(lens, shape.d_model, seed=17)
    prefixes = np.split(rows, np.cumsum(lens)[:-1])
    fed = workload.random_tokens(2, len(lens), shape.vocab, seed=5)
    print(f"causal attention edges: {n_head} heads, {len(lens)} prefixes", flush=True)
    res = helpers.run_gpu(dm, shape, prefixes, fed)
    model = ogpt.GPT(helpers.oracle_weights(inputs, "bf16"), shape.n_head, shape.d_head)
    for b in range(len(lens)):
        last, dec = helpers.oracle_teacher_forced(model, prefixes[b], fed[:, b])
        for got, ref in ((res["prefill"][b], last), (res["logits"][0, b], dec[0]), (res["logits"][1, b], dec[1])):
            ok, err = helpers.tolerance_ok(got, ref, "bf16")
            assert ok, (n_head, lens[b], err)


def test_the_cases_take_both_grids():
    assert [wide(2 * lens[:32], n_head) for n_head, lens in FULL] == [True, True, False, False]
    assert [wide(lens, n_head) for n_head, lens in RULE_EDGES] == [False, True] * 3


# (heads, lengths) of the unmasked calls: wide, wide, short, short
FULL = [SHORT, WIDE, (4, EDGES[::2]), (4, EDGES[1::2])]


# both sides of the rule's three lines: 24 groups per 64 keys of the longest sequence, 128, 768
RULE_EDGES = [(8, [500] * 5 + [300]), (8, [500] * 6), (8, [100] * 15), (8, [100] * 16),
              (8, [128 * 41] + [128] * 54), (8, [128 * 41] + [128] * 55)]


@pytest.mark.parametrize("n_head,lens", RULE_EDGES)
def test_causal_attention_around_the_rule(n_head, lens):
    from paper_2607_21042_amd import ftts
    shape = workload.ModelShape(n_layer=2, d_model=64 * n_head, n_head=n_head, d_head=64, d_ff=512, vocab=640)
    inputs = workload.bf16_weights(workload.master_weights(shape, seed=3))
    dm = ftts.DeviceModel(inputs, shape, ftts.BF16)
    rows = workload.prefix_embeddings(lens, shape.d_model, seed=17)
    prefixes = np.split(rows, np.cumsum(lens)[:-1])
    fed = workload.random_tokens(1, len(lens), shape.vocab, seed=5)
    print(f"causal attention around the rule: {n_head} heads, {len(lens)} prefixes", flush=True)
    res = helpers.run_gpu(dm, shape, prefixes, fed)
    model = ogpt.GPT(helpers.oracle_weights(inputs, "bf16"), shape.n_head, shape.d_head)
    for b in sorted({0, 1, len(lens) // 2, len(lens) - 1}):
        last, dec = helpers.oracle_teacher_forced(model, prefixes[b], fed[:, b])
        for got, ref in ((res["prefill"][b], last), (res["logits"][0, b], dec[0])):
            ok, err = helpers.tolerance_ok(got, ref, "bf16")
            assert ok, (n_head, lens[b], err)


@pytest.mark.parametrize("n_head,lens", FULL)
def test_full_attention_edges(n_head, lens):
    import torch
    from paper_2607_21042_amd import ftts
    shape = workload.DitShape(n_layer=2, d_model=64 * n_head, n_head=n_head, d_head=64, d_ff=512, n_mel=64, d_cond=128)
    w = workload.bf16_weights(workload.dit_master_weights(shape, seed=20))
    lens = lens[:32]
    dm, ora = ftts.DitDeviceModel(w, shape), odit.DiT(w, shape.n_head, shape.d_head, dtype=np.float32)
    x, cond = workload.dit_inputs(shape, sum(lens), seed=41)
    xg, cg = torch.from_numpy(x).cuda(), torch.from_numpy(cond).cuda().to(torch.bfloat16)
    xo, vo = torch.empty_like(xg), torch.empty_like(xg)
    ws = torch.empty(ftts.dit_workspace_bytes(dm.cfg, sum(lens)), dtype=torch.uint8, device="cuda")
    print(f"full attention edges: {n_head} heads, {len(lens)} utterances", flush=True)
    ftts.dit_step(dm, xg, cg, 0.4, 0.04, 1.5, xo, vo, ws, lens=lens)
    torch.cuda.synchronize()
    v, at = vo.cpu().numpy(), 0
    for n in lens:
        _, ref = ora.step(x[at:at + n], cond[at:at + n], 0.4, 0.04, 1.5)
        ok, rel, err = helpers.dit_tolerance_ok(v[at:at + n], ref)
        assert ok, (n_head, n, rel, err)
        at += n


@pytest.mark.parametrize("mode", ["f32", "bf16", "w8a16", "w4a16"])
@pytest.mark.parametrize("lens", [[1], [32, 33, 1, 200]])
def test_prefill_without_logits_fills_the_same_cache(mode, lens):
    """The last layer stops early without logits; the cached keys and values are the same bits."""
    import torch
    from paper_2607_21042_amd import ftts
    shape = workload.ModelShape(n_layer=2, d_model=256, n_head=4, d_head=64, d_ff=512, vocab=640)
    wd = {"f32": ftts.F32, "bf16": ftts.BF16, "w8a16": ftts.W8A16, "w4a16": ftts.W4A16}[mode]
    dm = ftts.DeviceModel(workload.quantisable_weights(workload.master_weights(shape, seed=3)), shape, wd)
    table, n_pages = helpers.make_block_table(lens)
    pt = ftts.PageTableView(torch.from_numpy(table).cuda(), torch.zeros(len(lens), dtype=torch.int32, device="cuda"))
    prefix = torch.from_numpy(workload.prefix_embeddings(lens, shape.d_model, seed=17)).cuda().to(ftts.act_dtype(wd))
    pools = []
    print(f"prefill without logits: {mode} {lens}", flush=True)
    for logits in (None, torch.empty((len(lens), shape.vocab), device="cuda")):
        kv = ftts.KVCache(shape, wd, n_pages)
        ws = torch.empty(ftts.workspace_bytes(dm.cfg, len(lens), sum(lens)), dtype=torch.uint8, device="cuda")
        ftts.prefill(dm, prefix, lens, pt, kv, logits, ws)
        torch.cuda.synchronize()
        pools.append(kv.pool)
    assert pools[0].abs().max() > 0 and torch.equal(*pools)


@pytest.mark.parametrize("n_head,seqs", [(4, 2), (8, 24)])
def test_non_finite_rows_stay_causal(n_head, seqs):
    """A NaN row of a prefix reaches later rows only, and the 32-row block that it is
    in (its masked probability is 0, and 0 x NaN is NaN inside one matrix product):
    the keys and values of every earlier block keep their bits, on the short grid and
    on the wide one, and so do the other sequences'."""
    import torch
    from paper_2607_21042_amd import ftts
    shape = workload.ModelShape(n_layer=3, d_model=64 * n_head, n_head=n_head, d_head=64, d_ff=512, vocab=640)
    dm = ftts.DeviceModel(workload.bf16_weights(workload.master_weights(shape, seed=3)), shape, ftts.BF16)
    lens = [230] * seqs
    assert wide(lens, n_head) == (n_head == 8)
    table, n_pages = helpers.make_block_table(lens)
    pt = ftts.PageTableView(torch.from_numpy(table).cuda(), torch.zeros(seqs, dtype=torch.int32, device="cuda"))
    clean = torch.from_numpy(workload.prefix_embeddings(lens, shape.d_model, seed=17)).cuda().to(torch.bfloat16)

    def cache(prefix):
        kv = ftts.KVCache(shape, ftts.BF16, n_pages)
        ws = torch.empty(ftts.workspace_bytes(dm.cfg, seqs, sum(lens)), dtype=torch.uint8, device="cuda")
        ftts.prefill(dm, prefix, lens, pt, kv, None, ws)
        torch.cuda.synchronize()
        # [layer][seq][k|v][head][row][dim]
        pool = kv.pool[:, torch.from_numpy(table).cuda().long()]
        return pool.permute(0, 1, 3, 4, 2, 5, 6).flatten(4, 5)[..., :lens[0], :].float()

    ref = cache(clean)
    assert torch.isfinite(ref).all()
    for bad in (45, 100, 190, 229):
        x = clean.clone()
        x[bad] = float("nan")  # a row of sequence 0
        print(f"non-finite row {bad}: {n_head} heads, {seqs} prefixes", flush=True)
        got = cache(x)
        assert torch.isnan(got[0, 0, :, :, bad]).all()
        rows = bad // 32 * 32
        others, earlier = torch.equal(got[:, 1:], ref[:, 1:]), torch.equal(got[:, 0, :, :, :rows], ref[:, 0, :, :, :rows])
        assert others and earlier, (bad, others, earlier)
