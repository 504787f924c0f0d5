"""GPU parity of the prefill and DiT linears over the launch shapes their plan
chooses: row counts at the edges of the 64-row tiles, and every tile shape of
either kernel with every epilogue that some row count gives it, with and without a
K split, and with the last rows left to the small kernel (tests/test_linear_plan.py
asks the plan whether these cases reach them all).  All through the public calls: a
two-layer model's prefill (its last layer goes on after QKV with each prefix's last
row only) followed by a decode step that reads every cached key and value back, and
a one-block DiT step.  Bars as in tests/helpers.py (bf16 storage: 3e-2 absolute on
logits; DiT: its own).
"""
import numpy as np
import pytest

from oracle import dit as odit
from oracle import gpt as ogpt
from paper_2607_21042_amd import workload
from tests import helpers

pytestmark = pytest.mark.gpu

SHAPE = workload.ModelShape(n_layer=2, d_model=1280, n_head=20, d_head=64, d_ff=5120, vocab=640)
DIT = workload.DitShape(n_layer=1, d_model=768, n_head=12, d_head=64, d_ff=3072, n_mel=128, d_cond=1280)
# (256 x 128 tiles come up at a width that leaves half of a 256-column tile idle)
SHAPE_640 = workload.ModelShape(n_layer=2, d_model=640, n_head=10, d_head=64, d_ff=2560, vocab=640)
DIT_640 = workload.DitShape(n_layer=1, d_model=640, n_head=10, d_head=64, d_ff=2560, n_mel=128, d_cond=896)

PREFILLS = [
    ("bf16", [1]), ("bf16", [64]), ("bf16", [65]), ("bf16", [257]), ("bf16", [333, 300]), ("bf16", [500, 511]),
    ("bf16", [512] * 4 + [51]), ("bf16", [700] * 7 + [120]), ("bf16", [640] * 11), ("bf16", [640] * 15 + [310]),
    ("w8a16", [1]), ("w8a16", [65]), ("w8a16", [257]), ("w8a16", [500, 500, 77]), ("w8a16", [640] * 4),
    ("w4a16", [1]), ("w4a16", [65]), ("w4a16", [257]), ("w4a16", [500, 500, 77]), ("w4a16", [640] * 4),
    ("bf16", [600, 700]), ("bf16", [650] * 6 + [97])]
PREFILLS_640 = [("bf16", [600] * 7), ("bf16", [700] * 14 + [99])]
DITS = [[1], [32], [33], [150, 91], [500], [700, 311], [512] * 4 + [117], [400] * 11 + [53], [640] * 12, [700] * 2,
        [500] * 7 + [199], [730, 170, 490, 615, 340, 512, 700, 433, 381, 290, 402, 514]]
DITS_640 = [[700] * 3, [610] * 8 + [70]]


@pytest.fixture(scope="module")
def master():
    return workload.master_weights(SHAPE, seed=0)


def wd(name):
    from paper_2607_21042_amd import ftts
    return {"bf16": ftts.BF16, "w8a16": ftts.W8A16, "w4a16": ftts.W4A16}[name]


@pytest.mark.parametrize("mode,lens", PREFILLS)
def test_prefill_linears(master, mode, lens):
    check_prefill(master, SHAPE, mode, lens)


@pytest.mark.parametrize("mode,lens", PREFILLS_640)
def test_prefill_linears_width_640(mode, lens):
    check_prefill(workload.master_weights(SHAPE_640, seed=0), SHAPE_640, mode, lens)


def check_prefill(master, shape, mode, lens):
    from paper_2607_21042_amd import ftts
    inputs = workload.bf16_weights(master) if mode == "bf16" else workload.quantisable_weights(master)
    dm = ftts.DeviceModel(inputs, shape, wd(mode))
    rows = workload.prefix_embeddings(lens, shape.d_model, seed=31)
    prefixes = np.split(rows, np.cumsum(lens)[:-1])
    fed = workload.random_tokens(1, len(lens), shape.vocab, seed=4)
    print(f"prefill linears: {mode} rows {sum(lens)} in {len(lens)} prefixes", flush=True)
    res = helpers.run_gpu(dm, shape, prefixes, fed)
    model = ogpt.GPT(helpers.oracle_weights(inputs, mode), shape.n_head, shape.d_head)
    for b in range(len(lens)):
        last, dec = helpers.oracle_teacher_forced(model, prefixes[b], fed[:, b])
        for got, ref in ((res["prefill"][b], last), (res["logits"][0, b], dec[0])):
            ok, err = helpers.tolerance_ok(got, ref, mode)
            assert ok, (mode, lens, b, err)


@pytest.mark.parametrize("lens", DITS)
def test_dit_linears(lens):
    check_dit(DIT, lens)


@pytest.mark.parametrize("lens", DITS_640)
def test_dit_linears_width_640(lens):
    check_dit(DIT_640, lens)


def check_dit(shape, lens):
    import torch
    from paper_2607_21042_amd import ftts
    w = workload.bf16_weights(workload.dit_master_weights(shape, seed=20))
    dm, ora = ftts.DitDeviceModel(w, shape), odit.DiT(w, shape.n_head, shape.d_head, dtype=np.float32)
    x, cond = workload.dit_inputs(shape, sum(lens), seed=41)
    xg, cg = torch.from_numpy(x).cuda(), torch.from_numpy(cond).cuda().to(torch.bfloat16)
    xo, vo = torch.empty_like(xg), torch.empty_like(xg)
    ws = torch.empty(ftts.dit_workspace_bytes(dm.cfg, sum(lens)), dtype=torch.uint8, device="cuda")
    print(f"dit linears: {sum(lens)} frames in {len(lens)} utterances", flush=True)
    ftts.dit_step(dm, xg, cg, 0.4, 0.04, 1.5, xo, vo, ws, lens=lens)
    torch.cuda.synchronize()
    v, at = vo.cpu().numpy(), 0
    for n in lens:
        _, ref = ora.step(x[at:at + n], cond[at:at + n], 0.4, 0.04, 1.5)
        ok, rel, err = helpers.dit_tolerance_ok(v[at:at + n], ref)
        assert ok, (lens, n, rel, err)
        at += n
