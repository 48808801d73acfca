"""GPU test of 256-row blocks that hold an expert's short tail: up to 64 rows they run the 64-row main loop, up to 128 the 128-row
one.  Tails on both sides of the limits, experts that have only a tail, ragged column tiles, both schedulers, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_00686_amd import workloads as W
from tests import parity

pytestmark = pytest.mark.gpu

# other options of the layer: signaling mode, fence group, destinations, rows an expert owns (0: ragged)
OPTIONS = [(0, 0, 1, 0), (1, 0, 3, 0), (0, 0, 6, 0), (1, 5, 6, 0), (1, 0, 2, 448), (0, 0, 3, 401)]

ROWS = {"behind": [257, 319, 320, 321, 384, 385], "alone": [64, 65, 1, 63, 128, 0, 300, 256]}


@pytest.mark.parametrize("sched", [0, 1], ids=["static", "ready_queue"])
@pytest.mark.parametrize("tile_m", [128, 64])
@pytest.mark.parametrize("rows", list(ROWS), ids=list(ROWS))
@pytest.mark.parametrize("d,f", [(320, 192), (64, 448)])
def test_tails_of_a_256_row_block(rows, d, f, tile_m, sched):
    from paper_2605_00686_amd import binding as B
    counts = ROWS[rows]
    E, T = len(counts), sum(counts)
    print(f"case short tails {rows} d={d} f={f} tile_m={tile_m} scheduler={sched}", flush=True)
    inp = W.make_inputs(dict(T=T, d=d, E=E, k=1, f=f, R=1, dtype="bf16", seed=d + T, tile_m=tile_m))
    gen = torch.Generator().manual_seed(T)
    idx = torch.repeat_interleave(torch.arange(E), torch.tensor(counts))[torch.randperm(T, generator=gen)].to(torch.int32).reshape(T, 1)
    w = torch.rand(T, 1, generator=gen) + 0.1
    p = B.problem(T, d, E, 1, f, 1, "bf16", tile_m=tile_m, scheduler=sched)
    dev = {n: inp[n].cuda() for n in ("x", "W1", "W3", "W2")}
    buf = B.Buffers(p)
    buf.topk_idx.copy_(idx)
    buf.topk_w.copy_(w)
    o = parity.oracle_arrays(inp)
    ref = oracle.forward(o["x"], o["Wg"], o["W1"], o["W3"], o["W2"], 1, idx=idx.numpy(), w=w.numpy())
    buf.staging.fill_(float("nan"))
    buf.out.fill_(float("nan"))
    B.forward(p, buf, dev["x"], None, None, dev["W1"], dev["W3"], dev["W2"])
    torch.cuda.synchronize()
    assert int(buf.stats[7].item()) == 0
    blocks = sum(-(-c // 256) for c in counts)  # (an expert of at most 128 rows is one block of the smaller height)
    assert int(buf.stats[4].item()) == blocks * -(-f // 128) and int(buf.stats[5].item()) == blocks * -(-d // 256)
    for name in ("staging", "out"):  # rows of bf16 products of bf16 operands: the tolerance of the layer's parity tests
        err = parity.row_err(getattr(buf, name).float().cpu().numpy(), ref[name]).max()
        assert err <= 2e-2, (name, err)


@pytest.mark.parametrize("mode,group,R,capacity", OPTIONS, ids=["m%d_g%d_R%d_c%d" % o for o in OPTIONS])
@pytest.mark.parametrize("sched", [0, 1], ids=["static", "ready_queue"])
def test_tails_with_other_options(mode, group, R, capacity, sched):
    """Per-tile signaling, fence groups, destinations that cut the tails, the padded layout: experts with and without full blocks."""
    from paper_2605_00686_amd import binding as B
    counts, d, f = [257, 64, 300, 65, 128, 1, 321, 384, 256, 130, 0, 60], 320, 192
    E, T = len(counts), sum(counts)
    T -= T % 6
    print(f"case short tails mode={mode} group={group} R={R} capacity={capacity} scheduler={sched}", flush=True)
    inp = W.make_inputs(dict(T=T, d=d, E=E, k=1, f=f, R=R, dtype="bf16", seed=T + R, tile_m=64))
    assert T % R == 0 and 96 <= T // E < 512  # (blocks of 256 rows; an expert's tail stays with them)
    gen = torch.Generator().manual_seed(T)
    idx = torch.repeat_interleave(torch.arange(E), torch.tensor(counts))[:T][torch.randperm(T, generator=gen)].to(torch.int32).reshape(T, 1)
    w = torch.rand(T, 1, generator=gen) + 0.1
    p = B.problem(T, d, E, 1, f, R, "bf16", tile_m=64, scheduler=sched, signal_mode=mode, group_size=group, capacity=capacity)
    dev = {n: inp[n].cuda() for n in ("x", "W1", "W3", "W2")}
    buf = B.Buffers(p)
    buf.topk_idx.copy_(idx)
    buf.topk_w.copy_(w)
    o = parity.oracle_arrays(inp)
    ref = oracle.forward(o["x"], o["Wg"], o["W1"], o["W3"], o["W2"], 1, idx=idx.numpy(), w=w.numpy(), capacity=capacity)
    plan = oracle.publish_plan(idx.numpy(), ref["offsets"], ref["inv_perm"], E, R, d, 64, 64)
    for epoch in (1, 2):
        p.epoch = epoch
        buf.staging.fill_(float("nan"))
        buf.out.fill_(float("nan"))
        B.forward(p, buf, dev["x"], None, None, dev["W1"], dev["W3"], dev["W2"])
        torch.cuda.synchronize()
        assert int(buf.stats[7].item()) == 0
        assert np.array_equal(buf.perm.cpu().numpy(), ref["perm"])
        assert np.array_equal(buf.slot_flag.cpu().numpy(), plan["slot_flag"])
        assert np.all(buf.flags.cpu().numpy()[:plan["n_flags"]] == epoch)
        assert int(buf.stats[0].item()) == parity.expected_fences(plan, mode, group)
        for name in ("staging", "out"):  # (as above)
            err = parity.row_err(getattr(buf, name).float().cpu().numpy(), ref[name]).max()
            assert err <= 2e-2, (name, err)
