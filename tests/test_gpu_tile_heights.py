"""GPU test of the layer's row blocks of two heights with a 32-row publish tile (64-row tiles, and 32-row ones for experts of at most
32 rows): experts on both sides of every height in one batch, an expert without rows, ragged column tiles, both schedulers and
signaling modes, both layouts of the rows, destinations that cut row blocks, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_00686_amd import workloads as W
from tests import parity

pytestmark = pytest.mark.gpu

# rows of the experts: 32 and more on average, all experts at most 32 rows (no 64-row block), none (no 32-row block)
ROWS = {"mixed": [1, 31, 32, 33, 63, 64, 65, 97, 0, 128, 129, 16], "short": [32, 32, 32], "tall": [33, 64, 95]}


@pytest.mark.parametrize("sched,mode,capacity", [(0, 1, 0), (0, 0, 0), (1, 1, 0), (0, 1, 129), (1, 0, 192)],
                         ids=["static_per_dest", "static_per_tile", "ready_queue", "padded", "padded_ready_queue_per_tile"])
@pytest.mark.parametrize("rows", list(ROWS), ids=list(ROWS))
@pytest.mark.parametrize("d,f", [(320, 192), (64, 448)])
def test_row_blocks_of_two_heights(rows, d, f, sched, mode, capacity):
    from paper_2605_00686_amd import binding as B
    counts = ROWS[rows]
    E, T = len(counts), sum(counts)
    R = 3 if T % 3 == 0 else 1
    assert T // E >= 32
    print(f"case tile heights {rows} d={d} f={f} R={R} scheduler={sched} mode={mode} capacity={capacity}", flush=True)
    inp = W.make_inputs(dict(T=T, d=d, E=E, k=1, f=f, R=R, dtype="bf16", seed=d + T, tile_m=32))
    gen = torch.Generator().manual_seed(T)
    idx = torch.repeat_interleave(torch.arange(E), torch.tensor(counts))[torch.randperm(T, generator=gen)].to(torch.int32).reshape(T, 1)
    w = torch.rand(T, 1, generator=gen) + 0.1
    p = B.problem(T, d, E, 1, f, R, "bf16", tile_m=32, scheduler=sched, signal_mode=mode, capacity=capacity)
    dev = {n: inp[n].cuda() for n in ("x", "W1", "W3", "W2")}
    buf = B.Buffers(p)
    buf.topk_idx.copy_(idx)
    buf.topk_w.copy_(w)
    o = parity.oracle_arrays(inp)
    ref = oracle.forward(o["x"], o["Wg"], o["W1"], o["W3"], o["W2"], 1, idx=idx.numpy(), w=w.numpy(), capacity=capacity)
    plan = oracle.publish_plan(idx.numpy(), ref["offsets"], ref["inv_perm"], E, R, d, 32, 64)
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
        assert int(buf.stats[0].item()) == parity.expected_fences(plan, mode, 0)
        blocks = sum(1 if c <= 32 else -(-c // 64) for c in counts if c)
        assert int(buf.stats[4].item()) == blocks * -(-f // 128) and int(buf.stats[5].item()) == blocks * -(-d // 256)
        for name in ("staging", "out"):  # rows of bf16 products of bf16 operands: the tolerance of the layer's parity tests
            err = parity.row_err(getattr(buf, name).float().cpu().numpy(), ref[name]).max()
            assert err <= 2e-2, (name, err)
