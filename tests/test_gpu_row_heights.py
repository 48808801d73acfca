"""GPU test of row blocks with fewer rows than their tile, which run the main loop of the next multiple of 32 rows: row counts on both
sides of every height, as an expert's only block, as its tail behind whole blocks and (many rows per expert) as a tail in a
block of its own, with a reduction of one stage up, ragged column tiles, both schedulers and signaling modes, against the oracle; and
the same bits as whole blocks give, with destinations, fence groups and padding."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_00686_amd import workloads as W
from tests import parity

pytestmark = pytest.mark.gpu

EDGES = [1, 32, 33, 64, 65, 96, 97, 128, 129, 160, 161, 192, 193, 224, 225, 256]
# 96 to 511 rows per expert on average: a tail stays with the big blocks; from 512 on one of at most 128 rows is a small block
ROWS = {"alone": EDGES, "behind_one": [256 + r for r in EDGES], "behind_many": [512 + r for r in EDGES]}


@pytest.mark.parametrize("sched,mode", [(0, 1), (1, 1), (0, 0)], ids=["static", "ready_queue", "static_per_tile"])
@pytest.mark.parametrize("d,f", [(64, 192), (320, 64), (192, 448)])
@pytest.mark.parametrize("rows", list(ROWS), ids=list(ROWS))
def test_row_heights(rows, d, f, sched, mode):
    from paper_2605_00686_amd import binding as B
    counts = ROWS[rows]
    E, T = len(counts), sum(counts)
    assert T // E >= 96 and (T // E >= 512) == (rows == "behind_many")
    print(f"case row heights {rows} d={d} f={f} scheduler={sched} mode={mode}", flush=True)
    inp = W.make_inputs(dict(T=T, d=d, E=E, k=1, f=f, R=1, dtype="bf16", seed=d + T))
    gen = torch.Generator().manual_seed(T)
    idx = torch.repeat_interleave(torch.arange(E), torch.tensor(counts))[torch.randperm(T, generator=gen)].to(torch.int32).reshape(T, 1)
    w = torch.rand(T, 1, generator=gen) + 0.1
    p = B.problem(T, d, E, 1, f, 1, "bf16", scheduler=sched, signal_mode=mode)
    dev = {n: inp[n].cuda() for n in ("x", "W1", "W3", "W2")}
    buf = B.Buffers(p)
    buf.topk_idx.copy_(idx)
    buf.topk_w.copy_(w)
    o = parity.oracle_arrays(inp)
    ref = oracle.forward(o["x"], o["Wg"], o["W1"], o["W3"], o["W2"], 1, idx=idx.numpy(), w=w.numpy())
    for epoch in (1, 2):
        p.epoch = epoch
        buf.staging.fill_(float("nan"))
        buf.out.fill_(float("nan"))
        B.forward(p, buf, dev["x"], None, None, dev["W1"], dev["W3"], dev["W2"])
        torch.cuda.synchronize()
        assert int(buf.stats[7].item()) == 0
        assert np.array_equal(buf.perm.cpu().numpy(), ref["perm"])
        for name in ("staging", "out"):  # rows of bf16 products of bf16 operands: the tolerance of the layer's parity tests
            err = parity.row_err(getattr(buf, name).float().cpu().numpy(), ref[name]).max()
            assert err <= 2e-2, (name, err)


# (scheduler, signal mode, flags per fence group, destinations, padded layout)
WAYS = [(0, 1, 0, 8, False), (1, 1, 0, 8, False), (0, 0, 0, 8, False), (0, 1, 5, 8, False), (1, 1, 5, 8, False), (0, 1, 0, 4, True), (1, 1, 5, 2, True)]


@pytest.mark.parametrize("d,f", [(320, 64), (192, 448)])
def test_same_bits_as_whole_blocks(d, f):
    """A row's result does not depend on how many rows its block has: 768 rows per expert, all in whole blocks of 256, against every
    number of rows above, of the same tokens."""
    from paper_2605_00686_amd import binding as B
    E, whole = len(EDGES), 768
    inp = W.make_inputs(dict(T=E * whole, d=d, E=E, k=1, f=f, R=1, dtype="bf16", seed=d + f))
    dev = {n: inp[n].cuda() for n in ("x", "W1", "W3", "W2")}
    order = torch.randperm(E * whole, generator=torch.Generator().manual_seed(d))
    expert = (order % E).to(torch.int32)  # 768 tokens each, in no order

    def run(tokens, scheduler, mode, group, R, capacity):
        print(f"case row heights, bits: {len(tokens)} tokens d={d} f={f} scheduler={scheduler} mode={mode} group={group} R={R} capacity={capacity}", flush=True)
        p = B.problem(len(tokens), d, E, 1, f, R, "bf16", scheduler=scheduler, signal_mode=mode, group_size=group, capacity=capacity)
        buf = B.Buffers(p)
        buf.topk_idx.copy_(expert[tokens].reshape(-1, 1))
        buf.topk_w.fill_(1.0)
        buf.staging.fill_(float("nan"))
        buf.out.fill_(float("nan"))
        B.forward(p, buf, dev["x"][tokens.cuda()].contiguous(), None, None, dev["W1"], dev["W3"], dev["W2"])
        torch.cuda.synchronize()
        assert int(buf.stats[7].item()) == 0 and int(buf.stats[1].item()) == int(buf.stats[2].item())
        assert bool((buf.flags[:int(buf.stats[1].item())] == 1).all())
        return buf.staging.view(torch.int16).cpu(), buf.out.view(torch.int16).cpu()

    want = run(torch.arange(E * whole), 0, 1, 0, 1, 0)
    for counts in ROWS.values():
        tokens = torch.cat([torch.nonzero(expert == e).reshape(-1)[:n] for e, n in enumerate(counts)]).sort().values
        for scheduler, mode, group, R, padded in WAYS:
            got = run(tokens, scheduler, mode, group, R, max(counts) if padded else 0)
            assert torch.equal(got[0], want[0][tokens]) and torch.equal(got[1], want[1][tokens])
