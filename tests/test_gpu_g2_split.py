"""GPU test of fp32 GEMM2 tiles that are cut along the reduction: numbers of parts from two to the most, reductions that do not
divide evenly, ragged column tiles, one to several row blocks per expert, the padded layout, destinations, and shapes on both
sides of the rule's limits, against the oracle; repeated calls and both schedulers give the same bits."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_00686_amd import workloads as W
from tests import parity

pytestmark = pytest.mark.gpu

# (T, d, E, k, f, R, capacity); GEMM2 tiles = row blocks x ceil(d / 64), parts = min(256 / tiles, 8, f / 128)
CASES = [(1, 64, 2, 2, 256, 1, 0), (3, 80, 4, 2, 272, 3, 0), (16, 528, 16, 2, 1040, 2, 0), (256, 512, 8, 2, 1024, 2, 0),
         (200, 512, 8, 2, 1024, 1, 72), (129, 208, 2, 1, 2064, 1, 0), (500, 64, 3, 2, 3072, 4, 0), (128, 1024, 8, 1, 400, 1, 0),
         (64, 4096, 2, 2, 384, 1, 0), (64, 4160, 2, 2, 384, 1, 0), (40, 64, 2, 2, 240, 1, 0)]


@pytest.mark.parametrize("T,d,E,k,f,R,capacity", CASES, ids=["T%d_d%d_E%d_k%d_f%d_R%d_c%d" % c for c in CASES])
def test_parts_of_a_tile(T, d, E, k, f, R, capacity):
    from paper_2605_00686_amd import binding as B
    print(f"case g2_split T={T} d={d} E={E} k={k} f={f} R={R} capacity={capacity}", flush=True)
    inp = W.make_inputs(dict(T=T, d=d, E=E, k=k, f=f, R=R, dtype="f32", seed=T + d))
    idx = w = None
    if capacity:  # balanced: the padded layout drops nothing
        idx = ((np.arange(T)[:, None] * k + np.arange(k)) % E).astype(np.int32)
        w = np.full((T, k), 1.0 / k, dtype=np.float32)
    dev = {n: inp[n].cuda() for n in ("x", "Wg", "W1", "W3", "W2")}
    o = parity.oracle_arrays(inp)
    ref = oracle.forward(o["x"], o["Wg"], o["W1"], o["W3"], o["W2"], k, idx=idx, w=w, capacity=capacity)
    first = None
    for scheduler in (0, 1):
        p = B.problem(T, d, E, k, f, R, "f32", capacity=capacity, scheduler=scheduler)
        buf = B.Buffers(p)
        if capacity:
            buf.topk_idx.copy_(torch.from_numpy(idx))
            buf.topk_w.copy_(torch.from_numpy(w))
        for epoch in (1, 2, 3):
            p.epoch = epoch
            buf.staging.fill_(float("nan"))
            buf.out.fill_(float("nan"))
            B.forward(p, buf, dev["x"], None if capacity else dev["Wg"], None, dev["W1"], dev["W3"], dev["W2"])
            torch.cuda.synchronize()
            assert int(buf.stats[7].item()) == 0
            blocks = sum(-(-int(c) // 128) for c in ref["counts"])
            assert int(buf.stats[5].item()) == blocks * -(-d // 64)  # a tile is counted once, whatever its parts
            if scheduler:
                assert int(buf.stats[16].item()) >= int(buf.stats[5].item())
            got = {n: getattr(buf, n).cpu().numpy() for n in ("staging", "out", "perm")}
            assert np.array_equal(got["perm"], ref["perm"])
            first = first or got
            for name in ("staging", "out"):
                assert np.array_equal(got[name], first[name]), name
                err = parity.row_err(got[name], ref[name]).max()
                print(f"  {name}: row-normalised error {err:.2e}", flush=True)
                assert err <= 2e-5, name  # (as in the test of the fp32 tiles: n * 2^-24 at most, n <= 3072 here)
