"""GPU test of fp32 GEMM2 tiles that are cut along the reduction, each shape with its number of parts, two to eight: reductions that do not
divide evenly, ragged column tiles, one to several row blocks per expert, the padded layout, destinations, and shapes on both
sides of the rule's limits (tests/test_g2_forms.py ties the rule to the library), against the oracle; repeated calls, both schedulers
and every way of signaling give the same bits."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_00686_amd import workloads as W
from tests import g2_forms, parity

pytestmark = pytest.mark.gpu

# (T, d, E, k, f, R, capacity): parts
CASES = {(256, 512, 8, 2, 512, 2, 0): 2, (200, 528, 2, 2, 272, 4, 0): 2, (512, 512, 8, 2, 768, 4, 0): 2, (576, 512, 8, 2, 768, 4, 0): 1,
         (256, 512, 8, 2, 784, 1, 0): 3, (1, 64, 1, 1, 768, 1, 0): 3, (256, 512, 8, 2, 1024, 2, 0): 4, (200, 512, 8, 2, 1024, 1, 72): 4,
         (64, 256, 4, 2, 896, 8, 0): 5, (64, 256, 4, 2, 1040, 1, 0): 6, (60, 256, 4, 2, 1232, 3, 48): 6, (64, 256, 4, 2, 1232, 2, 0): 7,
         (3, 80, 4, 2, 2064, 3, 0): 8, (129, 208, 2, 1, 2064, 1, 0): 8, (500, 64, 3, 2, 3072, 4, 0): 8,
         (1, 64, 2, 2, 256, 1, 0): 1, (16, 528, 16, 2, 1040, 2, 0): 1, (64, 4160, 2, 2, 384, 1, 0): 1, (40, 64, 2, 2, 240, 1, 0): 1}
# (scheduler, signal mode, flags per fence group)
WAYS = [(0, 1, 0), (1, 1, 0), (0, 0, 0), (1, 0, 0), (0, 1, 3), (1, 1, 3)]


@pytest.mark.parametrize("T,d,E,k,f,R,capacity", list(CASES), ids=["T%d_d%d_E%d_k%d_f%d_R%d_c%d" % c for c in CASES])
def test_every_number_of_parts(T, d, E, k, f, R, capacity):
    from paper_2605_00686_amd import binding as B
    print(f"case g2_parts T={T} d={d} E={E} k={k} f={f} R={R} capacity={capacity}", flush=True)
    assert g2_forms.parts(T, d, E, k, f) == CASES[T, d, E, k, f, R, capacity]
    inp = W.make_inputs(dict(T=T, d=d, E=E, k=k, f=f, R=R, dtype="f32", seed=T + d))
    idx = w = None
    if capacity:  # balanced: the padded layout drops nothing
        idx = ((np.arange(T)[:, None] * k + np.arange(k)) % E).astype(np.int32)
        w = np.full((T, k), 1.0 / k, dtype=np.float32)
    dev = {n: inp[n].cuda() for n in ("x", "Wg", "W1", "W3", "W2")}
    o = parity.oracle_arrays(inp)
    ref = oracle.forward(o["x"], o["Wg"], o["W1"], o["W3"], o["W2"], k, idx=idx, w=w, capacity=capacity)
    tiles = sum(-(-int(c) // 128) for c in ref["counts"]) * -(-d // 64)
    first = None
    for scheduler, mode, group in WAYS:
        p = B.problem(T, d, E, k, f, R, "f32", capacity=capacity, scheduler=scheduler, signal_mode=mode, group_size=group)
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
            stats = [int(v) for v in buf.stats.cpu()]
            assert stats[7] == 0
            assert stats[5] == tiles  # a tile is counted once, whatever its parts
            assert stats[16] == (tiles + g2_forms.combine_tasks(T, R) if scheduler else 0) and stats[17] <= (tiles if scheduler else 0)
            assert stats[1] == stats[2] and bool((buf.flags[:stats[1]] == epoch).all())
            got = {n: getattr(buf, n).cpu().numpy() for n in ("staging", "out", "perm")}
            assert np.array_equal(got["perm"], ref["perm"])
            first = first or got
            for name in ("staging", "out"):
                assert np.array_equal(got[name], first[name]), name
                err = parity.row_err(got[name], ref[name]).max()
                print(f"  {name}: row-normalised error {err:.2e}", flush=True)
                assert err <= 2e-5, name  # (as in the test of the fp32 tiles: n * 2^-24 at most, n <= 3072 here)
