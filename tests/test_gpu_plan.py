"""GPU test of the plan inside the megakernel on both sides of the rule that chooses between its two forms (every workgroup
derives it in LDS; one workgroup writes it to memory): destinations x experts and token blocks x experts at and just past
the limits, destinations that are and are not whole token blocks, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_00686_amd import workloads as W
from tests import parity

pytestmark = pytest.mark.gpu

# (T, E, R, k, tile_m, capacity): the tables' limits are 8 * E * R <= 32 KB and 4 * E * ceil(T / 64) <= 64 KB
CASES = [(192, 64, 64, 2, 32, 0), (195, 64, 65, 2, 32, 0), (4096, 256, 4, 2, 128, 0), (4100, 256, 4, 2, 128, 0),
         (640, 3, 10, 2, 64, 0), (640, 3, 10, 2, 64, 512), (77, 5, 7, 3, 128, 77)]


@pytest.mark.parametrize("T,E,R,k,tile_m,capacity", CASES, ids=["T%d_E%d_R%d_k%d_m%d_c%d" % c for c in CASES])
def test_plan_forms(T, E, R, k, tile_m, capacity):
    from paper_2605_00686_amd import binding as B
    print(f"case plan T={T} E={E} R={R} k={k} tile_m={tile_m} capacity={capacity}", flush=True)
    inp = W.make_inputs(dict(T=T, d=64, E=E, k=k, f=64, R=R, dtype="bf16", seed=T + R, bias_std=0.2, tile_m=tile_m))
    p = B.problem(T, 64, E, k, 64, R, "bf16", tile_m=tile_m, capacity=capacity)
    dev = {n: inp[n].cuda() for n in ("x", "Wg", "gate_bias", "W1", "W3", "W2")}
    buf = B.Buffers(p)
    B.forward(p, buf, dev["x"], dev["Wg"], dev["gate_bias"], dev["W1"], dev["W3"], dev["W2"])
    torch.cuda.synchronize()
    assert int(buf.stats[7].item()) == 0
    idx, w, _ = parity.oracle_routing(inp)
    o = parity.oracle_arrays(inp)
    ref = oracle.forward(o["x"], o["Wg"], o["W1"], o["W3"], o["W2"], k, idx=idx, w=w, capacity=capacity)
    plan = oracle.publish_plan(idx, ref["offsets"], ref["inv_perm"], E, R, 64, tile_m, 64)
    for name in ("counts", "offsets", "perm", "inv_perm"):
        assert np.array_equal(getattr(buf, name).cpu().numpy(), ref[name]), name
    assert np.array_equal(buf.slot_flag.cpu().numpy(), plan["slot_flag"])
    assert np.all(buf.flags.cpu().numpy()[:plan["n_flags"]] == 1)
    assert int(buf.stats[0].item()) == plan["fences_per_dest"]
