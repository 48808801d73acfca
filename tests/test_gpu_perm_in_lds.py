"""GPU test of the layer's permutation in LDS (at most 1024 slots, static order, no padding): slots on both sides of the limit,
partial token blocks, destinations that cut them, experts without rows, all slots on one expert, against the oracle and against
the general path (the same layer through the ready-queue scheduler, which reads the permutation from memory)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_00686_amd import workloads as W
from tests import parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,k,E,R,dtype", [
    (1, 1, 1, 1, "bf16"), (1, 8, 8, 1, "bf16"), (63, 2, 5, 3, "bf16"), (65, 3, 130, 5, "f32"), (128, 8, 128, 2, "bf16"),
    (341, 3, 6, 11, "bf16"), (205, 5, 24, 5, "bf16"), (1023, 1, 16, 1, "bf16"), (1024, 1, 256, 16, "bf16"), (1025, 1, 16, 1, "bf16"),
])
@pytest.mark.parametrize("spread", ["even", "skewed"])
def test_layer_on_its_own_permutation(T, k, E, R, dtype, spread):
    from paper_2605_00686_amd import binding as B
    d, f = 64, 64
    print(f"case perm in LDS T={T} k={k} E={E} R={R} {dtype} {spread}", flush=True)
    inp = W.make_inputs(dict(T=T, d=d, E=E, k=k, f=f, R=R, dtype=dtype, seed=T + E, tile_m=32))
    gen = torch.Generator().manual_seed(T * 7 + k)
    score = torch.rand(T, E, generator=gen)
    if spread == "skewed":
        score[:, E // 2] += 1.0  # one expert has every token
    idx = score.topk(k, dim=1).indices.to(torch.int32)
    w = torch.rand(T, k, generator=gen) + 0.1
    dev = {n: inp[n].cuda() for n in ("x", "W1", "W3", "W2")}
    o = parity.oracle_arrays(inp)
    ref = oracle.forward(o["x"], o["Wg"], o["W1"], o["W3"], o["W2"], k, idx=idx.numpy(), w=w.numpy())
    tol = 2e-2 if dtype == "bf16" else 1e-4  # the tolerances of the layer's parity tests
    outs = []
    for sched in (0, 1):
        p = B.problem(T, d, E, k, f, R, dtype, tile_m=32, scheduler=sched)
        buf = B.Buffers(p)
        buf.topk_idx.copy_(idx)
        buf.topk_w.copy_(w)
        for epoch in (1, 2):
            p.epoch = epoch
            buf.perm.fill_(-7)
            buf.out.fill_(float("nan"))
            B.forward(p, buf, dev["x"], None, None, dev["W1"], dev["W3"], dev["W2"])
            torch.cuda.synchronize()
            assert int(buf.stats[7].item()) == 0
            assert np.array_equal(buf.perm.cpu().numpy(), ref["perm"])
            assert np.array_equal(buf.inv_perm.cpu().numpy().reshape(-1), np.asarray(ref["inv_perm"]).reshape(-1))
            err = parity.row_err(buf.out.float().cpu().numpy(), ref["out"]).max()
            assert err <= tol, err
        outs.append(buf.out.clone())
    assert torch.equal(outs[0], outs[1])


def test_waits_behind_the_first_gemm_expire():
    """Routing that is an input and a bound of one tick for the waits: nothing is waited for before GEMM1, so the waits behind it are
    the ones that expire.  The call reports it, every workgroup leaves, and with the workspace initialised again the same
    buffers give the right result."""
    from paper_2605_00686_amd import binding as B
    T, k, E, R, d, f = 64, 2, 6, 2, 2048, 256
    print("case perm in LDS, wait limit 1 tick", flush=True)
    inp = W.make_inputs(dict(T=T, d=d, E=E, k=k, f=f, R=R, dtype="bf16", seed=9, tile_m=32))
    idx = torch.rand(T, E, generator=torch.Generator().manual_seed(1)).topk(k, dim=1).indices.to(torch.int32)
    w = torch.full((T, k), 0.5)
    dev = {n: inp[n].cuda() for n in ("x", "W1", "W3", "W2")}
    o = parity.oracle_arrays(inp)
    ref = oracle.forward(o["x"], o["Wg"], o["W1"], o["W3"], o["W2"], k, idx=idx.numpy(), w=w.numpy())
    p = B.problem(T, d, E, k, f, R, "bf16", tile_m=32, wait_ticks=1)
    buf = B.Buffers(p)
    buf.topk_idx.copy_(idx)
    buf.topk_w.copy_(w)
    B.forward(p, buf, dev["x"], None, None, dev["W1"], dev["W3"], dev["W2"])
    torch.cuda.synchronize()
    assert int(buf.stats[7].item()) == B.MOE_ERR_TIMEOUT and int(buf.stats[6].item()) > 0
    B.moe_workspace_init(p, buf.workspace)
    buf.flags.zero_()
    p.wait_ticks = 0
    B.forward(p, buf, dev["x"], None, None, dev["W1"], dev["W3"], dev["W2"])
    torch.cuda.synchronize()
    assert int(buf.stats[7].item()) == 0
    assert np.array_equal(buf.perm.cpu().numpy(), ref["perm"])
    assert parity.row_err(buf.out.float().cpu().numpy(), ref["out"]).max() <= 2e-2  # (as above)
