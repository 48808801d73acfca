"""GPU test of the layer's combine: one to five tokens per task, so that a wavefront has fewer pieces than it keeps in flight, a whole
number of rounds of them and a rest; wavefronts that share a row; rows of odd numbers of 16-byte pieces; k below, at and past a
unit's; destinations of an odd number of tokens under the ready-queue scheduler.  And the plan from the choices: numbers of slots
up to and just past those a workgroup counts by itself, with destinations that are and are not whole token blocks."""
import numpy as np
import pytest
import torch

from paper_2605_00686_amd import workloads as W
from tests import parity

pytestmark = pytest.mark.gpu

# (T, d, E, k, R, dtype, scheduler)
CASES = [(1, 64, 4, 1, 1, "bf16", 0), (256, 1088, 8, 2, 4, "bf16", 0), (257, 2048, 8, 8, 1, "bf16", 0), (700, 1984, 8, 5, 7, "bf16", 0),
         (1021, 576, 8, 8, 1, "bf16", 0), (1025, 2112, 4, 4, 5, "bf16", 0), (1030, 64, 16, 9, 2, "bf16", 0), (1024, 4096, 4, 1, 8, "bf16", 0),
         (600, 1040, 4, 3, 3, "f32", 0), (1019, 128, 8, 8, 1, "f32", 0), (1029, 1024, 8, 4, 7, "bf16", 1), (771, 640, 4, 2, 3, "bf16", 1),
         (514, 192, 4, 1, 2, "bf16", 1),
         # more rows per token than a wavefront loads at once, and exactly as many
         (5, 1984, 32, 32, 1, "bf16", 0), (300, 576, 24, 16, 3, "bf16", 0), (770, 1088, 20, 17, 7, "bf16", 0), (1030, 320, 16, 10, 5, "bf16", 1),
         (257, 272, 24, 24, 1, "f32", 0), (1200, 144, 16, 16, 4, "f32", 0),
         (4096, 64, 8, 2, 64, "bf16", 0), (4097, 64, 8, 2, 17, "bf16", 0), (1024, 64, 16, 8, 16, "bf16", 1), (1025, 64, 16, 8, 25, "bf16", 0)]


@pytest.mark.parametrize("T,d,E,k,R,dtype,sched", CASES, ids=["T%d_d%d_E%d_k%d_R%d_%s_s%d" % c for c in CASES])
def test_layer_combine(T, d, E, k, R, dtype, sched):
    from paper_2605_00686_amd import binding as B
    print(f"case combine chunks T={T} d={d} E={E} k={k} R={R} {dtype} scheduler={sched}", flush=True)
    inp = W.make_inputs(dict(T=T, d=d, E=E, k=k, f=64, R=R, dtype=dtype, seed=T + d + k))
    p = B.problem(T, d, E, k, 64, R, dtype, scheduler=sched)
    dev = {n: inp[n].cuda() for n in ("x", "Wg", "W1", "W3", "W2")}
    buf = B.Buffers(p)
    buf.staging.fill_(float("nan"))
    buf.out.fill_(float("nan"))
    B.forward(p, buf, dev["x"], dev["Wg"], None, dev["W1"], dev["W3"], dev["W2"])
    torch.cuda.synchronize()
    assert int(buf.stats[7].item()) == 0
    ridx, _, _ = parity.oracle_routing(inp)
    assert np.array_equal(buf.topk_idx.cpu().numpy(), ridx)
    order = np.argsort(ridx.reshape(-1), kind="stable")
    assert np.array_equal(buf.perm.cpu().numpy(), order)
    assert np.array_equal(buf.counts.cpu().numpy(), np.bincount(ridx.reshape(-1), minlength=E))
    terms = buf.staging.cpu().double().reshape(T, k, d) * buf.topk_w.cpu().double()[:, :, None]
    # k roundings of an fp32 sum, each at most 2^-24 of the sum of magnitudes, then one rounding to the output type
    bound = k * 2.0 ** -23 * terms.abs().sum(1) + (2.0 ** -8 if dtype == "bf16" else 2.0 ** -24) * terms.sum(1).abs()
    assert bool(((buf.out.cpu().double() - terms.sum(1)).abs() <= bound + 1e-30).all())


@pytest.mark.parametrize("T,k", [(8192, 1), (8193, 1)], ids=["by_itself", "by_gate_tasks"])
def test_invalid_choices_are_reported_by_the_plan(T, k):
    """Routing that is an input with an id outside [0, E): reported whoever counts the choices, and the next call works."""
    from paper_2605_00686_amd import binding as B
    print(f"case invalid choice T={T}", flush=True)
    E, d = 4, 64
    p = B.problem(T, d, E, k, 64, 1, "bf16")
    x = torch.randn(T, d, device="cuda").bfloat16()
    W1, W2 = torch.randn(E, d, 64, device="cuda").bfloat16(), torch.randn(E, 64, d, device="cuda").bfloat16()
    buf = B.Buffers(p)
    ids = torch.randint(0, E, (T, 1), dtype=torch.int32, device="cuda")
    buf.topk_w.fill_(1.0)
    for epoch, bad in ((1, E), (2, -1), (3, None)):
        p.epoch = epoch
        buf.topk_idx.copy_(ids)
        if bad is not None:
            buf.topk_idx[T // 2] = bad
        B.forward(p, buf, x, None, None, W1, W1, W2)
        torch.cuda.synchronize()
        assert int(buf.stats[7].item()) == (B.MOE_ERR_BAD_ROUTING if bad is not None else 0)
        if bad is None:
            assert torch.equal(buf.counts.cpu(), torch.bincount(ids.cpu().reshape(-1), minlength=E).int())
