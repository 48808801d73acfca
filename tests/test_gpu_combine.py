"""GPU test of how combine tasks share their work: tokens per task of 1, 2 and 4 (where the rule changes, and one past it), rows
of fewer 16-byte pieces than the sharing wavefronts have lanes and of odd numbers of them, k from 1 to past the loads in
flight; alone and, through the flags, at the end of a forward pass."""
import pytest
import torch

from paper_2605_00686_amd import workloads as W

pytestmark = pytest.mark.gpu

# (T, d, k, dtype)
CASES = [(1, 64, 1, "bf16"), (256, 192, 8, "bf16"), (257, 1088, 2, "bf16"), (512, 64, 4, "bf16"), (513, 320, 9, "bf16"),
         (515, 576, 17, "bf16"), (130, 7168, 8, "bf16"), (300, 16, 3, "f32"), (514, 1040, 1, "f32"), (3, 4112, 12, "f32"),
         (768, 2048, 2, "bf16"), (769, 2048, 3, "bf16"), (767, 1984, 5, "bf16"), (1536, 1024, 1, "bf16"), (1537, 2048, 2, "bf16"),
         (1535, 960, 4, "bf16"), (770, 512, 6, "f32"), (9, 1024, 2, "f32")]


@pytest.mark.parametrize("T,d,k,dtype", CASES, ids=["T%d_d%d_k%d_%s" % c for c in CASES])
def test_combine_shares(T, d, k, dtype):
    from paper_2605_00686_amd import binding as B
    print(f"case combine T={T} d={d} k={k} {dtype}", flush=True)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    p = B.problem(T, d, 32, k, 64, 1, dt)
    gen = torch.Generator().manual_seed(T + d + k)
    rows = torch.randn(T * k, d, generator=gen).to(dt)
    w = torch.rand(T, k, generator=gen)
    out = torch.full((T, d), float("nan"), dtype=dt, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    B.moe_combine(p, rows.cuda(), None, None, w.cuda(), out, status)
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    terms = rows.double().reshape(T, k, d) * w.double()[:, :, None]
    # k roundings of an fp32 sum, each at most 2^-24 of the sum of magnitudes, then one rounding to the output type
    bound = k * 2.0 ** -23 * terms.abs().sum(1) + (2.0 ** -8 if dtype == "bf16" else 2.0 ** -24) * terms.sum(1).abs()
    assert bool(((out.cpu().double() - terms.sum(1)).abs() <= bound + 1e-30).all())


@pytest.mark.parametrize("T,R,sched", [(258, 2, 0), (258, 3, 1), (516, 2, 1), (516, 4, 1), (514, 1, 0)])
def test_combine_in_forward(T, R, sched):
    from paper_2605_00686_amd import binding as B
    print(f"case forward T={T} R={R} scheduler={sched}", flush=True)
    inp = W.make_inputs(dict(T=T, d=192, E=8, k=3, f=64, R=R, dtype="bf16", seed=T + R))
    p = B.problem(T, 192, 8, 3, 64, R, "bf16", scheduler=sched)
    dev = {n: (inp[n].cuda() if inp[n] is not None else None) for n in ("x", "Wg", "gate_bias", "W1", "W3", "W2")}
    buf = B.Buffers(p)
    buf.out.fill_(float("nan"))
    B.forward(p, buf, dev["x"], dev["Wg"], dev["gate_bias"], dev["W1"], dev["W3"], dev["W2"])
    torch.cuda.synchronize()
    assert int(buf.stats[7].item()) == 0
    terms = buf.staging.cpu().double().reshape(T, 3, 192) * buf.topk_w.cpu().double()[:, :, None]
    bound = 3 * 2.0 ** -23 * terms.abs().sum(1) + 2.0 ** -8 * terms.sum(1).abs()  # as above
    assert bool(((buf.out.cpu().double() - terms.sum(1)).abs() <= bound + 1e-30).all())
