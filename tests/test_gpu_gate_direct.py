"""GPU test of the gate of few tokens (exact logits of all experts, a task per CU) at the edges of its forms: 1, 2 and 4 tokens per
task, experts in parts and whole, both selections, k up to 32, reductions of fewer groups of rows than threads and of uneven
batches, views of x and Wg between 16-byte boundaries; and against the other forms of the gate on the same tokens."""
import numpy as np
import pytest
import torch

from paper_2605_00686_amd import workloads as W
from tests import gate_forms, parity

pytestmark = pytest.mark.gpu


def route(B, T, d, E, k, x, Wg, bias):
    p = B.problem(T, d, E, k, 64, 1, "bf16")
    idx = torch.full((T, k), -1, dtype=torch.int32, device="cuda")
    w = torch.full((T, k), float("nan"), dtype=torch.float32, device="cuda")
    B.moe_route(p, x, Wg, bias, idx, w)
    torch.cuda.synchronize()
    return idx.cpu(), w.cpu()


CASES = [(1, 64, 8, 8), (3, 2048, 128, 8), (8, 2112, 256, 32), (64, 4096, 64, 6), (127, 2048, 144, 8), (128, 1088, 240, 5), (129, 2048, 128, 8),
         (256, 64, 72, 32), (257, 320, 56, 1), (511, 7168, 16, 4), (512, 576, 136, 8), (513, 640, 24, 7), (1023, 128, 256, 8), (1024, 1024, 48, 6),
         (80, 2048, 128, 8), (48, 2048, 136, 8), (85, 2048, 128, 32), (100, 4096, 72, 8)]  # (parts of different size)


@pytest.mark.parametrize("T,d,E,k", CASES, ids=["T%d_d%d_E%d_k%d" % c for c in CASES])
def test_direct_gate(T, d, E, k):
    from paper_2605_00686_amd import binding as B
    print(f"case direct gate T={T} d={d} E={E} k={k}", flush=True)
    assert gate_forms.is_direct(T, E, d, True) and gate_forms.is_direct(T, E, d, False) == (T <= 512 or E * d <= 1 << 16)
    inp = W.make_inputs(dict(T=T, d=d, E=E, k=k, f=64, R=1, dtype="bf16", seed=T + d + E, bias_std=0.3))
    inp["x"][T // 2] = 0  # a padded slot: its logits are the biases ...
    inp["gate_bias"][:] = inp["gate_bias"].round(decimals=1)  # ... among which there are ties
    ridx, rw, _ = parity.oracle_routing(inp)
    dev = {n: inp[n].cuda() for n in ("x", "Wg", "gate_bias", "W1", "W3", "W2")}
    got = [route(B, T, d, E, k, dev["x"], dev["Wg"], dev["gate_bias"])]
    room = torch.full((T * d + d * E + 64,), float("nan"), dtype=torch.bfloat16, device="cuda")
    xv, wv = room[3:3 + T * d].reshape(T, d), room[T * d + 8 + 5:T * d + 8 + 5 + d * E].reshape(d, E)
    xv.copy_(dev["x"])
    wv.copy_(dev["Wg"])
    got.append(route(B, T, d, E, k, xv, wv, dev["gate_bias"]))
    p = B.problem(T, d, E, k, 64, 1, "bf16")
    buf = B.Buffers(p)
    for epoch in (1, 2):  # (twice: the parts' counters are zero again)
        p.epoch = epoch
        buf.topk_idx.fill_(-1)
        B.forward(p, buf, dev["x"], dev["Wg"], dev["gate_bias"], dev["W1"], dev["W3"], dev["W2"])
        torch.cuda.synchronize()
        assert int(buf.stats[7].item()) == 0
        got.append((buf.topk_idx.cpu(), buf.topk_w.cpu()))
    for idx, w in got:
        assert np.array_equal(idx.numpy(), ridx)
        # fp64 sums in another order, rounded once: one unit in the last place of fp32 and a little
        np.testing.assert_allclose(w.numpy(), rw, rtol=1.5e-7, atol=0)


@pytest.mark.parametrize("d,E,k", [(256, 128, 8), (1024, 48, 6), (512, 8, 2), (320, 256, 4)])
def test_direct_gate_is_the_same_as_the_others(d, E, k):
    """The first tokens of a batch that is large enough for the screen or the exact form, and the same tokens alone."""
    from paper_2605_00686_amd import binding as B
    T = 2304
    print(f"case direct and other gates d={d} E={E} k={k}", flush=True)
    inp = W.make_inputs(dict(T=T, d=d, E=E, k=k, f=64, R=1, dtype="bf16", seed=d + E, bias_std=0.3), with_weights=False)
    x, Wg, bias = (inp[n].cuda() for n in ("x", "Wg", "gate_bias"))
    idx, w = route(B, T, d, E, k, x, Wg, bias)
    for n in (1, 100, 256, 512, 1000):
        i2, w2 = route(B, n, d, E, k, x[:n], Wg, bias)
        assert torch.equal(i2, idx[:n])
        np.testing.assert_allclose(w2.numpy(), w[:n].numpy(), rtol=1.5e-7, atol=0)


@pytest.mark.parametrize("T,d,E,k", [(80, 2048, 128, 8), (48, 2048, 136, 6), (100, 4096, 72, 8)])
def test_equal_columns_tie_across_parts(T, d, E, k):
    """Experts with the same gate weights have the same logit, whichever part of a task each lies in: the lower id comes first,
    alone and in the layer.  Entries of x and Wg are spread over so many orders of magnitude that a sum depends on the order of
    its terms, and the parts of a task are of different sizes."""
    from paper_2605_00686_amd import binding as B
    print(f"case equal columns T={T} d={d} E={E} k={k}", flush=True)
    pieces = gate_forms.part_pieces(E, gate_forms.direct_parts(T, E, d))
    assert gate_forms.is_direct(T, E, d, False) and min(pieces) != max(pieces)
    inp = W.make_inputs(dict(T=T, d=d, E=E, k=k, f=64, R=1, dtype="bf16", seed=T + E))
    gen = torch.Generator().manual_seed(T)
    for n in ("x", "Wg"):
        inp[n] = (inp[n].double() * torch.exp2(torch.randint(-12, 13, inp[n].shape, generator=gen).double())).bfloat16()
    inp["Wg"] = inp["Wg"][:, torch.randperm(E, generator=gen) % (E // 4)].contiguous()  # every column four times
    ridx, rw, _ = parity.oracle_routing(inp)
    assert (np.diff(ridx[:, :4], axis=1) > 0).all()  # (the first four choices are the same column)
    dev = {n: inp[n].cuda() for n in ("x", "Wg", "W1", "W3", "W2")}
    got = [route(B, T, d, E, k, dev["x"], dev["Wg"], None)]
    p = B.problem(T, d, E, k, 64, 1, "bf16")
    buf = B.Buffers(p)
    B.forward(p, buf, dev["x"], dev["Wg"], None, dev["W1"], dev["W3"], dev["W2"])
    torch.cuda.synchronize()
    assert int(buf.stats[7].item()) == 0
    got.append((buf.topk_idx.cpu(), buf.topk_w.cpu()))
    for idx, w in got:
        assert np.array_equal(idx.numpy(), ridx)
        # (1/4 each, and nothing for the others, whose logits are smaller by hundreds)
        np.testing.assert_allclose(w.numpy(), rw, rtol=1.5e-7, atol=0)
