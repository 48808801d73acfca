"""GPU test of the gate's code variants at the edges of their ranges: numbers of experts around the multiples at which
another variant takes over (and odd ones, whose weight rows are unaligned), reductions of one chunk and of many, tokens
per task of 4, 8 and 16 with a remainder; standalone and inside the megakernel, against the oracle."""
import numpy as np
import pytest
import torch

from paper_2605_00686_amd import workloads as W
from tests import gate_forms, parity

pytestmark = pytest.mark.gpu

# (T, d, E, k)
CASES = [(5, 64, 1, 1), (37, 128, 7, 3), (1030, 192, 16, 2), (16, 256, 17, 2), (2050, 128, 32, 4), (65, 320, 33, 6),
         (1025, 128, 64, 8), (40, 2880, 65, 4), (4100, 64, 128, 8), (33, 192, 129, 8), (130, 128, 192, 8), (70, 256, 200, 8),
         (2049, 64, 255, 5), (64, 1024, 256, 8),
         (2050, 1088, 16, 2), (2049, 64, 17, 3), (40, 1088, 16, 2), (40, 1024, 15, 2), (9, 1088, 3, 1),
         # both sides of the standalone gate's rule for short reductions, at 4, 8 and 16 tokens per task
         (130, 320, 24, 4), (65, 384, 32, 6), (70, 192, 48, 4), (130, 256, 33, 8), (9, 64, 96, 8), (70, 128, 64, 8), (1030, 448, 20, 2),
         (1025, 512, 32, 4), (1025, 256, 47, 4), (1025, 192, 64, 8), (1030, 128, 200, 4), (2049, 640, 17, 3), (2050, 704, 32, 4),
         (2049, 384, 47, 4), (2050, 448, 48, 6), (2049, 192, 64, 8), (2050, 256, 64, 8), (4100, 128, 128, 8), (4100, 192, 128, 8),
         (2049, 192, 255, 5), (2050, 2048, 8, 2), (2049, 2112, 16, 2), (2049, 1024, 12, 2), (2049, 1088, 15, 2),
         # both sides of the rules for the direct gate of few tokens; past them the layer screens with tasks of 4 tokens and aligned rows of Wg
         (512, 4096, 128, 8), (513, 512, 128, 8), (513, 576, 128, 8), (1024, 1024, 64, 8), (1024, 1088, 64, 8), (1025, 1024, 64, 8),
         (256, 4096, 256, 8), (257, 2048, 256, 8), (257, 2112, 256, 8), (600, 4096, 24, 4), (600, 2112, 32, 4), (600, 448, 192, 8)]


@pytest.mark.parametrize("T,d,E,k", CASES, ids=["T%d_d%d_E%d_k%d" % c for c in CASES])
def test_gate_variants(T, d, E, k):
    from paper_2605_00686_amd import binding as B
    print(f"case gate T={T} d={d} E={E} k={k}", flush=True)
    inp = W.make_inputs(dict(T=T, d=d, E=E, k=k, f=64, R=1, dtype="bf16", seed=T + E, bias_std=0.3))
    cfg = inp["cfg"]
    p = B.problem(T, d, E, k, 64, 1, "bf16", tile_m=cfg["tile_m"], tile_n=cfg["tile_n"])
    dev = {n: inp[n].cuda() for n in ("x", "Wg", "gate_bias", "W1", "W3", "W2")}
    ridx, rw, margin = parity.oracle_routing(inp)
    idx = torch.full((T, k), -1, dtype=torch.int32, device="cuda")
    w = torch.full((T, k), float("nan"), dtype=torch.float32, device="cuda")
    B.moe_route(p, dev["x"], dev["Wg"], dev["gate_bias"], idx, w)
    buf = B.Buffers(p)
    B.forward(p, buf, dev["x"], dev["Wg"], dev["gate_bias"], dev["W1"], dev["W3"], dev["W2"])
    torch.cuda.synchronize()
    assert int(buf.stats[7].item()) == 0
    # logits and softmax are fp64 on both sides and rounded once: one unit in the last place of fp32 (2^-23) and a little
    for i2, w2 in ((idx, w), (buf.topk_idx, buf.topk_w)):
        assert np.array_equal(i2.cpu().numpy(), ridx), f"min margin {margin.min()}"
        np.testing.assert_allclose(w2.cpu().numpy(), rw, rtol=1.5e-7, atol=0)
    assert np.array_equal(buf.counts.cpu().numpy(), np.bincount(ridx.reshape(-1), minlength=E))


@pytest.mark.parametrize("which", ["x", "Wg"])
@pytest.mark.parametrize("T,d,E,k", [(21, 1152, 16, 2), (70, 64, 128, 8), (33, 192, 129, 8)],
                         ids=lambda v: str(v))
def test_gate_of_views_off_16_bytes(T, d, E, k, which):
    """Contiguous views that start between 16-byte boundaries: the same choices as with the aligned tensors."""
    from paper_2605_00686_amd import binding as B
    print(f"case gate view T={T} d={d} E={E} k={k} {which}", flush=True)
    inp = W.make_inputs(dict(T=T, d=d, E=E, k=k, f=64, R=1, dtype="bf16", seed=T + E, bias_std=0.3))
    p = B.problem(T, d, E, k, 64, 1, "bf16")
    dev = {n: inp[n].cuda() for n in ("x", "Wg", "gate_bias", "W1", "W3", "W2")}
    room = torch.zeros(dev[which].numel() + 16, dtype=torch.bfloat16, device="cuda")
    view = room[1:1 + dev[which].numel()].reshape(dev[which].shape)
    view.copy_(dev[which])
    assert view.data_ptr() % 16 != 0
    off = {**dev, which: view}
    out = []
    for t in (dev, off):
        idx = torch.full((T, k), -1, dtype=torch.int32, device="cuda")
        w = torch.full((T, k), float("nan"), dtype=torch.float32, device="cuda")
        B.moe_route(p, t["x"], t["Wg"], t["gate_bias"], idx, w)
        out.append((idx.cpu(), w.cpu()))
    if which == "Wg":  # (the experts' products ask for aligned rows of x)
        buf = B.Buffers(p)
        B.forward(p, buf, dev["x"], view, dev["gate_bias"], dev["W1"], dev["W3"], dev["W2"])
        torch.cuda.synchronize()
        assert int(buf.stats[7].item()) == 0
        out.append((buf.topk_idx.cpu(), buf.topk_w.cpu()))
    for idx, w in out[1:]:
        assert torch.equal(idx, out[0][0])
        # fp64 sums in another order, rounded once: one unit in the last place of fp32 and a little
        np.testing.assert_allclose(w.numpy(), out[0][1].numpy(), rtol=1.5e-7, atol=0)


# (tests/test_gate_forms.py checks which forms of the gate these are)
UNALIGNED_CASES = [(9, 1152, 8, 2), (1030, 256, 64, 8), (2050, 576, 48, 6), (40, 1024, 256, 8), (130, 128, 72, 4),
                   (600, 4096, 24, 4), (600, 2112, 32, 4), (520, 1088, 64, 8), (600, 576, 128, 8), (600, 448, 192, 8), (520, 320, 256, 5),
                   (1030, 192, 128, 8)]


@pytest.mark.parametrize("offset", [1, 4, 7])
@pytest.mark.parametrize("T,d,E,k", UNALIGNED_CASES, ids=lambda v: str(v))
def test_unaligned_view_of_the_gate_weights(T, d, E, k, offset):
    """Wg as a view that starts `offset` elements past a 16-byte boundary, inside a tensor whose neighbours are no numbers:
    the oracle's choices, standalone and in the layer, in every code variant of the screen that takes whole pieces otherwise and
    in the direct gate."""
    from paper_2605_00686_amd import binding as B
    print(f"case gate weights off T={T} d={d} E={E} k={k} offset={offset}", flush=True)
    inp = W.make_inputs(dict(T=T, d=d, E=E, k=k, f=64, R=1, dtype="bf16", seed=T + E + offset, bias_std=0.3))
    p = B.problem(T, d, E, k, 64, 1, "bf16")
    dev = {n: inp[n].cuda() for n in ("x", "gate_bias", "W1", "W3", "W2")}
    room = torch.full((d * E + 16,), float("nan"), dtype=torch.bfloat16, device="cuda")
    view = room[offset:offset + d * E].reshape(d, E)
    view.copy_(inp["Wg"])
    ridx, rw, _ = parity.oracle_routing(inp)
    idx = torch.full((T, k), -1, dtype=torch.int32, device="cuda")
    w = torch.full((T, k), float("nan"), dtype=torch.float32, device="cuda")
    B.moe_route(p, dev["x"], view, dev["gate_bias"], idx, w)
    buf = B.Buffers(p)
    B.forward(p, buf, dev["x"], view, dev["gate_bias"], dev["W1"], dev["W3"], dev["W2"])
    torch.cuda.synchronize()
    assert int(buf.stats[7].item()) == 0
    for i2, w2 in ((idx, w), (buf.topk_idx, buf.topk_w)):
        assert np.array_equal(i2.cpu().numpy(), ridx)
        np.testing.assert_allclose(w2.cpu().numpy(), rw, rtol=1.5e-7, atol=0)  # (as above)


@pytest.mark.parametrize("T", [8, 600], ids=["direct", "screen"])
def test_unaligned_view_of_the_gate_weights_keeps_its_form(T):
    """The gate phase of the layer takes at most twice as long on such a view as on aligned weights, of a decode batch (the direct
    gate) and of 600 tokens (the screen, whose exact fallback, taken here with a row that is no number in every task, is outside
    that bound)."""
    from paper_2605_00686_amd import binding as B
    print(f"case gate weights off, time T={T}", flush=True)
    assert (gate_forms.form(T, 128, 2048, False) == "direct") == (T == 8)
    inp = W.make_inputs(dict(T=T, d=2048, E=128, k=8, f=64, R=1, dtype="bf16", seed=3, bias_std=0.3, tile_m=32))
    p = B.problem(T, 2048, 128, 8, 64, 1, "bf16", tile_m=32)
    buf = B.Buffers(p)
    dev = {n: inp[n].cuda() for n in ("x", "Wg", "gate_bias", "W1", "W3", "W2")}
    room = torch.zeros(dev["Wg"].numel() + 16, dtype=torch.bfloat16, device="cuda")
    view = room[1:1 + dev["Wg"].numel()].reshape(dev["Wg"].shape)
    view.copy_(dev["Wg"])
    spoiled = dev["x"].clone()
    spoiled[::4, 0] = float("nan")
    gate_us = []
    for x, wg in ((dev["x"], dev["Wg"]), (dev["x"], view), (spoiled, dev["Wg"])):
        seen = []
        for _ in range(12):
            p.epoch += 1
            B.forward(p, buf, x, wg, dev["gate_bias"], dev["W1"], dev["W3"], dev["W2"])
            torch.cuda.synchronize()
            seen.append(int(buf.stats[8].item()) / 1000)
        gate_us.append(sorted(seen)[len(seen) // 2])
    print(f"gate phase {gate_us[0]:.1f} us, on a view off 16 bytes {gate_us[1]:.1f} us, through the fallback {gate_us[2]:.1f} us", flush=True)
    assert gate_us[1] <= 2 * gate_us[0]
    if T == 600:
        assert gate_us[2] > 2 * gate_us[0]


def test_gate_weights_past_32_bits():
    """Gate weights of more than 4 GB whose rows are unaligned: x has a few entries per token, at both ends and on either side
    of the 2^32nd byte, so the logits are known from those rows of Wg alone."""
    from paper_2605_00686_amd import binding as B
    E, k, T = 255, 4, 3
    d = 8421568  # 64 * 131587; d * E * 2 bytes is just past 2^32
    assert d % 64 == 0 and d * E * 2 > 2 ** 32
    print(f"case gate weights past 32 bits d={d} E={E}", flush=True)
    gen = torch.Generator().manual_seed(1)
    at = [0, 77, d // 2 + 1, 2 ** 32 // (2 * E) - 3, 2 ** 32 // (2 * E) + 5, d - 1]
    rows = torch.randn(len(at), E, generator=gen).bfloat16()
    vals = torch.randn(T, len(at), generator=gen).bfloat16()
    x = torch.zeros(T, d, dtype=torch.bfloat16, device="cuda")
    Wg = torch.zeros(d, E, dtype=torch.bfloat16, device="cuda")
    for i, r in enumerate(at):
        x[:, r] = vals[:, i].cuda()
        Wg[r] = rows[i].cuda()
    logits = (vals.double() @ rows.double()).numpy()
    order = np.argsort(-logits, axis=1, kind="stable")[:, :k]
    chosen = np.take_along_axis(logits, order, axis=1)
    soft = np.exp(chosen - chosen[:, :1])
    soft /= soft.sum(axis=1, keepdims=True)
    p = B.problem(T, d, E, k, 64, 1, "bf16")
    idx = torch.full((T, k), -1, dtype=torch.int32, device="cuda")
    w = torch.full((T, k), float("nan"), dtype=torch.float32, device="cuda")
    B.moe_route(p, x, Wg, None, idx, w)
    torch.cuda.synchronize()
    assert np.array_equal(idx.cpu().numpy(), order)
    np.testing.assert_allclose(w.cpu().numpy(), soft, rtol=1.5e-7, atol=0)
