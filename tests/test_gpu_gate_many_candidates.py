"""GPU test of the screened gate where the screen orders little: equal logits (rows of zeros, as padded slots of a decode
step have, with and without biases that tie), logits closer together than the screen's error bound, 32 choices a token.
Tasks of 4, 8 and 16 tokens (up to 256, 128 and 64 candidates a token; past that the exact fallback), standalone (several
sweeps over the reduction) and inside the megakernel, against the oracle."""
import numpy as np
import pytest
import torch

from paper_2605_00686_amd import workloads as W
from tests import gate_forms, parity

pytestmark = pytest.mark.gpu


def make(T, d, E, k, kind):
    inp = W.make_inputs(dict(T=T, d=d, E=E, k=k, f=64, R=1, dtype="bf16", seed=T + E + k, bias_std=0.0))
    if kind == "zero_rows":  # every logit equal: the lowest expert ids
        inp["x"][T // 2] = 0
        inp["x"][T - 1] = 0
    elif kind == "all_zero":
        inp["x"][:] = 0
    elif kind == "tied_bias":  # zeros of either sign, equal biases, masked experts
        inp["x"][::3] = 0
        values = torch.tensor([0.0, -0.0, 0.5, -0.5, float("-inf"), 0.25])
        inp["gate_bias"] = values[torch.randint(0, 6, (E,), generator=torch.Generator().manual_seed(E))]
    elif kind == "tiny":  # products below the range of fp32: no magnitude, yet no row of zeros
        inp["x"][T // 3:] = 0
        inp["x"][T // 3:, d - 1] = 2.0 ** -133
    elif kind == "near":  # columns of Wg that differ in one element by one unit in the last place of 16: far below the bound
        w = inp["Wg"]
        w[:] = 0.5
        w[d // 2, ::3] = 0.5 + 2.0 ** -8
        inp["x"][T // 3:, d // 2] *= -1
    return inp


# (T, d, E, k, kind); d past what the standalone gate takes on exact logits of all experts
CASES = [(9, 128, 128, 8, "zero_rows"), (9, 192, 256, 8, "all_zero"), (130, 1024, 80, 6, "zero_rows"),
         (130, 128, 200, 8, "all_zero"), (8, 2048, 128, 8, "near"), (37, 128, 255, 5, "near"), (12, 320, 33, 6, "zero_rows"),
         (1030, 192, 128, 8, "all_zero"), (1030, 192, 129, 4, "zero_rows"), (1030, 256, 256, 32, "near"), (1030, 192, 200, 32, ""),
         (2050, 576, 40, 32, ""), (2050, 256, 65, 32, ""), (2050, 256, 256, 32, ""), (2050, 320, 64, 8, "zero_rows"),
         (2050, 256, 80, 8, "zero_rows"), (2050, 832, 17, 3, "all_zero"), (2050, 576, 48, 4, "near"),
         (9, 192, 64, 8, "tied_bias"), (130, 192, 129, 8, "tied_bias"), (1030, 7168, 24, 4, "tied_bias"), (2050, 256, 200, 8, "tied_bias"),
         (9, 1088, 48, 4, "tiny"), (2050, 576, 48, 4, "tiny"), (2050, 256, 256, 8, "tiny"),
         # tasks of 4 tokens with aligned rows of Wg (in the layer), every code variant
         (600, 4096, 24, 4, "tiny"), (600, 2112, 32, 4, "zero_rows"), (520, 1088, 64, 8, "all_zero"), (600, 576, 128, 8, "near"),
         (600, 448, 192, 8, "tied_bias"), (520, 320, 256, 32, ""), (520, 320, 256, 5, "near")]


@pytest.mark.parametrize("T,d,E,k,kind", CASES, ids=["T%d_d%d_E%d_k%d_%s" % c for c in CASES])
def test_many_candidates(T, d, E, k, kind):
    from paper_2605_00686_amd import binding as B
    print(f"case many candidates T={T} d={d} E={E} k={k} {kind}", flush=True)
    inp = make(T, d, E, k, kind)
    p = B.problem(T, d, E, k, 64, 1, "bf16")
    dev = {n: inp[n].cuda() for n in ("x", "Wg", "W1", "W3", "W2")}
    bias = None if inp["gate_bias"] is None else inp["gate_bias"].cuda()
    ridx, rw, _ = parity.oracle_routing(inp)
    idx = torch.full((T, k), -1, dtype=torch.int32, device="cuda")
    w = torch.full((T, k), float("nan"), dtype=torch.float32, device="cuda")
    B.moe_route(p, dev["x"], dev["Wg"], bias, idx, w)
    buf = B.Buffers(p)
    B.forward(p, buf, dev["x"], dev["Wg"], bias, dev["W1"], dev["W3"], dev["W2"])
    torch.cuda.synchronize()
    assert int(buf.stats[7].item()) == 0
    for i2, w2 in ((idx, w), (buf.topk_idx, buf.topk_w)):
        assert np.array_equal(i2.cpu().numpy(), ridx)
        # fp64 logits and softmax on both sides, rounded once: one unit in the last place of fp32 and a little
        np.testing.assert_allclose(w2.cpu().numpy(), rw, rtol=1.5e-7, atol=0)
    assert np.array_equal(buf.counts.cpu().numpy(), np.bincount(ridx.reshape(-1), minlength=E))


@pytest.mark.parametrize("T", [8, 128, 600])
def test_padded_slots_of_a_batch_keep_its_form(T):
    """Rows of zeros in a batch: the gate phase of the layer takes at most twice as long as without them.  8 and 128 tokens take the
    direct gate, 600 the screen with tasks of 4 tokens, whose exact fallback (taken here with a row that is no number in every
    task) is outside that bound."""
    from paper_2605_00686_amd import binding as B
    print(f"case padded slots T={T}", flush=True)
    assert (gate_forms.form(T, 128, 2048, False) == "direct") == (T <= 128)
    inp = W.make_inputs(dict(T=T, d=2048, E=128, k=8, f=64, R=1, dtype="bf16", seed=T, bias_std=0.0, tile_m=32))
    p = B.problem(T, 2048, 128, 8, 64, 1, "bf16", tile_m=32)
    buf = B.Buffers(p)
    dev = {n: inp[n].cuda() for n in ("x", "Wg", "W1", "W3", "W2")}
    gate_us = []
    for rows in ("full", "zeros", "nan"):
        x = dev["x"].clone()
        if rows == "zeros":
            x[T - 1] = 0
            x[3::4] = 0 if T > 128 else x[3::4]
        elif rows == "nan":
            x[3::4, 0] = float("nan")
        seen = []
        for _ in range(12):
            p.epoch += 1
            B.forward(p, buf, x, dev["Wg"], None, dev["W1"], dev["W3"], dev["W2"])
            torch.cuda.synchronize()
            seen.append(int(buf.stats[8].item()) / 1000)
            assert rows == "nan" or int(buf.stats[7].item()) == 0
        gate_us.append(sorted(seen)[len(seen) // 2])
    print(f"gate phase {gate_us[0]:.1f} us, with rows of zeros {gate_us[1]:.1f} us, with rows that are no numbers {gate_us[2]:.1f} us", flush=True)
    assert gate_us[1] <= 2 * gate_us[0]
    if T == 600:
        assert gate_us[2] > 2 * gate_us[0]
