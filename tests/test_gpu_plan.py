"""GPU test of the plan inside the megakernel on both sides of the rules that choose between its three forms (every workgroup
derives it in LDS, from the choices or from block histograms; one workgroup writes it to memory): destinations x experts, token blocks x experts and the decode tables at
and just past the limits, destinations that are and are not whole token blocks, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_00686_amd import workloads as W
from tests import parity

pytestmark = pytest.mark.gpu

# (T, E, R, k, tile_m, capacity)
CASES = [(192, 64, 64, 2, 32, 0), (195, 64, 65, 2, 32, 0), (4096, 256, 4, 2, 128, 0), (4100, 256, 4, 2, 128, 0),
         (640, 3, 10, 2, 64, 0), (640, 3, 10, 2, 64, 512), (77, 5, 7, 3, 128, 77),
         (8192, 128, 4, 2, 128, 0), (8196, 128, 4, 2, 128, 0), (47, 255, 1, 2, 32, 0), (48, 255, 1, 2, 32, 0),
         # 64-row blocks have fewer decode tables than 32-row ones (48 tokens above); both sides of the slots counted as choices
         (4096, 252, 4, 2, 32, 0), (4096, 16, 8, 2, 128, 0), (4098, 16, 6, 2, 128, 0), (4160, 8, 10, 3, 128, 4160), (4160, 8, 64, 3, 64, 4100),
         (4104, 6, 12, 2, 32, 0)]
# how each derives the plan: every workgroup from the choices, every workgroup from block histograms, one workgroup
FORMS = ["choices", "one", "one", "one", "choices", "choices", "choices", "histograms", "one", "choices", "one",
         "one", "choices", "histograms", "histograms", "histograms", "histograms"]


def plan_form(T, E, R, k, tile_m):
    """The rule of the launch: at most 32 KB of segment tables (8 * E * R), 64 KB of histograms (4 * E * ceil(T / 64)) and 6 KB of
    decode tables (4 * (6 * E + 4 + row blocks); with a 32-row publish tile row blocks of 32 rows below 32 rows per expert and of 64
    below 96, else of 256) for a plan in every workgroup, from the choices up to 8192 of them."""
    avg = T * k // E
    bm = 256 if avg >= 96 or tile_m > 32 else 64 if avg >= 32 else 32
    if 8 * E * R > 32768 or 4 * E * -(-T // 64) > 65536 or 4 * (6 * E + 4 + T * k // bm) > 6144:
        return "one"
    return "choices" if T * k <= 8192 else "histograms"


def test_cases_reach_every_form():
    assert [plan_form(*c[:5]) for c in CASES] == FORMS
    assert plan_form(192, 64, 64, 2, 32) == "choices" and plan_form(195, 64, 65, 2, 32) == "one" and plan_form(4160, 8, 10, 3, 32) == "histograms"


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


@pytest.mark.parametrize("T,E,R,k", [(192, 64, 64, 2), (4160, 8, 10, 3), (195, 64, 65, 2)], ids=["choices", "histograms", "one"])
@pytest.mark.parametrize("padded", [False, True], ids=["ragged", "padded"])
def test_plan_reports_slots_that_no_expert_counts(T, E, R, k, padded):
    """An id outside [0, E) among routing that is an input, every form of the plan and either layout: reported, nothing else
    written (perm keeps its poison), and the workspace is good for the next call.  Padded: so is an expert over its capacity."""
    from paper_2605_00686_amd import binding as B
    capacity = T * k // E + 100 if padded else 0
    print(f"case plan bad id T={T} E={E} R={R} k={k} capacity={capacity}", flush=True)
    inp = W.make_inputs(dict(T=T, d=64, E=E, k=k, f=64, R=R, dtype="bf16", seed=5, tile_m=32))
    p = B.problem(T, 64, E, k, 64, R, "bf16", tile_m=32, capacity=capacity)
    buf = B.Buffers(p)
    good = (torch.arange(T)[:, None] + torch.arange(k)[None, :] * 3) % E
    dev = {n: inp[n].cuda() for n in ("x", "W1", "W3", "W2")}
    buf.topk_w.fill_(0.5)
    buf.perm.fill_(-7)
    for bad_id in (E, -1, 1 << 20):
        ids = good.clone()
        ids[T // 2, 1] = bad_id
        buf.topk_idx.copy_(ids)
        B.forward(p, buf, dev["x"], None, None, dev["W1"], dev["W3"], dev["W2"])
        torch.cuda.synchronize()
        assert int(buf.stats[7].item()) == B.MOE_ERR_BAD_ROUTING
        assert bool((buf.perm == -7).all().item())
    if padded:
        full = good.clone()
        full[:capacity + 1, 0] = 0  # too many rows for expert 0
        for j in range(1, k):  # (the ids of a token stay distinct)
            full[:capacity + 1, j] = 1 + (torch.arange(capacity + 1) + j) % (E - 1)
        buf.topk_idx.copy_(full)
        B.forward(p, buf, dev["x"], None, None, dev["W1"], dev["W3"], dev["W2"])
        torch.cuda.synchronize()
        assert int(buf.stats[7].item()) == B.MOE_ERR_CAPACITY
        assert bool((buf.perm == -7).all().item())
        assert np.array_equal(buf.counts.cpu().numpy(), np.bincount(full.numpy().reshape(-1), minlength=E))
    buf.topk_idx.copy_(good)
    p.epoch = 2
    B.forward(p, buf, dev["x"], None, None, dev["W1"], dev["W3"], dev["W2"])
    torch.cuda.synchronize()
    assert int(buf.stats[7].item()) == 0
    counts, offsets, perm, inv = oracle.dispatch(good.to(torch.int32).numpy(), E, capacity)
    assert np.array_equal(buf.counts.cpu().numpy(), counts) and np.array_equal(buf.perm.cpu().numpy(), perm)
    assert np.array_equal(buf.offsets.cpu().numpy(), offsets) and np.array_equal(buf.inv_perm.cpu().numpy(), inv)
