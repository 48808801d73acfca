"""GPU test of the standalone gate of few tokens where its tasks have 512 threads, and where the partial sums of a logit are added up in
two steps: 1, 2 and 4 tokens per task, few experts (many partial sums) to many, numbers of experts that do not divide the threads,
weights just on either side of the 512 threads' limit, against the oracle; equal experts tie wherever they lie."""
import numpy as np
import pytest
import torch

from paper_2605_00686_amd import workloads as W
from tests import gate_forms, parity

pytestmark = pytest.mark.gpu

CASES = [(5, 16384, 16, 4), (300, 8192, 24, 8), (520, 6144, 32, 8), (1024, 1024, 136, 8), (1, 1024, 136, 3), (7, 2048, 64, 8), (7, 2112, 64, 8),
         (513, 2048, 64, 6), (257, 8192, 8, 2), (600, 64, 8, 8), (1000, 512, 16, 5), (33, 128, 248, 32),
         (600, 4096, 40, 4)]


@pytest.mark.parametrize("T,d,E,k", CASES, ids=["T%d_d%d_E%d_k%d" % c for c in CASES])
def test_direct_gate_alone(T, d, E, k):
    from paper_2605_00686_amd import binding as B
    print(f"case direct gate alone T={T} d={d} E={E} k={k}", flush=True)
    assert gate_forms.is_direct(T, E, d, True)
    inp = W.make_inputs(dict(T=T, d=d, E=E, k=k, f=64, R=1, dtype="bf16", seed=T + d + E, bias_std=0.3), with_weights=False)
    inp["Wg"][:, E - 1] = inp["Wg"][:, 0]  # two equal experts: the lower one comes first
    inp["gate_bias"][E - 1] = inp["gate_bias"][0]
    ridx, rw, _ = parity.oracle_routing(inp)
    x, Wg, bias = (inp[n].cuda() for n in ("x", "Wg", "gate_bias"))
    p = B.problem(T, d, E, k, 64, 1, "bf16")
    idx = torch.full((T, k), -1, dtype=torch.int32, device="cuda")
    w = torch.full((T, k), float("nan"), dtype=torch.float32, device="cuda")
    for _ in range(2):
        B.moe_route(p, x, Wg, bias, idx, w)
        torch.cuda.synchronize()
        assert np.array_equal(idx.cpu().numpy(), ridx)
        # fp64 sums in another order, rounded once: one unit in the last place of fp32 and a little
        np.testing.assert_allclose(w.cpu().numpy(), rw, rtol=1.5e-7, atol=0)
