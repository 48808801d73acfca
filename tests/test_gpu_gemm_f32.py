"""GPU test of the fp32 tile GEMM inside the whole layer, against the oracle: every number of 32-row blocks a tile can have and
the row counts next to them, reductions shorter than one piece per wavefront, ragged and narrow column tiles, both column
widths of GEMM1, more than one row block per expert."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_00686_amd import workloads as W
from tests import parity

pytestmark = pytest.mark.gpu

# (T, d, E, k, f): with one expert a tile's rows are T; f / 64 x row blocks < 256 takes 32-column GEMM1 tiles
CASES = ([(T, 80, 1, 1, 48) for T in (1, 31, 32, 33, 64, 65, 96, 97, 128, 129)]
         + [(T, 64, 1, 1, 16384) for T in (1, 33, 65, 97)]
         + [(5, 16, 2, 2, 16), (40, 16, 3, 2, 32), (70, 112, 4, 3, 16), (300, 192, 2, 2, 272), (257, 1024, 1, 1, 8192 + 16)])


@pytest.mark.parametrize("T,d,E,k,f", CASES, ids=["T%d_d%d_E%d_k%d_f%d" % c for c in CASES])
def test_fp32_tiles(T, d, E, k, f):
    from paper_2605_00686_amd import binding as B
    print(f"case gemm_f32 T={T} d={d} E={E} k={k} f={f}", flush=True)
    inp = W.make_inputs(dict(T=T, d=d, E=E, k=k, f=f, R=1, dtype="f32", seed=T + d))
    p = B.problem(T, d, E, k, f, 1, "f32")
    dev = {n: inp[n].cuda() for n in ("x", "Wg", "W1", "W3", "W2")}
    buf = B.Buffers(p)
    B.forward(p, buf, dev["x"], dev["Wg"], None, dev["W1"], dev["W3"], dev["W2"])
    torch.cuda.synchronize()
    assert int(buf.stats[7].item()) == 0
    o = parity.oracle_arrays(inp)
    ref = oracle.forward(o["x"], o["Wg"], o["W1"], o["W3"], o["W2"], k)
    assert np.array_equal(buf.perm.cpu().numpy(), ref["perm"])
    # fp32 sums of n terms: at most n * 2^-24 of the sum of magnitudes, in practice its square root; n <= 16384 here
    for name in ("staging", "out"):
        got = getattr(buf, name).cpu().numpy()
        assert np.isfinite(got).all()
        err = parity.row_err(got, ref[name]).max()
        print(f"  {name}: row-normalised error {err:.2e}", flush=True)
        assert err <= 2e-5, name
