"""GPU test of the gate on logits that are not finite: a token row or a gate column with a NaN, an infinity in a token row,
experts masked by a gate bias of -inf, more of them than leave k.  The selection is by rank: position j is the lowest expert
that exactly j logits beat (larger, or equal and lower id), or -1 where there is none.  Inside the layer a -1 is reported
as invalid routing."""
import numpy as np
import pytest
import torch

from paper_2605_00686_amd import workloads as W

pytestmark = pytest.mark.gpu

NAN, INF = float("nan"), float("inf")


def by_rank(logits, k):
    T, E = logits.shape
    want = np.full((T, k), -1, np.int32)
    for t in range(T):
        v = logits[t]
        beats = (v[None, :] > v[:, None]) | ((v[None, :] == v[:, None]) & (np.arange(E)[None, :] < np.arange(E)[:, None]))
        rank = beats.sum(axis=1)
        for j in range(k):
            at = np.flatnonzero(rank == j)
            if at.size:
                want[t, j] = at[0]
    return want


def spoil(inp, kind, E, k):
    T = inp["x"].shape[0]
    if kind == "nan_row":
        inp["x"][T // 2, 7] = NAN
    elif kind == "nan_column":
        inp["Wg"][11, E - 1] = NAN
    elif kind == "inf_row":
        inp["x"][T - 1, 3] = INF
    elif kind == "inf_bias":
        inp["gate_bias"][E // 2] = INF
    elif kind == "nan_bias":
        inp["gate_bias"][0] = NAN
    elif kind == "masked_finite":  # every second expert, with the lowest finite number
        inp["gate_bias"][1::2] = torch.finfo(torch.float32).min
    elif kind == "masked":  # every second expert
        inp["gate_bias"][1::2] = -INF
    elif kind == "all_but_few":  # fewer than k are left
        inp["gate_bias"][max(1, k - 1):] = -INF


def check(B, cfg, kind):
    print(f"case not finite {kind} {cfg}", flush=True)
    cfg = dict(cfg, f=64, R=1, bias_std=0.3)
    T, d, E, k = (cfg[n] for n in ("T", "d", "E", "k"))
    inp = W.make_inputs(cfg)
    spoil(inp, kind, E, k)
    p = B.problem(T, d, E, k, 64, 1, cfg["dtype"])
    dev = {n: inp[n].cuda() for n in ("x", "Wg", "gate_bias", "W1", "W3", "W2")}
    with np.errstate(invalid="ignore"):
        logits = (inp["x"].double() @ inp["Wg"].double() + inp["gate_bias"].double()).numpy()
        want = by_rank(logits, k)
    idx = torch.full((T, k), -7, dtype=torch.int32, device="cuda")
    w = torch.full((T, k), -7.0, dtype=torch.float32, device="cuda")
    B.moe_route(p, dev["x"], dev["Wg"], dev["gate_bias"], idx, w)
    buf = B.Buffers(p)
    buf.topk_idx.fill_(-7)
    for t in (buf.perm, buf.inv_perm):
        t.fill_(0)
    B.forward(p, buf, dev["x"], dev["Wg"], dev["gate_bias"], dev["W1"], dev["W3"], dev["W2"])
    torch.cuda.synchronize()
    assert np.array_equal(idx.cpu().numpy(), want)
    assert np.array_equal(buf.topk_idx.cpu().numpy(), want)
    ok = np.isfinite(logits[np.arange(T)[:, None], want]).all(axis=1) & (want >= 0).all(axis=1)
    chosen = logits[np.arange(T)[:, None], want][ok]
    soft = np.exp(chosen - chosen.max(axis=1, keepdims=True))
    soft /= soft.sum(axis=1, keepdims=True)
    for got in (w, buf.topk_w):  # fp64 softmax rounded once: one unit in the last place of fp32 and a little
        np.testing.assert_allclose(got.cpu().numpy()[ok], soft, rtol=1.5e-7, atol=0)
    status = int(buf.stats[7].item())
    assert status == (B.MOE_ERR_BAD_ROUTING if (want < 0).any() else 0)
    if status == 0:
        assert np.array_equal(buf.counts.cpu().numpy(), np.bincount(want.reshape(-1), minlength=E))
        assert all(len(set(r)) == k for r in want.tolist())
        assert np.array_equal(np.sort(buf.perm.cpu().numpy()), np.arange(T * k))
    # the workspace is clean: the next call, on clean inputs, works
    clean = W.make_inputs(cfg)
    p.epoch = 2
    B.forward(p, buf, clean["x"].cuda(), clean["Wg"].cuda(), clean["gate_bias"].cuda(), dev["W1"], dev["W3"], dev["W2"])
    torch.cuda.synchronize()
    assert int(buf.stats[7].item()) == 0 and int(buf.counts.sum().item()) == T * k


KINDS = ["nan_row", "nan_column", "inf_row", "inf_bias", "nan_bias", "masked", "masked_finite", "all_but_few"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("E,k", [(65, 1), (80, 8), (128, 8), (256, 5)])
def test_exact_gate_of_more_than_64_experts(E, k, kind):
    """fp32 problems: the selection on exact logits of all experts."""
    from paper_2605_00686_amd import binding as B
    check(B, dict(T=37, d=64, E=E, k=k, dtype="f32", seed=E + k), kind)


# (T, d, E, k): every code variant of the screen and tasks of 4, 8 and 16 tokens in the layer (the variants and 8 and 16 tokens alone too),
# rows of Wg off 16 bytes; experts few enough that all of a token's could pass as candidates, and more; and the direct gate of few
# tokens, which has neither screen nor fallback, standalone with 256 and 512 threads and with either way of adding up (see
# tests/test_gate_forms.py, which checks that each is here)
BF16_CASES = [(37, 1152, 8, 2), (9, 1088, 16, 4), (37, 320, 48, 8), (2050, 576, 48, 6), (70, 192, 64, 8), (1030, 256, 64, 3), (37, 128, 65, 8),
              (37, 128, 128, 8), (33, 128, 192, 8), (40, 128, 256, 5),
              (600, 4096, 24, 4), (600, 2112, 32, 4), (520, 1088, 64, 8), (600, 576, 128, 8), (600, 448, 192, 8), (520, 320, 256, 5),
              (1030, 1152, 16, 2), (2050, 2112, 16, 4), (1030, 192, 128, 8), (1030, 128, 192, 8), (1030, 128, 256, 5),
              (33, 2048, 128, 8), (300, 8192, 24, 8), (600, 4096, 40, 4)]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("T,d,E,k", BF16_CASES, ids=lambda v: str(v))
def test_bf16_gate(T, d, E, k, kind):
    """bf16 problems: bounds that are not finite select no candidates."""
    from paper_2605_00686_amd import binding as B
    check(B, dict(T=T, d=d, E=E, k=k, dtype="bf16", seed=E + k), kind)
