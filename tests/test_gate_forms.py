"""The gate tests run the forms of the gate that they name: both of the bf16 gate's rules (alone and in the layer), applied to their
lists of cases."""
from tests import gate_forms as G
from tests import test_gpu_gate, test_gpu_gate_direct, test_gpu_gate_direct_alone, test_gpu_gate_many_candidates, test_gpu_gate_nonfinite

FOUR_TOKENS = {("screen", v, 4) for v in (1, 2, 3, 4, 5, 6)}


def forms(cases, alone):
    return {G.form(c[0], c[2], c[1], alone) for c in cases}


def of_whole_pieces(cases):
    """Screens whose rows of Wg are whole 16-byte pieces."""
    return {G.form(c[0], c[2], c[1], False) for c in cases if c[2] % 8 == 0} - {"direct"}


def test_rule_of_the_direct_gate():
    assert G.is_direct(256, 256, 4096, False) and not G.is_direct(257, 256, 4096, False) and not G.is_direct(256, 256, 4160, False)
    assert G.is_direct(512, 64, 12288, False) and not G.is_direct(512, 64, 12352, False)  # (two rows of x in LDS)
    assert G.is_direct(513, 128, 512, False) and not G.is_direct(513, 128, 576, False) and G.is_direct(513, 128, 576, True)
    assert G.is_direct(1024, 64, 1024, False) and not G.is_direct(1025, 64, 1024, True) and not G.is_direct(8, 65, 1024, False)
    assert [G.direct_parts(*c) for c in ((8, 128, 2048), (80, 128, 2048), (128, 128, 2048), (129, 128, 2048), (8, 64, 2048))] == [8, 3, 2, 1, 1]
    assert G.part_pieces(128, 3) == [5, 5, 6] and G.part_pieces(136, 5) == [3, 3, 4, 3, 4]


def test_random_inputs_reach_every_form():
    layer, alone = forms(test_gpu_gate.CASES, False), forms(test_gpu_gate.CASES, True)
    assert FOUR_TOKENS <= of_whole_pieces(test_gpu_gate.CASES)
    assert "direct" in layer and "direct" in alone and "exact" in alone
    assert {f[2] for f in layer if f != "direct"} == {4, 8, 16} and {f[1] for f in layer if f != "direct"} == {1, 2, 3, 4, 5, 6}


def test_numbers_that_are_not_finite_reach_every_form():
    cases = test_gpu_gate_nonfinite.BF16_CASES
    layer, alone = forms(cases, False), forms(cases, True)
    assert FOUR_TOKENS <= of_whole_pieces(cases) and "direct" in layer and "direct" in alone
    assert {f[2] for f in layer if f != "direct"} == {4, 8, 16}
    screens = {f for f in alone if f not in ("direct", "exact")}
    assert {f[1] for f in screens} == {1, 2, 3, 4, 5, 6} and {f[2] for f in screens} >= {8, 16}


def test_equal_logits_reach_every_form():
    cases = test_gpu_gate_many_candidates.CASES
    assert FOUR_TOKENS <= of_whole_pieces(cases) and "direct" in forms(cases, False)
    assert {f[2] for f in forms(cases, False) if f != "direct"} == {4, 8, 16}


def test_unaligned_weights_reach_every_screen():
    assert {f[1] for f in of_whole_pieces(test_gpu_gate.UNALIGNED_CASES)} == {1, 2, 3, 4, 5, 6}
    assert "direct" in forms(test_gpu_gate.UNALIGNED_CASES, False)


def test_direct_gate_cases_are_direct_and_some_parts_uneven():
    uneven = 0
    for T, d, E, k in test_gpu_gate_direct.CASES:
        assert G.is_direct(T, E, d, True)
        if G.is_direct(T, E, d, False):
            pieces = G.part_pieces(E, G.direct_parts(T, E, d))
            uneven += min(pieces) != max(pieces)
    assert uneven >= 4


def test_standalone_direct_gate_cases_have_every_number_of_threads_and_runs():
    cases = test_gpu_gate_direct_alone.CASES
    assert all(G.is_direct(T, E, d, True) for T, d, E, k in cases)
    sums = {G.direct_sums_alone(T, E, d) for T, d, E, k in cases}
    assert {threads for threads, _ in sums} == {256, 512} and {runs for _, runs in sums} == {1, 2, 4, 8, 16}
    assert {E * d for T, d, E, k in cases} >= {1 << 17, (1 << 17) + 4096}  # either side of the rule


def test_numbers_that_are_not_finite_reach_the_standalone_direct_gate_with_either_number_of_threads():
    cases = test_gpu_gate_nonfinite.BF16_CASES
    sums = {(G.direct_tokens(T), *G.direct_sums_alone(T, E, d)) for T, d, E, k in cases if G.is_direct(T, E, d, True)}
    assert {t for t, threads, _ in sums if threads == 512} == {1, 2, 4}
    assert {(threads, runs > 1) for _, threads, runs in sums} == {(256, False), (256, True), (512, False), (512, True)}
