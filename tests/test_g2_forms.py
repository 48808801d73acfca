"""The rule by which fp32 layers cut their GEMM2 tiles: the numbers of parts it gives, and that the library follows it (a cut layer keeps
counters and the parts' sums in its workspace)."""
import pytest

from paper_2605_00686_amd import binding as B
from tests import g2_forms as G
from tests import test_gpu_g2_parts

# (T, d, E, k, f): parts
PARTS = {(256, 512, 8, 2, 1024): 4, (256, 512, 8, 2, 512): 2, (256, 512, 8, 2, 256): 1,
         # a part costs more than it takes off a short tile
         (16, 512, 8, 2, 512): 1, (16, 512, 8, 2, 768): 1, (16, 512, 8, 2, 1024): 2, (4, 512, 4, 2, 512): 1, (4, 512, 4, 2, 768): 3,
         (128, 768, 8, 1, 512): 1, (128, 768, 8, 1, 2048): 2, (1, 4096, 2, 2, 1024): 1, (128, 512, 4, 2, 256): 1, (128, 512, 4, 2, 512): 4,
         (64, 256, 4, 2, 896): 5, (64, 256, 4, 2, 1040): 6, (64, 256, 4, 2, 1232): 7, (64, 256, 4, 2, 2048): 8,
         # the bound on the tiles: (8 + 8) * 8 and (9 + 8) * 8
         (512, 512, 8, 2, 2048): 2, (576, 512, 8, 2, 2048): 1, (1, 64, 1, 1, 16): 1, (1, 64, 1, 1, 768): 3}


@pytest.mark.parametrize("shape", list(PARTS), ids=["T%d_d%d_E%d_k%d_f%d" % s for s in PARTS])
def test_parts_of_a_tile(shape):
    T, d, E, k, f = shape
    assert G.parts(*shape) == PARTS[shape]
    for capacity in (0, 128):
        large, small = (B.problem(T, d, E, k, f2, 1, "f32", capacity=capacity) for f2 in (f, 16))
        grown = B._lib.moe_workspace_bytes(large) - B._lib.moe_workspace_bytes(small)
        assert grown == G.workspace_growth(*shape, capacity=capacity)


def test_the_gpu_cases_are_cut_as_they_say():
    cases = test_gpu_g2_parts.CASES
    assert all(G.parts(*c[:5]) == n for c, n in cases.items()) and set(cases.values()) == set(range(1, 9))
    assert {G.most_tiles(*c[:4]): n > 1 for c, n in cases.items()}.items() >= {128: True, 136: False}.items()
