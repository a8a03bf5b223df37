"""GPU: the heat step with every width of its z tiles, few pencils and a ragged
last tile among them, against the FP64 oracle at the bars of test_gpu_heat."""
import pytest

from paper_1707_08500_amd import synth

from psatd_cases import say
from test_gpu_heat import TOL, heat_case

pytestmark = pytest.mark.gpu

# (N, boxes, guard): 4, 8, 16 and 32 pencils (tests/select_check.cpp); 4 with 126 pencils
SHAPES = [((16, 14, 96), (1, 1, 1), 0), ((60, 70, 12), (1, 1, 1), 0), ((96, 96, 20), (1, 1, 1), 0),
          ((72, 60, 48), (3, 3, 3), 8)]


@pytest.mark.parametrize("precision", ["f64", "f32", "bf16x6"])
@pytest.mark.parametrize("N,boxes,guard", SHAPES)
def test_heat_tile_widths(N, boxes, guard, precision):
    say(f"heat tiles, {N} in {boxes} boxes, {precision}")
    lo, n, g = synth.uniform_decomposition(N, boxes, guard)
    err = heat_case(N, lo, n, g, 8, 0.5, 0.3, precision, 3, 3)
    say(f"  rel-L2 {err:.3e}")
    assert err <= TOL[precision]
