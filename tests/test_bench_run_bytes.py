"""CPU: the bytes that bench.py counts for a step of a run, against counts made by
hand: the 256^3 grid cut into 4x4x4 boxes of 64^3 with 16 guard cells, whose
columns of 4 boxes share 256 planes of 96 x 96, and small columns."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402
from test_bench_bytes import FakePlan, cfg2  # noqa: E402


class Plan(FakePlan):
    def __init__(self, padded, precision, **tune):
        super().__init__(padded, precision)
        self.tune = dict(fuse_eb=0, pull_eb=1, batch_boxes=0, z_reg=0, **{})
        self.tune.update(tune)

    def tuning(self):
        return self.tune


def test_run_of_config2_counts_shared_planes_and_six_fields():
    lo, n, g, padded = cfg2()
    steps = 4
    out, kpoints = bench.algorithmic_bytes(Plan(padded, "f32"), lo, n, g, 4, run=((256, 256, 256), steps))
    P, I, H, boxes = 96, 64, 49, 64
    planes = 16 * 256  # 16 columns
    guard = P ** 3 - I ** 3
    assert kpoints == boxes * P * P * H
    assert out["exchange_J"] == boxes * guard * 3 * 2 * 4 / steps
    assert out["exchange_EB"] == boxes * guard * 6 * 2 * 4 / steps
    # nine fields in the first step, six in the other three
    assert out["fft_xy_fwd"] == (9 + 3 * 6) / steps * planes * (P * P * 4 + P * H * 8)
    assert out["z_update"] == 9 * planes * P * H * 8 + 6 * boxes * I * P * H * 8
    assert out["fft_xy_inv"] == boxes * (6 * I * P * H * 8 + 2 * 6 * I ** 3 * 4)


def test_run_of_a_batched_plan_counts_every_box_and_field():
    lo, n, g, padded = cfg2()
    one, _ = bench.algorithmic_bytes(Plan(padded, "f32"), lo, n, g, 4)
    out, _ = bench.algorithmic_bytes(Plan(padded, "f32", batch_boxes=8, pull_eb=0), lo, n, g, 4,
                                     run=((256, 256, 256), 2))
    assert out == dict(one, exchange_J=one["exchange_J"] / 2)


@pytest.mark.parametrize("Nz,boxes,planes", [
    (16, [(0, 16, 0)], 16),                     # one box
    (16, [(0, 16, 4)], 16),                     # wrapping onto itself: 24 padded planes
    (16, [(0, 8, 2), (8, 8, 2)], 16),           # 12 each
    (16, [(0, 4, 1), (8, 4, 1)], 12),           # a column with gaps: 6 each, none shared
    (16, [(4, 4, 2), (8, 4, 1)], 11),           # 2 .. 9 and 7 .. 12
    (16, [(0, 4, 16), (4, 12, 2)], 36 + 16),    # 36 padded planes wrap twice
])
def test_distinct_planes_of_a_column(Nz, boxes, planes):
    lo = [(0, 0, z) for z, _, _ in boxes]
    n = [(8, 6, m) for _, m, _ in boxes]
    g = [(1, 1, w) for _, _, w in boxes]
    padded = [(10, 8, m + 2 * w) for _, m, w in boxes]
    assert bench.distinct_planes((8, 6, Nz), lo, n, g, padded) == (planes * 8 * 6, planes * 8 * 10)
