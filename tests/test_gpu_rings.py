"""GPU: columns of boxes that share their spectral planes, the workspace layouts
they run in, and the launch shapes chosen by size.  Every pair of settings
compared below runs the same operations on the same values per transform, so
their results are byte-identical; one of each pair is checked against the FP64
oracle at the bars of the parity tests (FP64 1e-12, FP32 1e-5)."""
import numpy as np
import pytest

from paper_1707_08500_amd import synth
from psatd_cases import deposited_partition, random_fields, say, upload_boxes
from test_gpu_parity import check, run_both

pytestmark = pytest.mark.gpu
TOL = {"f64": 1e-12, "f32": 1e-5}


def column(zs, gz, nx=8, gx=2):
    """Boxes stacked along z with their own z guards."""
    lo, n, g, z = [], [], [], 0
    for nz, q in zip(zs, gz):
        lo.append([0, 0, z])
        n.append([nx, nx, nz])
        g.append([gx, gx, q])
        z += nz
    return (nx, nx, z), lo, n, g


def mixed():
    """Columns that cover part of the axis, next to columns of other guards."""
    lo, n, g = [], [], []
    for z in range(0, 20, 5):
        for x in (0, 6):
            lo.append([x, 0, z])
            n.append([6, 7, 5])
            g.append([[3, 2, 1], [2, 1, 3]][(z // 5 + x // 6) % 3 == 0])
    return (12, 7, 20), lo, n, g


LAYOUTS = {"wrap": column([16], [4]), "thin": column([2, 10, 4], [4, 5, 4]), "past": column([4, 12], [18, 2]),
           "mixed": mixed()}


def rerun(case, E, B, J, steps, **tuning):
    """The state after `steps` from the same start with other settings."""
    import torch
    case.plan.set_tuning(**tuning)
    for glob, pad in ((E, case.E), (B, case.B)):
        case.plan.scatter([torch.from_numpy(np.ascontiguousarray(glob[a])).to("cuda", case.dtype).reshape(-1)
                           for a in range(3)], pad)
    J(case)
    case.plan.run(case.E, case.B, case.J, steps)
    case.plan.sync()
    return torch.cat([x.clone() for x in case.E + case.B + case.J])


def state(case):
    import torch
    return torch.cat([x.clone() for x in case.E + case.B + case.J])


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("layout", sorted(LAYOUTS))
def test_shared_planes_equal_own_planes(precision, layout):
    import torch
    from oracle import psatd_oracle as O
    say(f"shared spectral planes ({layout}), {precision}")
    N, lo, n, g = LAYOUTS[layout]
    E, B, J = random_fields(N, 51, p=8)
    if precision == "f32":
        E, B, J = (x.astype(np.float32).astype(np.float64) for x in (E, B, J))
    dec = O.Decomposition(N, lo, n, g)
    parts = deposited_partition(J, dec, 5)
    case, eE, eB, _ = run_both(N, lo, n, g, 8, 0.5, 1.0, precision, "deposited", (E, B, J), 3, J_boxes=parts)
    check(case, eE, eB, precision, TOL[precision])
    first = state(case)
    put = lambda c: upload_boxes(c, c.J, parts)  # noqa: E731
    if len(lo) > 1:  # batches keep a box's planes to itself
        assert torch.equal(first, rerun(case, E, B, put, 3, batch_boxes=1))
        case.plan.set_tuning(batch_boxes=0)
    need = case.plan.workspace_bytes()  # the least a caller may hand over: planes back to back
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    case.plan.set_workspace(ws)
    assert torch.equal(first, rerun(case, E, B, put, 3))


@pytest.mark.parametrize("N,g", [((210, 201, 6), [3, 12, 2]), ((420, 1, 4), [0, 87, 1])])
def test_inverse_pass_in_halves_equals_split_passes(N, g):
    """Padded planes of 216 x 225 (odd interior rows) and 420 x 175 with one
    interior row; the fused exchange keeps the split passes."""
    import torch
    say(f"inverse pass in halves, {N} guards {g}")
    E, B, J = (x.astype(np.float32).astype(np.float64) for x in random_fields(N, 52, p=8))
    case, eE, eB, _ = run_both(N, [[0, 0, 0]], [list(N)], [g], 8, 0.5, 1.0, "f32", "replicated", (E, B, J), 2)
    assert case.plan.tuning()["split_xy"] == 1
    check(case, eE, eB, "f32", TOL["f32"])
    first = state(case)
    assert torch.equal(first, rerun(case, E, B, lambda c: None, 2, fuse_eb=1))


@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_narrow_z_tiles(precision):
    """27 boxes of 32^3 padded: more tiles than one round, run with 256 threads;
    z_threads 1024 keeps the wide kernels."""
    import torch
    say(f"narrow z tiles, {precision}")
    N = (72, 72, 72)
    lo, n, g = synth.uniform_decomposition(N, (3, 3, 3), 4)
    E, B, J = random_fields(N, 53, p=16)
    if precision == "f32":
        E, B, J = (x.astype(np.float32).astype(np.float64) for x in (E, B, J))
    case, eE, eB, _ = run_both(N, lo, n, g, 16, 0.5, 1.0, precision, "replicated", (E, B, J), 2)
    check(case, eE, eB, precision, TOL[precision])
    first = state(case)
    assert torch.equal(first, rerun(case, E, B, lambda c: None, 2, z_threads=1024))


# (N, boxes, guard): 8 pencils from the shortest z whose nine-field tiles do not share a
# compute unit to the longest whose held tiles do, odd lengths, two boxes that share
# planes; 4 pencils to the same end.  All with a ragged last tile but the boxes.
HELD = [((70, 75, 70), 1, 0), ((70, 75, 99), 1, 0), ((70, 75, 100), 1, 0), ((64, 64, 160), 2, 8),
        ((48, 45, 147), 1, 0), ((48, 45, 200), 1, 0)]


@pytest.mark.parametrize("N,boxes,guard", HELD)
@pytest.mark.parametrize("maxr", [16, 8])
def test_held_z_tiles(N, boxes, guard, maxr):
    """FP64 tiles with J's transform in registers: against the oracle, and against the
    nine-field tiles of 1024 threads within twice its bar (each is within one)."""
    say(f"held z tiles, {N}, {boxes} boxes, radix {maxr}")
    lo, n, g = synth.uniform_decomposition(N, (1, 1, boxes), guard)
    E, B, J = random_fields(N, 61, p=16)
    case, eE, eB, _ = run_both(N, lo, n, g, 16, 0.5, 1.0, "f64", "replicated", (E, B, J), 2)
    check(case, eE, eB, "f64", TOL["f64"])
    first = state(case)
    for nt in (512, 1024):
        other = rerun(case, E, B, lambda c: None, 2, z_threads=nt, max_radix_z=maxr)
        assert float((other - first).abs().max()) <= 2 * TOL["f64"] * float(first.abs().max())
