"""GPU parity of the shape descriptors (paper sec. 4; include/shape.h)
against the FP64 oracle (oracle/shape.py).

The inside decisions (C >= 1 at grid points) are taken in FP64 by both sides
with exact quotients in control-point order, so the volume's cell count is
equal; surface area and dimensions agree to rounding (1e-12, 1e-10).  The
projected area counts columns of a grid aligned with the principal axes:
for a body without symmetry the axes agree to rounding and so does the count
(within 2 columns, for a sample point within 1e-13 of the surface); for an
axisymmetric body two axes are any pair in a plane, the grids differ by a
rotation and the counts agree to the grid resolution (1 %).
"""
import numpy as np
import pytest

import workloads
from oracle import shape

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mdl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2209_10411_amd as m
    m.lib()
    return m


def _compare(g, o, h, exact_projection):
    assert g["cells_inside"] == int(round(o["V"] / h ** 3))
    assert g["S"] == pytest.approx(o["S"], rel=1e-12)
    assert np.allclose(g["dims"], o["dims"], rtol=1e-10, atol=0)
    assert np.allclose(g["centroid"], o["centroid"], rtol=0, atol=1e-10)
    if exact_projection:
        assert abs(g["A_p"] - o["A_p"]) <= 2 * h * h
        assert np.allclose(np.abs(np.sum(g["axes"] * o["axes"], 0)), 1.0, atol=1e-9)
    else:
        assert g["A_p"] == pytest.approx(o["A_p"], rel=1e-2)
    assert g["Phi"] == pytest.approx(o["Phi"], rel=1e-12)
    assert g["CSF"] == pytest.approx(o["CSF"], rel=1e-10)


@pytest.mark.parametrize("seed", [1, 2, 3])
def test_random_bodies(mdl, seed):
    cp, k = workloads.random_body(np.random.Generator(np.random.PCG64(90 + seed)), 6, 6.0)
    h = 0.25
    print(f"shape descriptors seed {seed}", flush=True)
    g = mdl.shape_descriptors(cp, k, h)
    o = shape.descriptors(cp, k, h)
    print(f"  V {g['V']:.3f} S {g['S']:.3f} A_p {g['A_p']:.3f}/{o['A_p']:.3f} dims {g['dims']} "
          f"Phi {g['Phi']:.4f} CSF {g['CSF']:.4f}", flush=True)
    _compare(g, o, h, True)


def test_sphere_and_dumbbell(mdl):
    h = 0.25
    g = mdl.shape_descriptors(np.zeros((1, 3)), np.array([64.0]), h)
    o = shape.descriptors(np.zeros((1, 3)), np.array([64.0]), h)
    _compare(g, o, h, False)
    assert g["Phi"] == pytest.approx(1.0, abs=3e-3) and g["CSF"] == pytest.approx(1.0, abs=1e-12)
    cp, k = np.array([[-3.0, 0.0, 0.0], [3.0, 0.0, 0.0]]), np.array([20.0, 20.0])
    g = mdl.shape_descriptors(cp, k, h)
    o = shape.descriptors(cp, k, h)
    _compare(g, o, h, False)
    assert g["CSF"] < 0.95


def test_rejects_bad_input(mdl):
    with pytest.raises(mdl.LbmError):
        mdl.shape_descriptors(np.zeros((1, 3)), np.array([-1.0]), 0.25)


def test_designed_particles_of_the_dkt_table(mdl):
    """The kernel on two-point bodies whose CSF is bisected onto P2-P5 of the
    paper's Table T:MP_particles (tests/golden/dkt_table.json; grid step 0.05,
    as the DKT benchmark uses): the table's sphericity and d_n/d_s follow to
    2e-3 (measured: Phi within 1.6e-3 for P2, printed as 1.0000, and 7e-4
    for P3-P5; d_n/d_s within 1.1e-3)."""
    import json
    import os

    tab = json.load(open(os.path.join(os.path.dirname(__file__), "golden", "dkt_table.json")))["particles"]
    for name in ("P2", "P3", "P4", "P5"):
        phi, dnds, csf = tab[name]
        lo, hi = 0.0, 4.9
        for _ in range(14):
            mid = 0.5 * (lo + hi)
            if mdl.shape_descriptors(*workloads.dkt_body(mid), 0.05)["CSF"] > csf:
                lo = mid
            else:
                hi = mid
        d = mdl.shape_descriptors(*workloads.dkt_body(0.5 * (lo + hi)), 0.05)
        print(f"{name}: CSF {d['CSF']:.4f} ({csf}) Phi {d['Phi']:.4f} ({phi}) d_n/d_s {d['d_n'] / d['d_s']:.4f} ({dnds})",
              flush=True)
        assert abs(d["CSF"] - csf) < 3e-3
        assert abs(d["Phi"] - phi) < 2e-3
        assert abs(d["d_n"] / d["d_s"] - dnds) < 2e-3


@pytest.mark.parametrize("n,R,h", [(3, 6.0, 0.9), (20, 4.0, 0.31), (64, 5.0, 0.4), (2, 3.0, 2.6)])
def test_patch_and_segment_edges(mdl, n, R, h):
    """Grids of a few cells (one patch), of several patches of 15 and segments
    of 32 cells with remainders, the most control points, a coarse grid."""
    cp, k = workloads.random_body(np.random.Generator(np.random.PCG64(200 + n)), n, R)
    print(f"shape edges n={n} R={R} h={h}", flush=True)
    _compare(mdl.shape_descriptors(cp, k, h), shape.descriptors(cp, k, h), h, True)


def test_long_thin_grid(mdl):
    """Two points far apart along one axis on a coarse grid: the rows of the
    grid do not fit the workspace beside the patches' results."""
    cp, k = np.array([[0.0, 0.1, 0.2], [90.0, 0.3, -0.1], [45.0, -0.2, 0.4]])[:, [1, 2, 0]], np.array([6.0, 9.0, 7.0])
    for order in ([0, 1, 2], [2, 0, 1], [1, 2, 0]):
        g = mdl.shape_descriptors(cp[:, order], k, 2.3)
        o = shape.descriptors(cp[:, order], k, 2.3)
        _compare(g, o, 2.3, False)


@pytest.mark.parametrize("scale", [1e-4, 1.0, 3e5])
def test_no_unit_of_length(mdl, scale):
    """The FP32 first decision works on coordinates scaled by the body's own
    size: a body in other units has the same cells, area and columns."""
    cp, k = workloads.random_body(np.random.Generator(np.random.PCG64(301)), 7, 5.0)
    g = mdl.shape_descriptors(cp * scale, k * scale ** 2, 0.3 * scale)
    o = shape.descriptors(cp * scale, k * scale ** 2, 0.3 * scale)
    assert g["cells_inside"] == int(round(o["V"] / (0.3 * scale) ** 3))
    assert g["S"] == pytest.approx(o["S"], rel=1e-12) and np.allclose(g["dims"], o["dims"], rtol=1e-10, atol=0)
    assert abs(g["A_p"] - o["A_p"]) <= 2 * (0.3 * scale) ** 2


@pytest.mark.parametrize("h", [0.31, 0.25])
@pytest.mark.parametrize("n", [2, 4])
def test_sphere_of_coincident_points(mdl, n, h):
    """n points of weight K / n in one place are the point of weight K (n a
    power of two: C is the same to the bit).  The roundings of a sphere's
    moments choose its axes: both bodies' must be summed alike."""
    for p in ([0.0, 0.0, 0.0], [0.1, 0.2, 0.3]):
        one = mdl.shape_descriptors(np.array([p]), np.array([64.0]), h)
        more = mdl.shape_descriptors(np.array([p] * n), np.full(n, 64.0 / n), h)
        assert more["cells_inside"] == one["cells_inside"] and more["columns_hit"] == one["columns_hit"]
        assert np.array_equal(more["dims"], one["dims"]) and np.array_equal(more["axes"], one["axes"])
        assert np.array_equal(more["centroid"], one["centroid"])
        assert more["S"] == pytest.approx(one["S"], rel=1e-12)


def test_light_point_far_from_the_rest(mdl):
    """A body so long (2e7 for a radius of 16) that FP32 no longer separates a
    cell's centre from the light control point 0.24 away: the centre lies
    inside.  The cells are counted in FP64 about each control point."""
    h, k = 16.0, np.array([255.6, 0.1, 0.2])
    r = np.sqrt(k.sum())
    lo = np.full(3, -r - h)
    cp = np.array([[0.0, 0.0, 0.0], [0.0, 0.0, 0.0], [3.0, 260.0, 251.0]])
    cp[1] = lo + h * (np.array([1249978, 2, 2]) + 0.5) + [-0.186, -0.143, 0.052]
    cells = set()
    for p in cp:
        mid = np.floor((p - lo) / h).astype(int)
        for d in np.ndindex(7, 7, 7):
            i = mid + np.array(d) - 3
            c = lo + h * (i + 0.5)
            if np.all(i >= 0) and (k / ((c - cp) ** 2).sum(1)).sum() >= 1.0:
                cells.add(tuple(i))
    assert (1249978, 2, 2) in cells
    g = mdl.shape_descriptors(cp, k, h)
    assert g["cells_inside"] == len(cells)
