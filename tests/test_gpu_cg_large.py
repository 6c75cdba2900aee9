"""CG operators of the sizes that take their own paths: Q1 by lattice sweeps (above 4.2 M cells), with cut
bricks and surrogate faces, against the operator of a corner of the same mesh, which goes cell by cell and
has the same rows; and the boundary sums of more than 2^22 points against a batch, which reads them
through the cache.  And which form the small meshes of the form tests take."""

import numpy as np
import pytest

from layout_util import brick_form
from paper_2507_17053_amd import inputs
from test_gpu_cg_forms import CASES

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
sbm = pytest.importorskip("paper_2507_17053_amd.sbm")

TOL = {torch.float64: 1e-12, torch.float32: 5e-6}  # as the apply parity tests


def _ids(op, lo, h, first, n):
    """Each DoF's number among the lattice points of the whole mesh (n cells per axis)."""
    m = np.rint((op.dof_points() - lo) / h).astype(np.int64) + np.asarray(first)
    return (m[:, 2] * (n[1] + 1) + m[:, 1]) * (n[0] + 1) + m[:, 0], m


def test_q1_sweeps_with_cut_bricks_and_faces():
    n, h, lo = np.array([176, 170, 165]), 1.0 / 64, np.array([-1.0] * 3)
    hi = lo + h * n
    # a slanted plane takes the corner x, z high off
    ls = inputs.halfspace((0.6, 0.0, 0.8), 0.6 * hi[0] + 0.8 * hi[2] - 0.45)
    op = sbm.Operator(3, n, lo, hi, ls, 1)
    first = n - np.array([52, 33, 60])  # the corner's low sides, away from the plane
    lo2 = lo + h * first
    part = sbm.Operator(3, n - first, lo2, hi, ls, 1)
    print(f"case cells={op.n_cells} faces={op.n_sbm_faces}, corner {part.n_cells}", flush=True)
    assert brick_form(op) == "sweeps" and brick_form(part) == "cells"
    ids, m = _ids(op, lo, h, (0, 0, 0), n)
    ids2, m2 = _ids(part, lo2, h, first, n)
    at = np.searchsorted(ids, ids2)  # DoFs are numbered in lattice order
    assert np.array_equal(ids[at], ids2)
    same = (m2 >= first + 2).all(axis=1)  # the cells on the corner's own low faces have rows of their own
    assert same.sum() > 50000
    atd, sd = torch.from_numpy(at).to("cuda"), torch.from_numpy(same).to("cuda")
    try:
        for dtype, tol in TOL.items():
            u = torch.from_numpy(inputs.uniform_vector(op.n_dofs, seed=5)).to("cuda").to(dtype)
            u2 = u[atd].contiguous()
            for parts in (None, sbm.PART_CELLS, sbm.PART_SBM_FACES):
                v, v2 = torch.full_like(u, float("nan")), torch.full_like(u2, float("nan"))
                for o, x, y in ((op, u, v), (part, u2, v2)):
                    o.apply(x, y) if parts is None else o.apply_parts(x, y, parts)
                a, b = v[atd][sd].double(), v2[sd].double()
                assert bool(torch.isfinite(v).all()) and float(b.abs().max()) > 0
                assert float((a - b).norm() / b.norm()) <= 2 * tol, (dtype, parts)
                assert float((a - b).abs().max() / b.abs().max()) <= 2 * tol, (dtype, parts)
    finally:
        op.close()
        part.close()


def test_boundary_sums_beyond_the_cache():
    op = sbm.Operator(3, 112, -1.0, 1.0, inputs.sphere((0, 0, 0), 0.75), 4)
    print(f"case boundary points={op.layout_stats()[1]}", flush=True)
    assert op.layout_stats()[1] >= 1 << 22
    u = torch.from_numpy(inputs.uniform_vector(op.n_dofs, seed=6)).to("cuda")
    v, w = torch.full_like(u, float("nan")), torch.full_like(u, float("nan"))
    op.apply(u, v)
    sbm.apply_batch([op], [u], [w])
    torch.cuda.synchronize()
    assert bool(torch.isfinite(v).all()) and torch.equal(v, w)
    op.close()


def test_form_cases_take_both_forms():
    forms = {}
    for d, p, n in CASES:
        h = 0.125
        ls = inputs.sphere([-1.0 + 0.5 * h * k for k in n], 0.98 * 0.5 * h * min(n))
        op = sbm.Operator(d, n, [-1.0] * d, [-1.0 + h * k for k in n], ls, p)
        forms.setdefault((d, p), set()).add(brick_form(op))
        op.close()
    assert all(f == {"cells", "sweeps"} for f in forms.values()), forms
