"""The two forms of the DG cell kernel against the assembled FP64 oracle: one wavefront's cells
per workgroup (a single apply of a small operator) and a full workgroup's cells (a batch), for
every degree.  The cell counts leave both with a partly filled last workgroup, and a half-space
cut gives cells whose neighbours are missing on the mesh boundary as well.  Bars as the apply
parity tests: relative 2-norm and row-scaled error within 1e-12 (FP64) and 5e-6 (FP32)."""

import numpy as np
import pytest

from oracle import sbm_oracle as O
from paper_2507_17053_amd import inputs
from parity_util import rel, row_scaled_excess

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
sbm = pytest.importorskip("paper_2507_17053_amd.sbm")

TOL = {torch.float64: 1e-12, torch.float32: 5e-6}


def _meshes(d, p):
    n = {2: 9, 3: 3 if p > 4 else 5}[d]
    hi = [-1.0 + 2.0 * (n + k) / n for k in range(d)]  # n, n+1, n+2 cells of one size
    return [([n + k for k in range(d)], [-1.0] * d, hi, inputs.sphere([0.1] * 3, 0.85)),
            ([n] * d, [-1.0] * d, [1.0] * d, inputs.halfspace((1.0, 0.0, 0.0), 0.3))]


@pytest.mark.parametrize("p", range(1, 9))
@pytest.mark.parametrize("d", [2, 3])
def test_dg_cell_forms(d, p):
    cases = _meshes(d, p)
    refs = [O.setup(d, n, lo, hi, ls, p, disc="dg") for n, lo, hi, ls in cases]
    mats = [O.assemble(r) for r in refs]
    ops = [sbm.Operator(d, n, lo, hi, ls, p, disc="dg") for n, lo, hi, ls in cases]
    try:
        for dtype, tol in TOL.items():
            print(f"case d={d} p={p} dtype={dtype}", flush=True)
            us = [torch.from_numpy(inputs.uniform_vector(o.n_dofs, seed=i)).to("cuda").to(dtype)
                  for i, o in enumerate(ops)]
            one = [torch.full_like(u, float("nan")) for u in us]
            many = [torch.full_like(u, float("nan")) for u in us]
            for o, u, v in zip(ops, us, one):
                o.apply(u, v)
            sbm.apply_batch(ops, us, many)
            torch.cuda.synchronize()
            for A, u, a, b in zip(mats, us, one, many):
                ui = u.double().cpu().numpy()
                vref = A @ ui
                for v in (a.double().cpu().numpy(), b.double().cpu().numpy()):
                    assert rel(v, vref) <= tol
                    ex, i = row_scaled_excess(v, vref, A, ui, tol)
                    assert ex <= 1.0, (i, v[i], vref[i])
                assert np.array_equal(a.cpu().numpy(), b.cpu().numpy())
    finally:
        for o in ops:
            o.close()
