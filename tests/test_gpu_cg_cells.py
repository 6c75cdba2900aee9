"""The CG brick kernel of the low 3D degrees (p + 1 lanes per cell) against the assembled FP64
oracle, on meshes that hold full and partial bricks, cells on the mesh boundary, and a last brick
cut by it: the whole apply, its cell term and its surrogate-face term.  Bars as the apply parity
tests: relative 2-norm and row-scaled error within 1e-12 (FP64) and 5e-6 (FP32); a batch and a
repeated apply are bitwise the first apply."""

import pytest

from oracle import sbm_oracle as O
from paper_2507_17053_amd import inputs
from parity_util import rel, row_scaled_excess

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
sbm = pytest.importorskip("paper_2507_17053_amd.sbm")

TOL = {torch.float64: 1e-12, torch.float32: 5e-6}


@pytest.mark.parametrize("p,n", [(1, (19, 18, 17)), (1, (8, 4, 4)), (2, (16, 14, 13)), (2, (7, 6, 5)), (3, (17, 9, 10)),
                                 (3, (3, 2, 4))], ids=lambda v: str(v))
def test_low_degree_bricks(p, n):
    h = 0.125
    hi = [-1.0 + h * k for k in n]
    # everything but a slanted corner: interior bricks are full, and the mesh boundary is a face
    ls = inputs.halfspace((0.6, 0.0, 0.8), 0.8 * hi[2] + 0.6 * hi[0] - 0.3)
    ref = O.setup(3, n, [-1.0] * 3, hi, ls, p)
    A_cell, A_sbm = O.assemble(ref, parts=("cell",)), O.assemble(ref, parts=("sbm",))
    op = sbm.Operator(3, n, [-1.0] * 3, hi, ls, p)
    try:
        assert op.n_dofs == ref.n_dofs
        for dtype, tol in TOL.items():
            print(f"case p={p} n={n} dtype={dtype}", flush=True)
            u = torch.from_numpy(inputs.uniform_vector(op.n_dofs, seed=p)).to("cuda").to(dtype)
            ui = u.double().cpu().numpy()
            first = torch.full_like(u, float("nan"))
            op.apply(u, first)
            for parts, M in ((None, A_cell + A_sbm), (sbm.PART_CELLS, A_cell), (sbm.PART_SBM_FACES, A_sbm)):
                v = torch.full_like(u, float("nan"))
                if parts is None:
                    sbm.apply_batch([op], [u], [v])
                    torch.cuda.synchronize()
                    assert torch.equal(v, first)
                else:
                    op.apply_parts(u, v, parts)
                    torch.cuda.synchronize()
                vn = v.double().cpu().numpy()
                assert rel(vn, M @ ui) <= tol, parts
                ex, i = row_scaled_excess(vn, M @ ui, M, ui, tol)
                assert ex <= 1.0, (parts, i)
    finally:
        op.close()
