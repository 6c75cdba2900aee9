"""Both forms of the CG brick kernel (cell by cell on small operators, lattice sweeps on large ones)
against the C oracle, on meshes that hold full and partial bricks and last bricks cut by the mesh: the whole apply, its cell term and its surrogate-face term.  Bars as the full-size
parity tests: relative 2-norm and largest error over largest value within 1e-12 (FP64) and 5e-6
(FP32); a batch is bitwise the single apply."""

import pytest

from oracle import native
from oracle import sbm_oracle as O
from paper_2507_17053_amd import inputs
from parity_util import rel, rel_inf

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
sbm = pytest.importorskip("paper_2507_17053_amd.sbm")

TOL = {torch.float64: 1e-12, torch.float32: 5e-6}

CASES = ([(2, p, (19, 14)) for p in range(1, 9)] + [(2, 3, (3, 4))]
         + [(2, p, (160, 155)) for p in range(1, 9)]
         + [(3, p, (11, 10, 9)) for p in range(4, 9)] + [(3, 4, (4, 3, 5))]
         + [(3, 4, (37, 35, 36)), (3, 5, (29, 30, 28)), (3, 6, (22, 24, 23)), (3, 7, (29, 28, 30)), (3, 8, (22, 24, 23))])


@pytest.mark.parametrize("d,p,n", CASES, ids=lambda v: str(v))
def test_brick_forms(d, p, n):
    native.build(force=False)
    h = 0.125
    hi = [-1.0 + h * k for k in n]
    # a ball that nearly fills the box: full bricks inside, cut ones around them
    half = [0.5 * h * k for k in n]
    ls = inputs.sphere([-1.0 + a for a in half], 0.98 * min(half))
    ref = O.setup(d, n, [-1.0] * d, hi, ls, p)
    oracle = native.NativeApply(ref)
    op = sbm.Operator(d, n, [-1.0] * d, hi, ls, p)
    try:
        assert op.n_dofs == ref.n_dofs
        for dtype, tol in TOL.items():
            print(f"case d={d} p={p} n={n} cells={op.n_cells} dtype={dtype}", flush=True)
            u = torch.from_numpy(inputs.uniform_vector(op.n_dofs, seed=p)).to("cuda").to(dtype)
            ui = u.double().cpu().numpy()
            first = torch.full_like(u, float("nan"))
            op.apply(u, first)
            v = torch.full_like(u, float("nan"))
            sbm.apply_batch([op], [u], [v])
            torch.cuda.synchronize()
            assert torch.equal(v, first)
            for parts, oparts in ((None, ("cell", "sbm")), (sbm.PART_CELLS, ("cell",)), (sbm.PART_SBM_FACES, ("sbm",))):
                if parts is None:
                    v = first
                else:
                    v = torch.full_like(u, float("nan"))
                    op.apply_parts(u, v, parts)
                    torch.cuda.synchronize()
                vn, vref = v.double().cpu().numpy(), oracle(ui, parts=oparts)
                assert rel(vn, vref) <= tol, parts
                assert rel_inf(vn, vref) <= tol, parts
    finally:
        op.close()
