"""The sum-factorised surrogate faces of the low Taylor orders (m <= 2) against the oracle's E_m
operator: the lowest and highest degree, orders above the degree, a face count that leaves the last
workgroup partly filled and a single face workgroup.  Bars as the apply parity tests."""

import pytest

from oracle import sbm_oracle as O
from paper_2507_17053_amd import inputs
from parity_util import rel, row_scaled_excess

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
sbm = pytest.importorskip("paper_2507_17053_amd.sbm")

TOL = {torch.float64: 1e-12, torch.float32: 5e-6}


@pytest.mark.parametrize("d,n,p", [(2, 11, 1), (2, 3, 1), (3, 7, 1), (3, 3, 1), (3, 3, 8), (2, 5, 8)])
@pytest.mark.parametrize("disc", ["cg", "dg"])
def test_low_order_faces(d, n, p, disc):
    ls = inputs.ellipsoid((0.02, 0.01, -0.03), (0.8, 0.75, 0.9)) if n > 3 else inputs.sphere((0.05, 0.0, 0.02), 0.85)
    for m in (0, 1, 2):
        ref = O.setup(d, n, -1.0, 1.0, ls, p, disc=disc, taylor_order=m)
        A = O.assemble(ref)
        assert ref.n_dofs > 0
        op = sbm.Operator(d, n, -1.0, 1.0, ls, p, disc=disc, taylor_order=m)
        try:
            for dtype, tol in TOL.items():
                print(f"case d={d} n={n} p={p} {disc} m={m} {dtype}", flush=True)
                u = torch.from_numpy(inputs.uniform_vector(op.n_dofs, seed=m)).to("cuda").to(dtype)
                ui = u.double().cpu().numpy()
                v = torch.full_like(u, float("nan"))
                op.apply(u, v)
                torch.cuda.synchronize()
                vn = v.double().cpu().numpy()
                assert rel(vn, A @ ui) <= tol
                ex, i = row_scaled_excess(vn, A @ ui, A, ui, tol)
                assert ex <= 1.0, i
        finally:
            op.close()
