"""The scratch of sbm_apply_noalloc: taken from the static device array for every accepted operator, also
where the bricks in use have more boundary DoFs than the fixed brick shape that decides acceptance
counts; the array's size, three times the limit, holds it for any domain."""

import numpy as np
import pytest

from paper_2507_17053_amd import inputs

torch = pytest.importorskip("torch")
sbm = pytest.importorskip("paper_2507_17053_amd.sbm")

FIXED = {1: (8, 8, 8), 2: (8, 4, 4), 3: (4, 4, 4)}  # brick shape (cells) that decides acceptance


def _bytes(op, fixed, lo, h):
    """FP64 scratch of an apply (halo planes and face results) by the bricks in use, and by `fixed`."""
    m = np.rint((op.dof_points() - lo) / h * op.p).astype(np.int64)
    on = np.zeros(m.shape[0], dtype=bool)
    for k in range(3):
        on |= m[:, k] % (fixed[k] * op.p) == 0
    faces = op.n_sbm_faces * 2 * op.nq_face * 8
    return 64 * op.layout_stats()[1] + faces, 64 * int(on.sum()) + faces


@pytest.mark.parametrize("p", [1, 2, 3])
def test_three_times_the_limit_holds_any_domain(p):
    n, lo, h = (43, 37, 34), -1.0, 1.0 / 16
    hi = [lo + h * k for k in n]
    rng = np.random.default_rng(5)
    c = np.array([lo + 0.5 * h * k for k in n])
    domains = [inputs.sphere(list(c), 0.9)]
    for axis in range(3):
        for cell in range(3, 13):  # sheets one cell thick, at every place against the brick planes
            a = [40.0] * 3
            a[axis] = 0.51 * h * 1.01
            cc = list(c)
            cc[axis] = lo + h * (cell + 0.5)
            domains.append(inputs.ellipsoid(cc, a))
    for k in (1, 12):  # single cells
        cs = lo + h * (rng.integers(1, 33, size=(k, 3)) + 0.5)
        domains.append({"kind": "sphere_union", "centres": cs.tolist(), "radii": [0.95 * h] * k})
    worst = 0.0
    for ls in domains:
        op = sbm.Operator(3, n, [lo] * 3, hi, ls, p, host_only=True)
        own, need = _bytes(op, FIXED[p], lo, h)
        assert op.n_cells > 0 and own <= 3 * need
        worst = max(worst, own / need)
        op.close()
    assert worst > 1.0  # some of them do need more than the fixed shape counts


@pytest.mark.gpu
@pytest.mark.parametrize("p,n", [(1, 156), (3, 60)])
def test_noalloc_leaves_the_handles_buffers_alone(p, n):
    """Within the limit by the fixed shape, beyond it by the bricks in use: the face results that the
    handle keeps from one of its own applies are still there after an apply_noalloc of another vector."""
    op = sbm.Operator(3, n, 0.0, 1.0, inputs.halfspace((1.0, 0.0, 0.0), 2.0), p)
    own, need = _bytes(op, FIXED[p], 0.0, 1.0 / n)
    assert need <= 96 << 20 < own
    print(f"case p={p} n={n} need={need} own={own}", flush=True)
    u1, u2 = (torch.from_numpy(inputs.uniform_vector(op.n_dofs, seed=s)).to("cuda") for s in (1, 2))
    a, b, ref, out = (torch.full_like(u1, float("nan")) for _ in range(4))
    op.apply(u2, ref)
    op.apply_parts(u1, a, sbm.PART_SBM_FACES)
    op.apply_noalloc(u2, out)
    op.apply_parts(u1, b, sbm.PART_SBM_FACES | sbm.PART_REUSE_FACES)
    torch.cuda.synchronize()
    assert torch.equal(out, ref) and bool(torch.isfinite(ref).all())
    assert torch.equal(a, b)
    op.close()
