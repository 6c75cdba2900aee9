"""One batch over CG operators whose bricks take different forms (cell by cell, lattice sweeps) at one
degree, with the full and a truncated extension, and DG batches by both workgroup sizes: every result is
bitwise the single apply's, on one stream, on several, and replayed on new inputs."""

import pytest

from layout_util import brick_form
from paper_2507_17053_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
sbm = pytest.importorskip("paper_2507_17053_amd.sbm")


def _check(ops, dtype, streams, graph):
    us = [torch.empty(o.n_dofs, dtype=dtype, device="cuda") for o in ops]
    vs = [torch.empty_like(u) for u in us]
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        with sbm.Batch(ops, us, vs, graph=graph, streams=streams) as b:
            for rep in range(3):
                for i, (o, u, v) in enumerate(zip(ops, us, vs)):
                    u.copy_(torch.from_numpy(inputs.uniform_vector(o.n_dofs, seed=10 * rep + i)))
                    v.fill_(float("nan"))
                b.run()
                torch.cuda.synchronize()
                for o, u, v in zip(ops, us, vs):
                    ref = torch.full_like(u, float("nan"))
                    o.apply(u, ref)
                    torch.cuda.synchronize()
                    assert torch.equal(v, ref), (o.n_dofs, rep)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("d,p,ns", [(3, 4, (12, 44, 20)), (3, 8, (6, 30)), (2, 3, (20, 180, 60)), (2, 1, (180, 9))],
                         ids=lambda v: str(v))
def test_batch_of_both_brick_forms(d, p, ns, dtype):
    ops = [sbm.Operator(d, n, -1.0, 1.0, inputs.sphere((0.02, -0.01, 0.03)[:d], 0.9), p, taylor_order=o)
           for n in ns for o in (None, 1)]
    print(f"case d={d} p={p} cells={[o.n_cells for o in ops]} dtype={dtype}", flush=True)
    assert {brick_form(o) for o in ops} == {"cells", "sweeps"}
    for streams, graph in ((1, False), (4, True)):
        _check(ops, dtype, streams, graph)
    for o in ops:
        o.close()


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("p,n,count", [(4, 36, 6), (5, 24, 8)])
def test_batch_of_many_bricks_by_cells(p, n, count, dtype):
    """More bricks than the device holds several times over: a part of a brick's cells at a time."""
    ops = [sbm.Operator(3, n, -1.0, 1.0, inputs.sphere((0.02, -0.01, 0.03), 0.84 + 0.01 * k), p, taylor_order=(None, 1)[k % 2])
           for k in range(count)]
    bricks = sum(o.layout_stats()[0] for o in ops)
    print(f"case p={p} bricks={bricks} dtype={dtype}", flush=True)
    assert {brick_form(o) for o in ops} == {"cells"} and bricks > (4096 if p == 4 else 1024)
    _check(ops, dtype, 1, True)
    for o in ops:
        o.close()


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("d,p,ns", [(3, 2, (5, 8, 6)), (3, 2, (5, 40, 44)), (2, 8, (9, 12)), (3, 7, (4, 5))],
                         ids=lambda v: str(v))
def test_dg_batch_of_few_and_many_cells(d, p, ns, dtype):
    ops = [sbm.Operator(d, n, -1.0, 1.0, inputs.sphere((0.02, -0.01, 0.03)[:d], 0.9), p, disc="dg") for n in ns]
    print(f"case dg d={d} p={p} cells={[o.n_cells for o in ops]} dtype={dtype}", flush=True)
    _check(ops, dtype, 1, True)
    for o in ops:
        o.close()
