"""Closing an operator waits for its own applies, also where they follow long work on their stream and where
several follow each other (the event that shows it then has no system-scope release)."""

import threading

import pytest

from paper_2507_17053_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
sbm = pytest.importorskip("paper_2507_17053_amd.sbm")


def _inside_one_brick():
    # four cells in the middle of an 8 x 8 brick: no point on a brick's boundary
    return sbm.Operator(2, 8, -1.0, 1.0, inputs.sphere((0.0, 0.0), 0.4), 1)


CASES = {
    "cg": (lambda: sbm.Operator(3, 20, -1.0, 1.0, inputs.sphere((0, 0, 0), 0.8), 4), "apply"),
    "cg_e1": (lambda: sbm.Operator(3, 20, -1.0, 1.0, inputs.sphere((0, 0, 0), 0.8), 2, taylor_order=1), "apply"),
    "cg_no_sums": (_inside_one_brick, "apply"),
    "cg_parts": (lambda: sbm.Operator(3, 20, -1.0, 1.0, inputs.sphere((0, 0, 0), 0.8), 4), "parts"),
    "cg_noalloc": (lambda: sbm.Operator(3, 20, -1.0, 1.0, inputs.sphere((0, 0, 0), 0.8), 4), "noalloc"),
    "dg": (lambda: sbm.Operator(3, 12, -1.0, 1.0, inputs.sphere((0, 0, 0), 0.8), 3, disc="dg"), "apply"),
}


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_close_waits_for_the_applies(name, dtype):
    make, how = CASES[name]
    a = torch.randn(8192, 8192, dtype=torch.float32, device="cuda")
    c = torch.empty_like(a)
    one = torch.ones(1, device="cuda")
    done = torch.zeros(1, pin_memory=True)
    stream = torch.cuda.Stream()
    ref = None
    for rep in range(3):
        op = make()
        assert name != "cg_no_sums" or (op.n_cells > 0 and op.layout_stats()[1] == 0)
        print(f"case {name} dtype={dtype} n_dofs={op.n_dofs} rep={rep}", flush=True)
        u = torch.from_numpy(inputs.uniform_vector(op.n_dofs, seed=1)).to("cuda").to(dtype)
        v = torch.full_like(u, float("nan"))
        done.zero_()
        torch.cuda.synchronize()

        def applies(n):
            for _ in range(n):
                if how == "parts":
                    op.apply_parts(u, v, sbm.PART_ALL | sbm.PART_NO_ASSEMBLY)
                elif how == "noalloc":
                    op.apply_noalloc(u, v)
                else:
                    op.apply(u, v)

        with torch.cuda.stream(stream):
            applies(1)  # (the first call of its kind loads the kernels)
            stream.synchronize()
            for _ in range(3):
                torch.mm(a, a, out=c)
            done.copy_(one, non_blocking=True)
            applies(4)
            assert float(done[0]) == 0.0  # the products are still running
        op.close()
        assert float(done[0]) == 1.0  # (what the applies wait for on their stream)
        got = v.cpu()
        if how != "parts":
            assert bool(torch.isfinite(got).all())
            assert ref is None or torch.equal(got, ref)
            ref = got


@pytest.mark.parametrize("other_thread", [True, False], ids=["other_thread", "same_thread"])
def test_applies_beside_a_capture(other_thread):
    """A series of applies on a stream of its own while a graph is captured on another, by another thread or
    by the same: neither disturbs the other."""
    op = sbm.Operator(3, 24, -1.0, 1.0, inputs.sphere((0, 0, 0), 0.8), 4)
    u = torch.from_numpy(inputs.uniform_vector(op.n_dofs, seed=1)).to("cuda")
    ref, v = torch.empty_like(u), torch.full_like(u, float("nan"))
    op.apply(u, ref)
    stream = torch.cuda.Stream()
    x = torch.zeros(1000, device="cuda")
    err = []

    def series():
        try:
            for _ in range(40):
                op.apply(u, v, stream=stream)
        except Exception as exc:
            err.append(repr(exc))

    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        x.add_(1.0)
        if other_thread:
            th = threading.Thread(target=series)
            th.start()
            th.join()
        else:
            series()
        x.add_(1.0)
    for rep in range(3):
        g.replay()
        torch.cuda.synchronize()
        assert float(x[0]) == 2.0 * (rep + 1) and float(x[-1]) == 2.0 * (rep + 1)
    assert not err and torch.equal(v, ref)
    op.close()
