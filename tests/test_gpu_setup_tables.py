"""What a CG operator keeps on the device: the tables of its own form of the brick kernel and no
others, by the device build and the host build alike."""

import pytest

from layout_util import brick_form
from paper_2507_17053_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
sbm = pytest.importorskip("paper_2507_17053_amd.sbm")


@pytest.mark.parametrize("host_build", [False, True], ids=["device", "host"])
@pytest.mark.parametrize("d,p,n,form", [(2, 1, 24, "cells"), (2, 3, 160, "sweeps"), (2, 8, 12, "cells"), (3, 1, 20, "cells"),
                                        (3, 2, 15, "cells"), (3, 3, 13, "cells"), (3, 4, 12, "cells"), (3, 5, 36, "sweeps"),
                                        (3, 8, 28, "sweeps")])
def test_tables_of_the_form_only(d, p, n, form, host_build):
    op = sbm.Operator(d, n, -1.0, 1.0, inputs.sphere((0.02, -0.01, 0.03)[:d], 0.93), p, host_build=host_build)
    print(f"case d={d} p={p} n={n} cells={op.n_cells}", flush=True)
    assert brick_form(op) == form
    op.close()
