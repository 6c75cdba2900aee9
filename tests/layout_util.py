"""The form of a CG operator's brick kernel, from the device bytes that the operator holds: by cells it
keeps one word per cell for the faces, by lattice sweeps the cells' run bases and the faces' places."""

# bricks (cells) by form: 3D by sweeps per degree; by cells the same but for degree 1 to 3; 2D
_SWEEPS3 = {1: (8, 8, 8), 2: None, 3: None, 4: (4, 2, 2), 5: (4, 2, 2), 6: (2, 2, 1), 7: (2, 2, 2), 8: (2, 2, 1)}
_CELLS3 = {**_SWEEPS3, 1: (8, 4, 4), 2: (7, 6, 4), 3: (8, 4, 2)}


def expected_bytes(op, form):
    """Device bytes of a CG operator set up in the given form ("cells" or "sweeps"); None if that form
    does not exist."""
    d, p = op.d, op.p
    if d == 2:
        b = 8 if p <= 2 else (4 if p <= 7 else 3)
        shape = (b, b, 1)
    else:
        shape = (_CELLS3 if form == "cells" else _SWEEPS3)[p]
        if shape is None:
            return None
    nbricks, nh, _ = op.layout_stats()
    nc, nf, np_ = op.n_cells, op.n_sbm_faces, op.nq_face
    rows = nbricks * (shape[1] * p + 1) * (shape[2] * p + 1 if d == 3 else 1)
    words = [nc * np_, nbricks + 1, nf * np_, nc, nbricks + 1]  # runs, cell offsets, face runs, cell places, face offsets
    words += [nc] if form == "cells" else [nc * np_, nf]
    words += [rows] * 4 + [2 * rows, nh, nf, nf]
    up = [4 * w for w in words] + [nh, (1 << d) * 8 * nh, nf * 2 * np_ * 8, nf * np_ * d * 8]
    return sum((b + 255) // 256 * 256 for b in up)


def brick_form(op):
    """"cells" or "sweeps"."""
    match = [f for f in ("cells", "sweeps") if expected_bytes(op, f) == op.device_bytes]
    assert len(match) == 1, (op.device_bytes, expected_bytes(op, "cells"), expected_bytes(op, "sweeps"))
    return match[0]
