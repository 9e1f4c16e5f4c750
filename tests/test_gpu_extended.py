"""The extended lengths a context reports, and the stored tensor read with them: its
octant is the oracle's spectrum on exactly those lengths, powers of two or with an odd
factor, scale included (rounded once in single precision)."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import newell as onewell  # noqa: E402
from oracle.params import Grid  # noqa: E402

D = (2e-9, 2.5e-9, 1.5e-9)
GRIDS = [(5, 3, 2), (73, 9, 2), (9, 75, 3), (90, 81, 4), (160, 6, 5), (8, 75, 1), (70, 9, 20), (73, 130, 7)]


def test_query_refuses_null():
    import os
    from paper_2602_12242_amd import magx
    if not os.path.exists(magx.LIB_PATH):
        pytest.skip("libmagx.so not built")
    P = (ctypes.c_int * 3)(7, 7, 7)
    assert magx.load().magx_extended_lengths(None, P) == -1
    assert tuple(P) == (7, 7, 7)


@pytest.mark.gpu
@pytest.mark.parametrize("n", GRIDS)
@pytest.mark.parametrize("dtype", [1, 0])
def test_stored_tensor_at_the_reported_lengths(n, dtype):
    from paper_2602_12242_amd import magx
    ctx = magx.Context(n, D, dtype=dtype)
    Px, Py, Pz = ctx.extended_lengths()
    for P, k in zip((Px, Py, Pz), n):
        p2 = max(2, 1 << (2 * k - 1).bit_length())
        assert P >= 2 * k and P in (p2, p2 // 8 * 5, p2 // 4 * 3)
    assert ctx.lib.magx_extended_lengths(ctx.h, None) == -1
    arr, P = ctx.spectrum_array()
    assert P == (Px, Py, Pz)
    got = arr.cpu().numpy()
    ref = onewell.spectrum(Grid(*n, *D), (Pz, Py, Px))[:, : Pz // 2 + 1, : Py // 2 + 1, :] / (Px * Py * Pz)
    assert got.shape == ref.shape
    assert np.abs(got - ref).max() <= (1e-11 if dtype == 1 else 1e-7) * np.abs(ref).max()
