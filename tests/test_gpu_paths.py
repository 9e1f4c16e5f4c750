"""Which kernels a grid's convolution takes, and the parity of grids at each of them:
the three passes (forward y, z product, inverse y) or one kernel in their place (the
column convolution, whose spectrum ends with a copy of the tensor in its own order, or
the film kernel).  Every grid names its path and extended lengths, so that a change of
a rule cannot take a kernel out of the tests unseen.

Bars as in test_gpu_parity.py: double precision 1e-11, single precision 1e-5 (ten
times that for the step's reverse mode)."""
import ctypes
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import adjoint as oadj  # noqa: E402
from oracle import field as ofield  # noqa: E402
from oracle import llg as ollg  # noqa: E402
from oracle import newell as onewell  # noqa: E402
from oracle.params import Grid, Params  # noqa: E402
from workloads import random_unit_field, random_vector_field  # noqa: E402

MAT = dict(Ms=1e6, A=1.6e-11, D=2.5e-3, Ku=8e5, eK=(0.0, 0.6, 0.8), alpha=0.1, Hbias=(1e3, -2e3, 5e3), terms=31)
D = (2e-9, 2.5e-9, 1.5e-9)
# films of at most eight cells along x: one kernel as long as a tile of the
# power-of-two column fits in 64 KiB (Py <= 256 single, 128 double precision)
FILMS = [((8, 64, 1), 0, "film"), ((8, 65, 1), 0, "film"), ((8, 75, 1), 0, "film"), ((5, 96, 1), 0, "film"),
         ((8, 97, 1), 0, "film"), ((1, 128, 1), 0, "film"), ((8, 64, 1), 1, "film"), ((8, 65, 1), 1, "passes"),
         ((8, 129, 1), 0, "passes"), ((1500, 75, 1), 0, "film")]


def _path(ctx, m, p):
    launches = {}
    for kind in ("yfwd", "zconv", "yinv"):
        ctx.profile_start(kind)
        ctx.heff(m, p)
        launches[kind] = ctx.profile_stop()[0]
    assert launches["zconv"] == 1 and launches["yfwd"] == launches["yinv"]
    if launches["yfwd"]:
        return "passes"
    dims = (ctypes.c_int * 5)()
    assert ctx.lib.magx_spectrum_layout(ctx.h, dims) == 0
    tiles = math.prod(dims) * (4 if ctx.dtype == 0 else 8)
    return "column" if ctx.sizes["spectrum_bytes"] > tiles else "film"


def _dev(a, dtype):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", torch.float32 if dtype == 0 else torch.float64)


def _err(a, b):
    a, b = np.asarray(a, dtype=np.float64), np.asarray(b, dtype=np.float64)
    return np.sqrt(((a - b) ** 2).sum(0)).max() / np.sqrt((b ** 2).sum(0)).max()


def _parity(ctx, q, n, dtype):
    g, p = Grid(*n, *D), Params(**MAT)
    spec = onewell.spectrum(g)
    tol = 1e-11 if dtype == 1 else 1e-5
    m = random_unit_field(n, 951, 2).astype(np.float32)
    m64 = m.astype(np.float64)
    assert _err(ctx.heff(_dev(m, dtype), q).cpu().numpy(), ofield.heff(g, p, m64, spec)) <= tol
    gH = random_vector_field(n, 952).astype(np.float32)
    dt = 5e-14
    mg, tape = _dev(m, dtype), ctx.tape(1)
    ctx.step(mg, q, dt, 1, tape=tape)
    assert np.abs(mg.cpu().numpy() - ollg.rk4_step(g, p, m64, dt, spec)).max() <= tol
    ref, refh = oadj.rk4_step_vjp(g, p, m64, dt, gH.astype(np.float64), spec)
    lam, gh = _dev(gH, dtype), torch.zeros(3, dtype=mg.dtype, device="cuda")
    ctx.step_backward(tape, 1, q, dt, lam, gh)
    assert _err(lam.cpu().numpy(), ref) <= 10 * tol
    assert np.abs(gh.cpu().numpy() - refh).max() <= 10 * tol * np.abs(refh).max()


@pytest.mark.parametrize("n,dtype,path", FILMS)
def test_narrow_and_long_films(n, dtype, path):
    from paper_2602_12242_amd import magx
    ctx, q = magx.Context(n, D, dtype=dtype), magx.make_params(**MAT)
    assert _path(ctx, _dev(random_unit_field(n, 950, 2), dtype), q) == path
    _parity(ctx, q, n, dtype)
