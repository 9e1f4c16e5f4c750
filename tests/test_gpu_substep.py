"""GPU parity of the multirate step where a fast substep is one kernel (thin grids
without a profile and the non-finite check): column tiles of 26 x 10 cells, their
edges and remainders, every plane count of its instances and the first one beyond,
against the FP64 oracle; a batch against its members; the checked call, which takes
the stage kernels, against the unchecked one.

Bars as in test_gpu_mri.py: double precision 1e-11, single precision 1e-5."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import mri as omri  # noqa: E402
from oracle import newell as onewell  # noqa: E402
from oracle.params import Grid, Params  # noqa: E402
from workloads import random_unit_field  # noqa: E402

MAT = dict(Ms=1e6, A=1.6e-11, D=2.5e-3, Ku=8e5, eK=(0.0, 0.6, 0.8), alpha=0.1, Hbias=(1e3, -2e3, 5e3), terms=31)
D = (2e-9, 2.5e-9, 1.5e-9)
GRIDS = [(26, 10, 1), (27, 11, 2), (25, 9, 3), (52, 20, 4), (53, 21, 5), (1, 30, 6), (30, 1, 7), (29, 13, 8),
         (27, 11, 9), (1, 1, 1)]


def _magx():
    from paper_2602_12242_amd import magx
    return magx


def _dev(a, dtype):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", torch.float32 if dtype == 0 else torch.float64)


def _err(a, b):
    a, b = np.asarray(a, dtype=np.float64), np.asarray(b, dtype=np.float64)
    return np.sqrt(((a - b) ** 2).sum(0)).max() / np.sqrt((b ** 2).sum(0)).max()


@pytest.mark.parametrize("n", GRIDS)
@pytest.mark.parametrize("dtype", [1, 0])
@pytest.mark.parametrize("renorm", [2, 0])
def test_step_matches_oracle(n, dtype, renorm):
    magx = _magx()
    g = Grid(*n, *D)
    m = random_unit_field(n, 701, 2).astype(np.float32)
    mg = _dev(m, dtype)
    # 3 + 4 + 2 substeps: an odd number of buffer changes
    magx.Context(n, D, dtype=dtype).step_mri(mg, magx.make_params(renorm=renorm, **MAT), 8e-14, 1, 1e-14)
    ref = omri.mri_run(g, Params(renorm=renorm, **MAT), m.astype(np.float64), 8e-14, 1e-14, 1, onewell.spectrum(g))
    assert _err(mg.cpu().numpy(), ref) <= (1e-11 if dtype == 1 else 1e-5)


@pytest.mark.parametrize("dtype", [1, 0])
def test_batch_equals_members_and_check_agrees(dtype):
    magx = _magx()
    n, B = (31, 12, 3), 3
    m = np.stack([random_unit_field(n, 710 + b, 2) for b in range(B)]).astype(np.float32)
    p = magx.make_params(**MAT)
    mb = _dev(m, dtype)
    magx.Context(n, D, dtype=dtype, nbatch=B).step_mri(mb, p, 1e-13, 2, 1e-14)
    for b in range(B):
        ctx, one = magx.Context(n, D, dtype=dtype), _dev(m[b], dtype)
        ctx.step_mri(one, p, 1e-13, 2, 1e-14)
        assert torch.equal(one, mb[b])
        chk = _dev(m[b], dtype)
        ctx.step_mri(chk, magx.make_params(check_finite=1, **MAT), 1e-13, 2, 1e-14)
        assert ctx.status() == 0
        assert _err(chk.cpu().numpy(), one.cpu().numpy()) <= (1e-12 if dtype == 1 else 2e-6)
