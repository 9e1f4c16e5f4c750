"""Calls that compute the same thing give the same bits: check_finite = 1 adds a flag
and leaves the computation unchanged, and a taped step records what the untaped one
computes, so a rollout's re-run segments repeat its forward pass.  Fields, steps
(single, and long enough to be replayed in two chunks), Euler and multirate steps, the
reverse mode, with and without a magnetisation profile, on every order and kind of
line; no tolerance."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from workloads import random_unit_field, random_vector_field  # noqa: E402

MAT = dict(Ms=1e6, A=1.6e-11, D=2.5e-3, Ku=8e5, eK=(0.0, 0.6, 0.8), alpha=0.1, Hbias=(1e3, -2e3, 5e3), terms=31)
D = (2e-9, 2.5e-9, 1.5e-9)
# column order: a film, lines of 64 and 128 values, odd lengths; row order: lines of 64,
# 256 (nx = 256 and below), odd lengths with one and two lines per block; long lines
GRIDS = [(128, 32, 1), (33, 20, 3), (128, 128, 2), (150, 60, 3), (37, 11, 5), (256, 20, 9), (251, 30, 10), (90, 40, 6),
         (73, 130, 7), (311, 75, 5), (1100, 6, 2)]
DT = 1e-13


def _cases():
    return [(n, t) for n in GRIDS for t in (0, 1) if t == 0 or n[0] <= 1024]


def _setup(n, dtype):
    from paper_2602_12242_amd import magx
    ctx = magx.Context(n, D, dtype=dtype)
    m = torch.from_numpy(random_unit_field(n, 901, 2)).to("cuda", ctx.tdtype)
    g = torch.from_numpy(random_vector_field(n, 902)).to("cuda", ctx.tdtype)
    return magx, ctx, m, g


def _profile(n, tdtype):
    # an ellipse with a weaker core and empty corners
    x = (np.arange(n[0]) + 0.5) / n[0] - 0.5
    y = (np.arange(n[1]) + 0.5) / n[1] - 0.5
    r = np.sqrt(x[None, :] ** 2 + y[:, None] ** 2)
    s = np.where(r < 0.2, 0.6, np.where(r < 0.45, 1.0, 0.0))
    return torch.from_numpy(np.broadcast_to(s, (n[2], n[1], n[0])).copy()).to("cuda", tdtype)


def _outputs(magx, ctx, m, g, check, profile):
    p = magx.make_params(check_finite=check, **MAT)
    out = {"heff": ctx.heff(m, p)}
    for name, call in (("step", lambda y: ctx.step(y, p, DT, 1)), ("steps", lambda y: ctx.step(y, p, DT, 18)),
                       ("euler", lambda y: ctx.step_euler(y, p, 0.1 * DT, 3)),
                       ("mri", lambda y: ctx.step_mri(y, p, DT, 2))):
        out[name] = m.clone()
        call(out[name])
        if check:
            assert ctx.status() == 0, name
    tape = ctx.tape(2)
    out["taped"] = m.clone()
    ctx.step(out["taped"], p, DT, 2, tape=tape)
    if not profile:
        out["gm"], out["gH"] = ctx.heff_backward(g, p)
        out["lam"], out["lamh"] = g.clone(), torch.zeros(3, dtype=ctx.tdtype, device="cuda")
        ctx.step_backward(tape, 2, p, DT, out["lam"], out["lamh"])
    return out


@pytest.mark.parametrize("n,dtype", _cases())
@pytest.mark.parametrize("profile", [0, 1])
def test_checked_calls_equal_unchecked(n, dtype, profile):
    magx, ctx, m, g = _setup(n, dtype)
    if profile:
        s = _profile(n, ctx.tdtype)
        ctx.set_ms_profile(s)
    plain, checked = (_outputs(magx, ctx, m, g, c, profile) for c in (0, 1))
    differ = [k for k in plain if not torch.equal(plain[k], checked[k])]
    assert not differ


@pytest.mark.parametrize("n", [(37, 11, 5), (40, 12, 2)])
@pytest.mark.parametrize("dtype", [0, 1])
def test_overflow_inside_a_call_is_reported(n, dtype):
    # the input is finite; a stage inside the call overflows
    magx, ctx, m, _ = _setup(n, dtype)
    p = magx.make_params(check_finite=1, renorm=0, **MAT)
    dt = 1e30 if dtype == 0 else 1e200
    for call in (lambda y: ctx.step(y, p, dt, 1), lambda y: ctx.step(y, p, dt, 18),
                 lambda y: ctx.step(y, p, dt, 1, tape=ctx.tape(1)), lambda y: ctx.step_euler(y, p, dt, 4),
                 lambda y: ctx.step_mri(y, p, dt, 1)):
        call(m.clone())
        assert ctx.status() == -6
    ctx.step(m, p, DT, 1)
    assert ctx.status() == 0


@pytest.mark.parametrize("n,dtype", _cases())
@pytest.mark.parametrize("profile", [0, 1])
def test_taped_steps_equal_untaped(n, dtype, profile):
    magx, ctx, m, _ = _setup(n, dtype)
    if profile:
        s = _profile(n, ctx.tdtype)
        ctx.set_ms_profile(s)
    p = magx.make_params(**MAT)
    for steps in (1, 18):
        a, b = m.clone(), m.clone()
        ctx.step(a, p, DT, steps)
        ctx.step(b, p, DT, steps, tape=ctx.tape(steps))
        assert torch.equal(a, b), steps


# enough members that the stage kernels of the batch are those of a full card, without
# loads ahead of the inverse x pass: (grid, members in single and in double precision)
FULL = [((8, 35, 1), 32, 16), ((128, 32, 1), 40, 20), ((33, 20, 3), 20, 10), ((90, 20, 3), 16, 12), ((37, 11, 5), 20, 11),
        ((250, 30, 2), 20, 10)]
TERMS = [(31, 2), (31, 0), (1, 2), (3, 1), (2, 2), (4 | 2, 2), (1 | 8, 0), (16, 2)]


@pytest.mark.parametrize("n,b32,b64", FULL)
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("terms,renorm", TERMS)
def test_members_of_full_batches_equal_single_systems(n, b32, b64, dtype, terms, renorm):
    from paper_2602_12242_amd import magx
    B, N = (b32, b64)[dtype], n[0] * n[1] * n[2]
    p = magx.make_params(renorm=renorm, **{**MAT, "terms": terms})
    one, many = magx.Context(n, D, dtype=dtype), magx.Context(n, D, dtype=dtype, nbatch=B)
    m = torch.stack([torch.from_numpy(random_unit_field(n, 910 + b, 2)) for b in range(B)]).to("cuda", one.tdtype)
    g = torch.stack([torch.from_numpy(random_vector_field(n, 950 + b)) for b in range(B)]).to("cuda", one.tdtype)

    def outputs(ctx, m, g):
        out, tape, lam = [ctx.heff(m, p)], ctx.tape(1), g.clone()
        for call in (lambda y: ctx.step(y, p, DT, 3), lambda y: ctx.step_euler(y, p, 0.1 * DT, 2),
                     lambda y: ctx.step(y, p, DT, 1, tape=tape)):
            out.append(m.clone())
            call(out[-1])
        tn = N * ctx.nbatch
        out.append(tape.view(ctx.tdtype)[12 * tn:24 * tn].view((4,) + ctx.shape).movedim(0, -5))      # H_1 ... H_4
        ctx.step_backward(tape, 1, p, DT, lam, torch.zeros(ctx.lead + (3,), dtype=ctx.tdtype, device="cuda"))
        return out + [lam]

    got = outputs(many, m, g)
    for b in (0, B // 2, B - 1):
        for k, (x, y) in enumerate(zip(outputs(one, m[b].contiguous(), g[b].contiguous()), got)):
            assert torch.equal(x, y[b]), (b, k)
