"""nb_run on states whose particle times are not those of the scheduler's last block step: moved by
shared steps, or bound to a new context in mid-run.  The block is every particle at the smallest
t_i + dt_i (Sec. 2), whichever path nb_run takes for the size, and no step is counted that moves
nothing."""
import numpy as np
import pytest
import torch

from paper_astro_ph_0702058_amd import nbody
from paper_astro_ph_0702058_amd.plummer import plummer

pytestmark = pytest.mark.gpu

LMAX, EPS, ETA = 26, 1 / 256, 0.01


def _context(n, prec, lmin=3):
    st = nbody.DeviceState(*plummer(n, 40 + n))
    ctx = nbody.Context(n, EPS, lmin=lmin, lmax=LMAX, precision=prec)
    ctx.nb_bind(st)
    return st, ctx


def _apart(ctx, n, t_end):
    """Block steps to t_end by the separate calls."""
    acc = torch.zeros((3, n), dtype=torch.float64, device="cuda")
    jerk, pot = torch.zeros_like(acc), torch.zeros(n, dtype=torch.float64, device="cuda")
    while True:
        ctx.nb_schedule_block(ETA)
        if ctx.nb_read_control().t_next > t_end * 2 ** LMAX:
            return
        idx, cnt = ctx.nb_active()
        ctx.nb_predict()
        ctx.nb_force(acc, jerk, pot, i_idx=idx, n_i=cnt, n_i_max=n)
        ctx.nb_correct(acc, jerk, pot)


# below, at and past the sizes that one workgroup holds, in each arithmetic's tiles
@pytest.mark.parametrize("prec,n", [("fp64", 300), ("fp64", 401), ("fp64", 1024), ("fp64", 1025),
                                    ("fp64", 3000)])
@pytest.mark.parametrize("shared", [1, 3])
def test_run_after_shared_steps(prec, n, shared):
    """Shared steps leave every tick ahead of the scheduler's time and, for steps above the shared
    one, off their multiples.  Summation order apart (1e-12) the run is that of separate calls,
    with its block steps; a step limit counts steps that are taken."""
    out = []
    for run in (True, False):
        st, ctx = _context(n, prec)
        with ctx:
            ctx.nb_init(ETA)
            ctx.nb_shared_step(2.0 ** -9, shared)
            if run:
                ctx.nb_run(ETA, 1 / 64, max_steps=5, chunk=2)
                assert ctx.nb_read_control().n_steps == 5
                ctx.nb_run(ETA, 1 / 64)
            else:
                _apart(ctx, n, 1 / 64)
            c = ctx.nb_read_control()
            out.append((c.n_steps, c.n_active_sum, c.t_cur, st.numpy()))
    a, b = out
    assert a[:3] == b[:3] and a[0] > 5
    for key in ("tick", "level"):
        assert np.array_equal(a[3][key], b[3][key]), key
    assert np.max(np.abs(a[3]["x"] - b[3]["x"])) < 1e-12


@pytest.mark.parametrize("prec,n", [("fp32", 513), ("fp64", 700), ("ds", 300), ("ds", 1700),
                                    ("fp64", 3000), ("fp32", 5000)])
def test_state_bound_in_mid_run(prec, n):
    """A run cut in two, its second part by a new context, ends as the run in one context does:
    bitwise on the sizes that take the same path, to rounding where one workgroup takes over."""
    out = []
    for cut in (False, True):
        st, ctx = _context(n, prec)
        with ctx:
            ctx.nb_init(ETA)
            ctx.nb_run(ETA, 1 / 64)
            first = ctx.nb_read_control().n_steps
            if not cut:
                ctx.nb_run(ETA, 1 / 32)
                out.append((ctx.nb_read_control().n_steps, st.numpy()))
        if cut:
            with nbody.Context(n, EPS, lmin=3, lmax=LMAX, precision=prec) as new:
                new.nb_bind(st)
                new.nb_run(ETA, 1 / 32)
                out.append((first + new.nb_read_control().n_steps, st.numpy()))
    (sa, a), (sb, b) = out
    if n > 1024:
        assert sa == sb
        for key in a:
            assert np.array_equal(a[key], b[key]), key
    elif prec != "fp32":
        assert sa == sb and np.array_equal(a["tick"], b["tick"])
        assert np.max(np.abs(a["x"] - b["x"])) < 1e-12
    else:
        assert abs(sa - sb) <= 0.02 * sa


def test_particle_behind_is_reported():
    """A particle whose next time is behind the scheduler's is NB_ESTATE, as for the launch chain."""
    st, ctx = _context(3000, "fp64")
    with ctx:
        ctx.nb_init(ETA)
        ctx.nb_run(ETA, 1 / 64)
        st.tick[7] = 0
        st.level[7] = LMAX
        with pytest.raises(nbody.NBodyError) as e:
            ctx.nb_run(ETA, 1 / 32)
        assert e.value.status == nbody.NB_ESTATE
