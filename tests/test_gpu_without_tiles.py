"""The paths that cooperative launches otherwise take the runs from: the resident workgroup of small
sets (nb_set_tiles(0)), and an ensemble's global steps in lanes and layouts (nb_ens_set_teams(0))."""
import numpy as np
import pytest

import oracle
from paper_astro_ph_0702058_amd import nbody
from paper_astro_ph_0702058_amd.plummer import plummer

pytestmark = pytest.mark.gpu


def _small(n, prec, resident, calls):
    st = nbody.DeviceState(*plummer(n, 27))
    with nbody.Context(n, 1 / 256, lmin=3, precision=prec) as ctx:
        ctx.nb_set_resident(resident)
        ctx.nb_set_tiles(0)
        ctx.nb_bind(st)
        ctx.nb_init(0.01)
        e0 = sum(ctx.nb_energy())
        for t_end, max_steps in calls:
            ctx.nb_run(0.01, t_end, max_steps=max_steps, chunk=16)
        c = ctx.nb_read_control()
        e1 = sum(ctx.nb_energy())
    return c, st.numpy(), abs(e1 / e0 - 1)


# one and several staging passes of the j-particles, and the most that a workgroup holds
@pytest.mark.parametrize("prec,n", [("ds", 64), ("ds", 256), ("ds", 257), ("ds", 1024), ("fp64", 400),
                                    ("fp64", 513), ("fp64", 1024), ("fp32", 512), ("fp32", 513),
                                    ("fp32", 1024)])
def test_resident_workgroup_against_the_chain(prec, n):
    """FP64 and double-single take the same block steps with positions to 1e-12 (only summation orders
    differ); FP32 the same steps within 2 % and an energy error of the same size.  A limit on the steps
    stops both at that step."""
    calls = [(1 / 16, 0)]
    (ca, a, da), (cb, b, db) = (_small(n, prec, r, calls) for r in (1024, 0))
    assert ca.t_cur == cb.t_cur and ca.n_steps > 10
    if prec == "fp32":
        assert abs(ca.n_steps - cb.n_steps) <= 0.02 * cb.n_steps
        assert da <= 3 * db + 1e-9 and db <= 3 * da + 1e-9
    else:
        assert ca.n_steps == cb.n_steps and ca.n_active_sum == cb.n_active_sum
        assert np.array_equal(a["level"], b["level"]) and np.array_equal(a["tick"], b["tick"])
        assert np.max(np.abs(a["x"] - b["x"])) < 1e-12
    c, *_ = _small(n, prec, 1024, [(1 / 8, 37)])
    assert c.n_steps == 37


def _ensemble(sizes, prec, t_end, graph=True, lanes=None, layout=None, split=None, max_steps=0, polls=0):
    parts = [plummer(int(k), 100 + c) for c, k in enumerate(sizes)]
    st = nbody.DeviceState(*(np.concatenate([p[k] for p in parts]) for k in range(3)))
    with nbody.Ensemble(sizes, [1.0 / k for k in sizes], lmin=3, precision=prec) as ens:
        ens.nb_ens_set_teams(polls)
        ens.nb_ens_bind(st)
        if layout:
            ens.nb_ens_set_layout(**layout)
        if split:
            ens.nb_ens_set_split(split)
        if lanes is not None:
            ens.nb_ens_set_lanes(lanes)
        ens.nb_ens_init(0.02)
        ens.nb_ens_run(0.02, t_end, steps_per_launch=8, max_steps=max_steps, use_graph=graph)
        assert ens.nb_ens_took_teams() == (polls > 0 and graph)
        ctl = ens.nb_ens_control()
        e = ens.nb_ens_energy()
    return [(c.n_steps, c.n_active_sum, c.t_cur) for c in ctl], st.numpy(), e, parts


def _same(a, b):
    assert a[0] == b[0]
    for key in a[1]:
        assert np.array_equal(a[1][key], b[1][key]), key
    assert np.array_equal(a[2][0], b[2][0]) and np.array_equal(a[2][1], b[2][1])


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("graph", [True, False])
def test_lanes_of_global_steps(prec, graph):
    """Lanes of one, two and three groups end bitwise where one lane does, with and without graphs, and
    stop after the same number of global steps."""
    sizes = [70, 600, 1300, 90, 2100, 300, 64]
    for t_end, max_steps in ((1 / 16, 0), (1.0, 16)):
        ref = _ensemble(sizes, prec, t_end, max_steps=max_steps)
        assert max_steps == 0 or all(s[0] == max_steps for s in ref[0])
        for lanes in (None, [1, 0, 0, 1, 0, 1, 1], [2, 0, 1, 2, 0, 2, 1]):
            if graph and lanes is None:
                continue
            _same(_ensemble(sizes, prec, t_end, graph, lanes, max_steps=max_steps), ref)


def test_layouts_of_global_steps():
    """Tiles per item, unroll and lanes per row only reorder sums: the same block steps in FP64,
    positions to 1e-12; and the layouts do reach the kernels (the bits of the larger clusters differ)."""
    sizes = [70, 600, 1300]
    outs = [_ensemble(sizes, "fp64", 1 / 32, layout=layout, split=split)
            for layout, split in ((dict(tiles_per_item=1, ipl=1, unroll=2), None),
                                  (dict(tiles_per_item=4, ipl=1, unroll=1), None),
                                  (dict(tiles_per_item=[1, 2, 3], ipl=1, unroll=2), None),
                                  (dict(tiles_per_item=1, ipl=1, unroll=2), 1),
                                  (dict(tiles_per_item=2, ipl=1, unroll=2), 16),
                                  (dict(tiles_per_item=1, ipl=1, unroll=1), 64))]
    for o in outs[1:]:
        assert o[0] == outs[0][0]
        assert np.max(np.abs(o[1]["x"] - outs[0][1]["x"])) < 1e-12
    assert any(not np.array_equal(o[1]["x"], outs[0][1]["x"]) for o in outs[1:])


@pytest.mark.parametrize("prec", ["fp64", "ds"])
@pytest.mark.parametrize("polls", [0, 1 << 20])
def test_both_paths_follow_oracle_runs(prec, polls):
    """Global steps and teams: every cluster's block steps, levels and ticks are its oracle run's."""
    sizes = [1, 64, 257, 700, 1000, 256]
    steps, g, _, parts = _ensemble(sizes, prec, 1 / 8, polls=polls)
    off = np.concatenate([[0], np.cumsum(sizes)])
    for c, (x, v, m) in enumerate(parts):
        ref = oracle.BlockIntegrator(x, v, m, eps=1.0 / sizes[c], nu=0.02, lmin=3)
        ref.run_until(1 / 8)
        sl = slice(off[c], off[c + 1])
        assert steps[c] == (ref.n_steps, ref.n_active_total, ref.t), c
        assert np.array_equal(g["level"][sl], ref.level) and np.array_equal(g["tick"][sl], ref.tick)
        assert np.max(np.abs(g["x"][sl] - ref.x)) < 1e-10, c
