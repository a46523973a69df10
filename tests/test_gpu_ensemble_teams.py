"""nb_ens_run in one launch of teams (graph runs) against global steps (eager runs): the same block
steps, the sums of clusters of more than four tiles in another order."""
import numpy as np
import pytest

from paper_astro_ph_0702058_amd import nbody
from paper_astro_ph_0702058_amd.plummer import plummer

pytestmark = pytest.mark.gpu


def _run(sizes, prec, calls):
    parts = [plummer(int(k), 300 + c) for c, k in enumerate(sizes)]
    st = nbody.DeviceState(*(np.concatenate([p[k] for p in parts]) for k in range(3)))
    eps = [1.0 / max(k, 16) for k in sizes]
    with nbody.Ensemble(sizes, eps, lmin=3, precision=prec) as ens:
        ens.nb_ens_bind(st)
        ens.nb_ens_init(0.02)
        for t_end, max_steps, graph in calls:
            ens.nb_ens_run(0.02, t_end, steps_per_launch=8, max_steps=max_steps, use_graph=graph)
        ctl = ens.nb_ens_control()
        e = ens.nb_ens_energy()
    return st.numpy(), [(c.n_steps, c.n_active_sum, c.t_cur, c.n_act) for c in ctl], e


# whole tiles, one particle past a tile, a lone particle, and the most tiles a team takes (32)
SIZES = [8192, 4097, 2000, 1024, 257, 256, 64, 2, 1]


@pytest.mark.parametrize("prec", ["fp64", "ds"])
def test_teams_take_the_same_steps(prec):
    """FP64 and double-single: block steps equal, positions to 1e-13 (summation order, 1e-16 of
    the forces over t = 1/32 and what close pairs make of it)."""
    a = _run(SIZES, prec, [(1 / 32, 0, True)])
    b = _run(SIZES, prec, [(1 / 32, 0, False)])
    assert a[1] == b[1]
    assert np.array_equal(a[0]["tick"], b[0]["tick"]) and np.array_equal(a[0]["level"], b[0]["level"])
    assert np.max(np.abs(a[0]["x"] - b[0]["x"])) < 1e-13


def test_small_clusters_keep_every_bit():
    """Up to four tiles the sums are in the same order too."""
    sizes = [1024, 900, 512, 300, 64, 5]
    a = _run(sizes, "fp32", [(1 / 32, 0, True)])
    b = _run(sizes, "fp32", [(1 / 32, 0, False)])
    assert a[1] == b[1]
    for key in a[0]:
        assert np.array_equal(a[0][key], b[0][key]), key


def test_teams_stop_go_on_and_hand_over():
    """A step limit stops every cluster after as many block steps as global steps; teams go on from
    there, and so do global steps, from the block the teams left selected; a run of clusters that
    are done changes nothing."""
    sizes = [1000, 700, 300, 64]
    a = _run(sizes, "fp64", [(1 / 16, 0, False)])
    for calls in ([(1 / 16, 20, True), (1 / 16, 0, True), (1 / 16, 0, True)],
                  [(1 / 16, 20, True), (1 / 16, 0, False)],
                  [(1 / 16, 20, False), (1 / 16, 0, True)]):
        b = _run(sizes, "fp64", calls)
        assert a[1] == b[1]
        for key in a[0]:
            assert np.array_equal(a[0][key], b[0][key]), (calls, key)
    c, d = (_run(sizes, "fp64", [(1 / 16, 20, graph)]) for graph in (True, False))
    assert c[1] == d[1] and all(s[0] == 24 for s in c[1])  # batches of 8 steps


def test_a_cluster_too_large_for_a_team():
    """More than 32 tiles: the whole ensemble takes global steps, bitwise the eager run."""
    a = _run([8193, 64], "fp64", [(1 / 64, 0, True)])
    b = _run([8193, 64], "fp64", [(1 / 64, 0, False)])
    assert a[1] == b[1]
    for key in a[0]:
        assert np.array_equal(a[0][key], b[0][key]), key
