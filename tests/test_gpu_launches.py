"""Cooperative launches of nb_run and nb_ens_run: their workgroups start together or leave to another
path, and their epochs last.  (The order of the launches is simulated in test_run_loop_cpu.py.)"""
import numpy as np
import pytest
import torch

from paper_astro_ph_0702058_amd import nbody
from paper_astro_ph_0702058_amd.plummer import plummer

pytestmark = pytest.mark.gpu


def _run(n, prec, calls, polls=None, resident=1024, lmin=3, seed=17, chunk=64, pending=0,
         variant=None):
    """(block steps, particle steps), state after nb_run calls of (t_end, max_steps)."""
    st = nbody.DeviceState(*plummer(n, seed))
    with nbody.Context(n, 1 / 256, lmin=lmin, precision=prec) as ctx:
        ctx.nb_set_resident(resident)
        if polls is not None:
            ctx.nb_set_tiles(polls)
        if variant is not None:
            ctx.nb_set_variant(1, variant)
        ctx.nb_bind(st)
        ctx.nb_init(2.5e-5 if pending else 0.01)
        if pending:  # steps by the separate calls, the last one's new levels to come
            acc = torch.zeros((3, n), dtype=torch.float64, device="cuda")
            jerk, pot = torch.zeros_like(acc), torch.zeros(n, dtype=torch.float64, device="cuda")
            for _ in range(pending):
                ctx.nb_schedule_block(2.5e-5)
                idx, cnt = ctx.nb_active()
                ctx.nb_predict()
                ctx.nb_force(acc, jerk, pot, i_idx=idx, n_i=cnt, n_i_max=n)
                ctx.nb_correct(acc, jerk, pot)
        for t_end, max_steps in calls:
            ctx.nb_run(0.01, t_end, max_steps=max_steps, chunk=chunk)
        c = ctx.nb_read_control()
    return (c.n_steps, c.n_active_sum, c.t_cur), st.numpy()


def _same(a, b):
    assert a[0] == b[0] and a[0][0] > 10
    for key in a[1]:
        assert np.array_equal(a[1][key], b[1][key]), key


def test_many_runs_of_the_largest_chunk():
    """Runs of one launch each (the largest chunk) do not use up the launches' epochs: 600 short ones
    end where a single run does, bitwise."""
    t = 600 * 2.0 ** -15
    cuts = [(t * (k + 1) / 600, 0) for k in range(600)]
    _same(_run(1100, "fp32", cuts, lmin=6, chunk=2 ** 31 - 1), _run(1100, "fp32", [(t, 0)], lmin=6))


@pytest.mark.parametrize("prec,n", [("fp32", 3000), ("fp64", 16384), ("ds", 2000), ("fp64", 700),
                                    ("ds", 300), ("fp32", 1024)])
def test_workgroups_that_do_not_start_together(prec, n):
    """Workgroups that look for each other once only leave before the first step, unless they chance to
    be together; the launch chain, or the resident workgroup of a set that it holds, takes the run:
    bitwise as without tiles, but for the resident workgroup's order of sums in FP64 and double-single
    (1e-12 in the positions)."""
    calls = [(1 / 128, 0), (1 / 32, 21)]
    a, b = (_run(n, prec, calls, polls=p) for p in (1, 0))
    if n <= 1024 and prec != "fp32":
        assert a[0] == b[0] and np.array_equal(a[1]["level"], b[1]["level"])
        assert np.array_equal(a[1]["tick"], b[1]["tick"])
        assert np.max(np.abs(a[1]["x"] - b[1]["x"])) < 1e-12
        return
    _same(a, b)
    if n > 1024:
        _same(_run(n, prec, calls, polls=1), _run(n, prec, calls, resident=0))


@pytest.mark.parametrize("n", [1300, 9000])
@pytest.mark.parametrize("pending", [1, 4, 16])
def test_pending_levels_before_the_chain_takes_over(n, pending):
    """A block corrected by the separate calls gets its new levels once, also where the tiled launch
    after that leaves to the chain: the run's eta allows steps 20 times those of the blocks before it,
    and a particle at a multiple of four steps would be doubled twice."""
    calls = [(1 / 64, 0)]
    _same(_run(n, "fp64", calls, polls=1, pending=pending),
          _run(n, "fp64", calls, resident=0, pending=pending))


@pytest.mark.parametrize("prec,n,lo,hi", [("fp64", 33023, 2049, 7168), ("fp32", 58000, 4609, 7168)])
def test_large_blocks_are_summed_in_one_order(prec, n, lo, hi):
    """Blocks of lo to hi rows, whose tiles the chain joins: whichever launch takes them, and wherever
    the launches are cut, the run's bits are the chain's."""
    st = nbody.DeviceState(*plummer(n, 17))
    with nbody.Context(n, 1 / 256, lmin=3, precision=prec) as ctx:
        ctx.nb_bind(st)
        ctx.nb_init(0.01)
        blocks = []
        for _ in range(24):
            ctx.nb_step(0.01, 1)
            blocks.append(ctx.nb_read_control().n_act)
    assert any(lo <= b <= hi for b in blocks), blocks
    calls = [(1.0, 24)]
    ref = _run(n, prec, calls, resident=0)
    for chunk in (64, 5, 1):
        _same(_run(n, prec, calls, chunk=chunk), ref)


@pytest.mark.parametrize("variant", [dict(ipl=2, unroll=2, target=2048, kmax=1 << 16),
                                     dict(ipl=1, unroll=1, target=1024, kmax=1 << 16),
                                     dict(ipl=1, unroll=2, target=4096, kmax=8)])
def test_block_variant_keeps_its_order(variant):
    """A caller's block-step variant decides the order of the sums on every path."""
    calls = [(1 / 128, 0)]
    a, b = (_run(5000, "fp32", calls, resident=r, variant=variant) for r in (1024, 0))
    _same(a, b)


def _ensemble(sizes, prec, calls, polls=None):
    parts = [plummer(int(k), 300 + c) for c, k in enumerate(sizes)]
    st = nbody.DeviceState(*(np.concatenate([p[k] for p in parts]) for k in range(3)))
    with nbody.Ensemble(sizes, [1.0 / max(k, 16) for k in sizes], lmin=3, precision=prec) as ens:
        if polls is not None:
            ens.nb_ens_set_teams(polls)
        ens.nb_ens_bind(st)
        ens.nb_ens_init(0.02)
        for t_end, max_steps, graph in calls:
            ens.nb_ens_run(0.02, t_end, steps_per_launch=8, max_steps=max_steps, use_graph=graph)
        ctl = ens.nb_ens_control()
    return [(c.n_steps, c.n_active_sum, c.t_cur, c.n_act) for c in ctl], st.numpy()


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("max_steps", [0, 20])
def test_teams_that_do_not_start_together(prec, max_steps):
    """Global steps take the run, unless the workgroups chance to be together, with or without a step
    limit: the same block steps as without teams, the positions to 1e-13 (FP64: the order of sums)."""
    sizes = [8192, 4097, 2000, 1024, 257, 64, 2, 1]
    calls = [(1 / 32, max_steps, True)] + [(1 / 32, 0, True)] * (max_steps > 0)
    a, b = (_ensemble(sizes, prec, calls, polls) for polls in (1, 0))
    assert a[0] == b[0]
    assert np.array_equal(a[1]["tick"], b[1]["tick"]) and np.array_equal(a[1]["level"], b[1]["level"])
    if prec == "fp32":
        for key in a[1]:
            assert np.array_equal(a[1][key], b[1][key]), key
    else:
        assert np.max(np.abs(a[1]["x"] - b[1]["x"])) < 1e-13
        assert a[0] == _ensemble(sizes, prec, calls)[0]


def test_polls_are_checked():
    with nbody.Context(64, 1 / 256) as ctx, nbody.Ensemble([64], 1 / 64) as ens:
        for bad in (-1, (1 << 24) + 1):
            for call in (ctx.nb_set_tiles, ens.nb_ens_set_teams):
                with pytest.raises(nbody.NBodyError, match="polls"):
                    call(bad)


def test_small_runs_from_many_threads():
    """Twelve contexts of small sets on streams of their own, more workgroups than the device holds:
    their launches run side by side or make room for each other, and each run ends as it does alone."""
    import threading
    n, count = 1024, 12

    def run(seed, stream):
        with torch.cuda.stream(stream):
            st = nbody.DeviceState(*plummer(n, seed))
            with nbody.Context(n, 1 / 256, lmin=6, precision="fp32", stream=stream) as ctx:
                ctx.nb_bind(st)
                for _ in range(3):
                    ctx.nb_init(0.01)
                    ctx.nb_run(0.01, 1 / 64, chunk=16)
                ctx.nb_sync()
                return st.numpy()

    alone = [run(k, torch.cuda.current_stream()) for k in range(count)]
    streams, got = [torch.cuda.Stream() for _ in range(count)], [None] * count
    torch.cuda.synchronize()
    threads = [threading.Thread(target=lambda k=k: got.__setitem__(k, run(k, streams[k]))) for k in range(count)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    for a, g in zip(alone, got):
        assert g is not None
        for key in a:
            assert np.array_equal(a[key], g[key]), key


def _blocks(sizes, prec, lmin, polls, max_steps=0):
    parts = [plummer(int(k), 300 + c) for c, k in enumerate(sizes)]
    st = nbody.DeviceState(*(np.concatenate([p[k] for p in parts]) for k in range(3)))
    with nbody.Ensemble(sizes, [1.0 / k for k in sizes], lmin=lmin, precision=prec) as ens:
        if polls is not None:
            ens.nb_ens_set_teams(polls)
        ens.nb_ens_bind(st)
        ens.nb_ens_init(0.02)
        while not all(c.flags for c in ens.nb_ens_control()):  # max_steps steps a call
            ens.nb_ens_run(0.02, 1 / 64, steps_per_launch=8, max_steps=max_steps)
    return st.numpy()


@pytest.mark.parametrize("sizes,lmin,teams", [([4096], 11, False), ([2048, 1500], 11, False),
                                              ([2048], 3, True), ([2000] * 12, 3, True)])
def test_large_blocks_of_few_clusters_take_the_whole_device(sizes, lmin, teams):
    """Where nearly every block is a whole cluster, a few workgroups would take five times as long
    over a block step as global steps: those take the run (their FP64 sums are in another order
    than teams', so the bits tell).  The choice is the start's: wherever the run is cut, its bits are
    the same."""
    ref = _blocks(sizes, "fp64", lmin, (1 << 20) if teams else 0)
    other = _blocks(sizes, "fp64", lmin, 0 if teams else 1 << 20)
    assert not np.array_equal(ref["x"], other["x"])
    for max_steps in (0, 8):
        got = _blocks(sizes, "fp64", lmin, None, max_steps)
        for key in ref:
            assert np.array_equal(got[key], ref[key]), (key, max_steps)
