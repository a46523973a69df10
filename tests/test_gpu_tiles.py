"""nb_run by one cooperative launch of tile owners (sets of 1025 to 65536 particles) against the
chain of launches per step (nb_set_resident(0)): the same sums in the same order, so times,
levels, blocks and the whole state must agree bitwise."""
import numpy as np
import pytest
import torch

from paper_astro_ph_0702058_amd import nbody
from paper_astro_ph_0702058_amd.plummer import plummer

pytestmark = pytest.mark.gpu


def _run(n, prec, resident, lmin, calls, eta=0.01, eps=1 / 256):
    x, v, m = plummer(n, 60 + n)
    st = nbody.DeviceState(x, v, m)
    with nbody.Context(n, eps, lmin=lmin, precision=prec) as ctx:
        ctx.nb_set_resident(resident)
        ctx.nb_bind(st)
        ctx.nb_init(eta)
        for t_end, max_steps, chunk in calls:
            ctx.nb_run(eta, t_end, max_steps=max_steps, chunk=chunk)
        c = ctx.nb_read_control()
        idx, cnt = ctx.nb_active()
        block = np.sort(nbody.read_device_int32(idx, c.n_act))
        # a force call may follow a run (the j-particle stream is the last step's)
        acc = torch.zeros((3, n), dtype=torch.float64, device="cuda")
        jerk, pot = torch.zeros_like(acc), torch.zeros(n, dtype=torch.float64, device="cuda")
        ctx.nb_force(acc, jerk, pot)
        ctx.nb_sync()
        g = st.numpy()
    return c, block, g, [q.cpu().numpy() for q in (acc, jerk, pot)]


def _same(a, b):
    (ca, ba, ga, fa), (cb, bb, gb, fb) = a, b
    assert (ca.t_cur, ca.n_steps, ca.n_active_sum, ca.n_act) == \
        (cb.t_cur, cb.n_steps, cb.n_active_sum, cb.n_act)
    assert np.array_equal(ba, bb)
    for key in ga:
        assert np.array_equal(ga[key], gb[key]), key
    for p, q in zip(fa, fb):
        assert np.array_equal(p, q)


# one particle past the one-workgroup limit, ragged last tiles (of 1, 136 and 255 particles), whole
# tiles, and enough tiles that each has a workgroup to itself; a run that ends at its time, one
# cut by a step limit in the middle of a launch, and one after it
@pytest.mark.parametrize("n,t", [(1025, 1 / 64), (1536, 1 / 64), (5000, 1 / 128), (16384, 1 / 256),
                                 (33023, 1 / 512), (65536, 1 / 512)])
@pytest.mark.parametrize("prec", ["fp32", "fp64", "ds"])
def test_tiled_run_equals_launch_chain(n, t, prec):
    calls = [(t, 0, 64), (2 * t, 37, 16), (2 * t, 5, 64)]
    a = _run(n, prec, 1024, 3, calls)
    assert a[0].n_steps > 40
    _same(a, _run(n, prec, 0, 3, calls))


@pytest.mark.parametrize("n,lmin", [(3000, 12), (20000, 13), (65536, 14)])
def test_blocks_too_large_for_the_tiled_path(n, lmin):
    """A largest step so small that nearly every block is the whole system: such blocks end the
    tiled launch and take the launch chain."""
    calls = [(8 * 2.0 ** -lmin, 0, 64)]
    a = _run(n, "fp32", 1024, lmin, calls)
    assert a[0].n_active_sum > 8 * 0.5 * n
    _same(a, _run(n, "fp32", 0, lmin, calls))


@pytest.mark.parametrize("n", [1300, 9000])
def test_pending_levels_before_a_tiled_run(n):
    """A block corrected by the separate calls has its new levels before the first tiled step."""
    out = []
    for resident in (1024, 0):
        x, v, m = plummer(n, 5)
        st = nbody.DeviceState(x, v, m)
        with nbody.Context(n, 1 / 256, precision="fp64") as ctx:
            ctx.nb_set_resident(resident)
            ctx.nb_bind(st)
            ctx.nb_init(0.01)
            acc = torch.zeros((3, n), dtype=torch.float64, device="cuda")
            jerk, pot = torch.zeros_like(acc), torch.zeros(n, dtype=torch.float64, device="cuda")
            idx, cnt = ctx.nb_active()
            ctx.nb_predict()
            ctx.nb_force(acc, jerk, pot, i_idx=idx, n_i=cnt, n_i_max=n)
            ctx.nb_correct(acc, jerk, pot)
            ctx.nb_run(0.01, 1 / 256)
            c = ctx.nb_read_control()
            out.append((c.n_steps, c.n_active_sum, st.numpy()))
    (sa, aa, ga), (sb, ab, gb) = out
    assert sa == sb > 5 and aa == ab
    for key in ga:
        assert np.array_equal(ga[key], gb[key]), key


@pytest.mark.parametrize("prec,n", [("ds", 257), ("fp64", 401), ("fp64", 1024), ("ds", 1000)])
def test_small_sets_tiled(prec, n):
    """Sets that one workgroup could hold take its slices (1024 lanes over the block) on the tiled
    path, so their sums differ from the launch chain's in order: the same steps, and coordinates
    within 8 ulp of the largest (16: 1.8e-15), far above what the forces' rounding moves them in
    t = 1/64 (1e-14 of an acceleration of order 10 over t^2 / 2: 1e-17)."""
    out = []
    for resident in (1024, 0):
        x, v, m = plummer(n, 17)
        st = nbody.DeviceState(x, v, m)
        with nbody.Context(n, 1 / 256, lmin=6, precision=prec) as ctx:
            ctx.nb_set_resident(resident)
            ctx.nb_bind(st)
            ctx.nb_init(0.01)
            ctx.nb_run(0.01, 1 / 64)
            c = ctx.nb_read_control()
            out.append((c.n_steps, c.n_active_sum, st.numpy()))
    (sa, aa, ga), (sb, ab, gb) = out
    assert sa == sb > 10 and aa == ab
    assert np.array_equal(ga["tick"], gb["tick"]) and np.array_equal(ga["level"], gb["level"])
    assert np.max(np.abs(ga["x"] - gb["x"])) < 1.5e-14


def test_tiled_runs_from_two_threads():
    """Two contexts on streams of their own, each wanting every compute unit: the cooperative
    launches never wait for each other half resident, and each run ends as it does alone."""
    import threading
    n, t = 16384, 1 / 256
    alone = [_run_state(n, seed, t, torch.cuda.current_stream()) for seed in (1, 2)]
    got, streams = [None, None], [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()

    def work(k):
        with torch.cuda.stream(streams[k]):
            for _ in range(3):
                got[k] = _run_state(n, k + 1, t, streams[k])

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    for a, g in zip(alone, got):
        assert g is not None
        for key in a:
            assert np.array_equal(a[key], g[key]), key


def _run_state(n, seed, t, stream):
    x, v, m = plummer(n, seed)
    st = nbody.DeviceState(x, v, m)
    with nbody.Context(n, 1 / 256, precision="fp32", stream=stream) as ctx:
        ctx.nb_bind(st)
        ctx.nb_init(0.01)
        ctx.nb_run(0.01, t, chunk=8)
        ctx.nb_sync()
        return st.numpy()
