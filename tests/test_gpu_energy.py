"""nb_energy and nb_ens_energy sum each pair once, in items of rows and tiles; against the FP64
oracle over the sizes where the items change: a lone particle, edges of a tile, the lanes per row,
and the blocks of two rows a lane (from 128 tiles)."""
import numpy as np
import pytest
import torch

import oracle
from paper_astro_ph_0702058_amd import nbody
from paper_astro_ph_0702058_amd.plummer import plummer

pytestmark = pytest.mark.gpu

# a pair term is off by a few units of 1.1e-16; 256 of them are summed plainly, the rest with
# compensation: at most 256 * 1.1e-16
TOL = 3e-14


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 1000, 2049, 5000, 32512, 32513, 33000])
@pytest.mark.parametrize("eps", [1 / 256, 0.0])
def test_energy_against_oracle(n, eps):
    x, v, m = plummer(n, 80 + n)
    if n > 2:
        x[1] = x[0]  # a pair at zero separation adds nothing without softening
        m = m * np.linspace(0.5, 1.5, n)
    if n == 1:
        x, v = x + 0.3, v + 0.2
    st = nbody.DeviceState(x, v, m)
    with nbody.Context(n, eps, precision="fp64") as ctx:
        ctx.nb_bind(st)
        first = ctx.nb_energy()
        assert first == ctx.nb_energy()
    ek, ep = oracle.energy(x, v, m, eps * eps)
    assert abs(first[0] - ek) <= TOL * abs(ek)
    assert abs(first[1] - ep) <= TOL * abs(ep)


def test_ensemble_energy_against_oracle():
    sizes = np.array([1, 2, 255, 256, 257, 700, 1500])
    parts = [plummer(int(k), 90 + c) for c, k in enumerate(sizes)]
    x, v, m = (np.concatenate([p[k] for p in parts]) for k in range(3))
    eps = 1.0 / (sizes + 1)
    st = nbody.DeviceState(x, v, m)
    with nbody.Ensemble(sizes, eps, precision="fp64") as ens:
        ens.nb_ens_bind(st)
        ens.nb_ens_init(0.01)
        ek, ep = ens.nb_ens_energy()
    for c, (px, pv, pm) in enumerate(parts):
        rk, rp = oracle.energy(px, pv, pm, eps[c] ** 2)
        assert abs(ek[c] - rk) <= TOL * abs(rk) and abs(ep[c] - rp) <= TOL * abs(rp), c
