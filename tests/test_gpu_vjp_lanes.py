"""The force VJP of small systems spreads each row over more lanes: four helpers in FP32, which
must not change a bit, and up to 64 slices of the j-slots in FP64, which only reorders the sums.
The same particles followed by massless ones with zero adjoints (exact zeros in every sum) fill
the chip and take one lane a row."""
import numpy as np
import pytest
import torch

from paper_astro_ph_0702058_amd import nbody
from paper_astro_ph_0702058_amd.plummer import plummer

pytestmark = pytest.mark.gpu


def _vjp(prec, eps, x, v, m, A, B):
    n = len(m)
    st = nbody.DeviceState(x, v, m)
    t = lambda a: torch.tensor(np.ascontiguousarray(a.T), dtype=torch.float64, device="cuda")
    with nbody.Context(n, eps, precision=prec) as ctx:
        ctx.nb_bind(st)
        ctx.nb_predict(torch.zeros(1, dtype=torch.int64, device="cuda"))
        xb = torch.zeros((3, n), dtype=torch.float64, device="cuda")
        vb, mb = torch.zeros_like(xb), torch.zeros(n, dtype=torch.float64, device="cuda")
        ctx.nb_force_vjp(t(A), t(B), xb, vb, mb)
        ctx.nb_sync()
    return [q.cpu().numpy() for q in (xb, vb, mb)]


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("eps", [1 / 128, 0.0])
@pytest.mark.parametrize("n", [1, 3, 63, 64, 65, 255, 257, 1000, 2047, 3000])
def test_lanes_of_small_vjps(prec, eps, n):
    """FP32 bitwise; FP64 within 1e-11 of the largest component (a few thousand terms reordered)."""
    total = 7000
    x, v, m = plummer(3000, 43)
    x, v, m = x[:n], v[:n], m[:n]
    rng = np.random.default_rng(n)
    A, B = rng.normal(size=(n, 3)), rng.normal(size=(n, 3))
    far = np.zeros((total - n, 3))
    far[:, 0] = 50.0 + 0.01 * np.arange(total - n)
    none = np.zeros((total - n, 3))
    got = _vjp(prec, eps, x, v, m, A, B)
    ref = _vjp(prec, eps, np.concatenate([x, far]), np.concatenate([v, none]),
               np.concatenate([m, np.zeros(total - n)]), np.concatenate([A, none]),
               np.concatenate([B, none]))
    for name, g, r in zip(("x", "v", "m"), got, ref):
        r = r[..., :n]
        if prec == "fp32":
            assert np.array_equal(g, r), name
        else:
            assert np.max(np.abs(g - r)) <= 1e-11 * np.max(np.abs(r)), name
