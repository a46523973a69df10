"""Short lists at the edges of the rules for lanes per row: helpers up to half the chip's lanes (FP32),
second slices while they spread the work (fixed point), and at most 8 or 32 slices on systems too
large for tiled runs (FP64, double-single)."""
import numpy as np
import pytest
import torch

from paper_astro_ph_0702058_amd import nbody
from paper_astro_ph_0702058_amd.plummer import plummer, sample_indices
from _parity import check, reference

pytestmark = pytest.mark.gpu


def _forces(prec, n, eps, lists):
    """Forces on each list (None: all particles), with a host and a device count."""
    x, v, m = plummer(n, 73)
    st = nbody.DeviceState(x, v, m)
    out = []
    with nbody.Context(n, eps, precision=prec) as ctx:
        ctx.nb_bind(st)
        ctx.nb_predict(torch.zeros(1, dtype=torch.int64, device="cuda"))
        for idx in lists:
            k = n if idx is None else len(idx)
            ii = None if idx is None else torch.as_tensor(idx.astype(np.int32), device="cuda")
            got = []
            for cnt in (None, torch.tensor([k], dtype=torch.int32, device="cuda")):
                acc = torch.zeros((3, k), dtype=torch.float64, device="cuda")
                jerk, pot = torch.zeros_like(acc), torch.zeros(k, dtype=torch.float64, device="cuda")
                if idx is not None or cnt is None:
                    ctx.nb_force(acc, jerk, pot, i_idx=ii, n_i=cnt)
                    got.append((acc, jerk, pot))
            ctx.nb_sync()
            out.append([[q.cpu().numpy() for q in g] for g in got])
    return (x, v, m), out


@pytest.mark.parametrize("prec,n,counts", [
    ("fp32", 5000, (256, 1638, 1639, 2500)),
    ("fp32", 20000, (256, 414, 415, 1000)),
    ("fp32fixed", 20000, (64, 65, 100, 400, 600, 800, 1000, 1500)),
    ("fp32fixed", 8000, (400, 600, 2048, 2500, 4000))])
def test_bits_do_not_depend_on_the_lanes(prec, n, counts):
    """FP32 tile sums of one slice keep their order (every tile has a plane of its own in all these
    calls), and fixed-point sums have none: the rows of the full call (FP32 at N = 20000, where that
    joins tiles: of the longest list), bitwise."""
    longest = sample_indices(n, max(counts), 5)
    lists = [longest if prec == "fp32" and n > 5000 else None] + [longest[:k] for k in counts]
    _, (full, *parts) = _forces(prec, n, 1 / 256, lists)
    rows = longest if lists[0] is None else np.arange(len(longest))
    for k, part in zip(counts, parts):
        for got in part:
            for f, p in zip(full[0], got):
                assert np.array_equal(f[..., rows[:k]], p), k


@pytest.mark.parametrize("prec", ["fp64", "ds"])
def test_lists_of_large_systems_against_oracle(prec):
    n, eps = 70000, 1 / 256
    lists = [sample_indices(n, k, k) for k in (1, 8, 10, 24, 33, 60, 100, 250, 300, 600)]
    (x, v, m), out = _forces(prec, n, eps, lists)
    for idx, got in zip(lists, out):
        assert all(np.array_equal(a, b) for a, b in zip(*got))
        acc, jerk, pot = got[0]
        ref, scale = reference(x, v, m, eps * eps, idx=idx)
        check(prec, (acc.T, jerk.T, pot), ref, scale, f"{prec} {len(idx)} rows")
