"""Short lists on small systems spread each row over more lanes: four helper lanes per slice in
FP32, which must not change a bit of the sums, and more slices in FP64, double-single and
fixed-point arithmetic, which only reorders them."""
import numpy as np
import pytest
import torch

from paper_astro_ph_0702058_amd import nbody
from paper_astro_ph_0702058_amd.plummer import plummer, sample_indices
from _parity import check, reference

pytestmark = pytest.mark.gpu

N = 5000


def _forces(prec, eps, lists):
    """Forces on each list (None: all particles) as numpy arrays with the rows last."""
    x, v, m = plummer(N, 71)
    st = nbody.DeviceState(x, v, m)
    out = []
    with nbody.Context(N, eps, precision=prec) as ctx:
        ctx.nb_bind(st)
        ctx.nb_predict(torch.zeros(1, dtype=torch.int64, device="cuda"))
        for idx in lists:
            k = N if idx is None else len(idx)
            acc = torch.zeros((3, k), dtype=torch.float64, device="cuda")
            jerk, pot = torch.zeros_like(acc), torch.zeros(k, dtype=torch.float64, device="cuda")
            ii = None if idx is None else torch.as_tensor(idx.astype(np.int32), device="cuda")
            cnt = None if idx is None else torch.tensor([k], dtype=torch.int32, device="cuda")
            ctx.nb_force(acc, jerk, pot, i_idx=ii, n_i=cnt)
            ctx.nb_sync()
            out.append([q.cpu().numpy() for q in (acc, jerk, pot)])
    return (x, v, m), out


@pytest.mark.parametrize("prec,eps", [("fp32", 1 / 256), ("fp32", 0.0), ("fp32fixed", 1 / 256)])
@pytest.mark.parametrize("count", [256, 257, 1000, 3276, 3277])
def test_helper_lanes_keep_every_bit(prec, eps, count):
    """The full call takes one lane per row (5000 rows fill the chip); FP32 lists of up to 3276
    rows (a quarter of the lanes that fill it) take four, the same tile sums, bitwise; so do
    fixed-point sums in any number of slices."""
    idx = sample_indices(N, count, count)
    _, (full, part) = _forces(prec, eps, [None, idx])
    for f, p in zip(full, part):
        assert np.array_equal(f[..., idx], p)


@pytest.mark.parametrize("prec", ["fp32", "fp64", "ds"])
@pytest.mark.parametrize("eps", [1 / 256, 0.0])
def test_short_lists_against_oracle(prec, eps):
    """Every lane split: 64 slices down to one, with and without helpers."""
    lists = [sample_indices(N, k, k) for k in (1, 3, 4, 5, 9, 16, 17, 64, 65, 129, 255, 300, 1025)]
    (x, v, m), out = _forces(prec, eps, lists)
    for idx, (acc, jerk, pot) in zip(lists, out):
        ref, scale = reference(x, v, m, eps * eps, idx=idx)
        check(prec, (acc.T, jerk.T, pot), ref, scale, f"{prec} eps={eps} {len(idx)} rows")


@pytest.mark.parametrize("prec", ["fp64", "ds"])
def test_lists_of_several_blocks_leave_little_padding(prec):
    """Lists longer than a workgroup in a system large enough that they fill the chip: one slice
    (1024 rows), two (881), four (300, 700, 1030, 2100) of the j-slots, host and device counts."""
    n, eps = 40000, 1 / 256
    x, v, m = plummer(n, 72)
    st = nbody.DeviceState(x, v, m)
    with nbody.Context(n, eps, precision=prec) as ctx:
        ctx.nb_bind(st)
        ctx.nb_predict(torch.zeros(1, dtype=torch.int64, device="cuda"))
        for k in (300, 700, 881, 1024, 1030, 2100):
            idx = sample_indices(n, k, k)
            ii = torch.as_tensor(idx.astype(np.int32), device="cuda")
            got = []
            for cnt in (None, torch.tensor([k], dtype=torch.int32, device="cuda")):
                acc = torch.zeros((3, k), dtype=torch.float64, device="cuda")
                jerk, pot = torch.zeros_like(acc), torch.zeros(k, dtype=torch.float64, device="cuda")
                ctx.nb_force(acc, jerk, pot, i_idx=ii, n_i=cnt)
                ctx.nb_sync()
                got.append([q.cpu().numpy() for q in (acc, jerk, pot)])
            assert all(np.array_equal(a, b) for a, b in zip(*got))
            acc, jerk, pot = got[0]
            ref, scale = reference(x, v, m, eps * eps, idx=idx)
            check(prec, (acc.T, jerk.T, pot), ref, scale, f"{prec} {k} rows of {n}")
