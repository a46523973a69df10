"""Force plans (csrc/plan.hpp) on the CPU: tiled runs take only blocks that the launch chain sums in
the same order."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# argv: n, target, kmax, ib_max, smax, hmax, fill, pack [, whole].  Prints the lengths of blocks that tiles
# take, and those up to 8192 that are taken although the chain's plan joins tiles (none).
SOURCE = r"""
#include "plan.hpp"
#include <cstdio>
#include <cstdlib>
using namespace nbody;
int main(int argc, char **argv) {
    int32_t v[9];
    for (int i = 1; i < 9; ++i) v[i] = atoi(argv[i]);
    Spread sp{v[5], v[6], v[7], WG, v[8]};
    const int32_t T = (v[1] + TJ - 1) / TJ, most = 8192;
    sp.hfill = v[6] > 1 ? v[7] : 0;
    sp.tq = v[6] > 1 ? 16 * T : 0;
    if (argc > 9) sp.whole = atoi(argv[9]);
    const BlockRows rows = rows_by_tiles(v[1], v[4], v[2], v[3], sp, sp, most);
    printf("%d %d %d", rows.lo, rows.hi, rows.most);
    for (int32_t m = 1; m <= most; ++m) {
        // the chain's own items: a plane of tps tiles each
        const ForcePlan p = make_plan(m, v[1], v[4], v[2], v[3], sp);
        if (rows.has(m) && (p.tps != 1 || p.K != T)) printf(" %d", m);
    }
    printf("\n");
}
"""


@pytest.fixture(scope="module")
def limits(tmp_path_factory):
    d = tmp_path_factory.mktemp("plans")
    src, exe = str(d / "a.cpp"), str(d / "a")
    open(src, "w").write(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
                    os.path.join(ROOT, "paper_astro_ph_0702058_amd", "csrc"), "-o", exe, src], check=True)

    def run(*args):
        r = subprocess.run([exe, *(str(a) for a in args)], capture_output=True, text=True, check=True)
        lo, hi, most, *joined = (int(w) for w in r.stdout.split())
        assert lo <= most and hi <= most and not joined
        return lo, hi, most

    return run


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [1025, 5000, 16384, 16385, 33023, 50000, 65536])
def test_tiled_blocks_join_no_tiles(limits, n, prec):
    """At 256 compute units the default gives every block that tiles take a plane per tile; its target
    alone joins tiles of some lengths."""
    tiles = (n + 255) // 256
    fill = 256 * 1024 // tiles
    spread = (64, 4, fill, 0) if prec == "fp32" else (64, 1, fill, 1)
    lo, hi, most = limits(n, 4096, 1 << 16, 256, *spread, 7168)
    assert lo == most == {33023: 31 * 256, 50000: 7168, 65536: 7168}.get(n, 8192)
    lo, hi, most = limits(n, 4096, 1 << 16, 256, *spread)
    assert lo == most or (prec == "fp64" and 1024 <= lo < hi < 4096)


@pytest.mark.parametrize("target,kmax,ib", [(1024, 1 << 16, 256), (4096, 8, 256), (4096, 1 << 16, 512), (64, 64, 1024)])
def test_limit_follows_the_variant(limits, target, kmax, ib):
    for n in (1300, 5000, 40000):
        lo, hi, most = limits(n, target, kmax, ib, 64, 1, 0, 0)
        if kmax < (n + 255) // 256:
            assert most == 0


# argv: n, target, kmax.  For every spread a context may have: lists whose plan needs more partial rows
# than the one without a spread, that the workspace is sized for, or whose lanes do not fit a wave.
ROWS = r"""
#include "plan.hpp"
#include <cstdio>
#include <cstdlib>
using namespace nbody;
int main(int, char **argv) {
    const int32_t n = atoi(argv[1]), target = atoi(argv[2]), kmax = atoi(argv[3]);
    const int32_t T = (n + TJ - 1) / TJ, fill = 256 * 1024 / T, tq = (int32_t)(((int64_t)T * 4096 + 255) / 256);
    Spread all[5] = {Spread{64, 4, fill}, Spread{64, 1, fill, WG, 1}, Spread{64, 1, fill, WG, 1},
                     Spread{64, 1, fill, WG, 1}, Spread{4, 1, fill}};
    all[0].hfill = fill; all[0].tq = tq;
    all[2].most = 8; all[2].tq = tq;
    all[3].most = 32; all[3].tq = tq;
    all[4].most = 4; all[4].tq = tq; all[4].scalar = 1;
    int bad = 0;
    for (int k = 0; k < 5; ++k)
        for (int32_t m = 1; m <= n; m += m < 20000 ? 1 : 977) {
            Spread held_by{all[k].smax, 1, 0};
            held_by.whole = all[k].whole = T <= 256 && target == 4096 && kmax >= T && k != 4 ? LONG_LIST : 0;
            const ForcePlan p = make_plan(m, n, WG, target, kmax, all[k]);
            const ForcePlan q = make_plan(m, n, WG, target, kmax, held_by);
            const int64_t need = p.K > 1 ? p.K * p.P : 0, held = q.K > 1 ? q.K * q.P : 0;
            const bool whole = (int64_t)p.K * p.tps >= p.ntiles && (int64_t)p.n_iblk * p.ib >= m &&
                               p.items == p.n_iblk * p.K && p.ib * p.S * p.H == WG;
            if (need > held || !whole || p.S * p.H > 64 || p.S < q.S)
                bad += printf("spread %d rows %d: %lld of %lld\n", k, m, (long long)need, (long long)held) > 0;
        }
    return bad != 0;
}
"""


@pytest.fixture(scope="module")
def rows_check(tmp_path_factory):
    d = tmp_path_factory.mktemp("rows")
    src, exe = str(d / "a.cpp"), str(d / "a")
    open(src, "w").write(ROWS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
                    os.path.join(ROOT, "paper_astro_ph_0702058_amd", "csrc"), "-o", exe, src], check=True)
    return exe


@pytest.mark.parametrize("n", [1, 100, 257, 1000, 5000, 20000, 65536, 100003, 1 << 20, 1 << 24])
@pytest.mark.parametrize("target,kmax", [(4096, 1 << 16), (65536, 64), (1024, 1 << 16)])
def test_spread_lists_fit_the_planes(rows_check, n, target, kmax):
    """Every list length: more lanes per row cover every tile and row, at most 64 a row, and need no
    more partial sums than the plan that the workspace is sized for."""
    r = subprocess.run([rows_check, str(n), str(target), str(kmax)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout[:400]
