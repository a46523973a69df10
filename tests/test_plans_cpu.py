"""Force plans (csrc/plan.hpp) on the CPU: tiled runs take only blocks that the launch chain sums in
the same order."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# argv: n, target, kmax, ib_max, smax, hmax, fill, pack.  Prints the lengths of blocks that tiles
# take, and those up to 8192 that are taken although the chain's plan joins tiles (none).
SOURCE = r"""
#include "plan.hpp"
#include <cstdio>
#include <cstdlib>
using namespace nbody;
int main(int argc, char **argv) {
    int32_t v[9];
    for (int i = 1; i < 9; ++i) v[i] = atoi(argv[i]);
    const Spread sp{v[5], v[6], v[7], WG, v[8]};
    const int32_t T = (v[1] + TJ - 1) / TJ, most = 8192;
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
    """At 256 compute units and the default targets, where no block that tiles take has joined ones:
    all up to a limit, but for the lengths of several i-blocks that take more slices."""
    fill = 256 * 1024 // ((n + 255) // 256)
    spread = (64, 4, fill, 0) if prec == "fp32" else (64, 1, fill, 1)
    lo, hi, most = limits(n, 4096, 1 << 16, 256, *spread)
    assert most == {33023: 31 * 256, 50000: 5120, 65536: 4096}.get(n, 8192)
    if prec == "fp32":
        assert lo == most
    else:
        assert lo == most or 1024 <= lo < hi < 4096


@pytest.mark.parametrize("target,kmax,ib", [(1024, 1 << 16, 256), (4096, 8, 256), (4096, 1 << 16, 512), (64, 64, 1024)])
def test_limit_follows_the_variant(limits, target, kmax, ib):
    for n in (1300, 5000, 40000):
        lo, hi, most = limits(n, target, kmax, ib, 64, 1, 0, 0)
        if kmax < (n + 255) // 256:
            assert most == 0
