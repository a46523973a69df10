"""The order of nb_run's launches (csrc/run_loop.hpp) against a simulated device, on the CPU: every
run ends, with its steps counted, whichever launches the device refuses or ends early."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# A device with 500 block steps to t_end, whose block `i` is too large for tiles where i % 7 < large,
# which refuses tiled launches from the refuse-th on and whose every miss-th does not start together
# (0: none): a run to the end and one of 37 steps for every refuse and miss.
SIMULATION = r"""
#include "run_loop.hpp"
#include <cstdio>
#include <cstdlib>
using namespace nbody;
static bool run(long large, RunLoop l, long refuse, long miss) {
    const long total = 500;
    long at = 0, launches = 0, turns = 0;
    bool done = false;
    RunLoop::Path p;
    for (int32_t k; l.next(p, k);) {
        if (++turns > 20 * total + 1000) return printf("endless\n"), false;
        int32_t steps = 0;
        if (p == RunLoop::TILES) {
            if (launches++ >= refuse) { l.refused(); continue; }
            if (miss && launches % miss == 0) { l.missed(); continue; }
            while (!done && steps < k && !(at < total && at % 7 < large)) {
                if (at == total) done = true;
                else ++at, ++steps;
            }
        } else {
            for (int32_t i = 0; i < k && !done; ++i) {
                if (at == total) done = true;
                else ++at;
            }
        }
        if (!l.enqueued(p, k)) continue;
        if (done) break;
        if (p == RunLoop::TILES) l.tiled(k, steps);
    }
    const bool right = l.max_steps > 0 ? at == l.max_steps && l.done_steps == at && !done
                                       : at == total && done;
    if (!right) printf("refuse %ld miss %ld: %ld steps, %ld counted\n", refuse, miss, at, (long)l.done_steps);
    return right;
}
int main(int, char **argv) {
    const long large = atol(argv[1]);
    const bool resident = argv[3][0] == '1';
    bool ok = true;
    for (long refuse : {0l, 1l, 3l, 1000000000l})
        for (long miss = 0; miss < 4; ++miss)
            for (long max_steps : {0l, 37l})
                ok = run(large, RunLoop{(int32_t)atol(argv[2]), max_steps, true, resident, resident}, refuse, miss) && ok;
    return !ok;
}
"""

EPOCHS = r"""
#include "run_loop.hpp"
#include <cstdio>
using namespace nbody;
int main() {
    // launches of the most steps, ten times as many as use up all epochs
    Epochs e;
    const uint64_t n = TL_STEPS + 2;
    uint64_t before = 0, over = 0;
    for (uint64_t launch = 0; launch < 10 * (Epochs::LAST / n); ++launch) {
        bool again;
        const uint64_t first = e.take(n, again), last = first + n - 1;
        if (first == 0 || last << TL_SHIFT >> TL_SHIFT != last) { printf("does not fit\n"); return 1; }
        if (!again && first <= before) { printf("used before\n"); return 1; }
        before = last;
        over += again;
    }
    printf("%d\n", (int)over);
}
"""


def _build(tmp_path_factory, name, text):
    d = tmp_path_factory.mktemp(name)
    src, exe = str(d / "a.cpp"), str(d / "a")
    open(src, "w").write(text)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I",
                    os.path.join(ROOT, "paper_astro_ph_0702058_amd", "csrc"), "-o", exe, src], check=True)
    return exe


@pytest.fixture(scope="module")
def simulation(tmp_path_factory):
    return _build(tmp_path_factory, "run_loop", SIMULATION)


@pytest.mark.parametrize("chunk", [1, 2, 64, 2 ** 31 - 1])
@pytest.mark.parametrize("large", [0, 1, 7])
@pytest.mark.parametrize("resident", [0, 1])
def test_every_run_ends(simulation, chunk, large, resident):
    r = subprocess.run([simulation, str(large), str(chunk), str(resident)], capture_output=True, text=True,
                       timeout=60)
    assert r.returncode == 0, r.stdout


def test_epochs_fit_their_words(tmp_path_factory):
    """However many launches there were, an epoch fits above the words' low bits and is new, or the
    words are zeroed for it."""
    r = subprocess.run([_build(tmp_path_factory, "epochs", EPOCHS)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
    assert 9 <= int(r.stdout) <= 10
