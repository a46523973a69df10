"""The order of nb_run's launches (csrc/run_loop.hpp) against a simulated device, on the CPU: every
run ends, with its steps counted, whichever launches the device refuses or ends early."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# A device with `total` block steps to t_end, whose block `i` is too large for tiles where
# i % 7 < large, and which refuses tiled launches from the refuse-th on.  Prints steps taken,
# steps the loop counted, whether it stopped for `done`, and the looks at the record.
SIMULATION = r"""
#include "run_loop.hpp"
#include <cstdio>
#include <cstdlib>
using namespace nbody;
int main(int argc, char **argv) {
    const long total = atol(argv[1]), refuse = atol(argv[2]), large = atol(argv[3]);
    RunLoop l{(int32_t)atol(argv[4]), atol(argv[5]), argv[6][0] == '1', argv[7][0] == '1'};
    long at = 0, launches = 0, looks = 0, turns = 0;
    bool done = false;
    RunLoop::Path p;
    for (int32_t k; l.next(p, k);) {
        if (++turns > 20 * total + 1000) { printf("endless\n"); return 1; }
        int32_t steps = 0;
        if (p == RunLoop::TILES) {
            if (launches++ >= refuse) { l.refused(); continue; }
            while (!done && steps < k && !(at < total && at % 7 < large)) {
                if (at == total) done = true;
                else ++at, ++steps;
            }
        } else {
            for (int32_t i = 0; i < k; ++i) {
                if (at == total) done = true;
                else ++at;
            }
        }
        if (!l.enqueued(p, k)) continue;
        ++looks;
        if (done) break;
        if (p == RunLoop::TILES) l.tiled(k, steps);
    }
    printf("%ld %lld %d %ld\n", at, (long long)l.done_steps, (int)done, looks);
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
def simulate(tmp_path_factory):
    exe = _build(tmp_path_factory, "run_loop", SIMULATION)

    def run(*args):
        r = subprocess.run([exe, *(str(int(a)) for a in args)], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, (args, r.stdout)
        return [int(w) for w in r.stdout.split()]

    return run


@pytest.mark.parametrize("chunk", [1, 2, 64, 2 ** 31 - 1])
@pytest.mark.parametrize("large", [0, 1, 7])
@pytest.mark.parametrize("resident", [0, 1])
def test_every_run_ends(simulate, chunk, large, resident):
    total = 500
    for refuse in (0, 1, 3, 10 ** 9):
        at, counted, done, looks = simulate(total, refuse, large, chunk, 0, 1, resident)
        assert at == total and done, (refuse, at, done)
        at, counted, done, looks = simulate(total, refuse, large, chunk, 37, 1, resident)
        assert at == counted == 37 and not done, (refuse, at, counted, done)


def test_epochs_fit_their_words(tmp_path_factory):
    """However many launches there were, an epoch fits above the words' low bits and is new, or the
    words are zeroed for it."""
    r = subprocess.run([_build(tmp_path_factory, "epochs", EPOCHS)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
    assert 9 <= int(r.stdout) <= 10
