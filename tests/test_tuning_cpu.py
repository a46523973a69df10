"""The ensemble's tuner on a stand-in whose runs take a made-up time: layouts are timed where they count,
and the fastest of the search, the default layout and the teams stays set."""
import types

import numpy as np
import pytest
import torch

from paper_astro_ph_0702058_amd import tuning


class Stand:
    """Teams take `teams` seconds (None: they cannot run) whatever the layout; global steps take less the
    nearer smin is to `best`."""

    def __init__(self, teams, best, clock, polls=None):
        self.offsets = np.array([0, 300, 1300, 5300])
        self.t_teams, self.best, self.clock, self.polls = teams, best, clock, polls
        self.smin, self.took = 8, False

    def nb_ens_set_teams(self, polls):
        self.polls = polls

    def nb_ens_took_teams(self):
        return self.took

    def nb_ens_set_layout(self, tpi, ipl, unroll):
        self.unroll = unroll

    def nb_ens_set_split(self, smin):
        self.smin = smin

    def nb_ens_init(self, eta):
        pass

    def nb_ens_run(self, eta, t_end, steps_per_launch):
        self.took = self.t_teams is not None and self.polls != 0 and self.smin >= 8
        steps = 1.0 + 0.1 * abs(np.log2(self.smin / self.best)) + 0.05 * (self.unroll == 1)
        self.clock[0] += self.t_teams if self.took else steps


@pytest.mark.parametrize("teams,best,polls,smin,on,beats", [
    (0.5, 4, None, 8, True, False),     # teams fastest: the default layout, which they need
    (0.5, 4, 0, 4, False, True),        # the caller has switched them off
    (2.0, 4, None, 4, False, True),     # the search's winner fastest
    (2.0, 8, None, 8, False, False),    # the default layout fastest
    (None, 16, None, 16, False, True),  # teams cannot run
])
def test_the_fastest_stays_set(monkeypatch, teams, best, polls, smin, on, beats):
    import time
    clock = [0.0]
    monkeypatch.setattr(time, "perf_counter", lambda: clock[0])
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    ens = Stand(teams, best, clock, polls)
    state = types.SimpleNamespace(x=torch.zeros(3), v=torch.zeros(3))
    out = tuning.ensemble_autotune(ens, state, torch.ones(3), torch.ones(3), 0.02)
    assert out["smin"] == ens.smin == smin and ens.unroll == 2
    assert out["teams"] == on == (ens.polls > 0) and out["beats_default"] == beats
    ens.nb_ens_run(0.02, 1.0, 128)
    assert ens.took == on
    assert torch.equal(state.x, torch.ones(3))
