"""The tuner's choices, with a library context that returns given solutions and times."""

import pytest

import stinputs
from paper_1911_06066_amd import autotune


@pytest.fixture
def fake(monkeypatch):
    import torch

    import paper_1911_06066_amd as lib
    from paper_1911_06066_amd import klmodes
    made = []

    class Context:
        off = {}      # (sweeps, ratio): distance of its solutions
        seconds = {}

        def __init__(self, wl, level_tuning=None, **kw):
            self.tuning, self.G = level_tuning, kw.get("team_size", 1)
            made.append([t[:2] for t in level_tuning if t])

        def __enter__(self):
            return self

        def __exit__(self, *exc):
            return False

        def close(self):
            pass

        def kl_synthesize(self, level, modes, xi):
            return xi

        def st_solve(self, level, sigma):
            key = next(t[:2] for t in self.tuning if t)
            st = dict(status=0, device_seconds=self.seconds.get(key, 1.0), newton_iters=1, krylov_iters=1)
            return torch.full((2, 3), 0.5 + self.off.get(key, 0.0), dtype=torch.float64), [st]

        def timings(self):
            return dict(solve_blocks=self.G, solve_teams=1)

        def mlmc_estimate(self, *a):
            pass

    monkeypatch.setattr(lib, "Context", Context)
    monkeypatch.setattr(klmodes, "workload_modes", lambda wl: [torch.zeros(1).numpy()] * len(wl["levels"]))
    monkeypatch.setattr(torch, "device", lambda name: "cpu")
    monkeypatch.setattr(torch.cuda, "get_device_name", lambda i: "none")
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    return Context, made


def _wl():
    return stinputs.workload("small_mc_2d", levels=[(17, 17)], steps=[4], n_modes=4, samples=[2])


@pytest.mark.parametrize("off,taken", [(1e-13, (13, 9.0)), (1e-10, (0, 0.0))])
def test_fixed_setting_is_taken_only_where_its_solutions_agree(fake, off, taken):
    Context, _ = fake
    Context.seconds = {(0, 0.0): 1.0, (11, 7.0): 2.0, (13, 9.0): 0.5}
    Context.off = {(13, 9.0): off}
    e = autotune.tune(_wl(), log=lambda s: None)["levels"][0]
    assert (e["smooth_sweeps"], e["cheb_ratio"]) == taken


def test_refine_leaves_automatic_levels_alone(fake):
    _, made = fake
    rec = {"precision": "fp64", "levels": [{"smooth_sweeps": 0, "cheb_ratio": 0.0, "team_seconds": []}]}
    autotune.refine(_wl(), rec, [None], [None], log=lambda s: None)
    assert made == [[(0, 0.0)]] and rec["levels"][0]["smooth_sweeps"] == 0
