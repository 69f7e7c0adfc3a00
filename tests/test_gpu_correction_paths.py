"""GPU: which way the defect corrections of a case go.

The results agree on every way, so these tests look at the counts: corrections
only where preconditioner applications equal Newton steps, teams by workgroups
per team, and the 2D sweeps with the stencil in registers by the algorithmic
bytes of a sample, which count their arrays once per correction and those of the
tiled sweep pairs once per pass.
"""

import numpy as np
import pytest

import oracle.api as oapi
import stinputs

pytestmark = pytest.mark.gpu


def _solve(shape, m, S, precision, **over):
    import torch
    from paper_1911_06066_amd import Context
    dim = len(shape)
    base = "small_mc_2d" if dim == 2 else "slab3d"
    wl = stinputs.workload(base, levels=[shape], steps=[m], n_modes=8, precision=precision,
                           kl_grid=(17, 17) if dim == 2 else (9, 9, 3), ic_radius=0.3, sigma_f0=4e-3)
    wl["T"] = m / 64.0
    basis = oapi.kl_basis(wl)
    sig = oapi.kl_synthesize(oapi.kl_modes(wl, 0, basis), stinputs.xi(base, 0, S, wl["n_modes"]), wl["sigma_f0"])
    with Context(wl, **over) as ctx:
        u, stats = ctx.st_solve(0, torch.from_numpy(sig).cuda())
        t = ctx.timings()
    U_ref, _ = oapi.st_solve(wl, 0, sig, mode="timestep")
    assert np.abs(u.cpu().numpy() - U_ref).max() < 1e-9
    return stats, t["solve_blocks"] / t["solve_teams"]


def _register_bytes(shape, m, precision, newton):
    """Bytes of a sample without a previous one whose corrections all run in registers."""
    n, ne = int(np.prod(shape)), int(np.prod([k - 1 for k in shape]))
    w = 4 if precision == "mixed" else 8
    start = (48 + w) * n + 40 * (5 * w * n + 8 * ne)  # state, power iteration
    return start + m * 56 * n + newton * ((24 + 3 * w) * n + 8 * ne + (4 * w + 32) * n + 8 * ne)


@pytest.mark.parametrize("c", [
    dict(shape=(33, 33), lds_kb=16), dict(shape=(33, 33), precision="mixed", lds_kb=12), dict(shape=(49, 49)),
    dict(shape=(33, 129), lds_kb=24),
])
def test_team_of_a_2d_solve_fits_the_register_sweeps(c):
    """One workgroup's rows do not fit: the team is one whose rows do."""
    p = c.get("precision", "fp64")
    over = dict(lds_kb=c["lds_kb"]) if "lds_kb" in c else {}
    stats, G = _solve(c["shape"], 4, 1, p, **over)
    assert G > 1
    s = stats[0]
    assert s["krylov_iters"] == s["newton_iters"]
    assert s["algorithmic_bytes"] == _register_bytes(c["shape"], 4, p, s["newton_iters"])


@pytest.mark.parametrize("c", [
    # 2D with the stencil in registers: bands of teams, deep and shallow halos, one
    # workgroup at the ends of what fits 256 and 512 threads
    dict(shape=(17, 31), G=4, register=True), dict(shape=(129, 40), G=5, register=True),
    dict(shape=(257, 23), precision="mixed", G=2, register=True), dict(shape=(5, 9), G=3, register=True),
    dict(shape=(3, 3), precision="mixed", G=1, register=True), dict(shape=(33, 33), G=1, register=True),
    dict(shape=(65, 65), G=1, register=True), dict(shape=(45, 45), G=1, register=True),
    dict(shape=(257, 11), G=1, register=True),
    # more columns of three nodes than the threads hold: 833 of 3 x 256, 1806 of 3 x 512, 2838 of 4 x 512
    dict(shape=(49, 49), G=1, register=False), dict(shape=(129, 40), G=1, register=False),
    dict(shape=(129, 65), precision="mixed", G=1, register=False),
    # 3D: bands of rows, groups of planes
    dict(shape=(9, 9, 5), G=1), dict(shape=(9, 9, 17), precision="mixed", G=3), dict(shape=(13, 13, 13), G=12),
])
def test_corrections_run_on_the_team_and_sweeps_meant(c):
    p = c.get("precision", "fp64")
    stats, G = _solve(c["shape"], 4, 1, p, team_size=c["G"])
    assert G == c["G"]
    s = stats[0]
    assert s["krylov_iters"] == s["newton_iters"]  # no GMRES
    if "register" in c:
        b = _register_bytes(c["shape"], 4, p, s["newton_iters"])
        assert (s["algorithmic_bytes"] == b) if c["register"] else (s["algorithmic_bytes"] > 1.2 * b)


@pytest.mark.parametrize("c", [
    dict(shape=(17, 17), smoother=1), dict(shape=(9, 9, 9), precision="mixed", smoother=1, smooth_omega=0.4),
    dict(shape=(17, 17), mg_levels=2), dict(shape=(17, 17, 9), mg_levels=-1),
])
def test_fixed_weights_and_v_cycles_take_gmres(c):
    over = {k: v for k, v in c.items() if k not in ("shape", "precision")}
    stats, _ = _solve(c["shape"], 4, 1, c.get("precision", "fp64"), **over)
    assert stats[0]["krylov_iters"] > 1.5 * stats[0]["newton_iters"]


def test_settings_for_gmres_do_not_make_failed_corrections():
    """A level's own settings that do not contract leave the corrections as they are without."""
    free, _ = _solve((17, 17), 8, 1, "fp64", team_size=1)
    for tuning in ((2, 5.0), (4, 10.0), (8, 30.0)):
        s, _ = _solve((17, 17), 8, 1, "fp64", team_size=1, level_tuning=[tuning])
        assert (s[0]["newton_iters"], s[0]["krylov_iters"]) == (free[0]["newton_iters"], free[0]["krylov_iters"])
