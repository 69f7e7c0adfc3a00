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
