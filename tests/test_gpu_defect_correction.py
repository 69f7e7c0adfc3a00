"""GPU: Newton steps by Chebyshev defect correction against the oracle.

The slab systems of single-grid levels are solved by corrections u += P(A) r
whose interval is adapted from slab to slab, with GMRES as the way back.  The
cases reach each branch: the spectrum's own interval with trials of narrower
ones over many slabs and a lane of several samples, a level's own degree and
ratio, a degree too small to contract (GMRES within the slab, then for the
sample), a ratio too wide for corrections, and a small Newton limit.
Tolerance: the solver's Newton tolerance is 1e-10 per slab in the max norm, and
errors of a slab are damped by the following ones, so 1e-9 relative (FP64) as in
the other parity tests; 1e-8 with float32 corrections.
"""

import numpy as np
import pytest

import oracle.api as oapi
import stinputs

pytestmark = pytest.mark.gpu


@pytest.fixture
def torch_dev():
    import torch
    return torch, torch.device("cuda:0")


CASES = [
    # 2D, spectrum's interval, 40 slabs and a lane of three samples: several trials
    dict(shape=(17, 13), m=40, S=3, precision="fp64", G=1, lanes=1),
    dict(shape=(33, 25), m=24, S=2, precision="mixed", G=3),
    # stencil in registers: deep and shallow halos, the widest rows, uneven bands,
    # rows that do not fill a column of three; grids that do not fit (teams and alone)
    dict(shape=(17, 31), m=6, S=2, precision="fp64", G=4),
    dict(shape=(129, 40), m=4, S=2, precision="fp64", G=5),
    dict(shape=(257, 23), m=4, S=1, precision="mixed", G=2),
    dict(shape=(65, 65), m=4, S=1, precision="fp64", G=1),
    dict(shape=(5, 9), m=6, S=2, precision="fp64", G=3),
    dict(shape=(3, 3), m=4, S=2, precision="mixed", G=1),
    dict(shape=(257, 11), m=4, S=1, precision="fp64", G=1),
    dict(shape=(129, 65), m=4, S=1, precision="mixed", G=1),
    dict(shape=(33, 33), m=6, S=2, precision="fp64", G=3, lds_kb=16),
    # 3D, rows split over members, planes split over members
    dict(shape=(9, 9, 5), m=24, S=2, precision="fp64", G=1),
    dict(shape=(9, 9, 17), m=20, S=2, precision="mixed", G=3),
    # team size from the grid: bands of rows and groups of planes
    dict(shape=(13, 13, 13), m=8, S=2, precision="fp64", G=0),
    dict(shape=(9, 7, 9), m=8, S=3, precision="mixed", G=0),
    # smooth initial state: narrower intervals are kept
    dict(shape=(17, 17), m=24, S=2, precision="fp64", G=1, ic_kind="gauss", ic_radius=0.5),
    # the level's own degree and ratio: enough, narrow, and too little to contract
    dict(shape=(33, 25), m=8, S=2, precision="fp64", G=2, tuning=(13, 9.0)),
    dict(shape=(17, 17), m=12, S=2, precision="fp64", G=1, tuning=(12, 3.0)),
    dict(shape=(17, 17), m=12, S=2, precision="fp64", G=1, tuning=(3, 30.0)),
    dict(shape=(9, 9, 5), m=8, S=2, precision="mixed", G=1, tuning=(4, 30.0)),
    # stiffness far above mass: GMRES from the first slab
    dict(shape=(17, 17), m=8, S=2, precision="fp64", G=1, sigma_f0=0.2),
    # fixed weights: GMRES only
    dict(shape=(17, 17), m=8, S=2, precision="fp64", G=1, smoother=1),
    dict(shape=(9, 9, 5), m=8, S=2, precision="fp64", G=1, smoother=1, smooth_omega=0.4),
    dict(shape=(9, 9, 9), m=8, S=2, precision="mixed", G=4, smoother=1, smooth_omega=0.4),
    # corrections do not count against the Newton limit
    dict(shape=(17, 17), m=32, S=2, precision="fp64", G=1, newton_max=2),
]


@pytest.mark.parametrize("c", CASES)
def test_defect_corrections_match_oracle(torch_dev, c):
    torch, dev = torch_dev
    from paper_1911_06066_amd import Context
    base = "small_mc_2d" if len(c["shape"]) == 2 else "slab3d"
    wl = stinputs.workload(base, levels=[c["shape"]], steps=[c["m"]], n_modes=8, precision=c["precision"],
                           kl_grid=(17, 17) if len(c["shape"]) == 2 else (9, 9, 3),
                           ic_radius=c.get("ic_radius", 0.3), ic_kind=c.get("ic_kind", "ball"),
                           sigma_f0=c.get("sigma_f0", 4e-3))
    basis = oapi.kl_basis(wl)
    sig = oapi.kl_synthesize(oapi.kl_modes(wl, 0, basis), stinputs.xi(base, 0, c["S"], wl["n_modes"]), wl["sigma_f0"])
    over = dict(team_size=c["G"])
    if "lanes" in c:
        over["max_lanes"] = c["lanes"]
    if "tuning" in c:
        over["level_tuning"] = [c["tuning"]]
    for k in ("smoother", "smooth_omega", "newton_max", "lds_kb"):
        if k in c:
            over[k] = c[k]
    with Context(wl, **over) as ctx:
        u, stats = ctx.st_solve(0, torch.from_numpy(sig).to(dev))
    assert all(s["status"] == 0 for s in stats), stats
    U_ref, _ = oapi.st_solve(wl, 0, sig, mode="timestep")
    d = np.abs(u.cpu().numpy() - U_ref).max() / np.abs(U_ref).max()
    assert d < (1e-9 if c["precision"] == "fp64" else 1e-8)
