"""States near the end of the float range (1e18, whose squared derivatives
overflow) on large Q2 boxes: where the small box's residual, shock-capturing
weights and stage are finite, its 5 x 5 x 5 copies' are."""
import numpy as np
import pytest

import synth
from synth import Params

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2601_16911_amd import cvw  # noqa: E402

EUL, BUR, ADV = (dict(flux=synth.EULER, flux_param=(1.4, 0, 0, 0)), dict(flux=synth.BURGERS, flux_param=(1.0, 0.8, 0.6, 0)),
                 dict(flux=synth.ADVECT_CONST, flux_param=(1.0, 0.5, 0.25, 0)))


def _run(mesh, u, prm):
    gm, cp = cvw.Mesh(mesh, 2, cvw.DG), cvw.make_params(prm)
    ws = cvw.alloc_workspace(gm, cp, 0)
    E, nv = mesh.n_cells, u.shape[0]
    d = torch.from_numpy(np.ascontiguousarray(u)).cuda().reshape(-1)
    R, S = torch.empty_like(d), torch.empty_like(d)
    gam, alpha = torch.empty(E, device="cuda"), torch.empty(E * 27, device="cuda")
    cand = torch.empty((mesh.n_vertices, 9), device="cuda")
    cvw.residual(gm, cp, d, R, gam, ws)
    cvw.vertex_candidates(gm, cp, d, cand, ws)
    cvw.rk_stage(gm, cp, d, cand, None, S, 1e-30, 0.0, 1.0, ws)
    cvw.sensor(gm, cp, d, gam, alpha, ws)
    return [np.isfinite(x.cpu().numpy()).reshape(-1, E, 27) for x in (R, S, alpha)]


@pytest.mark.parametrize("law", [EUL, BUR, ADV])
@pytest.mark.parametrize("extra", [{}, dict(sensor=2, fixed_gamma=0.5)])
def test_huge_states(law, extra):
    n, c = (5, 3, 5), 5
    prm = Params(**law, **extra)
    rng = np.random.default_rng(4)
    rho = 1.0 + 0.2 * rng.uniform(size=(75, 27)) + 0.4 * (np.arange(75) % 7 < 3)[:, None]
    nv = 5 if prm.flux == synth.EULER else 1
    u = np.float32(1e18) * np.stack([rho, 0.3 * rho, 0.3 * rho, 0.3 * rho, 2.0 + 2.0 * rho])[:nv].astype(np.float32)
    ijk = np.indices((5 * c, 3 * c, 5 * c))
    src = ((ijk[2] % 5) + 5 * ((ijk[1] % 3) + 3 * (ijk[0] % 5))).ravel()
    small = _run(synth.hex_mesh(*n, x1=1.0, y1=0.8, z1=0.6), u, prm)
    big = _run(synth.hex_mesh(5 * c, 3 * c, 5 * c, x1=1.0 * c, y1=0.8 * c, z1=0.6 * c), u[:, src], prm)
    for name, a, b in zip(("residual", "stage", "alpha"), small, big):
        assert b[a[:, src]].all(), name
