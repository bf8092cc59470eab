"""The workspace of a line holds what its kernels use and no more: on each
route a residual, a sensor call and a step stay inside exactly
cvw_workspace_bytes and give what they give in a larger one."""
import pytest

import synth
from synth import Params

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2601_16911_amd import cvw  # noqa: E402

ADV = dict(flux=synth.ADVECT_CONST, flux_param=(1.0, 0, 0, 0))
EUL = dict(flux=synth.EULER, flux_param=(1.4, 0, 0, 0))


@pytest.mark.parametrize("p,E,law", [(2, 130, ADV), (4, 33, ADV), (1, 9000, EUL), (3, 40, dict(ADV, r=3)), (8, 20, EUL)])
@pytest.mark.parametrize("space", [cvw.DG, cvw.CG])
def test_exact_workspace(p, E, law, space):
    mesh, prm = synth.segment_mesh(E), Params(**law)
    gm, cp = cvw.Mesh(mesh, p, space), cvw.make_params(prm, cvw.F64)
    nv = 3 if prm.flux == synth.EULER else 1
    n = gm.info["n_dof"] if space == cvw.CG else E * (p + 1)
    size = cvw.workspace_bytes(gm, cp, 1)
    # status, totals, candidates, the stage states; CG: element rows; conjugate gradients (degree > 4): six vectors, sums
    vec, pad = 8 * nv * n, 256
    most = 33280 + 8 * p * gm.info["n_vertices"] + 2 * vec + 12 * pad
    if space == cvw.CG:
        most += 8 * nv * E * (p + 1)
        if p > 4:
            most += 6 * vec + 8 * (n // 256 + 9)
    assert size <= most
    s = torch.sin(torch.arange(n, device="cuda", dtype=torch.float64) * 0.37) + 2.0
    u0 = torch.cat([s, 0.3 * s, 2.5 * s][:nv])
    res = []
    for extra in (1 << 20, 0):
        buf = torch.full((size + extra + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
        ws = buf[:size + extra]
        ws[:256] = 0
        u, R, g = u0.clone(), torch.empty_like(u0), torch.empty(E, device="cuda", dtype=torch.float64)
        cvw.residual(gm, cp, u, R, g, ws)
        g2 = torch.empty_like(g)
        cvw.sensor(gm, cp, u, g2, None, ws)
        cvw.step(gm, cp, u, 1e-3 / E, 2, ws)
        assert cvw.poll_status(gm, ws) == 0
        assert (buf[size:] == 0xA5).all()
        res.append((u, R, g, g2))
    assert all(torch.equal(a, b) for a, b in zip(*res))
