"""The limiter's out-of-place copy of the cells it leaves alone, and its lists,
at sizes that are no multiple of a block: against the in-place call, bit for
bit, with the cells of gamma_e >= threshold unchanged."""
import numpy as np
import pytest

import synth
from synth import Params

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2601_16911_amd import cvw  # noqa: E402


@pytest.mark.parametrize("path", ["fused", "twopass"])
@pytest.mark.parametrize("flux", [synth.EULER, synth.BURGERS])
@pytest.mark.parametrize("p,size,threshold", [(1, (5, 3), 0.9), (1, (70, 33), 0.9), (2, (33, 31), 0.9),
                                              (2, (64, 64), -1.0), (3, (37, 61), 0.9), (3, (4, 4), 1.0)])
def test_copy_and_lists(p, size, threshold, flux, path, monkeypatch):
    if path == "twopass":
        monkeypatch.setenv("CVW_SENSOR_PATH", "twopass")
    E, nv = size[0] * size[1], 4 if flux == synth.EULER else 1
    gm = cvw.Mesh(synth.quad_mesh(*size), p, cvw.DG)
    cp = cvw.make_params(Params(flux=flux, flux_param=(1.4, 0, 0, 0) if nv == 4 else (1.0, 1.0, 0, 0)))
    rng = np.random.default_rng(E)
    u = rng.uniform(-0.1, 0.1, size=(nv, E, (p + 1) ** 2)) * rng.uniform(size=(1, E, 1)) ** 6
    u[0] += 1.0 + 0.3 * np.sin(np.arange(E) / 7.0)[:, None]
    if nv == 4:
        u[3] += 2.5
    u = torch.from_numpy(u.astype(np.float32)).cuda()
    ws = cvw.alloc_workspace(gm, cp, 2)
    out, gam = torch.full_like(u, float("nan")), torch.empty(E, device="cuda")
    cvw.limit(gm, cp, u, out, threshold, gam, ws)
    inplace = u.clone()
    cvw.limit(gm, cp, inplace, inplace, threshold, None, ws)
    assert torch.equal(out, inplace)
    left = ~(gam.double() < threshold)
    assert torch.equal(out[:, left], u[:, left])
    if threshold < 0:
        assert left.all()
