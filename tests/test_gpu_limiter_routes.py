"""A scalar limiter with candidates at listed vertices (large P3 grids) against
the one with candidates everywhere: 8 x 8 copies of a small periodic grid have
its gamma and its limited cells, bit for bit away from the seams (there the
order of a vertex's cells changes)."""
import numpy as np
import pytest

import synth
from synth import Params

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2601_16911_amd import cvw  # noqa: E402

BUR = Params(flux=synth.BURGERS, flux_param=(1.0, 1.0, 0, 0))


def _limited(mesh, u, threshold, in_place):
    gm, cp = cvw.Mesh(mesh, 3, cvw.DG), cvw.make_params(BUR)
    d = torch.from_numpy(np.ascontiguousarray(u)).cuda()
    out = d if in_place else torch.full_like(d, float("nan"))
    g = torch.empty(mesh.n_cells, device="cuda")
    cvw.limit(gm, cp, d, out, threshold, g, cvw.alloc_workspace(gm, cp, 2))
    return out.cpu().numpy(), g.cpu().numpy()


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("threshold", [0.9, 0.9999, 2.0])
def test_copies_of_a_small_grid(threshold, in_place):
    n, c = 64, 8
    rng = np.random.default_rng(2)
    y, x = np.indices((n, n)) / n
    u = (1.0 + 0.3 * np.sin(2 * np.pi * x) + (x + y > 1.1))[..., None] + 0.02 * rng.uniform(size=(n, n, 16)) * (x < 0.5)[..., None]
    u = u.astype(np.float32)
    a, ga = _limited(synth.quad_mesh(n, n), u.reshape(n * n, 16), threshold, in_place)
    b, gb = _limited(synth.quad_mesh(c * n, c * n, 0.0, float(c), 0.0, float(c)), np.tile(u, (c, c, 1)).reshape(-1, 16),
                     threshold, in_place)
    inner = slice(2, n - 2)
    b, gb = b.reshape(c, n, c, n, 16)[:, inner, :, inner], gb.reshape(c, n, c, n)[:, inner, :, inner]
    a, ga = a.reshape(1, n, 1, n, 16)[:, inner, :, inner], ga.reshape(1, n, 1, n)[:, inner, :, inner]
    assert (ga < 0.9).any() and (ga > 0.9).any()
    assert np.array_equal(np.broadcast_to(ga, gb.shape), gb)
    assert np.array_equal(np.broadcast_to(a, b.shape), b)
