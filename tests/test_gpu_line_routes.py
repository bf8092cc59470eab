"""Lines whose vertex candidates come from a pass of their own (long lines,
high degrees, general exponents) against those that form them in the cell
kernel: two copies of a line just below the length where the route changes
have its values, bit for bit away from the seams (there the order of a
vertex's two cells changes), and general exponents meet the oracle."""
import numpy as np
import pytest

import synth
from oracle import build_space, nodal_interpolate, residual as o_residual
from synth import Params
from tests.parity_helpers import rel_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2601_16911_amd import cvw  # noqa: E402

ADV = Params(flux=synth.ADVECT_CONST, flux_param=(1.0, 0, 0, 0))
EUL = Params(flux=synth.EULER, flux_param=(1.4, 0, 0, 0))


def _residual(mesh, p, space, prm, u):
    gm, cp = cvw.Mesh(mesh, p, space), cvw.make_params(prm, cvw.F64)
    ws = cvw.alloc_workspace(gm, cp, 1)
    d = torch.from_numpy(np.ascontiguousarray(u)).cuda()
    R, g = torch.empty_like(d), torch.empty(mesh.n_cells, dtype=torch.float64, device="cuda")
    cvw.residual(gm, cp, d, R, g, ws)
    g2 = torch.empty_like(g)
    cvw.sensor(gm, cp, d, g2, None, ws)
    assert torch.equal(g, g2)
    cvw.step(gm, cp, d, 1e-7, 1, ws)            # the same dt on a line and on its copies
    assert cvw.poll_status(gm, ws) == 0
    return R.cpu().numpy(), g.cpu().numpy(), d.cpu().numpy()


@pytest.mark.parametrize("space", [cvw.DG, cvw.CG])
@pytest.mark.parametrize("p,prm", [(1, EUL), (3, EUL), (4, ADV), (12, ADV)])
def test_two_copies_of_a_shorter_line(p, prm, space):
    n, nv = 4096, 3 if prm.flux == synth.EULER else 1
    rng = np.random.default_rng(p)

    def field(k):                       # k values per cell, smooth with jumps
        x = np.arange(n * k) / (n * k)
        s = 1.0 + 0.2 * np.sin(2 * np.pi * x) + 0.5 * (np.floor(x * 37) % 2) + 1e-3 * rng.uniform(size=n * k)
        return np.stack([s, 0.3 * s, 2.5 * s])[:nv].reshape(nv, n, k)

    cols = [field(p + 1)] if space == cvw.DG else [field(1)] + ([field(p - 1)] if p > 1 else [])
    flat = [np.concatenate([np.tile(c, (1, k, 1)).reshape(nv, -1) for c in cols], axis=1).ravel() for k in (1, 2)]
    R1, g1, u1 = _residual(synth.segment_mesh(n), p, space, prm, flat[0])
    R2, g2, u2 = _residual(synth.segment_mesh(2 * n, 0.0, 2.0), p, space, prm, flat[1])
    assert (g1 < 0.9).any() and (g1 > 0.9).any()
    inner = slice(2, n - 2)             # the step passes three stages on: its seams reach further
    for a, b, keep in ((R1, R2, inner), (u1, u2, slice(128, n - 128))):
        if a is u1 and space == cvw.CG:
            continue                    # the conjugate gradients' sums (and the solve's reach) span the line
        a, b = a.reshape(nv, -1), b.reshape(nv, -1)
        at = 0
        for c in cols:
            k = c.shape[2]
            x = a[:, at:at + n * k].reshape(nv, 1, n, k)
            y = b[:, 2 * at:2 * (at + n * k)].reshape(nv, 2, n, k)
            assert np.array_equal(np.broadcast_to(x, y.shape)[:, :, keep], y[:, :, keep])
            at += n * k
    assert np.array_equal(np.tile(g1, (2, 1))[:, inner], g2.reshape(2, n)[:, inner])


@pytest.mark.parametrize("space", [cvw.DG, cvw.CG])
@pytest.mark.parametrize("p,N", [(2, 40), (4, 33)])
def test_general_exponents(p, N, space):
    prm = Params(flux=synth.ADVECT_CONST, flux_param=(1.0, 0, 0, 0), r=3, q_beta=1.5, q_sensor=1.25)
    mesh = synth.segment_mesh(N)
    sp = build_space(mesh, p, 0 if space == cvw.CG else 1)
    U = nodal_interpolate(sp, [lambda x: np.sin(2 * np.pi * x[..., 0]) + (x[..., 0] > 0.63)])
    R, g, _ = _residual(mesh, p, space, prm, U)
    Ro, parts = o_residual(sp, U, prm, return_parts=True)
    assert np.abs(g - parts["gamma"]).max() < 1e-9        # well conditioned float64 data
    assert rel_err(R, np.asarray(Ro).ravel()) < 1e-9
