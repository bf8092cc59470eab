"""Tetrahedra with their vertices in every orientation-keeping order, so that a
face meets every face of its neighbour under every permutation: residual
against the float64 oracle, 1e-5 of the largest entry as for the ordered mesh."""
import itertools

import numpy as np
import pytest

import synth
from oracle import build_space, residual as o_residual
from synth import Params
from tests.parity_helpers import f32, rel_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2601_16911_amd import cvw  # noqa: E402

EVEN = [q for q in itertools.permutations(range(4))
        if sum(q[i] > q[j] for i in range(4) for j in range(i + 1, 4)) % 2 == 0]


@pytest.mark.parametrize("flux", [synth.EULER, synth.BURGERS])
@pytest.mark.parametrize("p", [1, 2])
def test_every_face_pairing(p, flux):
    mesh = synth.tet_mesh(5, 4, 3, x1=1.0, y1=0.8, z1=0.6)
    rng = np.random.default_rng(3)
    for e in range(mesh.n_cells):
        q = list(EVEN[rng.integers(len(EVEN))])
        mesh.cell_vertices[e] = mesh.cell_vertices[e][q]
        mesh.cell_coords[e] = mesh.cell_coords[e][q]
    nv = 5 if flux == synth.EULER else 1
    prm = Params(flux=flux, flux_param=(1.4, 0, 0, 0) if nv == 5 else (1.0, 0.8, 0.6, 0))
    sp = build_space(mesh, p, 1, n_var=nv)
    x = sp.node_coords()
    rho = 1.0 + 0.3 * np.sin(2 * np.pi * x[..., 0]) * np.cos(2 * np.pi * x[..., 1] / 0.8) + (x[..., 2] < 0.25)
    u = f32(np.stack([rho, 0.4 * rho, -0.3 * rho, 0.2 * rho * x[..., 0], 2.5 + 2.0 * rho])[:nv])
    gm, cp = cvw.Mesh(mesh, p, cvw.DG), cvw.make_params(prm)
    R = torch.empty(u.size, dtype=torch.float32, device="cuda")
    cvw.residual(gm, cp, torch.from_numpy(u.astype(np.float32).ravel()).cuda(), R, None, cvw.alloc_workspace(gm, cp, 0))
    Ro, parts = o_residual(sp, u.ravel(), prm, return_parts=True)
    keep = np.repeat(np.abs(parts["gamma"] - 0.9) >= 1e-4, sp.ref.n_loc)
    assert keep.mean() > 0.9
    for v in range(nv):
        assert rel_err(R.cpu().numpy().reshape(nv, -1)[v][keep], Ro.reshape(nv, -1)[v][keep]) < 1e-5, v
