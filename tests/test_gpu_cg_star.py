"""CG quadrilaterals around a vertex of five cells: the conjugate gradients'
gather of a DOF that more than four cells share, in each launch form."""
import numpy as np
import pytest

import synth
from oracle import build_space
from tests.test_gpu_cg_mass import mass, stage_and_residual

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2601_16911_amd import cvw  # noqa: E402


def star(n):
    """Five sectors of n x n rhombi about the origin."""
    a = [np.array([np.cos(0.4 * np.pi * k), np.sin(0.4 * np.pi * k)]) for k in range(5)]
    j, i = np.indices((n, n))
    cc = np.stack([np.stack([(i + di)[..., None] * a[k] + (j + dj)[..., None] * a[(k + 1) % 5]
                             for di, dj in ((0, 0), (1, 0), (1, 1), (0, 1))], axis=2) for k in range(5)]) / n
    # vertex ids: node (i, j) of sector k with j < n; its row i = 0 is row j = 0 of the next sector
    def vid(k, i, j):
        on_next = (i == 0) & (j > 0)
        k, i, j = np.where(on_next, (k + 1) % 5, k), np.where(on_next, j, i), np.where(on_next, 0, j)
        return np.where(i == 0, 0, 1 + k * n * (n + 1) + (i - 1) * (n + 1) + j)
    cv = np.stack([np.stack([vid(np.full_like(i, k), i + di, j + dj) for di, dj in ((0, 0), (1, 0), (1, 1), (0, 1))],
                            axis=2) for k in range(5)])
    return synth.MeshDesc(2, synth.QUAD, 1 + 5 * n * (n + 1), cv.reshape(-1, 4).astype(np.int32),
                          np.ascontiguousarray(cc.reshape(-1, 4, 2)), (0, 0))


# partials of 256 DOFs: up to 1024 (apply + update), up to 4096 (three launches), above (scalar launches)
@pytest.mark.parametrize("p,n", [(1, 2), (2, 6), (2, 120), (1, 235), (1, 460)])
def test_vertex_of_five_cells(p, n):
    mesh = star(n)
    assert np.bincount(mesh.cell_vertices.ravel(), minlength=mesh.n_vertices)[0] == 5
    sp = build_space(mesh, p, 0)
    X = np.empty((sp.n_dof, 2))
    X[sp.cell_dof.ravel()] = sp.node_coords().reshape(-1, 2)
    U = (np.sin(4 * X[:, 0]) * np.cos(3 * X[:, 1]) + (X[:, 0] > 0.2)).astype(np.float32)
    prm = synth.Params(flux=synth.ADVECT_CONST, flux_param=(1.0, 0.5, 0, 0))
    out, R, status = stage_and_residual(mesh, p, prm, U, cvw.F32)
    assert status == 0
    x = U.astype(np.float64) - out
    M = mass(sp)
    d = 1.0 / np.asarray(M.sum(1)).ravel()
    res = R - M @ x
    # as on grids: the iteration's tolerance in this norm, the float32 rounding of the rows and of the update
    tol = 2e-7 + 64 * np.finfo(np.float32).eps * (1.0 + np.sqrt((U.astype(np.float64) ** 2).sum() / (x ** 2).sum()))
    assert np.sqrt((res * d * res).sum() / (R * d * R).sum()) <= tol
