"""Non-finite Euler states on CG lines, in one block and in several: a variable
whose assembled right-hand side holds a NaN (also one made where two infinite
element rows meet) keeps its state, one with infinities only has no finite
value left, and the others stay finite."""
import numpy as np
import pytest

from paper_2601_16911_amd import cvw
from tests.test_gpu_cg_mass import line_case, stage_and_residual

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,E", [(1, 50), (1, 700), (2, 64), (2, 2500), (4, 40), (4, 1500)])
@pytest.mark.parametrize("var", [0, 1, 2])
@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_each_variable_by_itself(p, E, var, bad):
    mesh, sp, prm, U = line_case(E, p, False, cvw.F64)
    n = U.size // 3
    U[var * n + E // 2] = bad
    out, R, status = stage_and_residual(mesh, p, prm, U, cvw.F64, 1e-9)
    assert status & 1
    for v in range(3):
        o, r, u = (x.reshape(3, n)[v] for x in (out, R, U))
        ok = np.isfinite(u)
        if np.isnan(r).any():
            assert np.array_equal(o[ok], u[ok]), v
        elif np.isinf(r).any():
            assert not np.isfinite(o).any(), v
        else:
            assert np.isfinite(o[ok]).all(), v
