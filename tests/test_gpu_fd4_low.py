"""Finite-difference steps on grids of a few rows, on either side of the rule
that chooses their tiles, against the oracle."""
import pytest

from gpu_util import TOL, max_rel_l2, to_gpu, to_np
from paper_2603_19789_amd import Solver, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("bc", ["periodic", "noflux"])
@pytest.mark.parametrize("nx,ny", [(13000, 1), (13001, 4), (12999, 5), (13000, 16), (13000, 17)])
def test_low_grids_against_oracle(nx, ny, bc, dtype):
    import oracle
    p = inputs.from_sigma_mu(0.5, 0.2, 0.1, 0.01, (2e-2, 1e-3, 5e-3, 1e-2, 3e-3))
    rho0 = inputs.random_state(nx, ny, 77)
    got = Solver(nx, ny, p, dtype=dtype, bc=bc).fd4_run(to_gpu(rho0, dtype), 3)
    want = oracle.load().fd4_rk4_run(rho0, p, 3, bc=bc)
    assert max_rel_l2(to_np(got), want) <= TOL[dtype]
