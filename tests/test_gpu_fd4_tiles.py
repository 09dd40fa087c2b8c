"""The finite-difference reference solver's tiles on the GPU, against the
oracle: grids that take each tile height, with a ragged last strip and last
row of tiles, and step counts that end in the state buffer each way (a copy
for one step, two buffers, three buffers)."""
import pytest

import oracle
from gpu_util import TOL, max_rel_l2, to_gpu, to_np
from paper_2603_19789_amd import inputs

pytestmark = pytest.mark.gpu


# tiles of 4, 8 and 32 output rows at 256 CUs; widths at, one under and one
# over a whole number of 48-column strips
SHAPES = [(96, 128), (97, 129), (239, 203), (335, 301), (337, 295), (481, 417), (575, 450)]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("bc", ["periodic", "noflux"])
@pytest.mark.parametrize("nx,ny", SHAPES)
def test_tiles_against_oracle(nx, ny, bc, dtype):
    from paper_2603_19789_amd import Solver
    orc = oracle.load()
    for d_dead, steps in ((0.0, 1), (0.0, 2), (4e-3, 3), (0.0, 5)):
        p = inputs.from_sigma_mu(0.5, 0.2, 0.1, 0.01, (2e-2, 1e-3, 5e-3, 1e-2, d_dead))
        rho0 = inputs.random_state(nx, ny, 31)
        s = Solver(nx, ny, p, dtype=dtype, bc=bc)
        got = to_np(s.fd4_run(to_gpu(rho0, dtype), steps))
        want = orc.fd4_rk4_run(rho0, p, steps, bc=bc)
        assert max_rel_l2(got, want) <= TOL[dtype], (d_dead, steps)
