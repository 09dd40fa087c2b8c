"""BGK runs of several steps per HBM pass, on the GPU: bit for bit the result of
single steps, at the sizes where the pass's strips, chunks and walls can go
wrong (grids large enough to take such passes), and the oracle on one of them."""
import pytest

from gpu_util import TOL, max_rel_l2, to_gpu, to_np
from paper_2603_19789_amd import inputs

pytestmark = pytest.mark.gpu


def _params():
    return inputs.from_sigma_mu(0.5, 0.2, 0.1, 0.01, (2e-2, 1e-3, 5e-3, 1e-2, 0.0))


# (nx, ny, steps): FP32 passes of 2..7 steps and FP64 passes of 2 and 3. Widths
# one column over and under a whole number of strips, ragged and odd sides,
# chunks of 6 rows with a remainder, one row of chunks, a grid as narrow as
# the rule allows, and grids of at least 1.5 million cells (seven steps).
CASES = [(432, 433, 10), (433, 325, 9), (431, 326, 7), (32, 4400, 6), (33, 4401, 5), (4403, 33, 4),
         (1251, 1200, 14), (1250, 1201, 13), (1249, 1202, 11)]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("bc", ["periodic", "noflux"])
@pytest.mark.parametrize("nx,ny,steps", CASES)
def test_passes_equal_single_steps(nx, ny, steps, bc, dtype):
    import torch
    from paper_2603_19789_amd import BGK
    s = BGK(nx, ny, _params(), dtype=dtype, bc=bc)
    f, d = s.init(to_gpu(inputs.random_state(nx, ny, 21), dtype))
    s.step(f.clone(), d.clone(), f, d)  # off equilibrium: every population its own value
    a, b = f.clone(), d.clone()
    for _ in range(steps):
        a, b = s.step(a, b)
    s.run(f, d, steps)
    assert torch.equal(f, a) and torch.equal(d, b)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("bc", ["periodic", "noflux"])
def test_passes_against_oracle(bc, dtype):
    import oracle
    from paper_2603_19789_amd import BGK
    nx, ny, steps = 450, 341, 10
    p = _params()
    rho0 = inputs.random_state(nx, ny, 22)
    s = BGK(nx, ny, p, dtype=dtype, bc=bc)
    f, d = s.run(*s.init(to_gpu(rho0, dtype)), steps)
    want = oracle.load().bgk_run_density(rho0, p, steps, bc=bc)
    assert max_rel_l2(to_np(s.density(f, d)), want) <= TOL[dtype]
