"""Recorded runs and reverse sweeps of small grids on the GPU (chunks of two
rows, register-tile segments) against the oracle: every interval gives the
same trajectory and checkpoints as plain runs, and the state and parameter
gradients of the oracle's adjoint steps."""
import numpy as np
import pytest

import oracle
from gpu_util import max_rel_l2, to_gpu, to_np
from paper_2603_19789_amd import Solver, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", ["periodic", "noflux"])
@pytest.mark.parametrize("nx,ny", [(3, 2), (61, 3), (65, 33), (130, 47)])
@pytest.mark.parametrize("every,steps", [(1, 4), (2, 9), (3, 7), (7, 20), (40, 23)])
def test_checkpoints_and_gradient(nx, ny, every, steps, bc):
    import torch
    orc = oracle.load()
    p = inputs.from_sigma_mu(0.5, 0.2, 0.1, 0.01, (2e-2, 1e-3, 5e-3, 1e-2, 4e-3))
    rho0 = inputs.random_state(nx, ny, 71)
    s = Solver(nx, ny, p, dtype="f64", bc=bc)
    start = to_gpu(rho0, "f64")
    rho = start.clone()
    cp = s.run_checkpointed(rho, steps, every)
    states = [rho0]
    for _ in range(steps):
        states.append(orc.sslbm_step(states[-1], p, bc=bc))
    march = Solver(nx, ny, p, dtype="f64", bc=bc)
    march.set_launch(2, 8, 1)
    assert torch.equal(rho, march.run(start.clone(), steps))
    for k in range(s.checkpoint_count(steps, every)):
        assert max_rel_l2(to_np(cp[k]), states[k * every]) <= 1e-12
    lam0 = np.random.default_rng(72).normal(size=rho0.shape)
    lam, grad = s.adjoint_run(cp, steps, every, to_gpu(lam0, "f64"))
    want, want_g = lam0, np.zeros(9)
    for n in range(steps - 1, -1, -1):
        want, g = orc.sslbm_adjoint_step(states[n], want, p, bc=bc)
        want_g += g
    assert max_rel_l2(to_np(lam), want) <= 1e-12
    assert np.linalg.norm(to_np(grad) - want_g) <= 1e-11 * np.linalg.norm(want_g)
