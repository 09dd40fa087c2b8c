"""Ensembles on register tiles of every height, with and without a diffusing D,
both walls: every instance bit for bit its single-grid march. That these sizes
take these heights is asserted without a GPU (test_launches.py)."""
import pytest

from paper_2603_19789_amd import inputs

pytestmark = pytest.mark.gpu

# (dtype, rows a lane, steps, sizes): ragged last tiles in both directions
HEIGHTS = [("f32", 2, 33, [(257, 255), (301, 199), (130, 120)]),
           ("f32", 3, 25, [(300, 201), (129, 255)] * 2),
           ("f32", 4, 33, [(512, 510), (384, 301)] * 3),
           ("f32", 5, 37, [(512, 510), (384, 301)] * 3),
           ("f32", 7, 29, [(600, 500)] * 4),
           ("f64", 1, 25, [(101, 67), (70, 45)]),
           ("f64", 2, 29, [(257, 255), (301, 199), (130, 120)]),
           ("f64", 3, 29, [(520, 510), (257, 129), (199, 200)])]


@pytest.mark.parametrize("bc", ["periodic", "noflux"])
@pytest.mark.parametrize("d_dead", [0.0, 3e-3])
@pytest.mark.parametrize("dtype,rows,steps,sizes", HEIGHTS)
def test_every_tile_height_equals_the_march(dtype, rows, steps, sizes, d_dead, bc):
    import torch
    from gpu_util import to_gpu
    from paper_2603_19789_amd import Ensemble, Solver
    params = [inputs.from_sigma_mu(0.3 + 0.02 * i, 0.2, 0.1, 0.01, (2e-2, 1e-3, 5e-3, 1e-2, d_dead))
              for i in range(len(sizes))]
    starts = [to_gpu(inputs.random_state(nx, ny, 71 + i), dtype) for i, (nx, ny) in enumerate(sizes)]
    ens = Ensemble(sizes, params, dtype=dtype, bc=bc)
    state = ens.empty()
    for v, x in zip(ens.views(state), starts):
        v.copy_(x)
    ens.run(state, steps)
    for i, v in enumerate(ens.views(state)):
        s = Solver(*sizes[i], params[i], dtype=dtype, bc=bc)
        s.set_launch(2, 8, 1)  # the march
        assert torch.equal(v, s.run(starts[i].clone(), steps)), sizes[i]
