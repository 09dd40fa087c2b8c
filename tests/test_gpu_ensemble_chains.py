"""Ensemble runs by chains of passes: register tiles over a small ensemble, one
merged march over all classes of a large one, and a class on its own. Every
instance bit for bit its single-grid march; graph replays with eager work in
between equal the eager run."""
import pytest

from gpu_util import to_gpu
from paper_2603_19789_amd import Ensemble, Solver, inputs

pytestmark = pytest.mark.gpu

SMALL = [(129, 127), (200, 96), (33, 300), (64, 64), (65, 66), (20, 7), (256, 255)]
# enough cells for marches, in three classes and two types
LARGE = [(512, 400), (384, 511), (500, 498), (256, 255), (200, 256), (129, 128), (100, 90),
         (64, 64), (512, 512), (510, 512), (600, 512), (512, 300)]


def _members(sizes, dtype, bc, seed):
    params = [inputs.from_sigma_mu(0.3 + 0.02 * i, 0.2, 0.1, 0.01,
                                   (2e-2, 1e-3, 5e-3, 1e-2, 3e-3 if i == 1 else 0.0))
              for i in range(len(sizes))]
    starts = [to_gpu(inputs.random_state(nx, ny, seed + i), dtype)
              for i, (nx, ny) in enumerate(sizes)]
    ens = Ensemble(sizes, params, dtype=dtype, bc=bc)
    state = ens.empty()
    for v, x in zip(ens.views(state), starts):
        v.copy_(x)
    return params, starts, ens, state


def _single(size, p, start, steps, dtype, bc):
    s = Solver(*size, p, dtype=dtype, bc=bc)
    s.set_launch(2, 8, 1)  # the march
    return s.run(start.clone(), steps)


@pytest.mark.parametrize("sizes", [SMALL, LARGE], ids=["small", "large"])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("bc", ["periodic", "noflux"])
@pytest.mark.parametrize("steps", [1, 23])
def test_every_instance_equals_its_single_grid(sizes, dtype, bc, steps):
    import torch
    params, starts, ens, state = _members(sizes, dtype, bc, 51)
    ens.run(state, steps)
    for i, v in enumerate(ens.views(state)):
        want = _single(sizes[i], params[i], starts[i], steps, dtype, bc)
        assert torch.equal(v, want), sizes[i]


@pytest.mark.parametrize("sizes", [SMALL, LARGE], ids=["small", "large"])
def test_replays_and_single_classes(sizes):
    import torch
    steps = 19
    _, _, ens, start = _members(sizes, "f32", "periodic", 61)
    want = start.clone()
    ens.run(want, steps)
    state, scratch = start.clone(), ens.empty()
    for _ in range(3):
        state.copy_(start)
        ens.run(state, steps, scratch, graph=True)
        torch.cuda.synchronize()
        scratch.zero_()  # eager work on the buffers between replays
        assert torch.equal(state, want)
    state.copy_(start)
    for c in range(len(ens.classes())):
        ens.run_class(c, state, steps, scratch)
    assert all(torch.equal(a, b) for a, b in zip(ens.views(state), ens.views(want)))
