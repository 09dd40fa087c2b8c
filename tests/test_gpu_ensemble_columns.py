"""Large ensembles some of whose classes have odd rows: two chains, with two and
with one column a lane. Every instance bit for bit its single-grid march, run
directly, as replayed graphs and class by class."""
import pytest

from gpu_util import to_gpu
from paper_2603_19789_amd import Ensemble, Solver, inputs

pytestmark = pytest.mark.gpu

SIZES = [(2048, 2048)] * 4 + [(511, 300), (1022, 1030), (20, 7), (129, 255)]


@pytest.mark.parametrize("bc", ["periodic", "noflux"])
@pytest.mark.parametrize("steps", [7, 12])
def test_two_chains_equal_single_grids(steps, bc):
    import torch
    params = [inputs.from_sigma_mu(0.3 + 0.02 * i, 0.2, 0.1, 0.01, (2e-2, 1e-3, 5e-3, 1e-2, 0.0))
              for i in range(len(SIZES))]
    starts = [to_gpu(inputs.random_state(nx, ny, 91 + i), "f32")
              for i, (nx, ny) in enumerate(SIZES)]
    ens = Ensemble(SIZES, params, dtype="f32", bc=bc)
    assert {c["launch"]["cols_per_lane"] for c in ens.classes() if not c["on_chip"]} == {1, 2}
    start, scratch = ens.empty(), ens.empty()
    for v, x in zip(ens.views(start), starts):
        v.copy_(x)
    want = []
    for size, p, x in zip(SIZES, params, starts):
        s = Solver(*size, p, dtype="f32", bc=bc)
        s.set_launch(2, 8, 1)  # the march
        want.append(s.run(x.clone(), steps))
    state = start.clone()

    def check(how):
        for size, v, w in zip(SIZES, ens.views(state), want):
            assert torch.equal(v, w), (how, size)
    ens.run(state, steps, scratch)
    check("direct")
    for i in range(3):
        state.copy_(start)
        ens.run(state, steps, scratch, graph=True)
        torch.cuda.synchronize()
        scratch.zero_()  # eager work between replays
        check(f"replay {i}")
    state.copy_(start)
    for c in range(len(ens.classes())):
        ens.run_class(c, state, steps, scratch)
    check("class by class")
