"""Register-tile passes on the GPU (the automatic choice on small and middle
grids): bit for bit the result of march passes, which the parity tests tie to
the oracle, at sizes that take every tile height, with ragged last tiles, grids
narrower than a tile, both walls, both types and a diffusing D."""
import pytest

from gpu_util import TOL, max_rel_l2, to_gpu, to_np
from paper_2603_19789_amd import Solver, inputs

pytestmark = pytest.mark.gpu


def _params(d_dead=0.0):
    return inputs.from_sigma_mu(0.5, 0.2, 0.1, 0.01, (2e-2, 1e-3, 5e-3, 1e-2, d_dead))


# (nx, ny, steps): 1x1 upwards; one column or row over and under a whole
# number of tiles; one wide and one tall grid; FP32 sizes for 2, 3, 4, 5 and 7
# rows a lane and FP64 sizes for 1, 2 and 3
SHAPES = [(1, 1, 9), (1, 70, 14), (70, 1, 15), (3, 5, 31), (36, 4, 28), (37, 33, 29), (64, 65, 16),
          (129, 127, 33), (200, 200, 40), (257, 255, 24), (512, 511, 20), (641, 640, 24),
          (770, 766, 16), (897, 895, 14), (1023, 1025, 18), (5000, 60, 17), (61, 5003, 13)]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("bc", ["periodic", "noflux"])
@pytest.mark.parametrize("nx,ny,steps", SHAPES)
def test_tiles_equal_the_march(nx, ny, steps, bc, dtype):
    import torch
    for d_dead in (0.0, 4e-3):
        start = to_gpu(inputs.random_state(nx, ny, 41), dtype)
        s = Solver(nx, ny, _params(d_dead), dtype=dtype, bc=bc)
        got = s.run(start.clone(), steps)
        s.set_launch(2, 8, 1)  # the march
        want = s.run(start.clone(), steps)
        assert torch.equal(got, want), d_dead


def test_every_tile_height_is_taken():
    """The sizes above cover the depths the choice takes: more steps per pass
    than any march pass, and the march again on grids past the limit."""
    longest = {n: Solver(n, n, _params(), dtype="f32").plan(1000)["longest"]
               for n in (128, 512, 768, 1024, 1300)}
    assert longest[128] > 8 and longest[1300] <= 8
    assert Solver(128, 128, _params(), dtype="f64").plan(1000)["longest"] >= 4


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("bc", ["periodic", "noflux"])
def test_tiles_against_oracle(bc, dtype):
    import oracle
    nx, ny, steps = 197, 143, 45
    p = _params()
    rho0 = inputs.random_state(nx, ny, 42)
    got = Solver(nx, ny, p, dtype=dtype, bc=bc).run(to_gpu(rho0, dtype), steps)
    want = oracle.load().sslbm_run(rho0, p, steps, bc=bc)
    assert max_rel_l2(to_np(got), want) <= TOL[dtype]


def test_tuned_context_keeps_the_bits():
    """After tuning, whichever of march and tiles won, runs give the same bits,
    and the reported shape is a valid one for another context."""
    import torch
    start = to_gpu(inputs.random_state(300, 200, 43), "f32")
    s = Solver(300, 200, _params(), dtype="f32")
    want = s.run(start.clone(), 37)
    best = s.tune(start.clone())
    assert best == s.launch()
    assert torch.equal(s.run(start.clone(), 37), want)
    other = Solver(300, 200, _params(), dtype="f32")
    other.set_launch(**best)
    assert other.launch() == best
    assert torch.equal(other.run(start.clone(), 37), want)
