"""Entry points without a stream argument run on torch's current stream of the
current device: eagerly on a side stream, and captured into a graph."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2603_19789_amd import Solver, binding, inputs  # noqa: E402


def test_the_handle_is_the_current_streams():
    main, side = torch.cuda.current_stream(), torch.cuda.Stream()
    assert (binding._stream(None).value or 0) == main.cuda_stream
    with torch.cuda.stream(side):
        assert binding._stream(None).value == side.cuda_stream
        assert (binding._stream(main).value or 0) == main.cuda_stream
    assert (binding._stream(None).value or 0) == main.cuda_stream


@pytest.mark.parametrize("capture", [False, True])
def test_steps_on_a_side_stream(capture):
    p = inputs.c2_params(3.0)
    s = Solver(128, 128, p, dtype="f64")
    rho = torch.rand(s.shape, dtype=torch.float64, device="cuda")
    want = s.step(s.step(rho.clone()))
    a, b = torch.empty_like(rho), torch.empty_like(rho)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    if capture:
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            s.step(rho, a)
            s.step(a, b)
        for _ in range(3):
            b.zero_()
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(b, want)
    else:
        with torch.cuda.stream(side):
            s.step(rho, a)
            s.step(a, b)
        side.synchronize()
        assert torch.equal(b, want)
