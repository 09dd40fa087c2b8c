"""Stores and mask loads of the halo-tile convolutions, whose lanes hold 4, 8
or 16 consecutive channels of a pixel: layers that end inside a lane's
channels or inside a channel group, in views that begin inside a wider
buffer, on ragged images. The view gets the bits of the same layer in a
buffer of its own, and nothing around it is written.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2603_19789_amd import binding  # noqa: E402
from paper_2603_19789_amd import surrogate as S  # noqa: E402
from test_gpu_surrogate import BF, bf16_array, lib, p  # noqa: E402

FILL = 12345.0


def split(buf, off, c):
    return buf[..., off:off + c], torch.cat([buf[..., :off], buf[..., off + c:]], dim=-1)


@pytest.mark.parametrize("kind", ["plain", "pool", "mask", "fp32"])
@pytest.mark.parametrize("cout", [8, 16, 24, 40, 56, 72, 104])
def test_ragged_layers_write_their_view_only(cout, kind):
    n, h, w, cin = 2, 10, 42, 24
    print(f"conv epilogue {kind} {cin}->{cout}", flush=True)
    L = lib()
    x, _ = bf16_array((n, h, w, cin))
    wt, _ = bf16_array((cout, 9, cin), scale=1.0 / np.sqrt(9 * cin))
    bias = torch.arange(cout, dtype=torch.float32, device="cuda") / 8
    fp32 = kind == "fp32"
    if fp32:
        cout -= 4  # FP32 outputs hold channels in fours
    flags = S.OUT_F32 if fp32 else S.LEAKY
    dt = torch.float32 if fp32 else BF
    off, pitch = 8, cout + 24
    y = torch.full((n, h, w, cout), FILL, dtype=dt, device="cuda")
    yv = torch.full((n, h, w, pitch), FILL, dtype=dt, device="cuda")
    act, _ = bf16_array((n, h, w, pitch))
    pool = torch.full((n, h // 2, w // 2, pitch), FILL, dtype=BF, device="cuda")
    if kind == "mask":
        plain = torch.zeros_like(y)
        assert L.sur_conv3x3_backward_data_flipped(p(x), cin, n, h, w, cin, p(wt), cout, p(plain),
                                                   cout, None, 0, 0.0, None) == binding.OK
        assert L.sur_leaky_backward(p(plain), cout, p(act, off), pitch, p(y), cout, n * h * w,
                                    cout, 0.1, None) == binding.OK
        assert L.sur_conv3x3_backward_data_flipped(p(x), cin, n, h, w, cin, p(wt), cout,
                                                   p(yv, off), pitch, p(act, off), pitch, 0.1,
                                                   None) == binding.OK
    else:
        assert L.sur_conv3x3_forward(p(x), cin, n, h, w, cin, p(wt), p(bias), p(y), cout, cout,
                                     flags, 0.1, None) == binding.OK
        if kind == "pool":
            assert L.sur_conv3x3_forward_pool(p(x), cin, n, h, w, cin, p(wt), p(bias), p(yv, off),
                                              pitch, cout, flags, 0.1, p(pool, off), pitch,
                                              None) == binding.OK
        else:
            assert L.sur_conv3x3_forward(p(x), cin, n, h, w, cin, p(wt), p(bias), p(yv, off),
                                         pitch, cout, flags, 0.1, None) == binding.OK
    torch.cuda.synchronize()
    got, rest = split(yv, off, cout)
    assert torch.equal(got, y)
    assert not bool((got == FILL).any())
    assert bool((rest == torch.tensor(FILL, dtype=dt)).all())
    if kind == "pool":
        got, rest = split(pool, off, cout)
        want = torch.empty((n, h // 2, w // 2, cout), dtype=BF, device="cuda")
        assert L.sur_pool2(p(y), cout, n, h, w, cout, p(want), cout, None) == binding.OK
        torch.cuda.synchronize()
        assert torch.equal(got, want)
        assert bool((rest == torch.tensor(FILL, dtype=BF)).all())
