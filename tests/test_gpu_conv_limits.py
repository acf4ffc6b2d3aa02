"""Single-layer convolution calls at the edge of what the copies address:
tensors whose z planes are past 32-bit byte offsets, tensors at odd addresses.
Small whole numbers make every sum exact in FP32, so results are compared for
equality."""
import pytest

from paper_1409_8336_amd import unet

pytestmark = pytest.mark.gpu


def _whole(g, *shape):
    import torch
    return torch.randint(-2, 3, shape, generator=g, device="cuda").to(torch.bfloat16)


@pytest.mark.parametrize("shape,cin,cout", [
    ((1, 2, 8200, 16385), 8, 16),     # the output gradient's plane: 4.3e9 bytes
    ((1, 1, 16390, 16385), 8, 8),     # both tensors'
])
def test_weight_gradient_of_planes_past_4_gib(shape, cin, cout):
    """Values in the first and the last eight rows only (zeros add nothing):
    the gradient is the sum of those of the two ends, whose planes are small.
    A sum has at most 32 x 16385 products of at most 4, below 2^24."""
    import torch
    print("case: weight gradient", shape, cin, cout, flush=True)
    n, d, h, w = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    x = torch.zeros(*shape, cin, dtype=torch.bfloat16, device="cuda")
    dy = torch.zeros(*shape, cout, dtype=torch.bfloat16, device="cuda")
    assert h * w * max(cin, cout) >= 2 ** 31
    want = torch.zeros(cout, unet.kp(cin), device="cuda")
    for rows in (slice(0, 8), slice(h - 8, h)):
        ends = []
        for t, c in ((x, cin), (dy, cout)):
            t[:, :, rows] = _whole(g, n, d, 8, w, c)
            ends.append(t[:, :, rows].contiguous())
        unet.pmc_nn_conv3d_backward_weight(ends[0], ends[1], want)
    dw = torch.zeros_like(want)
    unet.pmc_nn_conv3d_backward_weight(x, dy, dw)
    torch.cuda.synchronize()
    assert want.abs().max() > 0
    assert torch.equal(dw, want)


@pytest.mark.parametrize("shape,cin,cout", [
    ((1, 4, 9, 17), 8, 16),        # one 8-channel chunk a stage
    ((1, 5, 9, 17), 32, 32),       # two, pipelined
    ((2, 40, 40, 40), 32, 32),     # two, many tiles
])
@pytest.mark.parametrize("off", [1, 2, 4, 7])
def test_tensors_at_any_element_boundary(shape, cin, cout, off):
    """Views that start `off` BF16 elements past a 16-byte boundary (inputs,
    weights and outputs) give what aligned tensors give."""
    import torch
    print("case: unaligned tensors", shape, cin, cout, off, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    x, dy = _whole(g, *shape, cin), _whole(g, *shape, cout)
    w = torch.zeros(cout, unet.kp(cin), dtype=torch.bfloat16, device="cuda")
    w[:, :27 * cin] = _whole(g, cout, 27 * cin)
    bias = _whole(g, cout).float()

    def view(t, o):
        buf = torch.zeros(t.numel() + 64, dtype=t.dtype, device="cuda")
        v = buf[16 + o:16 + o + t.numel()].view(t.shape)
        v.copy_(t)
        assert v.data_ptr() % 16 == 2 * o % 16
        return v

    def run(o):
        xv, dyv, wv = view(x, o), view(dy, o), view(w, o)
        y, dx = view(torch.zeros_like(dy), o), view(torch.zeros_like(x), o)
        dw = torch.zeros(cout, unet.kp(cin), device="cuda")
        unet.pmc_nn_conv3d_forward(xv, wv, bias, y, True)
        unet.pmc_nn_conv3d_backward_weight(xv, dyv, dw)
        unet.pmc_nn_conv3d_backward_data_noalloc(dyv, wv, dx)
        torch.cuda.synchronize()
        return y, dw, dx

    for a, b in zip(run(0), run(off)):
        assert torch.equal(a, b)
