"""Weight gradients from single cells at the edges of the kernels' tiles, and of a grid
whose chunks of planes divide it for neither kind of layer: at 112^3 the 16 -> 16
layers march over 38, 38 and 36 planes and the first and last over 19 (the last chunk
17), in two grids of 80^3 over 27 (26) and 14 (10); tiles are 16 x 8 cells.

Reference: test_gpu_wgrad's, over the same rounded operands.  What is left is the FP32
accumulation (1e-6 of a layer's gradient) and the activations and layer gradients that
FP32 and FP64 sums round to different BF16 values: about 3 in 10^4 of them, each by
2^-8, which in a sum of many cells is below 1e-4 of a layer's gradient.  The bound
for whole grids is 2e-3 (a plane lost of 112 is 9e-3).  The gradient of a single
output cell rests on a few hundred cells, where one such operand weighs more: 1e-2,
while a lost or misplaced cell of the last layer changes order 1 and a lost plane of
the 7 that reach the first layer about a tenth.
"""
import pytest

from test_gpu_wgrad import CH, P, reference  # noqa: F401

pytestmark = pytest.mark.gpu


def compare(got, want, bound, what):
    at = 0
    for layer in range(4):
        k = CH[layer] * CH[layer + 1] * 27
        d = float((got[at:at + k].double() - want[at:at + k]).norm() / want[at:at + k].norm())
        print(f"{what} layer {layer + 1}: {d:.2e}")
        assert d <= bound, (what, layer, d)
        at += k


@pytest.mark.parametrize("n,batch", [(112, 1), (80, 2)])
def test_chunks_that_do_not_divide(P, n, batch):
    import torch
    from paper_1404_0959_amd import learn
    g = torch.Generator(device="cuda").manual_seed(n)
    w = torch.as_tensor(learn.init_weights(n), device="cuda")
    x = torch.randn((batch, n ** 3, 2), generator=g, device="cuda")
    t = 0.1 * torch.randn((batch, n ** 3), generator=g, device="cuda")
    t += torch.roll(x[..., 0], 1, dims=1) - 0.5 * x[..., 1]
    _, want = reference(w, x, t, n)
    _, got = P.Net(n, batch).grad(w, x, t)
    compare(got, want, 2e-3, f"{batch} x {n}")


@pytest.mark.parametrize("n,batch,crop,cells", [
    (112, 1, 14, [(0, 0, 0), (111, 111, 111), (15, 7, 18), (16, 8, 19), (95, 104, 37), (96, 103, 38),
                  (0, 111, 95), (50, 60, 75), (111, 0, 76)]),
    (80, 2, 20, [(0, 0, 0), (79, 79, 79), (15, 8, 13), (16, 7, 14), (64, 72, 26), (63, 71, 27), (40, 0, 69),
                 (0, 40, 70)]),
])
def test_single_cells(P, n, batch, crop, cells):
    """The target is the network's own output but for one cell of the last grid.  All that
    its gradient depends on lies within four cells of it, so the reference takes a
    periodic box around it (a power of two of which make the grids, so that the output
    gradient 2 d / cells rounds alike; the box's other outputs are off by order 1
    against 1e6)."""
    import torch
    from paper_1404_0959_amd import learn
    g = torch.Generator(device="cuda").manual_seed(n + 1)
    w = torch.as_tensor(learn.init_weights(n + 1), device="cuda")
    x = torch.randn((batch, n ** 3, 2), generator=g, device="cuda")
    net = P.Net(n, batch)
    y = net.forward(w, x)
    mid = crop // 2
    for cell in cells:
        at = cell[0] + n * (cell[1] + n * cell[2])
        t = y.clone()
        t[-1, at] += 1e6
        _, got = net.grad(w, x, t)
        shift = tuple(mid - c for c in cell[::-1])
        box = torch.roll(x[-1].reshape(n, n, n, 2), shift, dims=(0, 1, 2))[:crop, :crop, :crop]
        tb = torch.zeros((1, crop ** 3), device="cuda")
        tb[0, mid * (1 + crop + crop * crop)] = t[-1, at]
        _, want = reference(w, box.reshape(1, -1, 2), tb, crop)
        compare(got, want * crop ** 3 / (batch * n ** 3), 1e-2, f"{batch} x {n} cell {cell}")
