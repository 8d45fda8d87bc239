"""The weight-gradient kernels at the sizes where their split of the cells can go
wrong: one column per plane (16), chunks of planes that do not divide n (80),
several column tiles in x and y, and more units than blocks (17 grids of 64^3).

Reference: the network and its gradient in FP64 sums (torch) over the same
BF16-rounded weights, activations and layer gradients, so that what is left is
the FP32 accumulation and the rare operand it rounds the other way.  The bound
of 3e-2 of a layer's gradient is far above both; a misplaced cell, tap or channel
changes the gradient by order 1.  (Against an unrounded FP64 gradient the
rounding of the operands alone reaches 4e-2 at 16^3.)
"""
import pytest

pytestmark = pytest.mark.gpu

CH = (2, 16, 16, 16, 1)


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1404_0959_amd.pisoc as P
    P.lib()
    return P


def reference(w, x, t, n):
    """MSE loss and its gradient, x [batch, n^3, 2], t [batch, n^3]."""
    import torch

    def bf(v):
        return v.float().to(torch.bfloat16).double()

    def shifted(a, tap, sign):
        d = (tap // 9 - 1, (tap // 3) % 3 - 1, tap % 3 - 1)
        return torch.roll(a, tuple(-sign * s for s in d), dims=(1, 2, 3))

    acts, Ws, at = [bf(x).reshape(-1, n, n, n, 2)], [], 0
    for layer in range(4):
        ci, co = CH[layer], CH[layer + 1]
        W = bf(w[at:at + ci * co * 27]).reshape(co, ci, 27)
        at += ci * co * 27
        Ws.append(W)
        a = acts[-1]
        out = sum(shifted(a, tap, 1) @ W[:, :, tap].t() for tap in range(27))
        acts.append(bf(torch.relu(out)) if layer < 3 else out)
    d = acts[-1].reshape(x.shape[0], -1) - t.double()
    g = bf(2.0 / d.numel() * d).reshape(-1, n, n, n, 1)
    grads = []
    for layer in (3, 2, 1, 0):
        a, W = acts[layer], Ws[layer]
        flat = g.reshape(-1, W.shape[0])
        grads.append(torch.stack([flat.t() @ shifted(a, tap, 1).reshape(-1, W.shape[1])
                                  for tap in range(27)], dim=2).reshape(-1))
        if layer:
            back = sum(shifted(g, tap, -1) @ W[:, :, tap] for tap in range(27))
            g = bf(torch.where(a > 0, back, torch.zeros_like(back)))
    return float(d.square().mean()), torch.cat(grads[::-1])


@pytest.mark.parametrize("n,batch", [(16, 1), (16, 3), (48, 2), (80, 1), (64, 17)])
def test_gradient_of_every_layer(P, n, batch):
    import torch
    from paper_1404_0959_amd import learn
    g = torch.Generator(device="cuda").manual_seed(n + batch)
    w = torch.as_tensor(learn.init_weights(n), device="cuda")
    x = torch.randn((batch, n ** 3, 2), generator=g, device="cuda")
    t = torch.randn((batch, n ** 3), generator=g, device="cuda")
    # a target with structure: noise alone leaves a gradient of rounding size
    t = 0.1 * t + torch.roll(x[..., 0], 1, dims=1) - 0.5 * x[..., 1]
    want_loss, want = reference(w, x, t, n)
    loss, got = P.Net(n, batch).grad(w, x, t)
    assert abs(loss / want_loss - 1) <= 2e-2
    at = 0
    for layer in range(4):
        k = CH[layer] * CH[layer + 1] * 27
        d = (got[at:at + k].double() - want[at:at + k]).norm() / want[at:at + k].norm()
        print(f"n {n} batch {batch} layer {layer + 1}: {float(d):.2e}")
        assert d <= 3e-2, (layer, float(d))
        at += k
