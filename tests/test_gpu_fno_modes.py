"""The per-mode gradient kernel and the one-launch weight refresh of the
surrogate, at batch sizes around the kernel's 64-sample chunks and at several
mode counts, against the general GEMM path of the same network.

The two paths take the same BF16 operands; other stages between them may round
a few intermediates differently, by at most one BF16 unit in the last place
(2^-8) on a small part of the values, so the gradients agree to 1e-2 in
relative L2.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("modes,size", [(3, 32), (8, 32), (16, 64)])
@pytest.mark.parametrize("batch", [1, 63, 64, 65, 130])
def test_mode_gradients_match_the_general_path(gpu, modes, size, batch):
    import torch
    from paper_2304_03306_amd import fno as F
    print("[case] mode gradients", modes, size, batch, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(batch)
    x = torch.randn(batch, size, size, 3, device="cuda", generator=gen)
    t = torch.randn(batch, size, size, 2, device="cuda", generator=gen)
    y = torch.empty_like(t)
    out = []
    for special in (1, 0):
        net = F.FNO(width=32, modes=modes, layers=2, H=size, W=size, max_batch=batch, seed=5)
        net.set_option(F.FNO_OPT_SPECIALIZED, special)
        net.forward(x, y, train=True)
        net.loss(y, t)
        net.backward(batch)
        out.append(net.grads().astype(np.float64))
        net.close()
    nR = 2 * modes * modes * 32 * 32  # one part of a layer's mode matrices
    o = 3 * 32 + 32
    for _ in range(2):
        for _ in range(2):
            a, b = out[0][o:o + nR], out[1][o:o + nR]
            assert np.linalg.norm(a - b) < 1e-2 * np.linalg.norm(b)
            o += nR
        o += 32 * 32 + 32


def test_refreshed_weights_are_the_parameters(gpu):
    """A network whose parameters were set twice gives the output of a network
    created with the second set, bit for bit (every compute copy is renewed)."""
    import torch
    from paper_2304_03306_amd import fno as F
    for kw in (dict(width=32, modes=16), dict(width=32, modes=5), dict(width=24, modes=4)):
        print("[case] refresh", kw, flush=True)
        a, b = (F.FNO(layers=3, H=64, W=64, max_batch=2, seed=s, **kw) for s in (1, 2))
        a.set_params(b.params())
        x = torch.randn(2, 64, 64, 3, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))
        ya, yb = (torch.empty(2, 64, 64, 2, device="cuda") for _ in range(2))
        a.forward(x, ya)
        b.forward(x, yb)
        torch.cuda.synchronize()
        assert torch.equal(ya, yb)
        # backward uses the transposed copies
        t = torch.zeros_like(ya) + 0.5
        for net, y in ((a, ya), (b, yb)):
            net.forward(x, y, train=True)
            net.loss(y, t)
            net.backward(2)
        assert np.array_equal(a.grads(), b.grads())
        a.close()
        b.close()


@pytest.mark.parametrize("shift", [1, 2, 4])
@pytest.mark.parametrize("cin", [2, 3])
def test_input_alignment_does_not_matter(gpu, cin, shift):
    """The input at any 4-byte alignment gives the bits of a 16-byte aligned one."""
    import torch
    from paper_2304_03306_amd import fno as F
    print("[case] input alignment", cin, shift, flush=True)
    net = F.FNO(width=32, modes=4, layers=1, cin=cin, H=16, W=16, max_batch=3, seed=2)
    n = 3 * 16 * 16 * cin
    buf = torch.randn(n + 8, device="cuda", generator=torch.Generator(device="cuda").manual_seed(4))
    y = [torch.empty(3, 16, 16, 2, device="cuda") for _ in range(2)]
    net.forward(buf[shift:shift + n].view(3, 16, 16, cin), y[0])
    net.forward(buf[shift:shift + n].clone().view(3, 16, 16, cin), y[1])
    torch.cuda.synchronize()
    assert torch.equal(y[0], y[1])
    net.close()


@pytest.mark.parametrize("modes,size", [(3, 32), (8, 32), (16, 64)])
@pytest.mark.parametrize("batch", [1, 63, 64, 65, 130])
def test_mode_gradients_are_the_sums_of_the_captured_modes(gpu, modes, size, batch):
    """The per-mode products of the BF16 modes that the kernel read, summed in
    FP64: 2 batch terms added in FP32 with at most 2^-23 of the partial sum lost
    at each, so (2 batch + 4) 2^-23 of the sum of absolute terms."""
    import torch
    from paper_2304_03306_amd import fno as F
    print("[case] mode gradient sums", modes, size, batch, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(100 + batch)
    x = torch.randn(batch, size, size, 3, device="cuda", generator=gen)
    t = torch.randn(batch, size, size, 2, device="cuda", generator=gen)
    y = torch.empty_like(t)
    m, C = modes, 32
    net = F.FNO(width=C, modes=m, layers=2, H=size, W=size, max_batch=batch, seed=6)
    net.set_option(F.FNO_OPT_CAPTURE, 1)
    net.forward(x, y, train=True)
    net.loss(y, t)
    net.backward(batch)
    g = net.grads().astype(np.float64)
    nG = m * 4 * m * batch * C
    nR = 2 * m * m * C * C
    o = 3 * C + C
    for l in range(2):
        f, d = (net.capture(w, l, nG).reshape(m, 4 * m, batch, C) for w in (F.FNO_CAP_G, F.FNO_CAP_GG))
        f, d = ([a[:, :2 * m], a[:, 2 * m:]] for a in (f, d))

        def products(u, v):  # [kx][q][c][o] -> [q][kx][c][o]
            return np.matmul(u.swapaxes(2, 3), v).swapaxes(0, 1)

        for ref, size_ in ((products(f[0], d[0]) + products(f[1], d[1]),
                            products(abs(f[0]), abs(d[0])) + products(abs(f[1]), abs(d[1]))),
                           (products(f[0], d[1]) - products(f[1], d[0]),
                            products(abs(f[0]), abs(d[1])) + products(abs(f[1]), abs(d[0])))):
            got = g[o:o + nR].reshape(2 * m, m, C, C)
            assert (size_ > 0).any()
            assert (np.abs(got - ref) <= (2 * batch + 4) * 2.0 ** -23 * size_ + 1e-30).all()
            o += nR
        o += C * C + C
    net.close()
