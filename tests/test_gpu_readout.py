"""GPU parity of the read-out and projection kernels (fields, coarse fields,
order parameters, batched projection) at the sizes where their tiling changes,
against the FP64 oracle.

FP64 states and FP64 transforms: a float32 result is the correctly rounded
oracle value up to the transforms' own rounding (a few times 1e-15 of the
field's size, so at most one unit in the last place of float32); float64
results agree to 1e-12 of the field's size.
"""
import numpy as np
import pytest

from oracle import ttsh as O
from paper_2304_03306_amd import workloads as W

pytestmark = pytest.mark.gpu


def _solver(gpu, N, L, seed, prec=64):
    s = gpu.Solver([N], [L], O.workload_params(), prec)
    s.set_field(0, W.uniform_field(seed, N, 0.5, prec))
    M = N // 4
    return s, O.from_compact(s.state(0), N), M


@pytest.mark.parametrize("N", [64, 128, 256, 512, 1024, 2048])
def test_field_and_vorticity(gpu, N):
    L = 0.3 * N
    print("[case] field", N, flush=True)
    s, vhat, _ = _solver(gpu, N, L, N)
    v, w = s.field(0, omega=True)
    ref = O.field(vhat)
    kx, ky, _, _ = O.grid(N, L)
    wref = np.real(O.idft2(O.vorticity_hat(vhat, kx, ky)))
    assert np.abs(v - ref).max() < 1e-12 * np.abs(ref).max()
    assert np.abs(w - wref).max() < 1e-12 * np.abs(wref).max()
    s.close()


@pytest.mark.parametrize("N,Nc", [(64, 64), (512, 64), (256, 256), (1024, 128), (2048, 2048)])
@pytest.mark.parametrize("stride,shift", [(2, 0), (2, 1), (3, 0), (4, 2)])
def test_coarse_field_strides_and_alignment(gpu, N, Nc, stride, shift):
    """Pixel strides and base addresses with and without 8-byte alignment;
    values between the pixels' components stay untouched."""
    import torch
    print("[case] coarse field", N, Nc, stride, shift, flush=True)
    s, vhat, _ = _solver(gpu, N, 0.3 * N, N + 1)
    buf = torch.full((Nc * Nc * stride + shift,), 7.0, dtype=torch.float32, device="cuda")
    s.field_coarse(0, Nc, buf[shift:], stride)
    got = buf.cpu().numpy()
    assert (got[:shift] == 7.0).all()
    got = got[shift:].reshape(Nc, Nc, stride)
    assert (got[:, :, 2:] == 7.0).all()
    ref = O.field(O.resample(vhat, Nc))
    for c in range(2):
        assert np.abs(got[:, :, c] - ref[c]).max() < 1.2e-7 * np.abs(ref).max()
    s.close()


def test_coarse_field_finer_than_the_instance(gpu):
    """An instance read on a grid finer than its own (the context's largest)."""
    import torch
    print("[case] finer read-out 64 on 256", flush=True)
    s = gpu.Solver([64, 256], [20.0, 80.0], O.workload_params(), 64)
    s.set_field(0, W.uniform_field(3, 64, 0.5))
    vhat = O.from_compact(s.state(0), 64)
    out = torch.empty(256, 256, 2, dtype=torch.float32, device="cuda")
    s.field_coarse(0, 256, out, 2)
    ref = O.field(O.resample(vhat, 256))
    assert np.abs(out.cpu().numpy().transpose(2, 0, 1) - ref).max() < 1.2e-7 * np.abs(ref).max()
    s.close()


@pytest.mark.parametrize("N", [64, 256, 512, 2048])
def test_order_parameters(gpu, N):
    L = 0.3 * N
    print("[case] order", N, flush=True)
    s, vhat, _ = _solver(gpu, N, L, N + 2)
    v, w = s.field(0, omega=True)
    cen, D = (0.03 * L, -0.02 * L), 0.4 * L
    psi, psi2 = s.order(0, cen)
    assert abs(psi - O.vortex_order(v, L, cen)) < 1e-11
    assert abs(psi2 - O.vortex_order2(w, L, cen[0])) < 1e-11
    assert abs(s.order_dumbbell(0, D, cen) - O.vortex_order2(w, L, cen[0], D=D, center_y=cen[1])) < 1e-11
    s.close()


@pytest.mark.parametrize("N,B,ch,shift", [(64, 1, 2, 0), (64, 5, 3, 1), (128, 3, 4, 0), (512, 2, 2, 1), (1024, 1, 3, 0)])
def test_projection(gpu, N, B, ch, shift):
    """Batched projection in place with norms: the oracle's projected fields,
    and the other channels untouched."""
    import torch
    print("[case] project", N, B, ch, shift, flush=True)
    rng = np.random.default_rng(N + B)
    x = rng.standard_normal((B, N, N, ch)).astype(np.float32)
    buf = torch.zeros(B * N * N * ch + shift, dtype=torch.float32, device="cuda")
    buf[shift:] = torch.from_numpy(x.reshape(-1)).cuda()
    s = gpu.Solver([64], [20.0], O.workload_params(), 32)
    nrm = s.project_coarse(N, buf[shift:], ch, B, norms=True)
    got = buf[shift:].cpu().numpy().reshape(B, N, N, ch)
    assert (got[..., 2:] == x[..., 2:]).all()
    for b in range(B):
        vhat = O.project_field(x[b, :, :, :2].astype(np.float64).transpose(2, 0, 1), 2 * np.pi)
        ref = O.field(vhat)
        kx, ky, _, _ = O.grid(N, 2 * np.pi)
        w = np.real(O.idft2(O.vorticity_hat(vhat, kx, ky)))
        assert np.abs(got[b, :, :, :2].transpose(2, 0, 1) - ref).max() < 1.2e-7 * np.abs(ref).max()
        assert abs(nrm[b, 0] / (ref ** 2).sum() - 1) < 1e-12
        assert abs(nrm[b, 1] / (w ** 2).sum() - 1) < 1e-12
    s.close()


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("N", [64, 128, 256, 512])
def test_an_empty_region_gives_nan(gpu, N, prec):
    """Psi_2 where one region, left or right, or both hold no node (half-planes
    beside the box, disks between the nodes or off the grid), and a number
    where a region holds a single node."""
    L = 0.3 * N
    dx = L / N
    print("[case] empty region", N, prec, flush=True)
    s = gpu.Solver([N], [L], O.workload_params(), prec)
    s.set_field(0, W.uniform_field(N + 5, N, 0.5, prec))
    for cx in (-0.6 * L, 0.6 * L):
        psi, psi2 = s.order(0, (cx, 0.0))
        assert np.isfinite(psi) and np.isnan(psi2)
    xn, yn = 3 * dx, -5 * dx  # a node
    assert np.isnan(s.order_dumbbell(0, 0.5 * dx, (xn - 0.25 * dx, yn)))  # only the right disk has it
    assert np.isnan(s.order_dumbbell(0, 0.5 * dx, (xn + 0.25 * dx, yn)))  # only the left one
    assert np.isnan(s.order_dumbbell(0, 0.5 * dx, (xn - 0.25 * dx, yn + 0.5 * dx)))  # neither
    assert np.isnan(s.order_dumbbell(0, 0.2 * L, (-0.55 * L, 0.0)))  # the left one off the grid
    assert np.isnan(s.order_dumbbell(0, 0.2 * L, (0.52 * L, 0.0)))  # the right one
    assert np.isnan(s.order_dumbbell(0, 0.2 * L, (0.0, 2.0 * L)))  # both
    v, w = s.field(0, omega=True)
    i, j = N // 2 - 5, N // 2 + 3
    a, b = w[i, j], w[i, j + 1]  # one node in each disk
    assert abs(s.order_dumbbell(0, dx, (xn + 0.5 * dx, yn)) - abs(a + b) / (abs(a) + abs(b))) < 1e-11
    s.close()


def _plane_waves(s, N, L):
    """Sets a divergence-free state of a few modes (the mean, the m_x = 0 column,
    both axes' ends, the disk's rim, the lowest and some random ones) and
    returns its velocity and vorticity as sums of plane waves in FP64."""
    M = N // 4
    rng = np.random.default_rng(N)
    modes = [(0, M), (0, 1), (M, 0), (1, 0), (1, 1), (1, -1), (3 * M // 5, 4 * M // 5), (4 * M // 5, -(3 * M // 5))]
    while len(modes) < 16:
        m = (int(rng.integers(1, M)), int(rng.integers(-M, M)))
        if m[0] ** 2 + m[1] ** 2 <= M * M and m not in modes:
            modes.append(m)
    c = np.zeros((2, 2 * M + 1, M + 1), dtype=np.complex128)
    c[:, M, 0] = N * rng.standard_normal(2)  # the mean flow
    for mx, my in modes:
        a = N * complex(*rng.standard_normal(2)) / np.hypot(mx, my)
        c[:, my + M, mx] = -my * a, mx * a
        if mx == 0:
            c[:, M - my, 0] = np.conj(c[:, my + M, 0])
    s.set_state(0, c)
    c = s.state(0)
    dk = 2 * np.pi / L
    i = np.arange(N)
    left, right = [], []  # the fields are left.T @ right, per component
    for my, mx in np.argwhere(np.abs(c).max(0) > 0):
        my -= M
        ex = 2 * np.pi * ((mx * i) % N) / N
        ey = 2 * np.pi * ((my * i) % N) / N
        a = (1.0 if mx == 0 else 2.0) / N * c[:, my + M, mx]
        a = [a[0], a[1], 1j * dk * (mx * a[1] - my * a[0])]
        left.append([[(q * np.exp(1j * ey)).real, -(q * np.exp(1j * ey)).imag] for q in a])
        right += [np.cos(ex), np.sin(ex)]
    right = np.array(right)
    left = np.array(left).transpose(1, 0, 2, 3).reshape(3, -1, N)
    v = np.stack([left[q].T @ right for q in (0, 1)])
    return v, left[2].T @ right


@pytest.mark.parametrize("N,prec", [(2048, 64), (4096, 64), (8192, 96)])
def test_production_sizes(gpu, N, prec):
    """Velocity, vorticity, float pixels of either alignment and both order
    parameters where a workgroup has one row or one column, or one LDS region."""
    import torch
    L = 0.005 * N
    print("[case] production size", N, prec, flush=True)
    s = gpu.Solver([N], [L], O.workload_params(), prec)
    vr, wr = _plane_waves(s, N, L)
    v, w = s.field(0, omega=True)
    big = np.abs(vr).max()
    assert np.abs(v - vr).max() < 1e-12 * big
    assert np.abs(w - wr).max() < 1e-12 * np.abs(wr).max()
    for stride, shift in ((2, 0), (3, 1)):
        buf = torch.full((N * N * stride + shift,), 7.0, dtype=torch.float32, device="cuda")
        s.field_coarse(0, N, buf[shift:], stride)
        got = buf[shift:].view(N, N, stride)
        for c in range(2):
            assert np.abs(got[:, :, c].cpu().numpy() - vr[c]).max() < 1.2e-7 * big
        assert (got[:, :, 2:] == 7.0).all() and (buf[:shift] == 7.0).all()
        del buf, got
    cen, D = (0.03 * L, -0.02 * L), 0.4 * L
    psi, psi2 = s.order(0, cen)
    assert abs(psi - O.vortex_order(v, L, cen)) < 1e-11
    assert abs(psi2 - O.vortex_order2(w, L, cen[0])) < 1e-11
    assert abs(s.order_dumbbell(0, D, cen) - O.vortex_order2(w, L, cen[0], D=D, center_y=cen[1])) < 1e-11
    s.close()


@pytest.mark.parametrize("N,B,ch,shift", [(2048, 2, 3, 0), (4096, 1, 2, 1), (8192, 1, 2, 0)])
def test_projection_of_production_sizes(gpu, N, B, ch, shift):
    """As test_projection, with the reference's transforms by torch in FP64."""
    import torch
    print("[case] project", N, B, ch, shift, flush=True)
    buf = torch.zeros(B * N * N * ch + shift, dtype=torch.float32, device="cuda")
    buf[shift:] = torch.randn(B * N * N * ch, device="cuda", generator=torch.Generator(device="cuda").manual_seed(N))
    x = buf[shift:].view(B, N, N, ch).clone()
    s = gpu.Solver([64], [20.0], O.workload_params(), 32)
    nrm = s.project_coarse(N, buf[shift:], ch, B, norms=True)
    got = buf[shift:].view(B, N, N, ch)
    assert torch.equal(got[..., 2:], x[..., 2:])
    mx = torch.arange(N // 2 + 1, device="cuda", dtype=torch.float64)[None, :]
    my = torch.fft.fftfreq(N, 1.0 / N, device="cuda", dtype=torch.float64)[:, None]
    m2 = mx ** 2 + my ** 2
    keep = m2 <= (N // 4) ** 2
    for b in range(B):
        h = [torch.fft.rfft2(x[b, :, :, c].double()) * keep for c in range(2)]
        d = (mx * h[0] + my * h[1]) / m2.clamp_min(1.0)
        h = [h[0] - mx * d, h[1] - my * d]
        del d
        w = torch.fft.irfft2(1j * (mx * h[1] - my * h[0]), s=(N, N))
        assert abs(nrm[b, 1] / (w ** 2).sum().item() - 1) < 1e-12
        del w
        v = [torch.fft.irfft2(q, s=(N, N)) for q in h]
        big = max(q.abs().max().item() for q in v)
        for c in range(2):
            assert (got[b, :, :, c].double() - v[c]).abs().max().item() < 1.2e-7 * big
        assert abs(nrm[b, 0] / sum((q ** 2).sum().item() for q in v) - 1) < 1e-12
    s.close()
