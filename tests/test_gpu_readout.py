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
