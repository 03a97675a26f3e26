"""The resident time stepping of small grids against the two-pass stepping.

A context whose grids are all small enough steps in resident workgroups; with
a 256-point instance beside them the same instances go through the row and
column passes.  The two share their formulas and the transforms' stages; only
the order of the k = 0 row sums differs, so FP64 states agree to rounding
(bound 1e-12 after 60 steps of a flow that amplifies round-off by less than 10
per unit time) and FP32 states to a few units in the last place (1e-6).
"""
import numpy as np
import pytest

from paper_2304_03306_amd import workloads as W

pytestmark = pytest.mark.gpu


def _run(gpu, N, n, prec, params, steps, with_large, graph=20, groups=1):
    import torch
    Ns = [N] * n + ([256] if with_large else [])
    s = gpu.Solver(Ns, [0.4 * m for m in Ns], params, prec)
    s.option(gpu.TTSH_OPT_GRAPH_STEPS, graph)
    if groups > 1:
        s.option(gpu.TTSH_OPT_GROUPS, groups)
    for q in range(len(Ns)):
        L = 0.4 * Ns[q]
        s.mask_tanh(q, [(0.0, 0.0)], [L / 3.2], 0.5)
        gen = torch.Generator(device="cuda").manual_seed(17 + q)
        v = (torch.rand(2, Ns[q], Ns[q], generator=gen, device="cuda", dtype=torch.float64) - 0.5).float().double()
        s.set_field(q, v)
    for k in steps:
        s.step(k)
    s.sync()
    out = [s.state(q) for q in (0, n // 2, n - 1)]
    field = [s.field(q) for q in (0, n - 1)]
    s.close()
    return out + field


@pytest.mark.parametrize("preset", ["workload", "paper"])
@pytest.mark.parametrize("scheme", ["ifeuler", "etd1", "imex"])
@pytest.mark.parametrize("N,n,prec", [(64, 1, 64), (64, 3, 32), (64, 2, 96), (128, 96, 32), (128, 97, 96)])
def test_resident_steps_match_two_passes(gpu, N, n, prec, scheme, preset):
    import dataclasses
    print("[case] resident", N, n, prec, scheme, preset, flush=True)
    p = W.paper_coefficients() if preset == "paper" else W.workload_coefficients()
    p = dataclasses.replace(p, scheme=scheme)
    a = _run(gpu, N, n, prec, p, [60], False)
    b = _run(gpu, N, n, prec, p, [60], True)
    tol = 1e-12 if prec == 64 else 1e-6
    for x, y in zip(a, b):
        assert np.linalg.norm(x - y) < tol * np.linalg.norm(y)


@pytest.mark.parametrize("N,n,prec", [(64, 5, 64), (64, 5, 32), (128, 96, 32)])
def test_resident_steps_do_not_depend_on_the_chunks(gpu, N, n, prec):
    """Odd call lengths, plain launches, and two groups give the bits of one
    call of graph-replayed steps."""
    print("[case] resident chunks", N, n, prec, flush=True)
    p = W.paper_coefficients()
    ref = _run(gpu, N, n, prec, p, [53], False)
    for kw in (dict(steps=[1, 7, 45]), dict(steps=[53], graph=0), dict(steps=[3, 50], groups=2)):
        got = _run(gpu, N, n, prec, p, kw.pop("steps"), False, **kw)
        for x, y in zip(ref, got):
            assert np.array_equal(x, y)


def test_resident_guard_sees_a_non_finite_state(gpu):
    """A state that overflows within a resident run is reported by the sync."""
    import dataclasses
    print("[case] resident guard", flush=True)
    p = dataclasses.replace(W.workload_coefficients(), gamma_v=1e6)
    s = gpu.Solver([64], [25.6], p, 32)
    s.mask_tanh(0, [(0.0, 0.0)], [8.0], 0.5)
    s.set_field(0, W.uniform_field(1, 64, 0.5, 32))
    s.step(200)
    with pytest.raises(gpu.TTSHError):
        s.sync()
    s.close()


@pytest.mark.parametrize("preset,n128", [("workload", 130), ("paper", 170)])
@pytest.mark.parametrize("prec", [32, 96])
def test_two_resident_sizes_match_two_passes(gpu, preset, n128, prec):
    """64- and 128-point instances in one context, each size in a launch of its
    own, with one and two groups."""
    import torch
    print("[case] resident mixed", preset, n128, prec, flush=True)
    p = W.paper_coefficients() if preset == "paper" else W.workload_coefficients()

    def run(with_large, groups):
        Ns = [64] * 3 + [128] * n128 + ([256] if with_large else [])
        s = gpu.Solver(Ns, [0.4 * m for m in Ns], p, prec)
        if groups > 1:
            s.option(gpu.TTSH_OPT_GROUPS, groups)
        for q, N in enumerate(Ns):
            s.mask_tanh(q, [(0.0, 0.0)], [0.125 * N], 0.5)
            gen = torch.Generator(device="cuda").manual_seed(31 + q)
            v = torch.rand(2, N, N, generator=gen, device="cuda", dtype=torch.float64) - 0.5
            s.set_field(q, v.float().double())
        s.step(60)
        s.sync()
        out = [s.state(q) for q in (0, 2, 3, 4 + n128 // 2, n128 + 2)]
        s.close()
        return out

    ref = run(True, 1)
    for got in (run(False, 1), run(False, 2)):
        for x, y in zip(got, ref):
            assert np.linalg.norm(x - y) < 1e-6 * np.linalg.norm(y)


@pytest.mark.parametrize("graph", [0, 50])
@pytest.mark.parametrize("every,caught", [(7, True), (20, True), (21, False), (0, False)])
def test_resident_guard_looks_at_its_interval(gpu, every, caught, graph):
    """A state that overflows within a run of 20 steps and is replaced before
    the sync: only a check queued within the run can have seen it."""
    import dataclasses
    print("[case] resident guard interval", every, graph, flush=True)
    p = dataclasses.replace(W.workload_coefficients(), gamma_v=1e6)
    s = gpu.Solver([64, 64], [25.6, 25.6], p, 32)
    s.option(gpu.TTSH_OPT_GRAPH_STEPS, graph)
    s.option(gpu.TTSH_OPT_GUARD_EVERY, every)
    s.mask_tanh(0, [(0.0, 0.0)], [8.0], 0.5)  # the other instance has no wall
    for q in range(2):
        s.set_field(q, W.uniform_field(1, 64, 0.5, 32))
    s.step(20)
    s.set_field(0, W.uniform_field(1, 64, 0.5, 32))
    if caught:
        with pytest.raises(gpu.TTSHError, match="instance 0"):
            s.sync()
    s.sync()  # clean, or cleared by the report
    s.close()
