"""What the tuner chooses where candidates launch the same kernels: it keeps
what it cannot tell apart instead of picking by the noise of its timings."""
import dataclasses

import pytest

from paper_2304_03306_amd import workloads as W

pytestmark = pytest.mark.gpu


def _solver(gpu, Ns, prec=32, scheme="ifeuler"):
    p = dataclasses.replace(W.workload_coefficients(), scheme=scheme)
    s = gpu.Solver(Ns, [0.4 * n for n in Ns], p, prec)
    for q, n in enumerate(Ns):
        s.mask_tanh(q, [(0.0, 0.0)], [0.125 * n], 0.5)
        s.set_field(q, W.uniform_field(q, n, 0.05, prec if prec == 32 else 64))
    return s


@pytest.mark.parametrize("Ns,prec", [([64], 32), ([64] * 3, 64), ([64] * 5, 96), ([128] * 100, 32), ([64, *[128] * 130], 32)])
def test_resident_contexts_keep_the_passes_configuration(gpu, Ns, prec):
    """The steps launch neither pass: sizes, splits and schedules come back as
    they were set, only the number of groups is chosen."""
    print("[case] tune resident", len(Ns), prec, flush=True)
    s = _solver(gpu, Ns, prec)
    for cfg in ([128, 64, 0, 1, 8, 8, 1], [64, 128, 1, 0, 8, 8, 1]):
        s.set_tuning(cfg)
        got, us = s.tune(3)
        assert list(got[:6]) == cfg[:6] and got[6] in (1, 2) and us > 0
        assert list(s.get_tuning()) == list(got)
    s.step(5)
    s.sync()
    s.close()


@pytest.mark.parametrize("N,prec,scheme", [(64, 32, "etdrk2"), (128, 32, "ifeuler"), (256, 32, "ifeuler"), (256, 64, "ifeuler"),
                                           (512, 32, "etd1"), (512, 96, "ifeuler")])
def test_one_size_has_no_split_to_choose(gpu, N, prec, scheme):
    """A single grid size launches its own kernels with either split value."""
    print("[case] tune one size", N, prec, scheme, flush=True)
    s = _solver(gpu, [N] * 2, prec, scheme)
    got, _ = s.tune(3)
    assert list(got[2:4]) == [0, 0]
    s.close()
