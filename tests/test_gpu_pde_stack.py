"""Spectral passes over the time points of a PDE-LDDMM stack: one time step, stacks that
one pass holds, stacks cut into several passes with a remainder, and fields too large to
share one. With a data weight of 1e-30 the gradient is 2 L v, the product 2 L dv and the
energy the space-time sum of <L v, v>, each of which single-field calls give too."""

import math

import pytest
import torch

from paper_1807_04638_amd import Registration
from synth import phantom
from test_gpu_pde import T

pytestmark = pytest.mark.gpu


# spectra of a field / of a pass (96 MB): 25 kB, 6.5 MB (passes of 14 or 15 of the 18
# time points), 45 MB (two and one of three), 101 MB (one)
@pytest.mark.parametrize("n, nt, dtype", [((8, 6, 10), 1, torch.float64), ((20, 24, 30), 8, torch.float32),
                                          ((64, 64, 64), 17, torch.float64), ((128, 120, 120), 2, torch.float64),
                                          ((160, 160, 160), 1, torch.float64)])
def test_stack_passes(n, nt, dtype):
    tol = 1e-12 if dtype == torch.float64 else 2e-6  # the operator's own bound
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    v, dv = (torch.randn((nt + 1, 3, *n), generator=gen, device="cuda:0", dtype=dtype) * 1e-3 for _ in range(2))
    R = Registration(n, nt, 0.02, 2, 1e30, dtype=dtype)
    R.set_images(T(phantom(n, 4, (1.5, 3.0), False, 1), dtype), T(phantom(n, 4, (1.5, 3.0), False, 2), dtype))
    g, E = R.pde_gradient(v, False)
    hv = R.pde_hessvec(dv.clone(), False)
    want = 0.0
    for k in range(nt + 1):
        Lv, Ldv = R.apply_L(v[k].contiguous()), R.apply_L(dv[k].contiguous())
        assert float((g[k] - 2 * Lv).norm()) <= tol * float(Lv.norm())
        assert float((hv[k] - 2 * Ldv).norm()) <= tol * float(Ldv.norm())
        w = (0.5 if k in (0, nt) else 1.0) / nt
        want += w * float((Lv.double() * v[k].double()).sum()) * (2 * math.pi) ** 3 / (n[0] * n[1] * n[2])
    assert E == pytest.approx(want, rel=1e-6 if dtype == torch.float32 else 1e-12, abs=0)
    R.close()


def test_stack_on_the_split_path_with_a_long_first_axis():
    """128 x 8 x 8, 181 time points, split passes: the x1 pencils of all fields would be
    more than a launch's second dimension holds."""
    n, nt, dtype = (128, 8, 8), 180, torch.float64
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    v = torch.randn((nt + 1, 3, *n), generator=gen, device="cuda:0", dtype=dtype) * 1e-3
    R = Registration(n, nt, 0.02, 2, 1e30, dtype=dtype)
    R.set_option("fft.force_split", 1)
    R.set_images(T(phantom(n, 4, (1.5, 3.0), False, 1), dtype), T(phantom(n, 4, (1.5, 3.0), False, 2), dtype))
    g, _ = R.pde_gradient(v, False)
    for k in range(nt + 1):
        Lv = R.apply_L(v[k].contiguous())
        assert float((g[k] - 2 * Lv).norm()) <= 1e-12 * float(Lv.norm())
    R.close()
