"""Reductions read 16 bytes at a time where the address allows it: inner product, check
for NaN and Inf, smallest and largest value, at element counts that leave a remainder,
at aligned and unaligned inputs, against torch in double precision."""

import math

import pytest
import torch

from paper_1807_04638_amd import LddmmError, Registration
from synth import phantom
from test_gpu_pde import T

pytestmark = pytest.mark.gpu


def shifted(x):
    """The same values at an address one element past a 16-byte boundary."""
    buf = torch.empty(x.numel() + 1, dtype=x.dtype, device=x.device)
    out = buf[1:].view(x.shape)
    out.copy_(x)
    return out


# 3 N modulo 4: 2, 2, 0; fewer and more elements than one sweep of the grid
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("n", [(5, 7, 6), (63, 45, 50), (96, 100, 128)])
def test_reductions(n, dtype):
    gen = torch.Generator(device="cuda:0").manual_seed(11)
    v = torch.randn((3, *n), generator=gen, device="cuda:0", dtype=dtype) * 1e-3
    R = Registration(n, 2, 0.02, 2, 1e30, dtype=dtype)
    R.set_images(T(phantom(n, 4, (1.5, 3.0), False, 1), dtype), T(phantom(n, 4, (1.5, 3.0), False, 2), dtype))
    cell = (2 * math.pi) ** 3 / (n[0] * n[1] * n[2])
    for x in (v, shifted(v)):
        # the sum runs in double precision: 1e-12 is far above its rounding
        E, _ = R.pde_energy(x, True)
        Lx = R.apply_L(v)
        assert E == pytest.approx(float((Lx.double() * v.double()).sum()) * cell, rel=1e-12, abs=0)
        det, lo, hi = R.jacobian_det(x * 100)
        assert lo == float(det.min()) and hi == float(det.max())
        last = x.numel() - 1
        for at in (0, last, last - 1, last // 2):
            for bad in (math.nan, math.inf, -math.inf):
                y = x.clone() if x is v else shifted(x)
                y.view(-1)[at] = bad
                with pytest.raises(LddmmError):
                    R.pde_energy(y, True)
    R.close()
