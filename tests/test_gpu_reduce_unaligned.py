"""Inner product and smallest and largest value at a caller's own unaligned address (one
element per read), against torch in double precision."""

import math

import pytest
import torch

from paper_1807_04638_amd import Registration
from test_gpu_reduce import shifted

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("n", [(5, 7, 6), (63, 45, 50), (96, 100, 128)])
def test_reductions_at_unaligned_addresses(n, dtype):
    gen = torch.Generator(device="cuda:0").manual_seed(11)
    a, b = (torch.randn((3, *n), generator=gen, device="cuda:0", dtype=dtype) for _ in range(2))
    R = Registration(n, 2, 0.02, 2, 1.0, dtype=dtype)
    cell = (2 * math.pi) ** 3 / (n[0] * n[1] * n[2])
    # relative to the sum of magnitudes: the sum runs in double precision, whose rounding over
    # 4e6 terms stays below 1e-12 of it
    for x, y in ((shifted(a), b), (a, shifted(b)), (shifted(a), shifted(b))):
        want = float((a.double() * b.double()).sum()) * cell
        assert abs(R.dot(x, y) - want) <= 1e-12 * float((a.double() * b.double()).abs().sum()) * cell
        assert abs(R.dot(x[0], y[0]) - float((a[0].double() * b[0].double()).sum()) * cell) <= 1e-12 * float(
            (a[0].double() * b[0].double()).abs().sum()) * cell
    out = shifted(torch.zeros(n, device="cuda:0", dtype=dtype))
    assert out.data_ptr() % 16 != 0
    det, lo, hi = R.jacobian_det(a * 0.1, out=out)
    assert det.data_ptr() == out.data_ptr() and lo == float(out.min()) and hi == float(out.max())
    R.close()


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("n", [(12, 10, 48), (9, 8, 100), (6, 8, 180)])
def test_calls_on_unaligned_fields(n, dtype):
    """The same results from fields one element past an aligned address."""
    gen = torch.Generator(device="cuda:0").manual_seed(4)
    R = Registration(n, 3, 0.05, 2, 1.0, dtype=dtype)
    R.set_images(*(torch.rand(n, generator=gen, device="cuda:0", dtype=dtype) for _ in range(2)))
    v, dv = (R.apply_K(torch.randn((3, *n), generator=gen, device="cuda:0", dtype=dtype)) * 0.1 for _ in range(2))
    for newton in (False, True):
        want = R.hessvec(dv, v0=v, newton=newton)
        out = shifted(torch.zeros_like(dv))
        assert torch.equal(R.hessvec(shifted(dv), v0=shifted(v), out=out, newton=newton), want)
    assert torch.equal(R.apply_K(shifted(dv)), R.apply_K(dv))
    assert torch.equal(R.pde_displacement(shifted(v)), R.pde_displacement(v))
    R.close()
