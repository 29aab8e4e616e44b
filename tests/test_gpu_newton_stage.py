"""Newton stage kernels at every width of the row-vectorised forms (one voxel per lane
with both parts unrolled, wider lanes in two passes) against the oracle: paired and
whole-wave rows, full and partly idle lanes, N1 odd."""

import pytest
import torch

import oracle as O
from synth import random_field, random_velocity
from test_gpu_parity import DTYPES, TOL, T, images, make, rel, say

pytestmark = pytest.mark.gpu

# (grid, option, width); a velocity of 0.1 keeps the flow inside the FP32 tolerances on
# these thin grids
FORMS = [((6, 8, 32), "rowvec", 1), ((5, 7, 50), "rowvec", 1), ((6, 8, 64), "rowvec", 2), ((5, 7, 126), "rowvec", 2),
         ((6, 8, 96), "rowvec", 3), ((5, 6, 150), "rowvec", 3), ((4, 8, 128), "rowvec", 4), ((4, 7, 180), "rowvec", 4),
         ((6, 8, 48), "segments", 4), ((5, 8, 90), "segments", 2)]


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("n, form, width", FORMS)
def test_newton_stage_widths(n, form, width, dtype):
    I0, I1 = images(n)
    v0 = random_velocity(n, 31, 0.1, kc=2.0)
    dv = random_field(n, 7, kc=3.0)
    p = O.Params(tuple(n), 0.01, 2, 3, 0.05)
    _, lin = O.gradient(v0, I0, I1, p)
    R, _ = make(n, dtype, nt=3, sigma2=0.05)
    R.set_option("stencil." + form, width)
    R.set_images(T(I0, dtype), T(I1, dtype))
    R.linearize(T(v0, dtype))
    e = rel(R.hessvec(T(dv, dtype), newton=True), O.hessvec_newton(dv, lin, p))
    say(f"  {form}={width} newton {e:.2e}")
    assert e <= TOL[dtype]["hv"]
