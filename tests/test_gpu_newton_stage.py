"""Newton stage kernels at every width of the row-vectorised forms (one voxel per lane
with both parts unrolled, wider lanes in two passes) against the oracle: paired and
whole-wave rows, full and partly idle lanes, N1 odd; and the product for one to several time steps,
each trajectory policy, from one linearization to the next."""

import pytest
import torch

import oracle as O
from paper_1807_04638_amd import Registration
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


@pytest.mark.parametrize("every", [0, 2])
@pytest.mark.parametrize("nt", [1, 2, 5])
@pytest.mark.parametrize("n", [(8, 6, 10), (6, 8, 64)])  # one voxel per thread, row-vectorised
def test_newton_history(n, nt, every):
    """The stage histories are written by the sweeps themselves: products with two
    directions, then at another velocity, in the output's own memory too."""
    I0, I1 = images(n)
    p = O.Params(tuple(n), 0.01, 2, nt, 0.05)
    R = Registration(n, nt, 0.01, s=2, sigma2=0.05, dtype=torch.float64, checkpoint_every=every)
    R.set_images(T(I0, torch.float64), T(I1, torch.float64))
    for seed in (31, 32):
        v0 = random_velocity(n, seed, 0.1, kc=2.0)
        _, lin = O.gradient(v0, I0, I1, p)
        R.linearize(T(v0, torch.float64))
        for kd in (7, 8):
            dv = random_field(n, kd, kc=3.0)
            want = O.hessvec_newton(dv, lin, p)
            d = T(dv, torch.float64)
            assert rel(R.hessvec(d, newton=True), want) <= TOL[torch.float64]["hv"]
            assert rel(R.hessvec(d, newton=True, out=d), want) <= TOL[torch.float64]["hv"]
