"""The run-time transform kernels against the oracle: halves, thirds, quarters and
whole planes, odd rows, every radix, single-stage axes and ragged pencil tiles, in
both precisions, for vector and scalar fields.  Tolerances as for the operators of
the other parity tests (FP64 1e-12, FP32 2e-6, L by its symbol's growth)."""

import numpy as np
import pytest
import torch

import oracle as O
from paper_1807_04638_amd.lddmm import OP_K, apply_operator_noalloc
from synth import random_field
from test_gpu_parity import DTYPES, TOL, T, l_tol, make, rel, rounded, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, opts, cut", [
    ((24, 28, 50), {}, 1),                                            # halves of 14 rows, H = 25
    ((9, 8, 6), {}, 1),                                               # the smallest halves, H = 3, one stage along x0
    ((10, 45, 30), {}, 0),                                            # odd planes stay whole
    ((4, 7, 4), {}, 0),                                               # one stage on every axis
    ((63, 70, 90), {"fft.pencil_tb": 6}, 1),                          # ragged tiles of 3 groups
    ((60, 84, 70), {"fft.plane_threads": 256, "fft.pencil_threads": 512}, 1),
    ((30, 36, 42), {"fft.plane_halves": 0}, 0),                       # whole even planes
    ((180, 210, 180), {}, 1),                                         # halves of 153 KB in FP64
    ((128, 16, 128), {"fft.static": 0}, 1),                           # radix 16 along x0
    ((12, 256, 32), {"fft.static": 0}, 1),                            # and along x1
    ((8, 320, 288), {}, 1),                                           # quarters in FP32, split passes in FP64
    ((6, 256, 256), {}, 1),                                           # halves in FP32, quarters in FP64
    ((5, 225, 240), {}, 1),                                           # thirds
    ((50, 96, 100), {}, 1),                                           # radices 5 10, 6 8
    ((54, 36, 60), {}, 1),                                            # 6 9, 3 6, 5 6
    ((6, 210, 240), {}, 1),                                           # 7 15 and 10 12 (units over 80 KB)
    ((7, 224, 252), {}, 1),                                           # 8 14 and 9 14
])
@pytest.mark.parametrize("dtype", DTYPES)
def test_run_time_kernels(n, opts, cut, dtype):
    R, p = make(n, dtype, alpha=0.0025)
    for k, v in opts.items():
        R.set_option(k, v)
    used = R.get_option("fft.plane_halves_used")
    say(f"  {opts} cut={used} fused={R.get_option('fft.fused')} static={R.get_option('fft.static_kernels')}")
    if R.get_option("fft.fused"):
        assert used == cut
    f = rounded(random_field(n, 31, kc=max(n) / 4), dtype)
    Lf = O.apply_L(f, p)
    assert rel(R.apply_K(T(f, dtype)), O.apply_K(f, p)) <= TOL[dtype]["op"]
    assert rel(R.apply_L(T(f, dtype)), Lf) <= l_tol(p, f, Lf, dtype)
    s = T(f[1], dtype)
    R.apply_K(s, out=s)
    assert rel(s, O.apply_K(f[1], p)) <= TOL[dtype]["op"]
    assert np.isfinite(float(s.double().sum()))


def test_addend_of_the_run_time_inverse_pass():
    """The adjoint sweep adds K's term on the inverse pass: gradient and Hv on a
    grid without compile-time kernels."""
    n, dtype = (20, 18, 42), torch.float64
    R, p = make(n, dtype, nt=3)
    I0, I1 = random_field(n, 3, components=1)[0], random_field(n, 4, components=1)[0]
    v0, dv = 0.2 * random_field(n, 5), random_field(n, 6)
    R.set_images(T(I0, dtype), T(I1, dtype))
    lin = O.linearize(v0, I0, I1, p)
    g, _ = R.gradient(T(v0, dtype))
    assert rel(g, O.gradient(v0, I0, I1, p, lin)[0]) <= TOL[dtype]["grad"]
    assert rel(R.hessvec(T(dv, dtype)), O.hessvec(dv, lin, p)) <= TOL[dtype]["hv"]


@pytest.mark.parametrize("split", [0, 1])
@pytest.mark.parametrize("dtype", DTYPES)
def test_inverse_symbol_beyond_the_largest_float(dtype, split):
    """(1 + |k|^2)^13 reaches 966^13 = 6e38: K's coefficient there is 0 in FP32."""
    n, s = (24, 28, 50), 13
    R, p = make(n, dtype, alpha=1.0, s=s)
    R.set_option("fft.force_split", split)
    f = rounded(random_field(n, 7, kc=8.0), dtype)
    ref = O.apply_K(f, p)
    # rounding of about 2 log2(N) stages and of the power, on values of the input's size
    tol = (1.2e-7 if dtype == torch.float32 else 2.3e-16) * (8 * np.log2(np.prod(n)) + 2 * s) * np.linalg.norm(f)
    assert np.linalg.norm(R.apply_K(T(f, dtype)).double().cpu().numpy() - ref) <= tol
    got = apply_operator_noalloc(OP_K, T(f, dtype), 1.0, s)
    assert np.linalg.norm(got.double().cpu().numpy() - ref) <= tol


def test_long_axis_whose_pencils_leave_no_room_for_a_cut():
    """2304 x 2625 x 4 FP64: planes fit the LDS in thirds, but three sequences of 2304
    values beside their tables do not; two do, on the split path."""
    n, dtype = (2304, 2625, 4), torch.float64
    R, p = make(n, dtype, nt=1, alpha=0.0025)
    assert (R.get_option("fft.plane_halves_used"), R.get_option("fft.fused")) == (0, 0)
    f = np.random.default_rng(3).standard_normal(n)
    assert rel(R.apply_K(T(f, dtype)), O.apply_K(f, p)) <= TOL[dtype]["op"]
    R.close()


def operators_match(R, p, n, dtype):
    f = rounded(random_field(n, 31, kc=max(n) / 4), dtype)
    Lf = O.apply_L(f, p)
    assert rel(R.apply_K(T(f, dtype)), O.apply_K(f, p)) <= TOL[dtype]["op"]
    assert rel(R.apply_L(T(f, dtype)), Lf) <= l_tol(p, f, Lf, dtype)


# planes whose stages have radices 6, 9, 10, 12, 14 and 15, on the split path's kernels
@pytest.mark.parametrize("n", [(50, 96, 100), (54, 36, 60), (6, 210, 240), (7, 224, 252)])
@pytest.mark.parametrize("dtype", DTYPES)
def test_radices_on_the_split_path(n, dtype):
    R, p = make(n, dtype, alpha=0.0025)
    R.set_option("fft.force_split", 1)
    assert R.get_option("fft.fused") == 0
    operators_match(R, p, n, dtype)


def test_split_grids_keep_the_compile_time_rows():
    """16 x 490 x 180 FP32: no unit of the planes fits the LDS; rows of 180 and pencils
    of 16 points have compile-time kernels."""
    n, dtype = (16, 490, 180), torch.float32
    R, p = make(n, dtype, alpha=0.0025)
    assert (R.get_option("fft.fused"), R.get_option("fft.static_kernels")) == (0, 2)
    operators_match(R, p, n, dtype)


@pytest.mark.parametrize("n, dtype", [((6000, 16, 16), torch.float32), ((3000, 32, 32), torch.float64)])
def test_whole_planes_of_a_long_grid_keep_their_compile_time_kernels(n, dtype):
    """Pencils of two sequences do not fit the LDS: planes stay whole."""
    R, p = make(n, dtype, nt=1, alpha=0.0025)
    assert [R.get_option("fft." + k) for k in ("fused", "plane_halves_used", "static_kernels")] == [1, 0, 1]
    f = np.random.default_rng(3).standard_normal(n)
    f = rounded(f, dtype)
    assert rel(R.apply_K(T(f, dtype)), O.apply_K(f, p)) <= TOL[dtype]["op"]
    R.close()
