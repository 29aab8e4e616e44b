"""Semi-Lagrangian steps whose points stay within a voxel (gathered from a tile's
window in the LDS), go further (gathered from global memory) and both in one field,
against the oracle on edges and remainders of the tiles.  FP64 1e-11 (1e-10 for the
PDE gradient and Hessian product), FP32 1e-5 and 1e-4, as for the other parity tests."""

import numpy as np
import pytest
import torch

import oracle as O
import oracle.pde_lddmm as P
from synth import phantom, random_field
from test_gpu_parity import DTYPES, T, make, rel, rounded, say

pytestmark = pytest.mark.gpu


def velocity(n, vox, nt, seed):
    """|v| dt of `vox` voxels at most; "mixed": 0.3 with a patch of 2.5."""
    v = random_field(n, seed, kc=2.0)
    v /= np.sqrt((v * v).sum(0).max())
    if vox == "mixed":
        x = [np.arange(m) / m - 0.5 for m in n]
        bump = np.exp(-40 * (x[0][:, None, None] ** 2 + x[1][None, :, None] ** 2 + x[2][None, None, :] ** 2))
        v = v * (0.3 + 2.2 * bump)
    else:
        v = v * vox
    return v * nt * 2 * np.pi / max(n)


@pytest.mark.parametrize("n", [(4, 7, 6), (9, 30, 70), (21, 64, 50), (64, 64, 64), (6, 12, 126)])
@pytest.mark.parametrize("vox", [0.45, 3.0, "mixed"])
@pytest.mark.parametrize("dtype", DTYPES)
def test_steps_within_and_beyond_a_voxel(n, vox, dtype):
    nt = 3
    R, p = make(n, dtype, nt=nt, alpha=0.01)
    I0, I1 = phantom(n, 3, (1.0, 2.0), False, 5), phantom(n, 3, (1.0, 2.0), False, 6)
    v, dv = rounded(velocity(n, vox, nt, 3), dtype), rounded(0.1 * random_field(n, 4, kc=2.0), dtype)
    I0, I1 = rounded(I0, dtype), rounded(I1, dtype)
    R.set_images(T(I0, dtype), T(I1, dtype))
    u = R.pde_displacement(T(v, dtype), stationary=True)
    e = {"u1": rel(u, P.displacement([v] * (nt + 1), p))}
    g_ref, lin = P.gradient(v, I0, I1, p, True)
    g, E = R.pde_gradient(T(v, dtype), stationary=True)
    e["grad"] = rel(g, g_ref)
    e["hv"] = rel(R.pde_hessvec(T(dv, dtype), stationary=True), P.hessvec(dv, lin, p))
    say(f"  {vox} voxels a step", {k: f"{x:.2e}" for k, x in e.items()})
    f64 = dtype == torch.float64
    assert e["u1"] <= (1e-11 if f64 else 1e-5)
    assert e["grad"] <= (1e-10 if f64 else 1e-4) and e["hv"] <= (1e-10 if f64 else 1e-4)


# ragged along every axis (tiles of 4 x 63, 42 x 6 and 7 x 35 voxels), an odd number of planes.  The Hessian
# product in FP64 on the first grid: on the long ones L's symbol, and in FP32 the velocity, amplify its rounding
# (with plain gathers 1.5e-9 in FP64 on the second grid, 1.1e-4 in FP32 on the first)
@pytest.mark.parametrize("n, share, hv", [((98, 105, 126), 0.0005, True), ((98, 105, 126), 0.02, True),
                                          ((1575, 50, 6), 0.0005, False), ((243, 45, 70), 0.0005, False)])
@pytest.mark.parametrize("dtype", DTYPES)
def test_scattered_points_beyond_a_voxel(dtype, n, share, hv):
    """Tiles in which a few lanes of a wave, or lanes of most waves, leave the window:
    2.5 voxels a step on a share of the voxels, 0.3 elsewhere."""
    nt = 2
    R, p = make(n, dtype, nt=nt, alpha=0.01)
    r = np.random.default_rng(8)
    v = random_field(n, 3, kc=2.0)
    v *= 0.3 / np.sqrt((v * v).sum(0).max())
    v += np.where(r.random(n) < share, 2.5, 0.0) * r.choice([-1.0, 1.0], (3,) + n)
    v = rounded(v * nt * 2 * np.pi / max(n), dtype)
    dv = rounded(0.1 * random_field(n, 4, kc=2.0), dtype)
    I0, I1 = (rounded(phantom(n, 3, (1.0, 2.0), False, k), dtype) for k in (5, 6))
    R.set_images(T(I0, dtype), T(I1, dtype))
    f64 = dtype == torch.float64
    g_ref, lin = P.gradient(v, I0, I1, p, True)
    e = {"u1": rel(R.pde_displacement(T(v, dtype), stationary=True), P.displacement([v] * (nt + 1), p)),
         "grad": rel(R.pde_gradient(T(v, dtype), stationary=True)[0], g_ref)}
    if f64 and hv:
        e["hv"] = rel(R.pde_hessvec(T(dv, dtype), stationary=True), P.hessvec(dv, lin, p))
    say(f"  {share} of the voxels", {k: f"{x:.2e}" for k, x in e.items()})
    assert e["u1"] <= (1e-11 if f64 else 1e-5)
    assert e["grad"] <= (1e-10 if f64 else 1e-4) and e.get("hv", 0.0) <= 1e-10


@pytest.mark.parametrize("share", [0.0005, 0.02])
def test_tiles_of_four_planes(share):
    """4375 x 5 x 250 FP32, more than 16384 tiles: displacement and transported image."""
    n, nt, dtype = (4375, 5, 250), 2, torch.float32
    R, p = make(n, dtype, nt=nt, alpha=0.01)
    r = np.random.default_rng(8)
    v = random_field(n, 3, kc=2.0)
    v *= 0.3 / np.sqrt((v * v).sum(0).max())
    v += np.where(r.random(n) < share, 2.5, 0.0) * r.choice([-1.0, 1.0], (3,) + n)
    v = rounded(v * nt * 2 * np.pi / max(n), dtype)
    I0, I1 = (rounded(random_field(n, k, components=1)[0], dtype) for k in (5, 6))
    R.set_images(T(I0, dtype), T(I1, dtype))
    u = R.pde_displacement(T(v, dtype), stationary=True)
    m1 = R.pde_energy(T(v, dtype), stationary=True)[1]
    e = {"u1": rel(u, P.displacement([v] * (nt + 1), p)), "m1": rel(m1, P.state([v] * (nt + 1), I0, p)[-1])}
    say(f"  {share} of the voxels", {k: f"{x:.2e}" for k, x in e.items()})
    assert e["u1"] <= 1e-5 and e["m1"] <= 1e-5
    R.close()
