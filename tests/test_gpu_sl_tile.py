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
