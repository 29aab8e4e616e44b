"""The run-time transform kernels on the host (one host thread per lane, address
sanitizer, poisoned LDS) against numpy.fft, over lengths of every radix, one and
several stages, odd rows, ragged tiles and each number of units per plane."""

import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

# n0, n1, n2, components, units per plane, groups per pencil workgroup, lanes, XCD run, s, op (0 K, 1 L), add; plan
# (0: the compile-time kernels', 1: radices 2 to 10, 2: up to 16)
CASES = [
    ((6, 10, 14), 1, 2, 5, 32, 1, 2, 0, 0, 0),     # x2: one stage of radix 7; x0 two stages
    ((4, 7, 4), 1, 1, 3, 32, 1, 1, 0, 1, 0),       # whole odd planes, H = 2, one stage everywhere
    ((5, 12, 6), 3, 4, 4, 32, 2, 2, 1, 1, 0),      # quarters, single-stage x0, H = 3
    ((15, 9, 10), 1, 3, 4, 32, 8, 3, 0, 0, 0),     # thirds, ragged last tile
    ((21, 20, 70), 1, 2, 16, 64, 8, 2, 0, 1, 0),   # H = 35 (odd)
    ((18, 16, 36), 1, 2, 8, 64, 1, 2, 1, 0, 0),    # radix 9 and 2
    ((16, 30, 30), 1, 2, 16, 64, 2, 2, 0, 0, 0),   # radices 2, 3, 5; x0 = 16 (8 x 2)
    ((4, 256, 8), 1, 2, 4, 64, 1, 2, 0, 0, 0),     # a radix-16 stage along x1
    ((128, 4, 4), 1, 1, 1, 32, 1, 2, 0, 1, 0),     # a radix-16 stage along x0, one pencil per tile
    ((24, 28, 50), 1, 4, 3, 64, 4, 2, 0, 0, 0),    # quarters of 7 rows, H = 25
    ((10, 12, 60), 1, 2, 5, 32, 2, 2, 0, 1, 1),    # radices 10 (one stage along x0), 6, 5 x 6
    ((54, 18, 18), 1, 1, 4, 64, 1, 2, 1, 0, 1),    # 6 x 9, 3 x 6 whole planes, 9
    ((48, 20, 32), 1, 2, 4, 64, 1, 2, 0, 0, 1),    # 6 x 8, 10, 4 x 4
    ((15, 24, 28), 1, 2, 5, 32, 1, 2, 0, 1, 2),    # 15, 12, 14 in one stage each
    ((96, 10, 8), 1, 1, 2, 64, 1, 2, 0, 0, 2),     # 8 x 12
    ((7, 210, 24), 1, 2, 4, 64, 1, 2, 0, 0, 2),    # 7 x 15 along x1
]


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    cc = shutil.which("g++")
    if cc is None:
        pytest.skip("g++ not available")
    out = str(tmp_path_factory.mktemp("fftrt") / "fft_rt_host")
    subprocess.run([cc, "-O1", "-std=c++17", "-pthread", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", os.path.join(HERE, "native", "hip_host"), "-I",
                    os.path.join(ROOT, "paper_1807_04638_amd", "csrc"), "-I", os.path.join(ROOT, "include"), "-x", "c++",
                    os.path.join(HERE, "native", "fft_rt_host.cpp"), "-o", out], check=True)
    return out


@pytest.mark.parametrize("f64", [1, 0])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[0])) + f"-{c[2]}-{c[9]}")
def test_passes_match_numpy(exe, case, f64):
    n, ncomp, xs, tb, lanes, run, s, op, add, wide = case
    rng = np.random.default_rng(sum(n))
    f = rng.standard_normal((ncomp,) + n)
    q = rng.standard_normal((ncomp,) + n)
    if not f64:
        f, q = f.astype(np.float32).astype(np.float64), q.astype(np.float32).astype(np.float64)
    args = [*n, ncomp, xs, tb, lanes, run, s, op, f64, add, wide]
    r = subprocess.run([exe] + [str(int(a)) for a in args], input=f.tobytes() + (q.tobytes() if add else b""),
                       capture_output=True, timeout=120)
    assert r.returncode == 0, r.stderr.decode()[-2000:]
    got = np.frombuffer(r.stdout).reshape(f.shape)
    k2 = sum(np.meshgrid(*[np.fft.fftfreq(m, 1.0 / m) ** 2 for m in n], indexing="ij"))
    sym = (1.0 + 0.0025 * k2) ** (s if op else -s)
    ref = np.fft.ifftn(np.fft.fftn(f, axes=(1, 2, 3)) * sym, axes=(1, 2, 3)).real
    if add:
        ref = q + 0.3 * ref
    # rounding of about 2 log2(N) stages on values up to the symbol's range times the input's
    eps = 2.3e-16 if f64 else 1.2e-7
    tol = 8 * eps * np.log2(np.prod(n)) * max(1.0, np.sqrt(np.mean(sym**2)))
    assert np.linalg.norm(got - ref) <= tol * np.linalg.norm(f)


def test_quotient_by_reciprocal_is_exact(tmp_path):
    cc = shutil.which("g++")
    if cc is None:
        pytest.skip("g++ not available")
    src = tmp_path / "q.cpp"
    src.write_text('#include <initializer_list>\n#include "index_math.h"\nint main() { for (int d = 1; d < 2048; ++d) { const float i = 1.0f / float(d);'
                   "for (int b = 0; b < (1 << 20); b += (b < 4096 ? 1 : 97)) { const int q = b / d;"
                   "for (int x : {b, q * d, q * d + d - 1}) if (x < (1 << 20) && lddmm::index_quot(x, i) != x / d) return 1; }"
                   "} return 0; }\nvoid __syncthreads() {}\n")
    exe = str(tmp_path / "q")
    subprocess.run([cc, "-O2", "-std=c++17", "-I", os.path.join(HERE, "native", "hip_host"), "-I",
                    os.path.join(ROOT, "paper_1807_04638_amd", "csrc"), str(src), "-o", exe], check=True)
    assert subprocess.run([exe]).returncode == 0


# the highest frequencies' (1 + 0.0025 |k|^2)^s: beyond FP32's largest value for s = 80 (1e39), short of it for s = 70
@pytest.mark.parametrize("s", [70, 80])
@pytest.mark.parametrize("xs", [1, 2, 4])
def test_inverse_symbol_beyond_the_largest_float_is_zero(exe, xs, s):
    n = (6, 28, 50)
    f = np.random.default_rng(5).standard_normal((1,) + n).astype(np.float32).astype(np.float64)
    args = [*n, 1, xs, 16, 32, 1, s, 0, 0, 0, 1]
    r = subprocess.run([exe] + [str(a) for a in args], input=f.tobytes(), capture_output=True, timeout=120)
    assert r.returncode == 0, r.stderr.decode()[-2000:]
    got = np.frombuffer(r.stdout).reshape(f.shape)
    k2 = sum(np.meshgrid(*[np.fft.fftfreq(m, 1.0 / m) ** 2 for m in n], indexing="ij"))
    with np.errstate(over="ignore"):
        assert np.isinf(np.float32(1.0 + 0.0025 * k2.max()) ** np.float32(s)) == (s == 80)
    ref = np.fft.ifftn(np.fft.fftn(f, axes=(1, 2, 3)) * (1.0 + 0.0025 * k2) ** -s, axes=(1, 2, 3)).real
    # as above, and 2 s roundings of the power (of its base and its products)
    assert np.linalg.norm(got - ref) <= 1.2e-7 * (8 * np.log2(np.prod(n)) + 2 * s) * np.linalg.norm(f)
