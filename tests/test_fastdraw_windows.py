"""CPU check of the FP32 count estimates (csrc/fastdraw.hpp, Sec. 4.3.1) on cells of windows of 1
to 4.2 sigma: the estimates take the weights of the erf polynomial, the counts are defined by
those of the series (det_erf), whose error grows towards the edges of wide windows and, times
the electron count, passes any fixed margin.  Wherever the estimates claim certainty the count
equals the oracle's, with uniforms next to the cumulative sums and up to 2^31 electrons.  And
where the series gives weights below 0 and above 1."""
import os
import shutil
import subprocess

import numpy as np
import pytest
from scipy.special import erfinv

from oracle import fluct as OF
from oracle import normal as ON
from test_fastdraw_host import binom
from test_fastdraw_host import checker as plain_checker  # noqa: F401 (a fixture)

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SQRT_HALF = 0.5**0.5


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("fastdraw") / "fastdraw_window_check")
    subprocess.run([hipcc, "-std=c++17", "-O2", "-ffp-contract=off", "--offload-arch=gfx950", "-I",
                    os.path.join(ROOT, "paper_2104_08265_amd", "csrc"), "-x", "hip",
                    os.path.join(HERE, "sampler_host", "fastdraw_window_check.hip"), "-o", exe],
                   check=True, capture_output=True)
    return exe


def run(exe, mode, *columns):
    """Columns of numbers, one cell a line -> (sure, count)."""
    text = [[str(v) if isinstance(v, int) else v.hex() for v in np.asarray(c).tolist()] for c in columns]
    out = subprocess.run([exe, mode], input="\n".join(map(" ".join, zip(*text))), capture_output=True, text=True,
                         check=True).stdout.split()
    got = np.array(out, np.int64)
    return got[0::2] != 0, got[1::2]


def probability(cell):
    e = [OF.det_erf(x) for x in cell]
    return (0.5 * (e[1] - e[0])) * (0.5 * (e[3] - e[2]))


def edge_cells(rng, nsigma, N, mu):
    """Cells at the window's upper edge, N p about mu, on the other axis most of the window."""
    s = nsigma * SQRT_HALF
    b0, b1 = np.full(N.size, -s), np.where(rng.random(N.size) < 0.7, s, rng.uniform(0.0, s, N.size))
    density = np.exp(-s * s) / np.sqrt(np.pi) * 0.5 * (OF.det_erf(b1) - OF.det_erf(b0))
    return np.maximum(s - mu / N / density, 0.0), np.full(N.size, s), b0, b1


def next_to_sums(rng, N, p, most, each, lo, hi):
    """Indices and uniforms: `each` per cell, 10^lo to 10^hi beside one of its first sums."""
    i = np.repeat(np.arange(N.size), each)
    f, F, pick = np.exp(N * np.log1p(-p))[i], np.zeros(i.size), rng.integers(0, most, i.size)
    for k in range(most):
        F += np.where(pick >= k, f, 0.0)
        f *= (p / (1.0 - p))[i] * (N[i] - k) / (k + 1)
    u = F + rng.choice([-1.0, 1.0], i.size) * 10.0 ** rng.uniform(lo, hi, i.size)
    ok = (u > 0.0) & (u < 1.0)
    return i[ok], u[ok]


def assert_sure_counts(checker, mode, ref, N, cell, *last):
    sure, k = run(checker, mode, N, *cell, *last)
    bad = np.nonzero(sure & (k != ref))[0]
    assert bad.size == 0, [(int(N[i]), [float(c[i]) for c in cell], int(k[i]), int(ref[i])) for i in bad[:5]]
    return sure


@pytest.mark.parametrize("nsigma", [1.0, 3.0, 4.2])
@pytest.mark.parametrize("n_lo,n_hi", [(5e2, 1e7), (5e8, 2.1e9)])
def test_sure_binomial_counts_of_edge_cells(checker, nsigma, n_lo, n_hi):
    rng = np.random.default_rng(31)
    N = np.exp(rng.uniform(np.log(n_lo), np.log(n_hi), 3000)).astype(np.int64)
    cell = edge_cells(rng, nsigma, N, 10.0 ** rng.uniform(-3, 1.2, N.size))
    i, u = next_to_sums(rng, N, probability(cell), 4, 12, -5.0, -3.7)
    cell = [c[i] for c in cell]
    sure = assert_sure_counts(checker, "binom", OF.binomial(N[i], probability(cell), u), N[i], cell, u)
    if n_hi == 1e7:
        assert np.mean(sure) > 0.3


def test_sure_binomial_counts_near_one_half(checker):
    """Eleven to twenty electrons with p from 0.4 to 0.4999, u within 1e-5 to 5e-5 of a sum."""
    rng = np.random.default_rng(32)
    N = rng.integers(11, 21, 3000)
    s = 3.0 * SQRT_HALF
    p = rng.uniform(0.4, 0.4999, N.size)
    B = OF.det_erf(np.array(s))
    cell = np.full(N.size, -s), erfinv(2.0 * p / B - OF.det_erf(np.array(s))), np.full(N.size, -s), np.full(N.size, s)
    i, u = next_to_sums(rng, N, probability(cell), 15, 24, -5.0, -4.3)
    cell = [c[i] for c in cell]
    sure = assert_sure_counts(checker, "binom", OF.binomial(N[i], probability(cell), u), N[i], cell, u)
    assert np.mean(sure) > 0.3


@pytest.mark.parametrize("nsigma", [1.0, 4.2])
@pytest.mark.parametrize("n_lo,n_hi", [(5e2, 1e7), (5e8, 2.1e9)])
def test_sure_normal_counts_of_edge_cells(checker, nsigma, n_lo, n_hi):
    rng = np.random.default_rng(33)
    N = np.exp(rng.uniform(np.log(n_lo), np.log(n_hi), 60000)).astype(np.int64)
    cell = edge_cells(rng, nsigma, N, 10.0 ** rng.uniform(-3, 1.2, N.size))
    w = rng.integers(0, 2**32, (4, N.size), dtype=np.uint64)
    ref = ON.normal_count(N, probability(cell), ON.box_muller_words(*w)[0])
    sure = assert_sure_counts(checker, "normal", ref, N, cell, *w[:3].astype(np.int64))
    if n_hi == 1e7:
        assert np.mean(sure) > 0.9


@pytest.mark.parametrize("nsigma", [3.0, 4.2])
def test_sure_normal_counts_inside_one_cell(checker, nsigma):
    """p = erf(nsigma / sqrt 2)^2, x next to whole numbers around N: sd rests on 1 - p."""
    rng = np.random.default_rng(35)
    N = np.exp(rng.uniform(np.log(20), np.log(20000), 100000)).astype(np.int64)
    s = nsigma * SQRT_HALF
    cell = [np.full(N.size, v) for v in (-s, s, -s, s)]
    p = probability(cell)
    sd = np.sqrt(N * p * (1.0 - p))
    x = N - np.floor(np.abs(rng.normal(0, 1.5, N.size))) + rng.uniform(-3e-3, 3e-3, N.size) * np.maximum(sd, 0.05)
    z = (x - 0.5 - N * p) / sd
    ok = np.abs(z) < 6
    N, z, cell = N[ok], z[ok], [c[ok] for c in cell]
    w = np.zeros((4, N.size), np.uint64)  # the even cell's normal is r cos(0) or r cos(pi)
    w[0] = (1.0 - np.exp(-0.5 * z * z)) * 2.0**32
    w[1] = rng.integers(0, 2**32, N.size, dtype=np.uint64)
    w[2] = np.where(z < 0, 2**31, 0)
    ref = ON.normal_count(N, probability(cell), ON.box_muller_words(*w)[0])
    assert_sure_counts(checker, "normal", ref, N, cell, *w[:3].astype(np.int64))


def test_probabilities_outside_0_and_1(plain_checker):  # noqa: F811
    rng = np.random.default_rng(34)
    p = np.concatenate([-10.0 ** rng.uniform(-9, 4, 400), 10.0 ** rng.uniform(-0.5, 4, 400), [2.0, 4.0, -2.0]])
    N, p, u = (v.ravel() for v in np.meshgrid([1, 2, 3, 20, 5000], p, [0.0, 0.1, 0.6, 0.9999], indexing="ij"))
    sure, k = binom(plain_checker, N, p, u)
    ref = OF.binomial(N, p, u)
    bad = np.nonzero(sure & (k != ref))[0]
    assert bad.size == 0, [(int(N[i]), float(p[i]), float(u[i]), int(k[i]), int(ref[i])) for i in bad[:5]]
