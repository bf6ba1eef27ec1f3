"""CPU check of the FP32 count estimates (csrc/fastdraw.hpp, Sec. 4.3.1) against the oracle:
wherever they claim certainty the count equals the one the FP64 sampler defines, on seeded
and edge triples over both regimes, and they leave few cells undecided on the parameters of
real windows."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import fluct as OF
from oracle import normal as ON
from test_sampler_host import edge_triples, triples

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("fastdraw") / "fastdraw_host_check")
    subprocess.run([hipcc, "-std=c++17", "-O2", "-ffp-contract=off", "--offload-arch=gfx950",
                    "-DWCT_HOST_LOCKSTEP", "-I",
                    os.path.join(ROOT, "paper_2104_08265_amd", "csrc"), "-x", "hip",
                    os.path.join(HERE, "sampler_host", "fastdraw_host_check.hip"), "-o", exe],
                   check=True, capture_output=True)
    return exe


def run(exe, mode, lines):
    out = subprocess.run([exe, mode], input="".join(lines), capture_output=True, text=True, check=True).stdout.split()
    return np.array([int(v) for v in out], np.int64)


def binom(exe, N, p, u):
    got = run(exe, "binom", (f"{int(n)} {float(a).hex()} {float(b).hex()}\n" for n, a, b in zip(N, p, u)))
    return got[0::2] != 0, got[1::2]


def window_triples(seed, n):
    """Cells of 3-sigma windows: charges of 100 to 1e6 electrons over Gaussian weights."""
    rng = np.random.default_rng(seed)
    N = np.exp(rng.uniform(np.log(100), np.log(1e6), n)).astype(np.int64)
    peak = 0.16 / (rng.uniform(3, 20, n) * rng.uniform(1, 3, n))
    return N, peak * np.exp(-0.5 * rng.uniform(0, 3, n) ** 2 - 0.5 * rng.uniform(0, 3, n) ** 2), rng.random(n)


@pytest.mark.parametrize("make,seed", [(edge_triples, None), (triples, 11), (triples, 12), (window_triples, 13),
                                       (window_triples, 14)])
def test_sure_binomial_counts_equal_the_oracle(checker, make, seed):
    N, p, u = make() if seed is None else make(seed, 60000)
    sure, k = binom(checker, N, p, u)
    ref = OF.binomial(N, p, u)
    bad = np.nonzero(sure & (k != ref))[0]
    assert bad.size == 0, [(int(N[i]), float(p[i]), float(u[i]), int(k[i]), int(ref[i])) for i in bad[:5]]
    if make is window_triples:
        # means up to the search's limit: at most 0.4% near a sum, 1.2% near a rounding mode
        assert np.mean(~sure[N * p < 1000]) < 0.016


def test_sure_binomial_counts_next_to_the_sums(checker):
    """u placed at every cumulative sum of the inversion, and 1e-7 to 1e-3 to either side."""
    rng = np.random.default_rng(5)
    N, p, u = [], [], []
    for n, mu in [(1, 0.3), (3, 0.7), (20, 9.7), (50, 4.0), (700, 1.0), (5000, 9.9), (200000, 6.0)]:
        f = np.exp(n * np.log1p(-mu / n))
        F = 0.0
        for k in range(min(n, 40)):
            F += f
            f *= (mu / n) / (1 - mu / n) * (n - k) / (k + 1)
            for d in np.concatenate([[0.0], 10.0 ** rng.uniform(-7, -3, 6)]):
                for v in (F - d, F + d):
                    if 0.0 <= v < 1.0:
                        N.append(n), p.append(mu / n), u.append(v)
    sure, k = binom(checker, N, p, u)
    ref = OF.binomial(np.array(N), np.array(p), np.array(u))
    assert np.array_equal(k[sure], ref[sure]) and 0.1 < np.mean(sure) < 0.9


@pytest.mark.parametrize("seed", [21, 22])
def test_sure_normal_counts_equal_the_oracle(checker, seed):
    rng = np.random.default_rng(seed)
    n = 60000
    N, pe, _ = window_triples(seed, n)
    po = pe * rng.uniform(0.2, 1.2, n)
    w = rng.integers(0, 2**32, (4, n), dtype=np.uint64)
    w[0, :50] = rng.integers(0, 2**12, 50)  # u next to 0 (u1 next to 1)
    w[0, 50:100] = 2**32 - 1 - rng.integers(0, 2**12, 50)
    w[2, 100:140] = np.repeat(np.arange(8) * 2**29 % 2**32, 5)  # octant edges
    got = run(checker, "normal", (f"{a} {b} {c} {d} {m} {float(x).hex()} {float(y).hex()}\n"
                                  for a, b, c, d, m, x, y in zip(*w.tolist(), N.tolist(), pe, po)))
    ze, zo = ON.box_muller_words(*w)
    for sure, k, p, z in [(got[0::4] != 0, got[1::4], pe, ze), (got[2::4] != 0, got[3::4], po, zo)]:
        ref = ON.normal_count(N, p, z)
        bad = np.nonzero(sure & (k != ref))[0]
        assert bad.size == 0, [(int(N[i]), float(p[i]), float(z[i]), int(k[i]), int(ref[i])) for i in bad[:5]]
        assert np.mean(~sure) < 0.01
