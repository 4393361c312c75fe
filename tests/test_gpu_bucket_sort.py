"""The bucket sort of the values: one bucket, the edges of one and of several,
ties of every kind, and a bucket that outgrows its room.  The reorder map against
the oracle's, and the sorted values, which the fit reads, by the coefficients of a
constant over each of many short runs."""
import math
import re

import numpy as np
import pytest

import oracle
from paper_2102_03112_amd import binding as B
from _gpu_util import check_roundtrip, dev_tensor, host, log, run_roundtrip, sync, u64_scalar, workspace

pytestmark = pytest.mark.gpu

CAP, AVG, OVER = 4096, 1024, 16  # a bucket's room and mean size, samples per bucket


def _m32(x):
    return x & 0xFFFFFFFF


def sample_places(n):
    """Where the sort takes its sample of n > CAP values from."""
    S = -(-n // AVG) * OVER
    i = np.arange(S, dtype=np.uint64)
    a, e = i * np.uint64(n) // np.uint64(S), (i + np.uint64(1)) * np.uint64(n) // np.uint64(S)
    h = np.array([oracle.murmur3_32(int(q).to_bytes(4, "little"), 0x5EED) for q in i], dtype=np.uint64)
    return (a + (h * (e - a) >> np.uint64(32))).astype(np.int64)


def values(kind, n, rng):
    if kind == "normal":
        return rng.standard_normal(n)
    if kind == "equal":
        return np.full(n, 0.25)
    if kind == "zeros":  # signed zeros among values, as false positives with sparse values
        return np.where(rng.random(n) < 0.3, np.where(rng.random(n) < 0.5, 0.0, -0.0), rng.standard_normal(n))
    if kind == "coarse":
        return rng.integers(-9, 10, n) * 0.25
    if kind == "sorted":
        return np.sort(rng.standard_normal(n))
    if kind == "outgrown":  # every sampled value is the same, so one bucket gets all the others
        v = 2.0 + rng.random(n)
        v[sample_places(n)] = 1.0
        return v
    if kind == "ulps":  # 30 neighbouring floats, each many times, and two far off: one bin cut into 30 too full ones
        v = (np.float32(1.5).view(np.int32) + rng.integers(0, 30, n, dtype=np.int32)).view(np.float32)
        v[[0, n // 2]] = 1e30, -1e30
        return v
    if kind == "wide":  # both ends of the range of floats
        return rng.standard_normal(n) * 10.0 ** rng.integers(-40, 38, n)
    raise ValueError(kind)


SIZES = [1, 2, 63, 513, CAP - 1, CAP, CAP + 1, 8191, 20_000, 100_001, 512 * AVG, 512 * AVG + 1]
CASES = [(n, "normal") for n in SIZES] + [(n, "ulps") for n in (CAP, 30_000, 512 * AVG)]
CASES += [(n, k) for n in (CAP, 30_000) for k in ("equal", "zeros", "coarse", "sorted", "wide")]


def encode(v, degree, n_seg, ws):
    """The device's reorder map and coefficients."""
    import torch

    n = v.size
    nd = torch.tensor([n], dtype=torch.int64, device="cuda")
    coef = torch.zeros(n_seg * (degree + 1), dtype=torch.float32, device="cuda")
    sigma = torch.zeros((n * B.sigma_bits(n) + 31) // 32, dtype=torch.int32, device="cuda")
    B.curvefit_encode(dev_tensor(v), nd, n, degree, n_seg, coef, sigma, ws)
    sync()
    return host(sigma).view(np.uint32), host(coef)


def check_sorted_values(v, coef):
    """A run's constant is the mean of its sorted values, summed in double and
    rounded once: an ulp from the mean of their exact sum, and the sums' own
    rounding, at most (values - 1) 2^-53 of the sum of magnitudes each way."""
    order = np.sort(v.astype(np.float64))[::-1]
    n, runs = order.size, min(coef.size, order.size)
    at = np.arange(runs + 1, dtype=np.int64) * n // runs
    for s in range(runs):
        x = order[at[s]:at[s + 1]]
        mean = math.fsum(x) / x.size
        tol = float(np.spacing(np.float32(abs(mean)))) + 4 * x.size * 2.0 ** -53 * float(np.abs(x).sum()) / x.size
        assert abs(float(coef[s]) - mean) <= tol, (s, float(coef[s]), mean, tol)


@pytest.mark.parametrize("n,kind", CASES + [(30_000, "outgrown")])
def test_reorder_map(n, kind):
    log(f"sort n={n} kind={kind}")
    v = values(kind, n, np.random.default_rng(n)).astype(np.float32)
    ws = workspace(8 * n)
    sigma, coef = encode(v, 0, 4096, ws)
    np.testing.assert_array_equal(sigma, oracle.curvefit_encode(v, 3, 4).sigma)
    check_sorted_values(v, coef)


def test_workspace_without_room_for_buckets():
    """The exact workspace that the call asks for: the radix sort instead."""
    n = 50_000
    v = np.random.default_rng(1).standard_normal(n).astype(np.float32)
    with pytest.raises(B.DeepReduceError) as e:
        encode(v, 0, 4096, B.workspace(n)[:256])
    need = int(re.search(r"need (\d+)", str(e.value)).group(1))
    names = []
    for size in (need, B.workspace_bytes(n)):
        B.trace_begin()
        sigma, coef = encode(v, 0, 4096, B.workspace(n)[:size])
        names.append(set(B.trace_end()))
        np.testing.assert_array_equal(sigma, oracle.curvefit_encode(v, 3, 4).sigma)
        check_sorted_values(v, coef)
    assert "k_sort_pass" in names[0] and "k_bsort_bucket" in names[1]


@pytest.mark.parametrize("source", [B.VALUES_DENSE, B.VALUES_SPARSE], ids=["dense", "sparse"])
@pytest.mark.parametrize("sizes,ratio", [([700_000], (1, 50)), ([100, 400_000, 0, 41_000, 1, 900_000], (1, 20)),
                                         ([200_000], (1, 2))])
def test_round_trip(sizes, ratio, source):
    off = np.concatenate([[0], np.cumsum(sizes)])
    g = (np.random.default_rng(7).standard_normal(int(off[-1])) * 1e-3).astype(np.float32)
    cfg = B.Config(off, ratio, 1e-2, 3, 4, value_source=source)
    refs = oracle.roundtrip(g, off, ratio, 1e-2, 3, 4, value_source=source)
    check_roundtrip(g, cfg, run_roundtrip(g, cfg), refs)
