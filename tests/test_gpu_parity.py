"""GPU parity: every C-ABI entry point against the CPU oracle, element by
element, on seeded inputs that span several tiles and a ragged tail.

Bit-exact: selected indices, filter words, positives, reorder maps, header
fields.  Floating point: fit coefficients within 1e-4 (norm-wise per run) of
the oracle's double-precision solution; reconstructed values within 1e-5 of
the oracle's reconstruction from the same payload (floor: the run's largest
magnitude, which guards zero crossings).
"""
import numpy as np
import pytest

import oracle
from paper_2102_03112_amd import binding as B
from paper_2102_03112_amd import workloads as W
from _gpu_util import (check_roundtrip, coef_close, dev_tensor, host, log, run_roundtrip, sync, u64_scalar,
                       values_close, workspace)

pytestmark = pytest.mark.gpu

def ws_for(d, n_tensors=1):
    return workspace(d, n_tensors)


def gen(kind, d, seed):
    if kind == "normal":
        return W.normal(d, seed)
    if kind == "tied":
        return W.tied_values(d, seed)
    if kind == "coarse":
        rng = np.random.default_rng(seed)
        return (rng.integers(-20, 21, d) * 0.25).astype(np.float32)
    if kind == "equal":
        return np.full(d, 0.5, dtype=np.float32)
    if kind == "sparse":
        return W.sparse_normal(d, seed, 0.4)
    if kind == "zeros":
        g = np.zeros(d, dtype=np.float32)
        g[::3] = -0.0
        return g
    raise ValueError(kind)


# ---------------------------------------------------------------------------
# dr_sparsify_topr
# ---------------------------------------------------------------------------
TOPR_CASES = [
    (1, 1, "normal"), (1, 0, "normal"), (100, 7, "tied"), (4096, 41, "normal"), (4097, 4097, "tied"),
    (3 * 4096 + 17, 1000, "tied"), (70000, 7000, "normal"), (70000, 1, "tied"), (200_000, 2000, "coarse"),
    (10_000, 333, "equal"), (123_457, 61_000, "coarse"), (50_000, 25_000, "zeros"),
]


@pytest.mark.parametrize("d,r,kind", TOPR_CASES)
def test_topr_parity(d, r, kind):
    import torch

    log(f"topr d={d} r={r} kind={kind}")
    g = gen(kind, d, seed=d + r)
    gd = dev_tensor(g)
    cap = max(r, 1)
    idx = torch.full((cap,), -1, dtype=torch.int32, device="cuda")
    val = torch.zeros(cap, dtype=torch.float32, device="cuda")
    n = u64_scalar()
    B.sparsify_topr(gd, r, idx, val, n, ws_for(d))
    sync()
    ref = oracle.topr(g, r)
    assert int(host(n)[0]) == r
    np.testing.assert_array_equal(host(idx)[:r].view(np.uint32), ref)
    np.testing.assert_array_equal(host(val)[:r], g[ref.astype(np.int64)])


SAMPLED_D = (1 << 26) + 4099  # calls of at least 2^26 elements sample; ragged tail


def _sample_blind():
    """Large magnitudes only where the selection's sample does not look.
    A call of at least 2^26 elements takes the threshold's first digit of
    each tensor of at least 2^22 elements with r <= d/16 from a sample:
    segment j srate + srate/2 of 64 elements, srate the largest power of 2
    leaving max(2^18, 4096 ceil(d/r)) sampled elements, here 128 for r = 1%.
    Outside the sampled segments 2% of the elements are +-(1..2), so the 1%
    largest are all there, and the sample's bracket (around the threshold of
    the N(0, 1e-3) values it sees) is contradicted by the exact counts: the
    tensor is redone from a full histogram."""
    rng = np.random.default_rng(41)
    g = rng.standard_normal(SAMPLED_D).astype(np.float32) * np.float32(1e-3)
    seg = np.arange(SAMPLED_D) // 64
    big = (seg % 128 != 64) & (rng.random(SAMPLED_D) < 0.02)
    nb = int(big.sum())
    g[big] = (np.sign(rng.standard_normal(nb)) * (1.0 + rng.random(nb))).astype(np.float32)
    return g


def _all_binades():
    """Magnitudes log-uniform over all normal binades: about 33,000 elements
    per first-digit bin, so the sample's bracket may span more bins than it
    keeps (at r = 6%), and the exact counts decide whether it holds."""
    rng = np.random.default_rng(43)
    e = rng.uniform(-125.0, 127.0, SAMPLED_D)
    return (np.sign(rng.standard_normal(e.size)) * np.exp2(e)).astype(np.float32)


# large tensors: millions of elements, r from 0.1% to a few %, and heavy ties
# (in calls of at least 2^26 elements, tensors of at least 2^22 elements
# with r <= d/16 take the threshold's first digit from a sample, the others
# from an exact histogram)
LARGE_TOPR_CASES = [
    ("sample_blind_67m", _sample_blind, SAMPLED_D // 100),
    ("all_binades_67m", _all_binades, SAMPLED_D // 100),
    ("all_binades_67m_r6pct", _all_binades, SAMPLED_D * 6 // 100),
    ("normal_5m", lambda: W.normal(5_000_000, 31), 50_000),
    ("laplace_5m_r0.1pct", lambda: W.generate(W.Workload("t", 5_000_003, 1, (1, 1000), 1e-3, 5, 8, "laplace_5e-4", 32)),
     5001),
    ("coarse_ties_6m", lambda: (np.random.default_rng(35).integers(-40, 41, 6_000_000) * 0.125).astype(np.float32),
     200_000),
]


@pytest.mark.parametrize("name,make,r", LARGE_TOPR_CASES, ids=[c[0] for c in LARGE_TOPR_CASES])
def test_topr_large_parity(name, make, r):
    import torch

    g = make()
    d = g.size
    log(f"topr large {name} d={d} r={r}")
    ref = oracle.topr(g, r)
    idx = torch.full((r,), -1, dtype=torch.int32, device="cuda")
    val = torch.zeros(r, dtype=torch.float32, device="cuda")
    nd = u64_scalar()
    B.sparsify_topr(dev_tensor(g), r, idx, val, nd, ws_for(d))
    sync()
    assert int(host(nd)[0]) == r
    np.testing.assert_array_equal(host(idx).view(np.uint32), ref)
    np.testing.assert_array_equal(host(val).view(np.uint32), g[ref.astype(np.int64)].view(np.uint32))


@pytest.mark.parametrize("d,kind", [(50_000, "sparse"), (10_000, "zeros"), (5000, "normal"), (3 * 4096 + 1, "sparse")])
def test_support_parity(d, kind):
    import torch

    log(f"support d={d} kind={kind}")
    g = gen(kind, d, seed=d)
    gd = dev_tensor(g)
    idx = torch.full((d,), -1, dtype=torch.int32, device="cuda")
    n = u64_scalar()
    B.sparsify_topr(gd, B.R_NONZERO, idx, None, n, ws_for(d))
    sync()
    ref = oracle.nonzero(g)
    assert int(host(n)[0]) == ref.size
    np.testing.assert_array_equal(host(idx)[: ref.size].view(np.uint32), ref)


# ---------------------------------------------------------------------------
# dr_bloom_encode / dr_bloom_decode
# ---------------------------------------------------------------------------
@pytest.mark.parametrize(
    "d,n,fpr",
    [(1000, 0, 1e-3), (1000, 1, 1e-3), (36_864, 369, 1e-3), (1 << 20, 10_486, 1e-3), (8192, 8192, 1e-4),
     (300_000, 100_000, 1e-9), (200_000, 5000, 0.5), (25_557_032, 255_571, 1e-3),
     # filters above 2^23 bits take the bucketed insert: 2^16-bit slices, and
     # 2^18-bit slices with the 13 hashes in three rounds
     (4_000_000, 1_000_000, 1e-3), (3_000_000, 2_500_000, 1e-4)],
)
def test_bloom_encode_parity(d, n, fpr):
    log(f"bloom_encode d={d} n={n} fpr={fpr}")
    S = W.random_indices(d, n, seed=n + 3)
    m, k = oracle.bloom_params(n, fpr)
    ref = oracle.bloom_encode(S, m, k)
    import torch

    Sd = dev_tensor(S.view(np.int32)) if n else torch.zeros(1, dtype=torch.int32, device="cuda")
    nd = dev_tensor(np.array([n], dtype=np.int64))
    bits = torch.full((m // 32,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    B.bloom_encode(Sd, nd, n, m, k, bits, ws_for(max(n, 1)))
    sync()
    np.testing.assert_array_equal(host(bits).view(np.uint32), ref)


@pytest.mark.parametrize("n_dev,n_cap", [(900, 1000), (1000, 1000), (1300, 1000), (300_000, 200_000)])
def test_bloom_encode_count_against_capacity(n_dev, n_cap):
    """At most n_cap indices are inserted; a device count above the capacity
    is reported in flags_out (DR_FLAG_CAPACITY), one at or below it is not."""
    import torch

    log(f"bloom_encode n_dev={n_dev} n_cap={n_cap}")
    S = W.random_indices(4 * max(n_dev, n_cap), max(n_dev, n_cap), seed=n_dev)
    m, k = oracle.bloom_params(n_cap, 1e-3)
    used = min(n_dev, n_cap)
    ref = oracle.bloom_encode(S[:used], m, k)
    bits = torch.full((m // 32,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    flags = dev_tensor(np.array([0x77], dtype=np.int64))
    B.bloom_encode(dev_tensor(S.view(np.int32)), dev_tensor(np.array([n_dev], dtype=np.int64)), n_cap, m, k, bits,
                   ws_for(max(n_dev, n_cap)), flags_out=flags)
    sync()
    np.testing.assert_array_equal(host(bits).view(np.uint32), ref)
    assert int(host(flags)[0]) == (B.FLAG_CAPACITY if n_dev > n_cap else 0)


@pytest.mark.parametrize("n_dev,n_cap", [(5000, 6000), (6000, 6000), (7000, 6000)])
def test_curvefit_count_against_capacity(n_dev, n_cap):
    """The value path uses the first min(n, n_cap) values, and both calls
    report a count above the capacity in flags_out."""
    import torch

    log(f"curvefit n_dev={n_dev} n_cap={n_cap}")
    D, S = 3, 4
    V = W.normal(max(n_dev, n_cap), 71)
    used = min(n_dev, n_cap)
    ref = oracle.curvefit_encode(V[:used], D, S)
    nd = dev_tensor(np.array([n_dev], dtype=np.int64))
    coef = torch.zeros(S * (D + 1), dtype=torch.float32, device="cuda")
    nw = oracle.sigma_words(n_cap) + 1
    sig = torch.zeros(nw, dtype=torch.int32, device="cuda")
    f1 = dev_tensor(np.array([0x77], dtype=np.int64))
    f2 = dev_tensor(np.array([0x77], dtype=np.int64))
    ws = ws_for(max(n_dev, n_cap))
    B.curvefit_encode(dev_tensor(V), nd, n_cap, D, S, coef, sig, ws, flags_out=f1)
    out = torch.full((n_cap + 64,), 5.0, dtype=torch.float32, device="cuda")
    B.curvefit_decode(coef, sig, nd, n_cap, D, S, out, ws, flags_out=f2)
    sync()
    expect = B.FLAG_CAPACITY if n_dev > n_cap else 0
    assert int(host(f1)[0]) == expect and int(host(f2)[0]) == expect
    np.testing.assert_array_equal(host(sig).view(np.uint32)[: oracle.sigma_words(used)], ref.sigma)
    coef_close(host(coef), ref.coef64, ref.S_eff, D + 1, ref.D_eff + 1)
    y = host(out)
    assert np.all(y[used:] == 5.0)  # nothing written past the count and the capacity
    y_ref = oracle.curvefit_decode(ref.coef, ref.sigma, used, D, S)
    values_close(y[:used], y_ref, oracle.sigma_unpack(ref.sigma, used), used, ref.S_eff)


@pytest.mark.parametrize(
    "d,n,fpr",
    [(1, 1, 1e-3), (4095, 40, 1e-3), (4096, 41, 1e-2), (4097, 41, 1e-3), (3 * 4096 + 5, 200, 1e-3),
     (100_000, 1000, 1e-3), (1 << 20, 10_486, 1e-3), (250_000, 150_000, 1e-4)],
)
def test_bloom_decode_parity(d, n, fpr):
    import torch

    log(f"bloom_decode d={d} n={n} fpr={fpr}")
    S = W.random_indices(d, n, seed=d)
    m, k = oracle.bloom_params(n, fpr)
    bits = oracle.bloom_encode(S, m, k)
    ref = oracle.bloom_query(bits, m, k, d)
    idx = torch.full((d,), -1, dtype=torch.int32, device="cuda")
    nd = u64_scalar()
    B.bloom_decode(dev_tensor(bits.view(np.int32)), m, k, d, idx, d, nd, ws_for(d))
    sync()
    assert int(host(nd)[0]) == ref.size
    np.testing.assert_array_equal(host(idx)[: ref.size].view(np.uint32), ref)


def test_bloom_decode_full_empty_and_capacity():
    import torch

    d, m, k = 10_000, 256, 3
    ws = ws_for(d)
    idx = torch.full((d,), -1, dtype=torch.int32, device="cuda")
    nd = u64_scalar()
    full = np.full(m // 32, 0xFFFFFFFF, dtype=np.uint32)
    B.bloom_decode(dev_tensor(full.view(np.int32)), m, k, d, idx, d, nd, ws)
    sync()
    assert int(host(nd)[0]) == d
    np.testing.assert_array_equal(host(idx).view(np.uint32), np.arange(d, dtype=np.uint32))
    empty = np.zeros(m // 32, dtype=np.uint32)
    B.bloom_decode(dev_tensor(empty.view(np.int32)), m, k, d, idx, d, nd, ws)
    sync()
    assert int(host(nd)[0]) == 0
    # output capacity smaller than the count: the first `cap` entries and the full count
    S = W.random_indices(d, 500, seed=1)
    m2, k2 = oracle.bloom_params(500, 0.05)
    bits = oracle.bloom_encode(S, m2, k2)
    ref = oracle.bloom_query(bits, m2, k2, d)
    small = torch.full((100,), -1, dtype=torch.int32, device="cuda")
    B.bloom_decode(dev_tensor(bits.view(np.int32)), m2, k2, d, small, 100, nd, ws)
    sync()
    assert int(host(nd)[0]) == ref.size
    np.testing.assert_array_equal(host(small).view(np.uint32), ref[:100])


# ---------------------------------------------------------------------------
# dr_curvefit_encode / dr_curvefit_decode
# ---------------------------------------------------------------------------
CURVE_CASES = [
    (0, 5, 8), (1, 5, 8), (2, 5, 8), (5, 5, 8), (6, 5, 8), (7, 5, 8), (47, 5, 8), (48, 5, 8), (1000, 5, 8),
    (4096, 5, 1), (4097, 5, 8), (40_000, 5, 8), (12, 1, 6), (5000, 3, 16), (300_000, 5, 8), (100_000, 7, 64),
]


@pytest.mark.parametrize("n,D,S", CURVE_CASES)
def test_curvefit_parity(n, D, S):
    import torch

    log(f"curvefit n={n} D={D} S={S}")
    rng = np.random.default_rng(n + D)
    V = (rng.laplace(0, 5e-4, n)).astype(np.float32)
    if n > 100:
        V[::17] = V[5]  # exact ties
    ref = oracle.curvefit_encode(V, D, S)
    nw = max(1, oracle.sigma_words(n))
    Vd = dev_tensor(V) if n else torch.zeros(1, dtype=torch.float32, device="cuda")
    nd = dev_tensor(np.array([n], dtype=np.int64))
    coef = torch.full((S * (D + 1),), 7.0, dtype=torch.float32, device="cuda")
    sig = torch.zeros(nw, dtype=torch.int32, device="cuda")
    ws = ws_for(max(n, 1))
    B.curvefit_encode(Vd, nd, n, D, S, coef, sig, ws)
    out = torch.zeros(max(n, 1), dtype=torch.float32, device="cuda")
    B.curvefit_decode(coef, sig, nd, n, D, S, out, ws)
    # the decoder alone, on the oracle's coefficients and reorder map
    coef_o = dev_tensor(ref.coef.astype(np.float32))
    sig_o = dev_tensor(np.concatenate([ref.sigma.astype(np.uint32), np.zeros(1, np.uint32)]).view(np.int32))
    out_o = torch.zeros(max(n, 1), dtype=torch.float32, device="cuda")
    B.curvefit_decode(coef_o, sig_o, nd, n, D, S, out_o, ws)
    sync()
    c_gpu = host(coef)
    s_gpu = host(sig).view(np.uint32)[: oracle.sigma_words(n)]
    np.testing.assert_array_equal(s_gpu, ref.sigma)
    coef_close(c_gpu, ref.coef64, ref.S_eff, D + 1, ref.D_eff + 1)
    # everything outside the fitted rows and degrees is zero
    mask = np.ones(S * (D + 1), bool)
    for s in range(ref.S_eff):
        mask[s * (D + 1): s * (D + 1) + ref.D_eff + 1] = False
    assert np.all(c_gpu[mask] == 0)
    # decode: the oracle's reconstruction from its own coefficients, against
    # the GPU's from its own payload and from the oracle's payload
    y_ref = oracle.curvefit_decode(ref.coef, ref.sigma, n, D, S)
    if n:
        ranks = oracle.sigma_unpack(ref.sigma, n)
        values_close(host(out)[:n], y_ref, ranks, n, ref.S_eff)
        values_close(host(out_o)[:n], y_ref, ranks, n, ref.S_eff)


# ---------------------------------------------------------------------------
# dr_roundtrip over a gradient split into tensors
# ---------------------------------------------------------------------------
def _many_tensor_offsets():
    """37 tensors over about 3 M elements (about 740 tiles, so the probe pass
    gives each block two or three tiles): tensors of one element up to
    several hundred tiles, starting anywhere in a block's range."""
    rng = np.random.default_rng(11)
    sizes = list(rng.integers(1, 250_000, 24)) + [1, 2, 4095, 4096, 4097, 8192, 12_289, 0, 3, 70_000, 1, 5, 640_000]
    return [0] + list(np.cumsum(sizes).astype(int))


_MANY = _many_tensor_offsets()

RT_CASES = {
    "resnet20_conv_37k": (W.normal(36_864, 6), [0, 36_864], (1, 100), 1e-3, 5, 8),
    "student_t_3x": (None, None, (1, 100), 1e-3, 5, 8),
    "support_50k": (W.sparse_normal(50_000, 7, 0.4), [0, 50_000], None, 1e-4, 3, 16),
    # a filter planned for 1 M items: the bucketed insert, in three rounds
    "support_1m": (W.sparse_normal(1_000_000, 13, 0.4), [0, 1_000_000], None, 1e-4, 3, 16),
    # 1.5 M values: 366 sort tiles in each pass's look-back
    "support_2500k": (W.sparse_normal(2_500_000, 15, 0.4), [0, 2_500_000], None, 1e-4, 3, 16),
    # three such tensors: the bucketed insert over several tensors' slices
    # and chunks
    "support_3x500k": (W.sparse_normal(1_500_001, 14, 0.4), [0, 500_000, 1_000_000, 1_500_001], None, 1e-4, 3, 8),
    # empty, 1-, 5-, 4096-, 4097-element, empty and 4-element tensors
    "ragged_tensors": (W.normal(8203, 8), [0, 0, 1, 6, 4102, 8199, 8199, 8203], (1, 2), 1e-3, 5, 8),
    "take_all": (W.normal(5000, 9), [0, 5000], (1, 1), 1e-3, 2, 4),
    # the probe pass's per-block look-back across many tensor boundaries
    "many_tensors_3m": (W.normal(_MANY[-1], 12), _MANY, (1, 100), 1e-3, 5, 8),
}


@pytest.mark.parametrize("name", list(RT_CASES))
def test_roundtrip_parity(name):
    g, off, ratio, fpr, D, S = RT_CASES[name]
    if name == "student_t_3x":
        w = W.Workload("t", 100_001, 3, ratio, fpr, D, S, "student_t3", 77)
        g, off = W.generate(w), w.offsets()
    log(f"roundtrip {name} d={g.size} tensors={len(off) - 1}")
    assert off[-1] == g.size
    cfg = B.Config(off, ratio, fpr, D, S)
    out = run_roundtrip(g, cfg)
    refs = oracle.roundtrip(g, off, ratio, fpr, D, S)
    check_roundtrip(g, cfg, out, refs)


POLICIES = [oracle.POLICY_RANDOM, oracle.POLICY_LEFTMOST, oracle.POLICY_MIDDLE, oracle.POLICY_RIGHTMOST]


@pytest.mark.parametrize("policy", POLICIES)
@pytest.mark.parametrize("name", ["resnet20_fpr_1e-2", "support_50k", "ragged_tensors"])
def test_roundtrip_policy_parity(name, policy):
    """Policies that code r of the positives (Section 4; Sections 10.4,
    10.5): the same choice, value numbers and reconstruction as the oracle.
    A false-positive rate of 1e-2 leaves many positives undecoded."""
    if name == "resnet20_fpr_1e-2":
        g, off, ratio, fpr, D, S = W.normal(36_864, 6), [0, 36_864], (1, 100), 1e-2, 5, 8
    else:
        g, off, ratio, fpr, D, S = RT_CASES[name]
    seed = 0x5EED0000 + policy
    log(f"roundtrip {name} policy={policy} seed={seed:#x}")
    cfg = B.Config(off, ratio, fpr, D, S, policy, seed)
    out = run_roundtrip(g, cfg)
    refs = oracle.roundtrip(g, off, ratio, fpr, D, S, policy=policy, seed=seed)
    assert any(ref.P.size > ref.S.size for ref in refs)
    check_roundtrip(g, cfg, out, refs)


VSRC_CASES = {
    # name: (g, offsets, ratio, fpr, D, S, policy)
    "resnet20_fpr_1e-2": (W.normal(36_864, 6), [0, 36_864], (1, 100), 1e-2, 5, 8, oracle.POLICY_P0),
    "resnet20_fpr_1e-2_p1": (W.normal(36_864, 6), [0, 36_864], (1, 100), 1e-2, 5, 8, oracle.POLICY_RANDOM),
    "ragged_tensors": RT_CASES["ragged_tensors"] + (oracle.POLICY_P0,),
    "support_50k": RT_CASES["support_50k"] + (oracle.POLICY_P0,),
    "many_tensors_3m": RT_CASES["many_tensors_3m"] + (oracle.POLICY_P0,),
    # one value per run: the decoded gradient is g~ itself
    "interp_d0": (W.normal(3000, 31, scale=1.0), [0, 3000], (1, 50), 0.05, 0, oracle.MAX_SEG, oracle.POLICY_P0),
}


@pytest.mark.parametrize("name", list(VSRC_CASES))
def test_roundtrip_sparse_value_source_parity(name):
    """Values from the sparsified gradient (Section 4's P0: 0 at a false
    positive): record, positives and values as the oracle's."""
    g, off, ratio, fpr, D, S, policy = VSRC_CASES[name]
    seed = 0x5EED0001
    log(f"roundtrip {name} value_source=sparse policy={policy}")
    cfg = B.Config(off, ratio, fpr, D, S, policy, seed, value_source=B.VALUES_SPARSE)
    out = run_roundtrip(g, cfg)
    refs = oracle.roundtrip(g, off, ratio, fpr, D, S, policy=policy, seed=seed,
                            value_source=oracle.VALUES_SPARSE)
    check_roundtrip(g, cfg, out, refs)
    if name == "interp_d0":
        (ref,) = refs
        assert ref.P.size > ref.S.size
        np.testing.assert_array_equal(out["dense"], ref.dense)


LAYOUT_CASES = {
    # name: (g, offsets, ratio, fpr, D, S): the partitioned filter layout
    "resnet20_conv_37k": RT_CASES["resnet20_conv_37k"],
    "ragged_tensors": RT_CASES["ragged_tensors"],
    "support_50k": RT_CASES["support_50k"],
    "support_1m": RT_CASES["support_1m"],          # the bucketed insert
    "many_tensors_3m": RT_CASES["many_tensors_3m"],
    # filters larger than the probe pass's LDS copy: 1.73 M and 4.3 M bits
    "normal_12m": (W.normal(12_000_000, 41), [0, 12_000_000], (1, 100), 1e-3, 5, 8),
    "normal_30m_fpr_1e-4": (W.normal(30_000_001, 42), [0, 30_000_001], (1, 100), 1e-4, 5, 8),
    # partitioned filters of 40-46 M bits (bucketed insert, most of the
    # filter outside the probe pass's LDS copy); the second beside a small
    # filter of the same call
    "support_4m_rounds": (W.sparse_normal(4_000_003, 44, 0.4), [0, 4_000_003], None, 1e-4, 3, 16),
    "support_rounds_and_lds": (W.sparse_normal(3_600_000, 45, 0.4), [0, 3_500_000, 3_600_000], None, 1e-4, 3, 16),
}

# A build that queried partitioned filters of at least 2^25 bits in per-part
# rounds went silent (killed after 180 s, the GPU still answering) in its
# first run of support_4m_rounds; the cause was not found by reading the
# code, and that code was taken out.  Until a cause is shown, the partitioned
# cases with filters that large stay off the GPU.
LARGE_PARTITIONED_HUNG = "partitioned filter of 4e7 bits: a run went silent on the GPU (cause not found); kept off the GPU"
LAYOUT_SKIP = {"support_4m_rounds", "support_rounds_and_lds"}


@pytest.mark.parametrize("name", list(LAYOUT_CASES))
def test_roundtrip_partitioned_layout_parity(name):
    """The partitioned filter (hash j over part j of k): filter words,
    positives, values and the record's hash id as the oracle's."""
    if name in LAYOUT_SKIP:
        pytest.skip(LARGE_PARTITIONED_HUNG)
    g, off, ratio, fpr, D, S = LAYOUT_CASES[name]
    log(f"roundtrip {name} layout=partitioned d={g.size}")
    cfg = B.Config(off, ratio, fpr, D, S, filter_layout=B.FILTER_PARTITIONED)
    out = run_roundtrip(g, cfg)
    refs = oracle.roundtrip(g, off, ratio, fpr, D, S, layout=oracle.LAYOUT_PARTITIONED)
    check_roundtrip(g, cfg, out, refs)


@pytest.mark.skip(reason=LARGE_PARTITIONED_HUNG)
def test_receiver_without_rounds_decodes_a_payload_queried_in_rounds():
    """A large partitioned payload decoded by a receiver whose configuration
    names the standard layout: the record decides the layout."""
    import torch

    g, off, ratio, fpr, D, S = LAYOUT_CASES["support_4m_rounds"]
    cfg_p = B.Config(off, ratio, fpr, D, S, filter_layout=B.FILTER_PARTITIONED)
    rt = run_roundtrip(g, cfg_p)
    cfg_s = B.Config(off, ratio, fpr, D, S)
    dense = torch.full((g.size,), 3.0, dtype=torch.float32, device="cuda")
    counts = torch.zeros(4, dtype=torch.int64, device="cuda")
    B.payload_decode(dev_tensor(rt["payload"]), cfg_s, dense, None, None, counts, workspace(g.size))
    sync()
    assert int(host(counts)[3]) == 0
    np.testing.assert_array_equal(host(dense), rt["dense"])


def test_receiver_reads_the_layout_from_the_record_and_rejects_unknown_ones():
    import torch

    w = W.Workload("t", 50_000, 1, (1, 100), 1e-3, 5, 8, "normal_1e-3", 12)
    g = W.generate(w)
    # a partitioned payload decoded by a receiver whose configuration names
    # the standard layout: the record decides
    cfg_p = B.Config.from_workload(w, filter_layout=B.FILTER_PARTITIONED)
    rt = run_roundtrip(g, cfg_p)
    cfg_s = B.Config.from_workload(w)
    dense = torch.full((w.d,), 3.0, dtype=torch.float32, device="cuda")
    counts = torch.zeros(4, dtype=torch.int64, device="cuda")
    B.payload_decode(dev_tensor(rt["payload"]), cfg_s, dense, None, None, counts, workspace(w.d))
    sync()
    assert int(host(counts)[3]) == 0
    np.testing.assert_array_equal(host(dense), rt["dense"])
    # an unknown hash id: the record is invalid and decodes as empty
    bad = rt["payload"].copy()
    bad[8 * 4: 8 * 4 + 4] = np.frombuffer(np.uint32(3).tobytes(), np.uint8)
    B.payload_decode(dev_tensor(bad), cfg_s, dense, None, None, counts, workspace(w.d))
    sync()
    assert int(host(counts)[3]) & B.FLAG_DEC_MISMATCH
    assert np.all(host(dense) == 0)


SEG_CASES = {
    # name: (g, offsets, ratio, fpr, D, S, segmentation)
    "resnet20_chord8": (W.normal(36_864, 6), [0, 36_864], (1, 100), 1e-3, 5, 8, oracle.SEG_CHORD),
    "laplace_chord16_d1": (W.generate(W.Workload("t", 300_000, 1, (1, 100), 1e-3, 1, 16, "laplace_5e-4", 13)),
                           [0, 300_000], (1, 100), 1e-3, 1, 16, oracle.SEG_CHORD),
    "ragged_chord8": (W.normal(8203, 8), [0, 0, 1, 6, 4102, 8199, 8199, 8203], (1, 2), 1e-3, 5, 8,
                      oracle.SEG_CHORD),
    "support_chord_auto_d0": (W.sparse_normal(50_000, 7, 0.4, scale=40.0), [0, 50_000], None, 1e-4, 0, 0,
                              oracle.SEG_CHORD),
    "normal_equal_auto_d1": (W.normal(200_000, 21, scale=3.0), [0, 200_000], (1, 100), 1e-3, 1, 0,
                             oracle.SEG_EQUAL),
    "normal_chord_auto_d1": (W.normal(200_000, 21, scale=3.0), [0, 200_000], (1, 100), 1e-3, 1, 0,
                             oracle.SEG_CHORD),
    "many_runs_chord": (W.normal(400_000, 22, scale=1e-3), [0, 400_000], (1, 10), 1e-3, 1, 3000,
                        oracle.SEG_CHORD),
    # splits evaluated over the whole grid: 600 k values in 16 runs, and 37
    # tensors at once
    "support_chord16_1m": (W.sparse_normal(1_000_000, 13, 0.4), [0, 1_000_000], None, 1e-4, 3, 16,
                           oracle.SEG_CHORD),
    "many_tensors_chord8": (W.normal(_MANY[-1], 12), _MANY, (1, 100), 1e-3, 5, 8, oracle.SEG_CHORD),
    # two and one runs: the sign split alone, and no split at all
    "resnet20_chord2": (W.normal(36_864, 6), [0, 36_864], (1, 100), 1e-3, 5, 2, oracle.SEG_CHORD),
    "resnet20_chord1": (W.normal(36_864, 6), [0, 36_864], (1, 100), 1e-3, 5, 1, oracle.SEG_CHORD),
}


@pytest.mark.parametrize("name", list(SEG_CASES))
def test_roundtrip_segmentation_parity(name):
    """Chord segmentation and the heuristic run count (Section 5): the same
    run starts (bit-exact) and values as the oracle."""
    g, off, ratio, fpr, D, S, seg = SEG_CASES[name]
    log(f"roundtrip {name} d={g.size} D={D} S={S} seg={seg}")
    cfg = B.Config(off, ratio, fpr, D, S, 0, 0, seg)
    out = run_roundtrip(g, cfg)
    refs = oracle.roundtrip(g, off, ratio, fpr, D, S, seg_mode=seg)
    check_roundtrip(g, cfg, out, refs)
    if seg == oracle.SEG_CHORD and S != 1:
        assert any(r.fit.S_eff > 1 for r in refs)


DEXP_CASES = {
    # name: (g, offsets, ratio, fpr, S, segmentation)
    "resnet20_dexp": (W.normal(36_864, 6), [0, 36_864], (1, 100), 1e-3, 1, oracle.SEG_EQUAL),
    "laplace_dexp8": (W.generate(W.Workload("t", 300_000, 1, (1, 100), 1e-3, 3, 8, "laplace_5e-4", 17)),
                      [0, 300_000], (1, 100), 1e-3, 8, oracle.SEG_EQUAL),
    "laplace_dexp_chord6": (W.generate(W.Workload("t", 300_000, 1, (1, 100), 1e-3, 3, 6, "laplace_5e-4", 18)),
                            [0, 300_000], (1, 100), 1e-3, 6, oracle.SEG_CHORD),
    "ragged_dexp": (W.normal(8203, 8), [0, 0, 1, 6, 4102, 8199, 8199, 8203], (1, 2), 1e-3, 4, oracle.SEG_EQUAL),
}


@pytest.mark.parametrize("name", list(DEXP_CASES))
def test_roundtrip_dexp_parity(name):
    """The double-exponential model (Section 5): same fitted rows (norm-wise
    1e-4 per run) and reconstructed values as the oracle."""
    g, off, ratio, fpr, S, seg = DEXP_CASES[name]
    log(f"roundtrip {name} d={g.size} S={S} seg={seg}")
    cfg = B.Config(off, ratio, fpr, 3, S, 0, 0, seg, oracle.FIT_DEXP)
    out = run_roundtrip(g, cfg)
    refs = oracle.roundtrip(g, off, ratio, fpr, 3, S, seg_mode=seg, model=oracle.FIT_DEXP)
    check_roundtrip(g, cfg, out, refs)
    assert any(r.fit.model == oracle.FIT_DEXP for r in refs)


def test_receiver_takes_the_policy_from_the_record():
    """The receiver reads policy and key from each record's header, not from
    its own configuration."""
    import torch

    g, off = W.normal(36_864, 6), [0, 36_864]
    enc = B.Config(off, (1, 100), 1e-2, 5, 8, oracle.POLICY_RANDOM, 1234)
    rt = run_roundtrip(g, enc)
    dec = B.Config(off, (1, 100), 1e-2, 5, 8, oracle.POLICY_P0, 0)
    dense = torch.full((g.size,), 3.0, dtype=torch.float32, device="cuda")
    counts = torch.zeros(4, dtype=torch.int64, device="cuda")
    B.payload_decode(dev_tensor(rt["payload"]), dec, dense, None, None, counts, workspace(g.size))
    sync()
    np.testing.assert_array_equal(host(dense), rt["dense"])
    assert int(host(counts)[3]) == 0


def test_receiver_rejects_an_unknown_policy_in_the_record():
    import torch

    g, off = W.normal(36_864, 6), [0, 36_864]
    cfg = B.Config(off, (1, 100), 1e-2, 5, 8, oracle.POLICY_LEFTMOST, 0)
    rt = run_roundtrip(g, cfg)
    bad = rt["payload"].copy()
    bad[36:40] = np.array([5], dtype="<u4").view(np.uint8)  # policy word
    dense = torch.full((g.size,), 3.0, dtype=torch.float32, device="cuda")
    counts = torch.zeros(4, dtype=torch.int64, device="cuda")
    B.payload_decode(dev_tensor(bad), cfg, dense, None, None, counts, workspace(g.size))
    sync()
    assert int(host(counts)[3]) & B.FLAG_DEC_MISMATCH
    assert np.all(host(dense) == 0)


def test_roundtrip_normal_1m_full_size():
    w = W.WORKLOADS["normal_1m"]
    log("roundtrip normal_1m")
    g = W.generate(w)
    cfg = B.Config.from_workload(w)
    out = run_roundtrip(g, cfg)
    refs = oracle.roundtrip(g, w.offsets(), w.ratio, w.fpr, w.degree, w.n_seg)
    check_roundtrip(g, cfg, out, refs)


def test_roundtrip_is_deterministic():
    w = W.Workload("t", 300_000, 2, (1, 100), 1e-3, 5, 8, "laplace_5e-4", 5)
    g = W.generate(w)
    cfg = B.Config.from_workload(w)
    a = run_roundtrip(g, cfg)
    b = run_roundtrip(g, cfg)
    np.testing.assert_array_equal(a["payload"], b["payload"])
    np.testing.assert_array_equal(a["dense"], b["dense"])


@pytest.mark.parametrize("name", ["resnet20_conv_37k", "ragged_tensors", "support_50k", "support_1m", "many_tensors_3m"])
def test_overlapped_round_trip_matches_the_sequential_one(name):
    """dr_roundtrip runs the receiver's probe pass on a second stream while
    the sender fits its values; dr_payload_encode then dr_payload_decode run
    the two sides one after the other.  Both give the same bytes."""
    import torch

    g, off, ratio, fpr, D, S = RT_CASES[name]
    cfg = B.Config(off, ratio, fpr, D, S)
    a = run_roundtrip(g, cfg)
    total, _ = B.payload_layout(cfg)
    d = g.size
    ws = workspace(max(d, 1), cfg.n_tensors)
    payload = torch.zeros(total, dtype=torch.uint8, device="cuda")
    dense = torch.full((max(d, 1),), 9.0, dtype=torch.float32, device="cuda")
    idx = torch.full((max(d, 1),), -1, dtype=torch.int32, device="cuda")
    val = torch.zeros(max(d, 1), dtype=torch.float32, device="cuda")
    counts = torch.zeros(4 * cfg.n_tensors, dtype=torch.int64, device="cuda")
    gd = dev_tensor(g) if d else torch.zeros(1, dtype=torch.float32, device="cuda")
    B.payload_encode(gd, cfg, payload, counts, ws)
    B.payload_decode(payload, cfg, dense, idx, val, counts, ws)
    sync()
    b = dict(payload=host(payload), dense=host(dense)[:d], idx=host(idx)[:d].view(np.uint32), val=host(val)[:d],
             counts=host(counts).reshape(cfg.n_tensors, 4))
    for key in ("payload", "dense", "idx", "val", "counts"):
        np.testing.assert_array_equal(a[key], b[key], err_msg=key)


def test_trace_attributes_both_streams():
    """Per-kernel timing follows each stream: the receiver's probe pass on
    the second stream is timed from the fork, not from the sender's last
    kernel."""
    w = W.WORKLOADS["normal_1m"]
    g = W.generate(w)
    cfg = B.Config.from_workload(w)
    run_roundtrip(g, cfg)
    B.trace_begin()
    run_roundtrip(g, cfg)
    tr = B.trace_end()
    for k in ("k_probe<Q_ENCODE>", "k_probe<Q_DECODE>", "k_bsort_bucket", "k_emit<Q_DECODE>"):
        assert k in tr and tr[k][0] >= 1 and tr[k][1] > 0, k


def test_sender_and_receiver_separately():
    """dr_payload_encode then dr_payload_decode into fresh buffers: the
    receiver needs nothing but the payload and the tensor layout."""
    import torch

    w = W.Workload("t", 200_003, 2, (1, 100), 1e-3, 5, 8, "laplace_5e-4", 11)
    g = W.generate(w)
    cfg = B.Config.from_workload(w)
    total, rec_off = B.payload_layout(cfg)
    ws = workspace(w.d, 2)
    payload = torch.zeros(total, dtype=torch.uint8, device="cuda")
    counts = torch.zeros(8, dtype=torch.int64, device="cuda")
    B.payload_encode(dev_tensor(g), cfg, payload, counts, ws)
    sync()
    sent = host(payload).copy()
    # a different workspace and a copy of the payload on the receiver side
    ws2 = B.workspace(w.d, 2)
    payload2 = dev_tensor(sent)
    dense = torch.full((w.d,), 3.0, dtype=torch.float32, device="cuda")
    counts2 = torch.zeros(8, dtype=torch.int64, device="cuda")
    B.payload_decode(payload2, cfg, dense, None, None, counts2, ws2)
    sync()
    rt = run_roundtrip(g, cfg)
    np.testing.assert_array_equal(host(dense), rt["dense"])
    np.testing.assert_array_equal(sent, rt["payload"])
    c1, c2 = host(counts).reshape(2, 4), host(counts2).reshape(2, 4)
    np.testing.assert_array_equal(c2[:, 2], c1[:, 1])
    assert np.all(c2[:, 3] == 0)


def test_receiver_flags_a_damaged_header():
    import torch

    w = W.Workload("t", 50_000, 1, (1, 100), 1e-3, 5, 8, "normal_1e-3", 12)
    g = W.generate(w)
    cfg = B.Config.from_workload(w)
    rt = run_roundtrip(g, cfg)
    bad = rt["payload"].copy()
    bad[0] ^= 0xFF  # magic
    dense = torch.full((w.d,), 3.0, dtype=torch.float32, device="cuda")
    counts = torch.zeros(4, dtype=torch.int64, device="cuda")
    B.payload_decode(dev_tensor(bad), cfg, dense, None, None, counts, workspace(w.d))
    sync()
    assert int(host(counts)[3]) & B.FLAG_DEC_MISMATCH
    assert np.all(host(dense) == 0)  # an invalid record decodes as empty


def test_per_kernel_trace():
    w = W.WORKLOADS["resnet20_conv_37k"]
    g = W.generate(w)
    cfg = B.Config.from_workload(w)
    B.trace_begin()
    run_roundtrip(g, cfg)
    tr = B.trace_end()
    assert "k_probe<Q_ENCODE>" in tr and "k_emit<Q_DECODE>" in tr
    assert all(n >= 1 and ms >= 0 for n, ms in tr.values())


# ---------------------------------------------------------------------------
# The bucketed query (rounds of one hash routed to filter slices in LDS),
# which the library takes for filters of at least 2^25 bits: with the
# threshold lowered to 1024 bits it runs on these small cases, for the
# sender (which skips its own selection) and the receiver, in the round
# trip and in a standalone decode of the same payload.
# ---------------------------------------------------------------------------
QB_CASES = {
    "resnet20_conv_37k": RT_CASES["resnet20_conv_37k"],
    "ragged_tensors": RT_CASES["ragged_tensors"],
    "support_50k": RT_CASES["support_50k"],
    # several index regions and filter slices, the bucketed insert before it
    "support_1m": RT_CASES["support_1m"],
    # more tensors than the path takes (16): the rest are probed as usual
    "many_tensors_3m": RT_CASES["many_tensors_3m"],
    # a 1.73 M-bit filter: four slices, 47 regions
    "normal_12m": LAYOUT_CASES["normal_12m"],
}


@pytest.mark.parametrize("layout", [B.FILTER_STANDARD, B.FILTER_PARTITIONED], ids=["standard", "partitioned"])
@pytest.mark.parametrize("name", list(QB_CASES))
def test_roundtrip_bucketed_query_parity(name, layout, monkeypatch):
    import torch

    monkeypatch.setenv("DR_QUERY_BUCKET_MIN_BITS", "1024")
    g, off, ratio, fpr, D, S = QB_CASES[name]
    log(f"roundtrip {name} bucketed query layout={layout} d={g.size} tensors={len(off) - 1}")
    cfg = B.Config(off, ratio, fpr, D, S, filter_layout=layout)
    out = run_roundtrip(g, cfg)
    refs = oracle.roundtrip(g, off, ratio, fpr, D, S,
                            layout=oracle.LAYOUT_PARTITIONED if layout == B.FILTER_PARTITIONED else oracle.LAYOUT_STANDARD)
    check_roundtrip(g, cfg, out, refs)
    # the same payload through the standalone receiver
    dense = torch.full((g.size,), 3.0, dtype=torch.float32, device="cuda")
    counts = torch.zeros(4 * cfg.n_tensors, dtype=torch.int64, device="cuda")
    B.payload_decode(dev_tensor(out["payload"]), cfg, dense, None, None, counts, workspace(g.size, cfg.n_tensors))
    sync()
    c = host(counts).reshape(cfg.n_tensors, 4)
    assert np.all(c[:, 3] == 0)
    np.testing.assert_array_equal(host(dense), out["dense"])
