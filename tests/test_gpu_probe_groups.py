"""The full-range query over the forms its hash groups take, and one hash at a
time: filters that the LDS copy holds whole, to the last word, or in part, one to
thirteen hashes, ragged windows, and filters so full that the survivor queues
overflow.  Bit-exact against the oracle's query."""
import numpy as np
import pytest

import oracle
from paper_2102_03112_amd import binding as B
from _gpu_util import check_roundtrip, dev_tensor, host, log, run_roundtrip, sync, u64_scalar, workspace

pytestmark = pytest.mark.gpu

LDS_BITS = 35072 * 32  # the filter bits that the probe pass keeps in LDS

# (m bits, k, share of set bits, d)
FILTERS = [
    (32, 1, 0.5, 1), (96, 3, 0.5, 4097), (4096, 2, 0.9, 2048), (40_000, 10, 0.5, 36_864),
    (LDS_BITS, 10, 0.5, 70_001), (LDS_BITS + 32, 10, 0.5, 70_001), (LDS_BITS + 32, 3, 0.5, 20_481),
    (LDS_BITS * 2, 10, 0.5, 100_003), (LDS_BITS * 2 + 32, 7, 0.5, 100_003), (LDS_BITS * 3, 1, 0.5, 9000),
    (LDS_BITS * 3, 5, 0.97, 50_000), (LDS_BITS * 6, 13, 0.6, 33_000), (LDS_BITS * 6 + 32, 13, 0.6, 33_000),
    (LDS_BITS * 9, 2, 0.98, 12_289), (LDS_BITS * 2, 13, 1.0, 8193), (LDS_BITS * 9, 13, 1.0, 8193),
    (LDS_BITS, 13, 1.0, 8193),
    # few members, so that groups of four, of three and (96 steps a block) of three again read memory
    (LDS_BITS * 3, 10, 0.5, 2_000_003), (LDS_BITS * 4 + 32, 13, 0.55, 2_200_001), (LDS_BITS * 12, 13, 0.5, 6_000_001),
    (LDS_BITS * 2 - 32, 10, 0.5, 12_700_001),
]


@pytest.mark.parametrize("m,k,fill,d", FILTERS)
def test_query_of_any_filter(m, k, fill, d):
    import torch

    log(f"query m={m} k={k} fill={fill} d={d}")
    rng = np.random.default_rng(m + k + d)
    words = np.packbits(rng.random(m) < fill, bitorder="little").view("<u4")
    ref = oracle.bloom_query(words, m, k, d)
    idx = torch.full((d,), -1, dtype=torch.int32, device="cuda")
    n = u64_scalar()
    B.bloom_decode(dev_tensor(words.view(np.int32)), m, k, d, idx, d, n, workspace(d))
    sync()
    assert int(host(n)[0]) == ref.size
    np.testing.assert_array_equal(host(idx)[: ref.size].view(np.uint32), ref)


# (d, ratio, fpr, layout): both directions, with the sender's own selection
TRIPS = [
    (300_000, (1, 4), 1e-3, 0), (300_000, (1, 2), 1e-2, 0), (300_000, (1, 4), 1e-3, 1), (300_000, (1, 8), 1e-3, 1),
    (300_000, (1, 3), 0.3, 1), (70_000, (1, 2), 1e-4, 1), (1_200_000, (1, 2), 1e-3, 0),
]


@pytest.mark.parametrize("d,ratio,fpr,layout", TRIPS)
def test_round_trip_with_large_filters(d, ratio, fpr, layout):
    log(f"round trip d={d} ratio={ratio} fpr={fpr} layout={layout}")
    g = (np.random.default_rng(d).standard_normal(d) * 1e-3).astype(np.float32)
    cfg = B.Config([0, d], ratio, fpr, 3, 4, filter_layout=layout)
    refs = oracle.roundtrip(g, [0, d], ratio, fpr, 3, 4, layout=layout)
    check_roundtrip(g, cfg, run_roundtrip(g, cfg), refs)


@pytest.mark.parametrize("layout", [0, 1], ids=["standard", "partitioned"])
@pytest.mark.parametrize("tensors,spread", [(300, 4000), (67, 40_000), (40, 1)])
def test_round_trip_of_many_tensors(tensors, spread, layout):
    """Blocks whose share holds a few tensors, empty and one-element tensors
    among them (40), and set-up over several launches."""
    rng = np.random.default_rng(tensors)
    sizes = rng.integers(0, spread + 1, tensors)
    sizes[tensors // 2] = 300_000  # a filter larger than what LDS keeps
    off = np.concatenate([[0], np.cumsum(sizes)])
    log(f"{tensors} tensors, {int(off[-1])} elements")
    g = (rng.standard_normal(int(off[-1])) * 1e-3).astype(np.float32)
    cfg = B.Config(off, (1, 4), 1e-3, 3, 2, filter_layout=layout)
    refs = oracle.roundtrip(g, off, (1, 4), 1e-3, 3, 2, layout=layout)
    check_roundtrip(g, cfg, run_roundtrip(g, cfg), refs)


@pytest.fixture(scope="module")
def shared():
    """Shares of 41 tiles over 9400 tensors, so that runs are shared and end at 32
    tensors, at a full LDS copy (10 tensors of 8 to 20 K elements, 14.4 bits
    each), at a filter larger than it and at the end of the share; empty and
    one-element tensors among them."""
    rng = np.random.default_rng(9)
    sizes = rng.integers(0, 41, 9400)
    mid = np.concatenate([np.arange(200, 500), rng.choice(np.arange(600, 9000), 100, replace=False)])
    sizes[mid] = rng.integers(8000, 20_001, mid.size)
    sizes[[100, 4700]] = 90_000
    off = np.concatenate([[0], np.cumsum(sizes)])
    cfg = B.Config(off, (1, 2), 1e-6, 2, 2)
    gs = [(np.random.default_rng(90 + p).standard_normal(cfg.d) * 1e-3).astype(np.float32) for p in range(2)]
    refs = [oracle.roundtrip(g, off, (1, 2), 1e-6, 2, 2) for g in gs]
    return cfg, gs, refs, np.sort(mid)


def traced(call):
    """The kernels that the call launched."""
    B.trace_begin()
    call()
    sync()
    return B.trace_end()


def test_round_trip_of_shared_runs(shared):
    cfg, gs, refs, _ = shared
    log(f"{cfg.n_tensors} tensors, {cfg.d} elements")
    outs = []
    kernels = traced(lambda: outs.append(run_roundtrip(gs[0], cfg)))
    assert {"k_probe_many<Q_ENCODE>", "k_probe_many<Q_DECODE>"} <= set(kernels)
    check_roundtrip(gs[0], cfg, outs[0], refs[0])


def test_damaged_records_among_shared_runs(shared):
    """A record with a damaged header inside a run is flagged and left out, by
    the receiver and by the summing receiver; the others are whole."""
    import torch

    cfg, gs, refs, mid = shared
    T, off = cfg.n_tensors, cfg.offsets.astype(np.int64)
    ws = workspace(cfg.d, T)
    outs = [run_roundtrip(g, cfg) for g in gs]
    pays = [o["payload"] for o in outs]
    damaged = [int(mid[40]), 5000, 9399]
    for t in damaged:
        pays[1][outs[1]["rec_off"][t]] ^= 0xFF  # magic
    pays = [dev_tensor(p) for p in pays]
    dense = torch.full((cfg.d,), 9.0, device="cuda")
    counts = torch.zeros(4 * T, dtype=torch.int64, device="cuda")
    kernels = traced(lambda: B.payload_decode(pays[1], cfg, dense, None, None, counts, ws))
    assert "k_probe_many<Q_DECODE>" in kernels
    want = outs[1]["dense"].copy()
    for t in damaged:
        want[off[t]:off[t + 1]] = 0.0
    np.testing.assert_array_equal(host(dense), want)
    flags = host(counts).reshape(T, 4)[:, 3]
    assert sorted(np.flatnonzero(flags)) == sorted(damaged) and all(flags[t] & B.FLAG_DEC_MISMATCH for t in damaged)

    total = torch.full((cfg.d,), 9.0, device="cuda")
    counts = torch.zeros(8 * T, dtype=torch.int64, device="cuda")
    ws2 = B.workspace(2 * cfg.d, 2 * T)
    kernels = traced(lambda: B.payload_decode_sum(pays, cfg, 0.5, total, counts, ws2))
    assert "k_probe_many<Q_SUM>" in kernels
    np.testing.assert_array_equal(host(total), np.float32(0.5) * (outs[0]["dense"] + want))
    flags = host(counts).reshape(2, T, 4)[:, :, 3]
    assert not flags[0].any() and sorted(np.flatnonzero(flags[1])) == sorted(damaged)


@pytest.mark.parametrize("tensors,d,layout", [(14, 4_800_003, 0), (14, 4_800_003, 1), (6, 12_000_001, 0),
                                              (6, 12_000_001, 1), (3, 23_000_001, 0)])
def test_groups_and_single_hashes_agree(tensors, d, layout):
    """A batch long enough for groups of hashes against its tensors one by one,
    which are tested one hash at a time or, the largest, in other groups: the same
    records, dense values and positives."""
    import torch

    log(f"{tensors} x {d} layout={layout}")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d + layout)
    off = [d * t for t in range(tensors + 1)]
    g = torch.randn(off[-1], generator=gen, device="cuda") * 1e-3
    cfg, one = B.Config(off, (1, 100), 1e-3, 3, 4, filter_layout=layout), B.Config([0, d], (1, 100), 1e-3, 3, 4,
                                                                                filter_layout=layout)

    def trip(x, c):
        total, rec = B.payload_layout(c)
        pay = torch.zeros(total, dtype=torch.uint8, device="cuda")
        dense = torch.full((c.d,), 9.0, device="cuda")
        counts = torch.zeros(4 * c.n_tensors, dtype=torch.int64, device="cuda")
        B.roundtrip(x, c, pay, dense, None, None, counts, workspace(c.d, c.n_tensors))
        sync()
        return pay, rec, dense, counts

    pay, rec, dense, counts = trip(g, cfg)
    for t in range(tensors):
        p1, _, d1, c1 = trip(g[off[t]:off[t + 1]], one)
        n = B.parse_record(host(p1), 0).rec_bytes
        assert torch.equal(counts[4 * t:4 * t + 4], c1) and int(c1[3]) == 0
        assert torch.equal(pay[rec[t]:rec[t] + n], p1[:n])
        assert torch.equal(dense[off[t]:off[t + 1]], d1)
