"""Stage 4 between 2^18 and 2^22 requests on the GPU against the oracle.

In this range FIFO and SJF are sample sorts by (key, position) with exact
bucket sizes (a bucket larger than the in-LDS limit is sorted through global
memory by the same block). Sizes around the range's ends, key layouts that
crowd a bucket's bins (heavy ties, constant keys, clusters, both zeros),
sequences already in order, and inputs arranged against the sampling so that
one bucket takes almost every request; every policy must match the oracle
exactly.
"""
import numpy as np
import pytest
import torch

from tests.gpu_util import dev
from tests.test_gpu_order import POLICIES, _batch, check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ds():
    from paper_2606_02982_amd import driftsched
    return driftsched


@pytest.mark.parametrize("pol", POLICIES)
@pytest.mark.parametrize("n", [262145, 300001, 524411, 1048575, 1048576, 1048577])
def test_sizes(ds, oracle, pol, n):
    tier, arr, bud = _batch(n + 1, n)
    check(ds, oracle, pol, tier, arr, bud, t_now=10.0, aging_rate=0.1)


def _layout(pattern, n, rng):
    j = np.arange(n)
    tier = rng.integers(0, 3, n).astype(np.uint8)
    arr = rng.uniform(0.0, 100.0, n)
    bud = np.round(rng.uniform(1, 3000, n), 1)
    if pattern == "ties":
        arr = np.round(arr / 5.0) * 5.0
        bud = np.round(bud / 500.0) * 500.0
        arr[:1000] = 0.0
        arr[1000:2000] = -0.0
    elif pattern == "constant":
        arr[:] = 7.25
        bud[:] = 100.0
    elif pattern == "in_order":
        arr = j * 1e-3
        bud = 1.0 + (j % 977) * 0.5
    elif pattern == "descending":
        arr = (n - j) * 1e-3
        bud = np.round((n - j) / 64.0)
    elif pattern == "skewed":
        arr = np.where(rng.random(n) < 0.99, 5.0, rng.uniform(-1e6, 1e6, n) * 10.0 ** rng.integers(-30, 30, n))
        bud = np.where(rng.random(n) < 0.99, 100.0, rng.standard_cauchy(n))
    elif pattern in ("repeated", "repeated_in_order"):
        # keys of 100 to 2,000 requests each, so that a bucket holds a few
        # whole keys and parts of two; zeros of both signs among them
        arr = np.floor(rng.normal(0.0, n / 1500.0, n)) / 4.0
        arr[rng.random(n) < 0.01] = -0.0
        bud = np.round(rng.uniform(1, n / 300.0, n)) * 0.5
        if pattern == "repeated_in_order":
            arr.sort()
            bud.sort()
    elif pattern == "clusters":
        arr = rng.choice([0.0, 50.0], n) + rng.uniform(0.0, 1e-9, n)
        bud = rng.choice([100.0, 100.5, 5000.0], n) + np.where(rng.random(n) < 0.5, 0.0,
                                                               rng.uniform(0.0, 1e-9, n))
    return tier, arr, bud


@pytest.mark.parametrize("pol", POLICIES)
@pytest.mark.parametrize("pattern", ["ties", "constant", "in_order", "descending", "skewed", "clusters", "repeated", "repeated_in_order"])
def test_layouts(ds, oracle, pol, pattern):
    n = 400003
    rng = np.random.default_rng(n + len(pattern))
    tier, arr, bud = _layout(pattern, n, rng)
    t_now = float(np.max(arr))
    check(ds, oracle, pol, tier, arr, bud, t_now=t_now, aging_rate=0.01, aging_floor=-np.inf)


def sample_positions(n):
    """The positions the sample sort of this range draws its sample from:
    one per stratum of [0, n), offset by a fixed integer hash."""
    B = max(2, -(-n // 1024))
    S = min(8192, -(-8 * B // 64) * 64)
    s = np.arange(S, dtype=np.uint64)
    lo = s * np.uint64(n) // np.uint64(S)
    hi = (s + np.uint64(1)) * np.uint64(n) // np.uint64(S)
    m = np.uint64(0xFFFFFFFF)
    h = (s * np.uint64(0x9E3779B1) + np.uint64(0x7F4A7C15)) & m
    h ^= h >> np.uint64(15)
    h = (h * np.uint64(0x85EBCA77)) & m
    h ^= h >> np.uint64(13)
    return (lo + h % (hi - lo)).astype(np.int64), S


@pytest.mark.parametrize("target", ["fifo", "sjf"])
@pytest.mark.parametrize("spread", [0.0, 1e-7])
def test_one_bucket_takes_almost_all(ds, oracle, target, spread):
    # the sampled positions get distinct keys 0, 1, ..., the others keys
    # between two of them: one bucket receives all but the sample (far over
    # the in-LDS limit) and is sorted through global memory; spread > 0
    # makes those keys differ, so that the passes cover key bytes as well as
    # positions
    n = 1048576 - 3
    rng = np.random.default_rng(5 if target == "fifo" else 6)
    pos, S = sample_positions(n)
    tier = rng.integers(0, 3, n).astype(np.uint8)
    fill = S / 2.0 + 0.25 + rng.uniform(0.0, spread, n)
    if target == "fifo":
        arr = fill.copy()
        arr[pos] = np.arange(S, dtype=np.float64)
        bud = np.round(rng.uniform(1, 3000, n), 1)
    else:
        # arrivals in index order: the FIFO sequence is the identity, so SJF
        # samples the same positions
        arr = np.arange(n) * 1e-3
        bud = fill.copy()
        bud[pos] = np.arange(S, dtype=np.float64)
    for pol in POLICIES:
        check(ds, oracle, pol, tier, arr, bud, t_now=float(np.max(arr)), aging_rate=0.01)


@pytest.mark.parametrize("n", [300007, 1048577])
@pytest.mark.parametrize("shares", ["even16", "tiny", "one", "gap"])
def test_aging_places(ds, oracle, n, shares):
    # each request's place from its run and the entries below it in the other
    # runs: many classes, runs of a few entries beside runs of all the others
    # (stretches searched in memory), empty classes, and a floor that cuts a
    # tile (its clamped entries tie with their neighbours in time, the others
    # follow every clamped one, far away)
    rng = np.random.default_rng(n + len(shares))
    tier, arr, bud = _batch(n + 7, n)
    k = 16 if shares == "even16" else 4
    p = {"even16": np.full(16, 1 / 16), "tiny": np.array([0.9, 0.0999, 0.0001, 0.0]),
         "one": np.array([0.0, 0.0, 1.0, 0.0]), "gap": np.array([0.4, 0.3, 0.2, 0.1])}[shares]
    tier = rng.choice(k, n, p=p).astype(np.uint8)
    arr = rng.uniform(0.0, 1000.0, n)
    check(ds, oracle, ds.AGING, tier, arr, bud, n_tiers=k, weights=(1,) * k,
          tier_priority=tuple(float(q) for q in range(k)), t_now=1000.0, aging_rate=0.004)


# the larger tiles and tables above 2^20, up to the last size before the radix
# passes and the first one with them
@pytest.mark.parametrize("n,pols", [(1500001, POLICIES), (4194304, (0, 3)), (4194305, (0, 3))])
def test_sizes_above_2_20(ds, oracle, n, pols):
    tier, arr, bud = _batch(n + 3, n)
    for pol in pols:
        check(ds, oracle, pol, tier, arr, bud, t_now=10.0, aging_rate=0.1)


@pytest.mark.parametrize("pol", POLICIES)
@pytest.mark.parametrize("pattern", ["ties", "constant", "skewed", "clusters", "repeated", "repeated_in_order"])
def test_layouts_above_2_20(ds, oracle, pol, pattern):
    n = 1100003
    rng = np.random.default_rng(n + len(pattern))
    tier, arr, bud = _layout(pattern, n, rng)
    check(ds, oracle, pol, tier, arr, bud, t_now=100.0, aging_rate=0.01, aging_floor=-np.inf)


# what ds_order took before the sample sorts of more than 2^20 requests, which
# then have no room
@pytest.mark.parametrize("n,nbytes", [(1048577, 64411136), (2097152, 65057536), (4194304, 127972096),
                                      (4194305, 127981568)])
@pytest.mark.parametrize("pol", POLICIES)
def test_smaller_workspaces(ds, n, nbytes, pol):
    """A workspace of that size is taken still, nothing behind it touched, and
    the order and keys are those of a workspace with room for the fast way,
    with the FIFO order given and without."""
    print("workspace n=%d bytes=%d policy=%d" % (n, nbytes, pol), flush=True)
    tier, arr, bud = (dev(x) for x in _batch(n, n))
    kw = dict(key=True, aging_rate=0.5, t_now=10.0)
    full = torch.empty(ds.workspace_bytes(ds.OP_ORDER, n), dtype=torch.uint8, device="cuda")
    fifo = ds.order(ds.FIFO, tier, arr, bud, ws=full, **kw)[0].clone()
    buf = torch.full((nbytes + 65536,), 0xA5, dtype=torch.uint8, device="cuda")
    for given in (None, fifo):
        want = ds.order(pol, tier, arr, bud, fifo=given, ws=full, **kw)
        got = ds.order(pol, tier, arr, bud, fifo=given, ws=buf[:nbytes], **kw)
        assert ds.wait_status(buf) == 0
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
        assert bool((buf[nbytes:] == 0xA5).all())


@pytest.mark.parametrize("shares", [(0.99, 0.01), (0.001, 0.999), (0.9, 0.06, 0.04), (0.5, 0.3) + (0.04,) * 5,
                                    (0.1,) * 10, (1 / 11,) * 11, (0.9,) + (0.1 / 12,) * 12, (1 / 16,) * 16,
                                    (0.6, 0.0, 0.0, 0.0) + (0.4 / 12,) * 12],
                         ids=lambda s: "%d classes" % len(s))
@pytest.mark.parametrize("rate,floor", [(0.0, -np.inf), (10.0, -np.inf), (0.1, 0.5)])
def test_aging_class_mixes(ds, oracle, shares, rate, floor):
    """Runs of every ratio (tiles of 1,024, 512 and 256 entries and runs too
    short for tiles), at 11 classes and more merged in two steps: apart, fully
    overlapping, and cut by the floor; with and without a given FIFO order."""
    n, k = 300007, len(shares)
    print("mix %s rate %g floor %g" % (shares, rate, floor), flush=True)
    rng = np.random.default_rng(k + int(10 * rate))
    tier = rng.choice(k, n, p=np.array(shares) / sum(shares)).astype(np.uint8)
    arr = np.round(rng.uniform(0.0, 60.0, n), 4)
    kw = dict(n_tiers=k, weights=(1,) * k, tier_priority=tuple(float(q) for q in range(k)), t_now=60.0,
              aging_rate=rate, aging_floor=floor)
    check(ds, oracle, ds.AGING, tier, arr, arr, **kw)
    fifo = dev(np.lexsort((np.arange(n), arr)).astype(np.uint32))
    want = oracle.order(ds.AGING, tier, arr, **{a: b for a, b in kw.items() if a != "n_tiers"})[0]
    got = ds.order(ds.AGING, dev(tier), dev(arr), fifo=fifo, **kw)[0]
    assert np.array_equal(got.cpu().numpy().view(np.uint32), want)


@pytest.mark.parametrize("n", [300001, 1048577])
@pytest.mark.parametrize("tiers", [3, 16])
def test_partitions_over_a_given_order(ds, oracle, n, tiers):
    # the digits and budgets are gathered through the given order, not read from
    # copies in FIFO order; both tile sizes, the last tier and shared classes
    rng = np.random.default_rng(n + tiers)
    tier = rng.integers(0, tiers, n).astype(np.uint8)
    arr = rng.uniform(0.0, 100.0, n)
    bud = np.round(rng.uniform(1, 3000, n), 1)
    kw = dict(weights=tuple(1 + q % 4 for q in range(tiers)), tier_priority=tuple(float(q % 5) for q in range(tiers)),
              aging_rate=0.1, t_now=100.0)
    fifo = dev(np.lexsort((np.arange(n), arr)).astype(np.uint32))
    pols = (ds.PRIORITY, ds.WEIGHTED, ds.SJF, ds.AGING)
    got, _ = ds.order_multi(pols, dev(tier), dev(arr), dev(bud), fifo=fifo, n_tiers=tiers, **kw)
    for pol in pols:
        want = oracle.order(pol, tier, arr, bud, **kw)[0].astype(np.int32)
        assert np.array_equal(got[pol].cpu().numpy(), want), pol
        one = ds.order(pol, dev(tier), dev(arr), dev(bud), fifo=fifo, n_tiers=tiers, **kw)[0]
        assert np.array_equal(one.cpu().numpy(), want), pol
