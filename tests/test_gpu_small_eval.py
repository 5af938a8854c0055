"""Evaluation of small partitions (one table in LDS, one workgroup for the
relabelling) at the limits of that path, against the oracle and closed
forms; what the path does not take gives the same through the general one."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mcc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2408_11331_amd as m
    m.lib()
    oracle.build(force=False)
    return m


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()


# n around the int16 / int32 counts, the limit of the path and beyond;
# clusters around its limit; labels with and without gaps
@pytest.mark.parametrize("n", [1, 2, 1000, 32767, 32768, 65536, 65537])
@pytest.mark.parametrize("clusters,labels,gap", [(1, 1, 1), (10, 10, 1), (256, 96, 1),
                                                 (257, 5, 1), (30, 20, 3)])
def test_tables(mcc, n, clusters, labels, gap):
    print(f"[gpu-case] small eval n={n} clusters={clusters} labels={labels}", flush=True)
    rng = np.random.default_rng(n + clusters)
    c = np.sort(rng.choice(n, min(n, clusters), replace=False))[rng.integers(0, min(n, clusters), n)]
    parts = rng.integers(0, labels, (3, n)) * gap
    assert mcc.objective(dev(c), dev(parts)) == oracle.objective(c.astype(np.int32),
                                                                 parts.astype(np.int32))
    assert mcc.mirkin(dev(c), dev(parts[0])) == oracle.mirkin(c.astype(np.int32),
                                                              parts[0].astype(np.int32))
    got = mcc.compare(dev(c), dev(parts[1]))
    want = oracle.compare(c.astype(np.int32), parts[1].astype(np.int32))
    for key in ("mirkin", "split_join_ab", "split_join_ba", "split_join", "clusters_a",
                "clusters_b"):
        assert got[key] == want[key], key
    # double sums in another order: a few ulp of sums of n ln n
    assert abs(got["vi"] - want["vi"]) <= 1e-12 * max(1.0, np.log(max(n, 2)))
    assert got["rand"] == pytest.approx(want["rand"], rel=1e-15, abs=0)
    assert mcc.compare(dev(c), dev(parts[1])) == got  # the same bits on every call


def test_ids_beyond_the_range(mcc):
    # any label value is allowed in mirkin and compare, not in an objective
    a, b = np.array([5, 5, 900, 7]), np.array([1, 1, 0, 0])
    assert mcc.mirkin(dev(a), dev(b)) == oracle.mirkin(a.astype(np.int32), b.astype(np.int32))
    assert mcc.compare(dev(a), dev(b))["clusters_a"] == 3
    for bad in (np.array([0, 4, 0, 0]), np.array([0, -1, 0, 0])):
        with pytest.raises(mcc.MccError) as e:
            mcc.objective(dev(bad), dev(b[None]))
        assert e.value.code == mcc.MCC_EINVAL
        with pytest.raises(mcc.MccError) as e:
            mcc.canonicalize(dev(bad))
        assert e.value.code == mcc.MCC_EINVAL
    for neg in ((np.array([-1, 0, 0, 0]), b), (b, np.array([0, 0, -7, 0]))):
        for f in (mcc.mirkin, mcc.compare):
            with pytest.raises(mcc.MccError) as e:
                f(dev(neg[0]), dev(neg[1]))
            assert e.value.code == mcc.MCC_EINVAL


@pytest.mark.parametrize("n", [1, 63, 1024, 1025, 16383, 16384, 16385])
@pytest.mark.parametrize("ids", [1, 50, 10**9])
def test_canonical(mcc, n, ids):
    print(f"[gpu-case] canonical n={n} ids={ids}", flush=True)
    rng = np.random.default_rng(n)
    x = rng.integers(0, n, min(ids, n))[rng.integers(0, min(ids, n), n)]
    out, clusters = mcc.canonicalize(dev(x))
    vals, first = np.unique(x, return_index=True)
    rank = np.empty(vals.size, np.int64)
    rank[np.argsort(first)] = np.arange(vals.size)
    assert clusters == vals.size
    assert np.array_equal(out.cpu().numpy(), rank[np.searchsorted(vals, x)])
    y = dev(x)  # in place
    again, _ = mcc.canonicalize(y, out=y)
    assert np.array_equal(again.cpu().numpy(), out.cpu().numpy())
