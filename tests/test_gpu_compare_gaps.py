"""Comparison of small partitions whose label values have gaps: the same bits
as the general comparison (which the same partition takes with its values far
apart), at the limits of the small table, and at the cost of one without."""
import time

import numpy as np
import pytest

import oracle

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


# (n, clusters, label values that occur, span of the values)
@pytest.mark.parametrize("n,clusters,labels,span", [
    (1, 1, 1, 1), (1, 1, 1, 24576), (40, 2, 3, 12288), (1000, 10, 10, 28), (5000, 96, 200, 256),
    (32767, 1, 255, 24576), (32768, 256, 40, 96), (65536, 250, 57, 98), (65536, 3, 3000, 8192)])
def test_equals_general(mcc, n, clusters, labels, span):
    print(f"[gpu-case] compare with gaps n={n} labels={labels} of {span}", flush=True)
    rng = np.random.default_rng(n + span)
    a = rng.integers(0, clusters, n)
    values = np.sort(rng.choice(span, min(labels, span), replace=False))
    values[-1] = span - 1
    b = values[rng.integers(0, values.size, n)]
    b[-1] = span - 1
    far = np.searchsorted(values, b) * 100_003 + 30_000  # the same partition, the general path
    got, want = mcc.compare(dev(a), dev(b)), mcc.compare(dev(a), dev(far))
    assert got == want
    ref = oracle.compare(a.astype(np.int32), b.astype(np.int32))
    for key in ("mirkin", "split_join_ab", "split_join_ba", "clusters_a", "clusters_b"):
        assert got[key] == ref[key], key


def test_time(mcc):
    print("[gpu-case] compare with gaps, time", flush=True)
    rng = np.random.default_rng(1)
    a, b = rng.integers(0, 50, 30000), rng.integers(0, 50, 30000)

    def best(x, y):
        t = []
        for _ in range(30):
            t0 = time.perf_counter()
            mcc.compare(x, y)
            t.append(time.perf_counter() - t0)
        return min(t)

    plain, gaps = best(dev(a), dev(b)), best(dev(a), dev(2 * b))
    assert gaps < 2 * plain, (gaps, plain)
