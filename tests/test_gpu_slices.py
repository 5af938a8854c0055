"""Many vertices with few clusters, whose passes read one partition's counts
at a time: the whole trace against the oracle, with few and with many
candidates a vertex, at the edges of the candidate masks (32 clusters a
word) and of the label words (4 partitions)."""
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


@pytest.mark.parametrize("symmetric", [False, True])
@pytest.mark.parametrize("clusters,k,graph", [(2, 1, "near"), (32, 2, "far"), (33, 5, "mixed"),
                                              (64, 4, "near"), (60, 7, "far"), (51, 9, "hubs")])
def test_many_vertices(mcc, symmetric, clusters, k, graph):
    print(f"[gpu-case] slices {clusters} {k} {graph} symmetric={symmetric}", flush=True)
    import torch
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    n = (1 << 19) + 777
    rng = np.random.default_rng(clusters)
    m = 8 * n
    u = rng.integers(0, n, m)
    v = (u + rng.integers(1, 2000, m)) % n
    far = rng.random(m) < {"near": 0.0, "far": 0.9, "mixed": 0.1, "hubs": 0.02}[graph]
    v[far] = rng.integers(0, n, int(far.sum()))
    if graph == "hubs":
        u[:40000] = rng.integers(0, 40, 40000) * 1000
    rp, col = synth.graph.csr_from_edges(n, u, v)
    base = np.arange(n) * clusters // n
    labels = np.tile(base, (k, 1))
    noise = rng.random((k, n)) < 0.25
    labels[noise] = rng.integers(0, clusters, int(noise.sum()))
    for i in range(k):
        labels[i] = rng.permutation(clusters)[labels[i]]
    labels = labels.astype(np.int32)
    init = base.copy()
    moved = rng.random(n) < 0.3
    init[moved] = rng.integers(0, clusters, int(moved.sum()))
    init = (init * 3 + 1).astype(np.int32)
    out, st, tr = mcc.consensus(dev(rp), dev(col), dev(labels), dev(init), trace=True,
                                flags=mcc.MCC_F_SYMMETRIC if symmetric else 0, max_rounds=5)
    eo, est, et = oracle.consensus(rp, col, labels, init, trace=True, max_rounds=5)
    assert st["tables"] == 1
    assert [tuple(t) for t in et][:st["passes"]] == tr
    assert np.array_equal(out.cpu().numpy(), eo)
    for key in ("passes", "clusters", "moves", "candidate_evals", "objective_init", "objective"):
        assert st[key] == est[key], key


@pytest.mark.parametrize("n,groups,k", [(4000, 600, 1), (20000, 1900, 4), (600001, 4000, 3)])
def test_many_clusters_aligned(mcc, n, groups, k):
    """Tables far larger than the sample their labels are aligned from (all
    vertices, or runs of 64): home clusters looked up by the sampled members;
    labels that no sampled vertex has."""
    print(f"[gpu-case] align n={n} groups={groups} k={k}", flush=True)
    import torch
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    rng = np.random.default_rng(n)
    u = rng.integers(0, n, 5 * n)
    v = (u + rng.integers(1, 40, 5 * n)) % n
    rp, col = synth.graph.csr_from_edges(n, u, v)
    base = np.arange(n) * groups // n
    labels = np.stack([rng.permutation(groups + 50)[
        np.where(rng.random(n) < 0.2, rng.integers(0, groups + 50, n), base)]
        for _ in range(k)]).astype(np.int32)
    init = np.where(rng.random(n) < 0.2, rng.integers(0, groups, n), base).astype(np.int32)
    out, st, tr = mcc.consensus(dev(rp), dev(col), dev(labels), dev(init), trace=True,
                                max_rounds=4)
    eo, est, et = oracle.consensus(rp, col, labels, init, trace=True, max_rounds=4)
    assert st["tables"] == 1
    assert [tuple(t) for t in et][:st["passes"]] == tr
    assert np.array_equal(out.cpu().numpy(), eo)
    assert st["objective"] == est["objective"] and st["objective_init"] == est["objective_init"]
