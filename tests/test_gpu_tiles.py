"""The tiled scorer's variants (vertices a tile, labels a lane) and the
staged first-occurrence search at the sizes where they change, against the
oracle."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu
KEYS = ("passes", "converged", "fallback_rounds", "clusters", "moves", "candidate_evals",
        "objective_init", "objective")


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
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def planted(n, k, groups, seed):
    """Ring graph with chords and k noisy copies of a planted partition."""
    rng = np.random.default_rng(seed)
    v = np.arange(n)
    u = np.concatenate([v, v, rng.integers(0, n, n)])
    w = np.concatenate([(v + 1) % n, (v + 7) % n, rng.integers(0, n, n)])
    row_ptr, col = synth.graph.csr_from_edges(n, u, w)
    truth = v * groups // n
    labels = np.tile(truth, (k, 1))
    noise = rng.random((k, n)) < 0.3
    labels[noise] = rng.integers(0, groups, int(noise.sum()))
    return row_ptr, col, labels.astype(np.int32)


# n at the edges of a tile and of the ranges of tile sizes; k at the edges of
# the labels a lane holds; more than 256 clusters above 2^18 vertices
@pytest.mark.parametrize("n,k,groups", [
    (63, 16, 4), (64, 17, 5), (65, 32, 6), (129, 33, 7), (1000, 64, 9), (1001, 65, 9),
    (1 << 18, 3, 100), ((1 << 18) + 1, 3, 100), ((1 << 18) + 1, 3, 300)])
@pytest.mark.parametrize("symmetric", [False, True])
def test_tile_variants(mcc, n, k, groups, symmetric):
    print(f"[gpu-case] tiles n={n} k={k} groups={groups} symmetric={symmetric}", flush=True)
    row_ptr, col, labels = planted(n, k, groups, n + k)
    init = labels[0].copy()
    flags = mcc.MCC_F_SYMMETRIC if symmetric else 0
    out, st = mcc.consensus(dev(row_ptr), dev(col), dev(labels), dev(init), flags=flags,
                            max_rounds=4)
    eo, est, _ = oracle.consensus(row_ptr, col, labels, init, max_rounds=4)
    assert np.array_equal(out.cpu().numpy(), eo)
    for key in KEYS:
        assert st[key] == est[key], key


@pytest.mark.parametrize("n", [1, 64, 1023, 1024, 1025, 2048, 32767, 32768, 66000])
@pytest.mark.parametrize("kind", ["few", "runs", "singletons"])
def test_canonicalize_ranges(mcc, n, kind):
    print(f"[gpu-case] canonicalize n={n} {kind}", flush=True)
    rng = np.random.default_rng(n)
    if kind == "few":  # an id that covers most vertices, and rare ones
        x = np.where(rng.random(n) < 0.9, n - 1, rng.integers(0, n, n))
    elif kind == "runs":  # long runs of one id, in decreasing order of id
        x = (n - 1 - np.arange(n)) // 300
    else:
        x = rng.permutation(n)
    out, clusters = mcc.canonicalize(dev(x.astype(np.int32)))
    ids, first = np.unique(x, return_index=True)
    rank = np.empty(ids.size, np.int64)
    rank[np.argsort(first)] = np.arange(ids.size)
    assert clusters == ids.size
    assert np.array_equal(out.cpu().numpy(), rank[np.searchsorted(ids, x)])
