"""Batches that the level-by-level kernels take in several waves: every
instance equals the oracle's solve of it.  The instances are copies of a few,
whose graphs and labels they share, each with an output of its own."""
import time

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


def copies(mcc, items, count):
    """count instances, cycling through the items (equal n), which they share."""
    import torch
    m = len(items)
    pick = np.arange(count) % m
    one = mcc.pack_batch(items)
    at = lambda sizes: np.concatenate([[0], np.cumsum(sizes)[:-1]]).astype(np.int64)[pick]
    n = one.n[pick]
    init = torch.from_numpy(np.stack([i.init for i in items])).cuda()[torch.from_numpy(pick).cuda()]
    return mcc.PackedBatch(one.row_ptr, one.col, one.labels, init.reshape(-1).contiguous(),
                           torch.full((int(n.sum()) + 1,), -3, dtype=torch.int32, device="cuda"),
                           n, one.nnz[pick], one.k[pick], at(one.n + 1), at(one.nnz),
                           at(one.n * one.k), np.ones(count, bool))


def check(pb, items, info, max_rounds, fits=True):
    assert info["rc"] == 0 and info["solved_in_batch"] == (pb.count if fits else 0)
    m = len(items)
    out = pb.out[:-1].cpu().numpy().reshape(pb.count, -1)
    for j, i in enumerate(items):
        eo, est, _ = oracle.consensus(i.row_ptr, i.col, i.labels, i.init, max_rounds=max_rounds)
        assert (out[j::m] == eo).all()
        for c in range(j, pb.count, max(m, pb.count // 50 // m * m)):
            st = pb.stats[c].as_dict()
            for key in KEYS:
                assert st[key] == est[key], (c, key)


def many_clusters(seed):
    """100 vertices in clusters of their own, 42 labels, 64 partitions: tables of
    half a megabyte, more than a workgroup of the persistent launch takes."""
    inst = synth.random_instance(100, 64, 6.0, 42, seed=seed, init="random")
    inst.labels[:, 0] = 41
    inst.init = np.random.default_rng(seed).permutation(100).astype(np.int32)
    return inst


def test_waves_of_full_tables(mcc):
    """Waves of 512 instances, whose tables fill them: eight times the
    instances take eight times the time, not up to 64."""
    import torch
    print("[gpu-case] batch waves of full tables", flush=True)
    items = [many_clusters(80 + j) for j in range(3)]
    t = []
    for count in (1000, 8000):
        pb = copies(mcc, items, count)
        best = float("inf")
        for _ in range(3):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            info = mcc.consensus_batch_packed(pb, max_rounds=4)
            best = min(best, time.perf_counter() - t0)
        check(pb, items, info, 4, fits=False)
        t.append(best)
    assert t[1] < 16 * t[0], t


def test_many_instances(mcc):
    """66 000 instances with 64 partitions each: 4.3 million label ranges, more
    workgroups of 1024 threads than one launch may hold."""
    print("[gpu-case] batch of 66000 x 100 vertices, k = 64", flush=True)
    items = [many_clusters(90 + j) for j in range(3)]
    pb = copies(mcc, items, 66_000)
    check(pb, items, mcc.consensus_batch_packed(pb, max_rounds=3), 3, fits=False)
    assert all(pb.stats[j].lanes_used == 0 for j in range(0, pb.count, 1000))


@pytest.mark.parametrize("count,n,k", [(15000, 30, 64), (3000, 100, 64), (15000, 100, 8),
                                       (200, 30, 3)])
def test_tiny_instances_time(mcc, count, n, k):
    """Many tiny instances take no longer than 1.5 times the persistent launch
    that lanes=4 asks for."""
    import torch
    print(f"[gpu-case] batch of {count} tiny instances {n} x {k}, time", flush=True)
    items = [synth.random_instance(n, k, 8.0, 2, seed=60 + j) for j in range(3)]
    pb = copies(mcc, items, count)

    def best(**kw):
        t = []
        for _ in range(8):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            info = mcc.consensus_batch_packed(pb, **kw)
            t.append(time.perf_counter() - t0)
        check(pb, items, info, 0)
        return min(t)

    mine, persistent = best(), best(lanes=4)
    assert mine < 1.5 * persistent, (mine, persistent)


@pytest.mark.parametrize("count", [127, 128, 400])
def test_tiny_instances_mixed(mcc, count):
    """Tiny instances on both sides of the number that goes to the persistent
    launch, among them tables too large for it, label values too large for it,
    singleton starts and a negative label, beside larger ones."""
    print(f"[gpu-case] batch of {count} tiny instances, mixed", flush=True)
    import torch
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    items = [synth.random_instance(20 + j % 90, 5 + j % 60, 4.0, 1 + j % 7, seed=j,
                                   init=["p0", "singleton", "random"][j % 3])
             for j in range(count)]
    for j in (3, 40, 99):
        items[j] = many_clusters(j)
    items[5].labels[2] *= 70_001
    items[6].labels[1, 4] = -2
    items += [synth.random_instance(3000, 9, 6.0, 8, seed=7 + j) for j in range(3)]
    single = lambda j: j < count and j % 3 == 1 and j not in (40,)
    probs = [{"row_ptr": dev(i.row_ptr), "col": dev(i.col), "labels": dev(i.labels),
              "init": None if single(j) else dev(i.init)} for j, i in enumerate(items)]
    outs, stats, codes, info = mcc.consensus_batch(probs, max_rounds=20)
    assert codes == [mcc.MCC_EINVAL if j == 6 else 0 for j in range(len(items))]
    for j, i in enumerate(items):
        if j == 6:
            continue
        eo, est, _ = oracle.consensus(i.row_ptr, i.col, i.labels, None if single(j) else i.init,
                                      max_rounds=20)
        assert np.array_equal(outs[j].cpu().numpy(), eo), j
        for key in KEYS:
            assert stats[j][key] == est[key], (j, key)
    # as many as its workgroups hold, whichever kernels solved them
    assert info["solved_in_batch"] == len(items) - 5
