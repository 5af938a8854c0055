"""The persistent launch of batched solves: what it takes beside instances that
the level-by-level kernels solve."""
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
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()


def problem(inst, init):
    return {"row_ptr": dev(inst.row_ptr), "col": dev(inst.col), "labels": dev(inst.labels),
            "init": dev(init)}


def check(inst, init, out, st, max_rounds=0):
    eo, est, _ = oracle.consensus(inst.row_ptr, inst.col, inst.labels, init,
                                  max_rounds=max_rounds)
    assert np.array_equal(out.cpu().numpy(), eo)
    for key in KEYS:
        assert st[key] == est[key], key


def test_labels_beyond_a_small_instance(mcc):
    """A singleton start whose labels pass 2 n + 1024 beside a large instance
    that the level-by-level kernels solve: the launch's label flags are sized
    for the batch, so it takes the small one all the same."""
    print("[gpu-case] batch: label flags sized for the batch", flush=True)
    large = synth.random_instance(20_000, 50, 6.0, 5, seed=1)
    small = synth.random_instance(300, 1, 6.0, 4, seed=2)
    small.labels[0] = small.labels[0] % 4 * 900
    small.labels[0, 0] = 2999
    items = [(large, large.init), (small, None)]
    outs, stats, codes, info = mcc.consensus_batch([problem(*i) for i in items], max_rounds=9)
    assert codes == [0, 0] and info["solved_in_batch"] == 2
    assert stats[1]["lanes_used"] == 4
    for (inst, init), out, st in zip(items, outs, stats):
        check(inst, init, out, st, 9)


def blocks(n, k, clusters, seed):
    """Ring graph with chords, an initial partition of exactly `clusters`
    clusters and k noisy copies of it."""
    rng = np.random.default_rng(seed)
    v = np.arange(n)
    rp, col = synth.graph.csr_from_edges(n, np.concatenate([v, v, v]), np.concatenate(
        [(v + 1) % n, (v + 5) % n, rng.integers(0, n, n)]))
    base = v * clusters // n
    lab = np.tile(base, (k, 1))
    noise = rng.random((k, n)) < 0.2
    lab[noise] = rng.integers(0, clusters, int(noise.sum()))
    init = base.copy()
    some = rng.random(n) < 0.2
    some[np.unique(base, return_index=True)[1]] = False
    init[some] = rng.integers(0, clusters, int(some.sum()))
    return type("Inst", (), dict(row_ptr=rp, col=col, labels=lab.astype(np.int32), n=n,
                                 init=init.astype(np.int32)))


FORCED = [{"lanes": 8}, {"wg_per_cu": 2}]


@pytest.mark.parametrize("kw", FORCED)
def test_counts_widths(mcc, kw):
    """Counts in int16 below 2^15 vertices and in int32 from there, in one
    launch."""
    print(f"[gpu-case] persistent widths {kw}", flush=True)
    items = [blocks(n, k, c, n) for n, k, c in ((40_000, 3, 20), (700, 9, 6), (32_767, 3, 30),
                                                (32_768, 4, 8))]
    outs, stats, codes, info = mcc.consensus_batch([problem(i, i.init) for i in items],
                                                   max_rounds=4, **kw)
    assert codes == [0] * 4 and info["solved_in_batch"] == 4
    for inst, out, st in zip(items, outs, stats):
        assert st["lanes_used"] > 0
        check(inst, inst.init, out, st, 4)


@pytest.mark.parametrize("kw", FORCED)
def test_fallback_and_errors(mcc, kw):
    """Labels beyond a slot, a negative label, an initial id outside the range
    and more than 256 partitions, found by the launch itself."""
    print(f"[gpu-case] persistent errors {kw}", flush=True)
    items = [synth.random_instance(100 + j, 3, 5.0, 4, seed=7 + j) for j in range(4)]
    items.append(synth.random_instance(40, 300, 4.0, 3, seed=20))
    items[1].labels[1] = items[1].labels[1] * 1_000_003 + 5
    items[2].labels[0, 3] = -1
    items[3].init[7] = items[3].n
    outs, stats, codes, info = mcc.consensus_batch([problem(i, i.init) for i in items],
                                                   max_rounds=50, **kw)
    assert codes == [0, 0, mcc.MCC_EINVAL, mcc.MCC_EINVAL, 0]
    assert info["solved_in_batch"] == 1 and info["rc"] == mcc.MCC_EINVAL
    for j in (0, 1, 4):
        check(items[j], items[j].init, outs[j], stats[j], 50)


def test_tuned(mcc):
    """A tune table shapes the persistent launch: with its workgroups asked
    for, every instance runs with the lanes of its bucket."""
    print("[gpu-case] persistent, tuned", flush=True)
    items = [synth.random_instance(80 + 90 * j, 3 + 7 * (j % 5), 6.0, 5, seed=40 + j)
             for j in range(14)]
    probs = [problem(i, i.init) for i in items]
    table = mcc.batch_tune(probs)
    lanes = {(b["n_log2"], b["k_class"]): b["lanes"] for b in table.as_dict()["buckets"]}
    outs, stats, codes, info = mcc.consensus_batch(probs, tune=table, wg_per_cu=table.wg_per_cu)
    assert codes == [0] * len(items) and info["solved_in_batch"] == len(items)
    for inst, out, st in zip(items, outs, stats):
        k = inst.labels.shape[0]
        kc = 0 if k <= 8 else 1 if k <= 16 else 2 if k <= 32 else 3
        assert st["lanes_used"] == lanes[(inst.n.bit_length() - 1, kc)]
        check(inst, inst.init, out, st)


@pytest.mark.parametrize("kw", FORCED)
def test_packed(mcc, kw):
    print(f"[gpu-case] persistent, packed {kw}", flush=True)
    items = [synth.random_instance(60 + 50 * j, 3 + j, 6.0, 5, seed=80 + j,
                                   init=["p0", "random"][j % 2]) for j in range(12)]
    pb = mcc.pack_batch(items)
    info = mcc.consensus_batch_packed(pb, **kw)
    assert info["rc"] == 0 and info["solved_in_batch"] == len(items)
    for j, inst in enumerate(items):
        st = pb.stats[j].as_dict()
        assert st["lanes_used"] > 0
        check(inst, inst.init, pb.output(j), st)


@pytest.mark.parametrize("n,clusters", [(65_538, 200), (300_000, 257), (1 << 20, 400),
                                        ((1 << 20) + 1, 400)])
def test_large_instances(mcc, n, clusters):
    """Instances whose clusters the level-by-level kernels only count (up to
    2^20 vertices), beside a small one and one with an invalid initial id."""
    print(f"[gpu-case] batch, large instance n={n}", flush=True)
    bad = blocks(70_001, 1, 9, 3)
    bad.init[70_000] = 70_001
    items = [blocks(n, 2, clusters, 5), blocks(900, 4, 9, 4), bad]
    outs, stats, codes, info = mcc.consensus_batch([problem(i, i.init) for i in items],
                                                   max_rounds=2)
    assert codes == [0, 0, mcc.MCC_EINVAL]
    for j in (0, 1):
        check(items[j], items[j].init, outs[j], stats[j], 2)
