"""Small instances with few clusters whose passes fall back: a random initial
partition, from which whole batches do not lower the objective.  The whole
trace against the oracle for int16 and int32 counts, for two and for 256
clusters (proposals that are few against a slice among them), alone and in a
batch where some instances fall back and others do not; and the time of such a
solve against the general kernels."""
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


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def random_start(n, k, clusters, labels, seed=3):
    rng = np.random.default_rng(seed)
    u = np.repeat(np.arange(n), 8)
    v = (u + rng.integers(1, 50, u.size)) % n
    rp, col = synth.graph.csr_from_edges(n, u, v)
    lab = np.tile(np.arange(n) * labels // n, (k, 1))
    noise = rng.random((k, n)) < 0.3
    lab[noise] = rng.integers(0, labels, int(noise.sum()))
    return rp, col, lab.astype(np.int32), rng.integers(0, clusters, n).astype(np.int32)


def problem(inst):
    return dict(zip(("row_ptr", "col", "labels", "init"), map(dev, inst)))


SHAPES = [(300, 5, 2, 1), (5000, 7, 40, 40), (3000, 3, 256, 96), (32767, 4, 30, 30),
          (32768, 4, 30, 30), (65536, 2, 250, 90)]


@pytest.mark.parametrize("n,k,clusters,labels", SHAPES)
def test_trace(mcc, n, k, clusters, labels):
    print(f"[gpu-case] levels fall back n={n} k={k} clusters={clusters}", flush=True)
    inst = random_start(n, k, clusters, labels)
    p = problem(inst)
    for most in (1, 6):
        out, st, tr = mcc.consensus(p["row_ptr"], p["col"], p["labels"], p["init"], trace=True,
                                    max_rounds=most)
        eo, est, et = oracle.consensus(*inst, max_rounds=most, trace=True)
        assert [tuple(t) for t in et][:st["passes"]] == tr
        assert np.array_equal(out.cpu().numpy(), eo)
        for key in KEYS:
            assert st[key] == est[key], key
    if clusters > 2:
        assert st["fallback_rounds"] > 0


def test_batch(mcc):
    print("[gpu-case] levels fall back, in a batch", flush=True)
    insts = [random_start(*s, seed=9 + j) for j, s in enumerate(SHAPES)]
    planted = synth.sbm_small()
    insts += [(planted.row_ptr, planted.col, planted.labels, planted.init)] * 2
    outs, stats, codes, _ = mcc.consensus_batch([problem(i) for i in insts], max_rounds=7)
    assert all(c == 0 for c in codes)
    for inst, out, st in zip(insts, outs, stats):
        eo, est, _ = oracle.consensus(*inst, max_rounds=7)
        assert np.array_equal(out.cpu().numpy(), eo)
        for key in KEYS:
            assert st[key] == est[key], key


def test_time(mcc):
    """20 000 vertices and 256 partitions, every pass falls back: no slower
    than twice the general kernels (lanes=16 takes those)."""
    import torch
    print("[gpu-case] levels fall back, time", flush=True)
    p = problem(random_start(20000, 256, 20, 20))

    def best(**kw):
        t = []
        for _ in range(4):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            out, st = mcc.consensus(p["row_ptr"], p["col"], p["labels"], p["init"], max_rounds=10,
                                    **kw)
            t.append(time.perf_counter() - t0)
        assert st["fallback_rounds"] == 10
        return min(t), out

    mine, out = best()
    general, ref = best(lanes=16)
    assert torch.equal(out, ref)
    assert mine < 2 * general, (mine, general)
