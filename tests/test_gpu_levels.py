"""Instances with few clusters, solved level by level: every way of scoring
them (rows of up to 32 and 64 clusters, gathers from LDS and from memory,
tiles of 256 and 1024 vertices, int16 and int32 counts) at the sizes where it
changes, alone with the per-pass trace and in a batch, against the oracle."""
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


def planted(n, k, clusters, labels, seed, hub=False, gap=1):
    """Random graph (a hub joined to every fourth vertex on request), an
    initial partition of exactly min(n, clusters) clusters with ids spread
    over [0, n), and k noisy partitions with `labels` values `gap` apart."""
    rng = np.random.default_rng(seed)
    m = min(n, clusters)
    u, v = rng.integers(0, n, 4 * n), rng.integers(0, n, 4 * n)
    near = rng.random(4 * n) < 0.7
    v[near] = np.minimum(n - 1, u[near] + rng.integers(0, 5, int(near.sum())))
    if hub:
        u = np.concatenate([u, np.zeros(n // 4, np.int64)])
        v = np.concatenate([v, np.arange(n // 4) * 4])
    row_ptr, col = synth.graph.csr_from_edges(n, u, v)
    ids = np.sort(rng.choice(n, m, replace=False))
    base = np.arange(n) * m // n
    noise = rng.random(n) < 0.2
    init = base.copy()
    init[noise] = rng.integers(0, m, int(noise.sum()))
    init[np.unique(base, return_index=True)[1]] = np.arange(m)  # every cluster occurs
    parts = np.tile(base * labels // m, (k, 1))
    noise = rng.random((k, n)) < 0.25
    parts[noise] = rng.integers(0, labels, int(noise.sum()))
    return row_ptr, col, (parts * gap).astype(np.int32), ids[init].astype(np.int32)


def problem(inst):
    rp, col, lab, init = inst
    return {"row_ptr": dev(rp), "col": dev(col), "labels": dev(lab), "init": dev(init)}


def check(out, st, inst, max_rounds=0):
    eo, est, tr = oracle.consensus(*inst, max_rounds=max_rounds, trace=True)
    assert np.array_equal(out.cpu().numpy(), eo)
    for key in KEYS:
        assert st[key] == est[key], key
    return tr


# (n, k, clusters, labels, hub, gap)
SHAPES = [
    (1, 1, 1, 1, False, 1), (2, 3, 2, 1, False, 5), (255, 5, 7, 3, False, 1),
    (256, 4, 31, 9, True, 1), (257, 9, 32, 8, True, 1), (700, 3, 33, 33, True, 1),
    (1500, 6, 64, 20, True, 2), (1500, 7, 65, 20, True, 1), (3000, 5, 96, 96, True, 1),
    (4000, 4, 255, 30, True, 1), (4001, 4, 256, 96, True, 1), (4001, 3, 257, 40, True, 1),
    (16383, 4, 3, 3, False, 1), (16384, 5, 3, 3, False, 1), (32767, 5, 2, 2, False, 1),
    (32768, 5, 2, 2, False, 1), (40000, 3, 60, 50, True, 1), (65536, 2, 40, 30, False, 1),
    (65537, 2, 40, 30, False, 1)]


@pytest.mark.parametrize("n,k,clusters,labels,hub,gap", SHAPES)
def test_alone(mcc, n, k, clusters, labels, hub, gap):
    print(f"[gpu-case] levels alone n={n} k={k} clusters={clusters}", flush=True)
    inst = planted(n, k, clusters, labels, n + clusters, hub, gap)
    p = problem(inst)
    most = 0 if n <= 20000 else 12  # passes
    out, st, tr = mcc.consensus(p["row_ptr"], p["col"], p["labels"], p["init"], trace=True,
                                max_rounds=most)
    assert [tuple(t) for t in check(out, st, inst, most)][:st["passes"]] == tr
    out, st = mcc.consensus(p["row_ptr"], p["col"], p["labels"], p["init"], max_rounds=1)
    check(out, st, inst, max_rounds=1)


def test_together(mcc):
    # all shapes in one call
    print("[gpu-case] levels together, tiles of 256", flush=True)
    insts = [planted(*s[:4], 7 + j, s[4], s[5]) for j, s in enumerate(SHAPES)]
    outs, stats, codes, _ = mcc.consensus_batch([problem(i) for i in insts], max_rounds=3)
    assert all(c == 0 for c in codes)
    for inst, out, st in zip(insts, outs, stats):
        check(out, st, inst, max_rounds=3)


def test_together_large_tiles(mcc):
    # more than 2 x 1024 vertices a compute unit: tiles of 1024, every
    # scoring mode among them; each instance twice
    print("[gpu-case] levels together, tiles of 1024", flush=True)
    insts = [planted(65000, 2, c, 20, c) for c in (20, 200)]
    insts += [planted(30000, 2, c, l, c, True)
              for c, l in ((30, 20), (60, 40), (90, 60), (140, 160), (2, 2))]
    outs, stats, codes, _ = mcc.consensus_batch([problem(i) for i in insts * 2], max_rounds=2)
    assert all(c == 0 for c in codes)
    for j, inst in enumerate(insts):
        check(outs[j], stats[j], inst, max_rounds=2)
        again = j + len(insts)
        assert np.array_equal(outs[j].cpu().numpy(), outs[again].cpu().numpy())
        assert all(stats[j][key] == stats[again][key] for key in KEYS)


def test_fallback_passes(mcc):
    # two equal halves that would swap: the batch does not lower the
    # objective, and only the owners of their clusters move
    print("[gpu-case] levels fallback", flush=True)
    k6 = [(a, b) for a in range(6) for b in range(6) if a != b]
    rp, col = synth.graph.csr_from_edges(6, np.array([a for a, _ in k6]),
                                         np.array([b for _, b in k6]))
    one = (rp, col, np.zeros((3, 6), np.int32), np.array([0, 0, 0, 1, 1, 1], np.int32))
    rng = np.random.default_rng(5)
    ring = np.arange(400)
    rp, col = synth.graph.csr_from_edges(400, ring, (ring + 1) % 400)
    many = (rp, col, np.zeros((5, 400), np.int32), (ring // 2).astype(np.int32))
    swap = (rp, col, rng.integers(0, 2, (4, 400)).astype(np.int32), (ring % 2).astype(np.int32))
    fell = 0
    for inst in (one, many, swap):
        p = problem(inst)
        out, st, tr = mcc.consensus(p["row_ptr"], p["col"], p["labels"], p["init"], trace=True)
        assert [tuple(t) for t in check(out, st, inst)][:st["passes"]] == tr
        fell += st["fallback_rounds"]
    assert fell > 0
    outs, stats, codes, _ = mcc.consensus_batch([problem(i) for i in (one, many, swap)])
    for inst, out, st in zip((one, many, swap), outs, stats):
        check(out, st, inst)
