"""Workspace of batched calls: what admission is told (host only), and that the
calls keep to it whichever kernels take their instances."""
import ctypes

import numpy as np
import pytest

import oracle
import synth


def mcc_module():
    import paper_2408_11331_amd as m
    m.lib()
    return m


def told(m, specs):
    """mcc_batch_workspace_bytes for instances of (vertices, partitions)."""
    arr = (m.Problem * len(specs))()
    for j, (n, k) in enumerate(specs):
        arr[j].g = m.Csr(n, 20 * n, None, None)
        arr[j].k = k
    opts, out = m.BatchOpts(), ctypes.c_int64(0)
    assert m.lib().mcc_batch_workspace_bytes(arr, len(specs), ctypes.byref(opts),
                                             ctypes.byref(out)) == 0
    return out.value


@pytest.mark.parametrize("specs", [[(20, 3)], [(1000, 10)], [(200, 8)] * 10, [(200, 64)] * 10,
                                   [(5000, 3)] * 3, [(50_000, 8)] * 3])
def test_told_follows_the_instances(specs):
    """Twice a slot of the persistent launch for each (five int32 and two int64
    arrays over the vertices, the label rows, flags, 2^18 cells at least) and a
    chunk of 16 MiB, a few KiB for the rest."""
    m = mcc_module()
    n, k = max(s[0] for s in specs), max(s[1] for s in specs)
    slot = 4 * (n * (4 + 4 + k + 2) + 1024 + max(n * k, 1 << 18))
    want = 2 * len(specs) * slot + (16 << 20)
    assert want <= told(m, specs) <= want + (64 << 10)


def dev(a):
    import torch
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()


def wide_table(seed):
    inst = synth.random_instance(150, 40, 6.0, 42, seed=seed, init="random")
    inst.init = np.random.default_rng(seed).permutation(150).astype(np.int32)
    return inst


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["tiny", "few clusters", "tables", "one table", "alone",
                                  "large alone", "mixed"])
def test_calls_keep_to_it(kind):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m = mcc_module()
    oracle.build(force=False)
    print(f"[gpu-case] batch workspace, {kind}", flush=True)
    few = [synth.random_instance(900 + 50 * j, 7, 6.0, 6, seed=j) for j in range(12)]
    items = {
        "tiny": [synth.random_instance(30 + j % 9, 6, 4.0, 3, seed=j) for j in range(40)],
        "few clusters": few,
        "tables": [wide_table(j) for j in range(9)],  # more than a wave's budget
        "one table": [wide_table(3)],
        "alone": [synth.lfr(n=15_000, k=4 + j) for j in range(3)],
        "large alone": [synth.lfr(n=80_000, k=5)],
        "mixed": few + [wide_table(1), synth.lfr(n=15_000, k=4),
                        synth.random_instance(2000, 5, 6.0, 6, seed=5, init="singleton")],
    }[kind]
    probs = [{"row_ptr": dev(i.row_ptr), "col": dev(i.col), "labels": dev(i.labels),
              "init": dev(i.init)} for i in items]
    bytes_told = m.batch_workspace_bytes(probs)
    m.release_workspace()
    outs, stats, codes, info = m.consensus_batch(probs, max_rounds=12)
    assert all(c == 0 for c in codes)
    # (tables beyond a slot are not foreseen; these are counted as solved there)
    if info["solved_in_batch"] == len(items) or kind in ("tables", "one table"):
        assert info["workspace_bytes"] <= bytes_told, (info, bytes_told)
    for inst, out, st in zip(items, outs, stats):
        eo, est, _ = oracle.consensus(inst.row_ptr, inst.col, inst.labels, inst.init,
                                      max_rounds=12)
        assert np.array_equal(out.cpu().numpy(), eo)
        assert st["objective"] == est["objective"] and st["passes"] == est["passes"]
