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
