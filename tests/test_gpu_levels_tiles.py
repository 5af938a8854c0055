"""Several instances in one call of the level-by-level kernels, with fewer
vertices than take tiles of 1024: tiles of 256 in every scoring mode, the
widest candidate masks and slice buffers beside the narrowest; and the slice
scorer at the most clusters its masks hold beside a label a cluster."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_levels import KEYS, check, dev, planted, problem

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


# rows of 32 and of 64 clusters, gathers from LDS (slices of up to 8 KiB) and
# from memory, one to eight mask words; int16 and int32 counts
SMALL = [(1, 1, 1, 1), (2, 3, 2, 1), (257, 9, 32, 8), (700, 3, 33, 33), (1500, 6, 64, 20),
         (1500, 7, 65, 20), (3000, 5, 96, 40), (4000, 4, 255, 15), (4001, 4, 256, 96),
         (2049, 5, 130, 30), (1023, 3, 200, 100)]
WIDE = [(32768, 2, 60, 30), (32769, 2, 250, 90)]


@pytest.mark.parametrize("shapes", [SMALL, SMALL + WIDE, WIDE])
def test_together_small_tiles(mcc, shapes):
    total = sum(s[0] for s in shapes)
    print(f"[gpu-case] levels together, {total} vertices in tiles of 256", flush=True)
    assert total < 131072  # 1024 vertices for half of 256 compute units
    insts = [planted(*s, 70 + j, s[0] > 300, 1 + j % 2) for j, s in enumerate(shapes)]
    outs, stats, codes, _ = mcc.consensus_batch([problem(i) for i in insts], max_rounds=3)
    assert all(c == 0 for c in codes)
    for inst, out, st in zip(insts, outs, stats):
        check(out, st, inst, max_rounds=3)


@pytest.mark.parametrize("clusters,k", [(64, 3), (65, 6), (66, 2)])
def test_slices_widest_mask(mcc, clusters, k):
    """65 clusters and as many labels are the largest slice that fits with
    three mask words; 66 are scored by tiles."""
    print(f"[gpu-case] slices {clusters} clusters", flush=True)
    n = (1 << 19) + 321
    rng = np.random.default_rng(clusters)
    u = rng.integers(0, n, 5 * n)
    v = np.where(rng.random(5 * n) < 0.3, rng.integers(0, n, 5 * n),
                 (u + rng.integers(1, 900, 5 * n)) % n)
    rp, col = synth.graph.csr_from_edges(n, u, v)
    base = np.arange(n) * clusters // n
    lab = np.tile(base, (k, 1))
    noise = rng.random((k, n)) < 0.25
    lab[noise] = rng.integers(0, clusters, int(noise.sum()))
    init = np.where(rng.random(n) < 0.3, rng.integers(0, clusters, n), base).astype(np.int32)
    lab = lab.astype(np.int32)
    out, st, tr = mcc.consensus(dev(rp), dev(col), dev(lab), dev(init), trace=True, max_rounds=4)
    eo, est, et = oracle.consensus(rp, col, lab, init, trace=True, max_rounds=4)
    assert [tuple(t) for t in et][:st["passes"]] == tr
    assert np.array_equal(out.cpu().numpy(), eo)
    for key in KEYS:
        assert st[key] == est[key], key
