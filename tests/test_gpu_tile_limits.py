"""The tiled scorer on both sides of the size where few clusters take tiles of
256 vertices, with the candidates carried over or not, against the oracle."""
import numpy as np
import pytest

import oracle
from test_gpu_tiles import KEYS, dev, planted

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [5 << 15, (5 << 15) + 1])
@pytest.mark.parametrize("groups,symmetric", [(60, True), (256, False), (257, False)])
def test_few_clusters(n, groups, symmetric):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2408_11331_amd as mcc
    oracle.build(force=False)
    print(f"[gpu-case] tile limits n={n} groups={groups}", flush=True)
    row_ptr, col, labels = planted(n, 3, groups, n + groups)
    init = labels[0].copy()
    out, st = mcc.consensus(dev(row_ptr), dev(col), dev(labels), dev(init), max_rounds=5,
                            flags=mcc.MCC_F_SYMMETRIC if symmetric else 0)
    eo, est, _ = oracle.consensus(row_ptr, col, labels, init, max_rounds=5)
    assert np.array_equal(out.cpu().numpy(), eo)
    for key in KEYS:
        assert st[key] == est[key], key
