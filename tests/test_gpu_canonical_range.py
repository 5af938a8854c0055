"""Relabelling of more vertices than one workgroup takes: ids outside [0, n)
are refused wherever they stand, and all others accepted."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [16385, 65537, 1_000_003])
def test_ids(n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2408_11331_amd as mcc
    print(f"[gpu-case] canonical range n={n}", flush=True)
    dev = lambda a: torch.from_numpy(a.astype(np.int32)).cuda()
    rng = np.random.default_rng(n)
    x = rng.integers(0, n, n)
    x[0], x[-1] = n - 1, 0
    out, clusters = mcc.canonicalize(dev(x))
    ids, first = np.unique(x, return_index=True)
    rank = np.empty(ids.size, np.int64)
    rank[np.argsort(first)] = np.arange(ids.size)
    assert clusters == ids.size
    assert np.array_equal(out.cpu().numpy(), rank[np.searchsorted(ids, x)])
    for at in (0, 63, 1024, n // 2, n - 1):
        for bad in (-1, n, 2**31 - 1):
            y = x.copy()
            y[at] = bad
            with pytest.raises(mcc.MccError) as e:
                mcc.canonicalize(dev(y))
            assert e.value.code == mcc.MCC_EINVAL
