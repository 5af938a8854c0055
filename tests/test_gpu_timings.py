"""Times in the statistics: the pass loop is a part of the call, the scoring a
part of the pass loop, and asking for the scoring's time does not change which
kernels a solve runs."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mcc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2408_11331_amd as m
    m.lib()
    return m


def dev(a):
    import torch
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("kind", ["small", "small, falls back", "general", "singletons"])
def test_times(mcc, kind):
    print(f"[gpu-case] timings {kind}", flush=True)
    inst = {"small": lambda: synth.sbm_small(),
            "small, falls back": lambda: synth.random_instance(2000, 5, 6.0, 8, seed=3,
                                                               init="random"),
            "general": lambda: synth.lfr(n=20_000, k=8),
            "singletons": lambda: synth.sbm_small()}[kind]()
    if kind == "small, falls back":
        inst.init = (inst.init % 16).astype(np.int32)
    args = [dev(inst.row_ptr), dev(inst.col), dev(inst.labels),
            None if kind == "singletons" else dev(inst.init)]
    for flags in (0, mcc.MCC_F_PROFILE):
        mcc.consensus(*args, flags=flags)
    _, plain = mcc.consensus(*args)
    _, st = mcc.consensus(*args, flags=mcc.MCC_F_PROFILE)
    assert plain["ms_score"] == 0
    assert 0 < plain["ms_passes"] < plain["ms_total"]
    assert 0 < st["ms_score"] < st["ms_passes"] < st["ms_total"]
    # the kernels are the same: so is the workspace, and the layout of the tables
    assert st["workspace_bytes"] == plain["workspace_bytes"] and st["tables"] == plain["tables"]
