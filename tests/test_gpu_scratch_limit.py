"""mcc_consensus_noalloc near the limit of its scratch array.  The trace takes
32 bytes a round of the cap, so the cap sets how much of the array is left for
the arrays that a solve can do without (compact label rows, carried-over
candidates, label words, the dense table a singleton start goes on with): from
room for all of them down to none.  A solve is accepted until the array is
full to the last few KiB, and every accepted one gives the same result."""
import ctypes

import numpy as np
import pytest

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
    return m


def dev(a):
    import torch
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()


class Caller:
    """noalloc calls with the trace, the host trace array kept (a cap of
    millions of rounds makes it long)."""

    def __init__(self, mcc, args, flags, most):
        import torch
        self.mcc, self.args, self.flags = mcc, [dev(a) for a in args], flags
        row_ptr, col, labels, init = self.args
        self.n = row_ptr.numel() - 1
        self.out = torch.empty(self.n, dtype=torch.int32, device="cuda")
        self.trace = np.zeros(4 * most, np.int64)
        self.arr = (ctypes.c_void_p * labels.shape[0])(
            *[labels.data_ptr() + 4 * self.n * i for i in range(labels.shape[0])])

    def __call__(self, rounds):
        """(return code, stats, out, the passes' trace)"""
        import torch
        row_ptr, col, labels, init = self.args
        st = self.mcc.Stats()
        st.max_rounds, st.flags = rounds, self.flags | self.mcc.MCC_F_TRACE
        st.stream = torch.cuda.current_stream().cuda_stream
        st.trace = self.trace.ctypes.data
        g = self.mcc.Csr(self.n, col.numel(), row_ptr.data_ptr(), col.data_ptr())
        rc = self.mcc.lib().mcc_consensus_noalloc(
            ctypes.byref(g), self.arr, labels.shape[0],
            init.data_ptr() if init is not None else None, self.out.data_ptr(), ctypes.byref(st))
        return rc, st.as_dict(), self.out.cpu().numpy(), self.trace[:4 * st.passes].copy()


def sweep(mcc, args, flags, caps):
    """Calls with growing caps: accepted, with equal results, up to some cap
    and refused from there on.  Returns the workspace of the accepted ones."""
    call = Caller(mcc, args, flags, max(caps))
    row_ptr, col, labels, init = call.args
    ref, rst, rtr = mcc.consensus(row_ptr, col, labels, init, flags=flags, trace=True)
    rtr = np.array(rtr).ravel()
    held, refused = [], None
    for cap in sorted(caps):
        rc, st, out, tr = call(cap)
        if rc == mcc.MCC_ESCRATCH:
            refused = refused or cap
            continue
        assert rc == 0, rc
        assert refused is None, f"{refused} rounds refused, {cap} accepted"
        assert np.array_equal(out, ref.cpu().numpy())
        assert np.array_equal(tr, rtr)
        for key in KEYS:
            assert st[key] == rst[key], key
        held.append(st["workspace_bytes"])
    assert held and refused
    return held


SCRATCH = 256 << 20


def caps_between(lo, hi, step):
    """Caps whose traces take lo to hi bytes in steps."""
    return [b // 32 for b in range(lo, hi, step)]


def largest_trace(mcc, args, flags):
    """Bytes, to 1 MiB, of the largest trace that is accepted (up to windows
    below it, which a sweep finds)."""
    call = Caller(mcc, args, flags, SCRATCH // 32)
    lo, hi = 0, SCRATCH >> 20
    while hi - lo > 1:  # refused at hi, accepted at lo
        mid = (lo + hi) // 2
        if call((mid << 20) // 32)[0] == 0:
            lo = mid
        else:
            hi = mid
    return (lo + 1) << 20


@pytest.mark.parametrize("flags", ["", "MCC_F_HASH_KEYS", "MCC_F_SYMMETRIC"])
def test_singletons(mcc, flags):
    """Hashed tables: compact rows beside the narrow copy of the clusters
    (2 bytes a vertex), carried-over sets, the dense table of a later pass."""
    print(f"[gpu-case] scratch limit, singletons {flags}", flush=True)
    inst = synth.lfr(n=50_000, k=13)
    bits = getattr(mcc, flags) if flags else 0
    args = (inst.row_ptr, inst.col, inst.labels, None)
    top = largest_trace(mcc, args, bits)
    # the megabytes around the largest trace, then the optional arrays' range
    # (compact rows of 16 to 32 bytes a vertex) around it
    held = sweep(mcc, args, bits, caps_between(top - (6 << 20), top + (1 << 20), 48 << 10) +
                 caps_between(1 << 20, top - (6 << 20), 3 << 20))
    assert max(held) > SCRATCH - (128 << 10)


def test_label_words(mcc):
    """Few clusters and many vertices: label words and slices, then the
    carried-over sets."""
    print("[gpu-case] scratch limit, label words", flush=True)
    n, k, c = (1 << 19) + 5, 30, 40
    rng = np.random.default_rng(2)
    u = rng.integers(0, n, 3 * n)
    rp, col = synth.graph.csr_from_edges(n, u, (u + rng.integers(1, 300, u.size)) % n)
    lab = np.tile(np.arange(n) * c // n, (k, 1))
    noise = rng.random((k, n)) < 0.1
    lab[noise] = rng.integers(0, c, int(noise.sum()))
    args = (rp, col, lab.astype(np.int32), lab[0].astype(np.int32))
    top = largest_trace(mcc, args, mcc.MCC_F_SYMMETRIC)
    held = sweep(mcc, args, mcc.MCC_F_SYMMETRIC,
                 caps_between(max(1 << 15, top - (130 << 20)), top - (2 << 20), 5 << 20) +
                 caps_between(top - (2 << 20), top + (1 << 19), 64 << 10))
    assert max(held) > SCRATCH - (256 << 10)


def test_small_instance(mcc):
    """An instance of the level-by-level kernels whose table of them, with
    labels far apart, is larger than all that the general ones take."""
    print("[gpu-case] scratch limit, few clusters", flush=True)
    rng = np.random.default_rng(4)
    n, k = 2000, 256
    u = rng.integers(0, n, 5 * n)
    rp, col = synth.graph.csr_from_edges(n, u, (u + rng.integers(1, 30, u.size)) % n)
    base = np.arange(n) * 2 // n
    lab = np.where(rng.random((k, n)) < 0.2, rng.integers(0, 2, (k, n)), base) * 6140
    args = (rp, col, lab.astype(np.int32), (rng.random(n) < 0.5).astype(np.int32))
    top = largest_trace(mcc, args, 0)
    # the small table alone takes 256 partitions x 6141 labels x 8 int16 counts
    assert top > SCRATCH - (24 << 20)
    held = sweep(mcc, args, 0, caps_between(top - (24 << 20), top, 1 << 20) +
                 caps_between(top - (1 << 20), top + (1 << 20), 128 << 10))
    assert max(held) > SCRATCH - (256 << 10)
