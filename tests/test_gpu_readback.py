"""Results and small host instances that travel through the pinned blocks
(16 KiB each, a pool of 32): at the block's size, just past it, and from
several threads and streams at a time; with every block taken, and after calls
that a stream capture refuses. Compared exactly with the oracle."""
import ctypes
import threading
from types import SimpleNamespace

import numpy as np
import pytest
import torch

import oracle
from paper_2609_13692_amd import mpt
from paper_2609_13692_amd import workloads as wl

pytestmark = pytest.mark.gpu


def instance(m, u, k, seed):
    rng = np.random.default_rng([seed, m, u])
    return wl.from_sets([rng.choice(u, size=k, replace=False).tolist() for _ in range(m)],
                        rng.integers(1, 300, size=u, dtype=np.int64), u)


def check(got, inst):
    ref = oracle.solve(inst)
    assert got["opt"] == ref["opt"]
    assert got["savings"] == int(inst.weights[inst.req_chunks].sum()) - ref["opt"]
    assert np.array_equal(np.asarray(got["orders"]), np.asarray(ref["orders"]))


# orders of 16380, 16384 and 16388 bytes; then host instances around 16 KiB
# (8 (m + 1) + 4 nnz + 8 u, each padded to 256 bytes)
@pytest.mark.parametrize("m,u,k", [(5, 1500, 819), (4, 1500, 1024), (1, 5000, 4097), (7, 1800, 20), (7, 1952, 20),
                                   (7, 2100, 20)])
def test_sizes_around_a_block(m, u, k):
    inst = instance(m, u, k, 1)
    print(f"[gpu] read-back m={m} u={u} nnz={inst.nnz}", flush=True)
    ctx = mpt.Context("cuda")
    check(ctx.run(inst), inst)
    check(ctx.run((inst.m, inst.n_chunks, torch.as_tensor(inst.weights).cuda(), torch.as_tensor(inst.req_off).cuda(),
                   torch.as_tensor(inst.req_chunks).cuda())), inst)
    ctx.close()


def test_threads_and_streams():
    insts = [[instance(4 + t % 5, 60 + 300 * i, 6 + t, 10 * t + i) for i in range(4)] for t in range(8)]
    failed = []

    def work(t):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                ctx = mpt.Context("cuda")
                for _ in range(5):
                    for inst in insts[t]:
                        check(ctx.run(inst), inst)
                        g = mpt.Greedy(inst)
                        out = g.run()
                        assert out["savings"] == int(g.gain[:inst.m - 1].sum())
                ctx.close()
        except BaseException as e:      # reported by the main thread
            failed.append((t, repr(e)))

    threads = [threading.Thread(target=work, args=(t,)) for t in range(len(insts))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed


class Blocks:
    """Takes every block that is left, for as long as it lives (the library's
    own mptlib::HostSlot, a class of one pointer)."""

    def __init__(self):
        lib = mpt.load()
        self._end = lib._ZN6mptlib8HostSlotD1Ev
        self.slots = []
        while True:
            slot = ctypes.c_void_p()
            lib._ZN6mptlib8HostSlotC1EP12ihipStream_t(ctypes.byref(slot), None)
            if not slot.value:
                break
            self.slots.append(slot)

    def close(self):
        for slot in self.slots:
            self._end(ctypes.byref(slot))
        self.slots = []


def everything(inst):
    """The results of one call of every kind that reads something back."""
    ctx, p, g = mpt.Context("cuda"), mpt.Problem(inst), mpt.Greedy(inst)
    out = [mpt.Context.run(ctx, inst), p.run(), p.orders.cpu().numpy(), g.run(), g.orders.cpu().numpy()]
    L = mpt.Layouts(inst, n_configs=2)
    pop = L.global_order(mpt.MPT_ORDER_POPULARITY)
    out += [L.cost(pop), L.simulate(pop, [0, 1], [500, 2000])]
    r = mpt.pinned_layout(inst, 1, "greedy")
    out += [r["orders"].cpu().numpy(), r["cost"], r["n_distinct"]]
    ctx.close()
    return out


def equal(a, b):
    if isinstance(a, dict):
        return a.keys() == b.keys() and all(equal(a[k], b[k]) for k in a)
    if isinstance(a, (list, tuple)):
        return len(a) == len(b) and all(equal(x, y) for x, y in zip(a, b))
    return np.array_equal(a, b)


def test_every_block_taken():
    insts = [instance(9, 60, 4, 2), instance(12, 300, 9, 2), instance(14, 900, 12, 3), instance(5, 20000, 800, 4)]
    want = [everything(inst) for inst in insts]
    held = Blocks()
    try:
        assert held.slots
        for inst, ref in zip(insts, want):
            print(f"[gpu] no blocks left, m={inst.m}", flush=True)
            assert equal(everything(inst), ref)
            check(mpt.Context("cuda").run(inst), inst)
    finally:
        held.close()


def test_refused_captures_keep_the_blocks():
    """A call that returns a host value cannot be captured: it fails, and the
    block it would have used is there for the next one."""
    hip = ctypes.CDLL("libamdhip64.so.7")
    inst = instance(6, 60, 4, 5)
    p = mpt.Problem(inst)
    want = p.run()
    free = Blocks()
    n = len(free.slots)
    free.close()
    torch.cuda.synchronize()
    for i in range(4):
        graph, handle = ctypes.c_void_p(), ctypes.c_void_p()
        assert hip.hipStreamCreate(ctypes.byref(handle)) == 0     # (a stream whose capture failed takes no other)
        assert hip.hipStreamBeginCapture(handle, 2) == 0          # 2: relaxed
        with pytest.raises(mpt.MptError) as e:
            p.solve(stream=SimpleNamespace(cuda_stream=handle.value))
        assert e.value.name == "MPT_E_DEVICE"
        assert hip.hipStreamEndCapture(handle, ctypes.byref(graph)) != 0 and not graph.value
        hip.hipGetLastError()
        assert hip.hipStreamDestroy(handle) == 0
    print("[gpu] captures refused", flush=True)
    assert p.solve() == want
    free = Blocks()
    assert len(free.slots) == n
    free.close()
