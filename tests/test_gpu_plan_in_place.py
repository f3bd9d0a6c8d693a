"""Plans read in place in the staging ring, or copied into the workspace (needs an MI355X).

A small call's kernel reads its work list where it was staged; debug checks keep the copy.
Both must give the same bits, over more calls than the ring has slots.  Under graph capture the
work list goes into the graph, and a captured call must give its bits at every replay.
"""
import numpy as np
import pytest
import torch

import workloads as W
from gpu_harness import DeviceWorkload, dev_bf16

pytestmark = pytest.mark.gpu

CASES = {
    "small": (28, 4, 128, [300, 17, 900, 0], [40, 1, 65, 33]),
    "one_key": (8, 8, 64, [0], [1]),
    "many_tasks": (8, 2, 64, [5 + 3 * i for i in range(90)], [1 + i % 7 for i in range(90)]),
}


@pytest.fixture(params=sorted(CASES))
def case(request):
    hq, hkv, d, prefix, extend = CASES[request.param]
    wl = W.custom_workload(hq, hkv, d, prefix, extend, seed=3)
    dw = DeviceWorkload(wl)
    dw.append_extend()
    q = dev_bf16(wl.packed("q", wl.extend_ranges()))
    last = torch.as_tensor(np.cumsum(wl.extend_lens) - 1, device="cuda")
    k = dev_bf16(wl.packed("k", wl.extend_ranges()))
    v = dev_bf16(wl.packed("v", wl.extend_ranges()))
    return wl, dw.kv, q, q[last].contiguous(), k, v


def bits(*ts):
    return [t.view(torch.int16).clone() for t in ts]


def in_place(kv, call):
    """call()'s result, and whether it left the workspace's header alone: a copied plan begins
    with zeros there, and a plan read in the staging slot does not touch it."""
    head = kv._ws[:256]
    head.fill_(0x5A)
    got = call()
    torch.cuda.synchronize()
    kept = bool((head == 0x5A).all())
    assert kept or not head.any()
    return got, kept


def test_in_place_equals_copied(case, monkeypatch):
    wl, kv, q, qd, k, v = case
    monkeypatch.setenv("TIDE_EXTEND_SPLIT", "0")  # a split plan is always copied
    got = []
    for checks in ("0", "1"):
        monkeypatch.setenv("TIDE_DEBUG_CHECKS", checks)
        for _ in range(20):
            kv.append(k, v, wl.prefix_lens, wl.extend_lens)
            e = kv.extend(q, wl.prefix_lens, wl.extend_lens)
            d = kv.decode(qd, wl.seq_lens)
        got.append(bits(e, d, kv.k_pool, kv.v_pool))
        for call in (lambda: kv.append(k, v, wl.prefix_lens, wl.extend_lens),
                     lambda: kv.extend(q, wl.prefix_lens, wl.extend_lens),
                     lambda: kv.decode(qd, wl.seq_lens)):
            assert in_place(kv, call)[1] == (checks == "0")
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("op, tasks, want", [
    ("append", 512, True), ("append", 513, False),   # one workgroup a page of 4 kv heads
    ("extend", 128, True), ("extend", 129, False),   # one a task and kv head
    ("decode", 512, True), ("decode", 513, False),   # 512 runs of a step; 257 of two steps
])
def test_where_plans_are_read_in_place(op, tasks, want, monkeypatch):
    """The largest calls whose plan at most 512 workgroups read once each, and the next."""
    wl = W.custom_workload(8, 4, 64, [3 + i % 9 for i in range(tasks)], [2] * tasks, seed=tasks)
    kv = DeviceWorkload(wl).kv
    q, k, v = (dev_bf16(wl.packed(x, wl.extend_ranges())) for x in "qkv")
    kv.append(k, v, wl.prefix_lens, wl.extend_lens)
    qd = q[1::2].contiguous()
    call = {"append": lambda: kv.append(k, v, wl.prefix_lens, wl.extend_lens),
            "extend": lambda: kv.extend(q, wl.prefix_lens, wl.extend_lens),
            "decode": lambda: kv.decode(qd, wl.seq_lens)}[op]
    monkeypatch.setenv("TIDE_DEBUG_CHECKS", "0")
    call()  # its workspace is large enough from here on
    out, kept = in_place(kv, call)
    assert kept == want
    pools = bits(kv.k_pool, kv.v_pool)
    monkeypatch.setenv("TIDE_DEBUG_CHECKS", "1")
    other, kept = in_place(kv, call)
    assert not kept
    assert all(torch.equal(a, b) for a, b in zip(pools, bits(kv.k_pool, kv.v_pool)))
    assert out is None or torch.equal(*bits(out, other))


def test_captured_call_replays(case):
    """Every replay gives the captured calls' bits, whatever was called in between: here more
    calls than the ring has slots, of other lengths, before the first replay and after each."""
    wl, kv, q, qd, k, v = case
    hq, hkv, d = wl.spec.num_q_heads, wl.spec.num_kv_heads, wl.spec.head_dim
    n = wl.num_tasks
    owl = W.custom_workload(hq, hkv, d, [40 + 7 * i % 50 for i in range(n)], [2 + i % 3 for i in range(n)], seed=5)
    odw = DeviceWorkload(owl)
    odw.append_extend()
    oq = dev_bf16(owl.packed("q", owl.extend_ranges()))
    oqd = oq[:n].contiguous()

    def others():
        for _ in range(12):
            odw.kv.extend(oq, owl.prefix_lens, owl.extend_lens)
            odw.kv.decode(oqd, owl.seq_lens)
        odw.kv.decode_noalloc(oqd, owl.seq_lens)

    want = bits(kv.extend(q, wl.prefix_lens, wl.extend_lens), kv.decode(qd, wl.seq_lens),
                kv.decode_noalloc(qd, wl.seq_lens, num_splits=2))
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    outs = e, d, dn = torch.empty_like(q), torch.empty_like(qd), torch.empty_like(qd)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        kv.extend(q, wl.prefix_lens, wl.extend_lens, out=e)
        kv.decode(qd, wl.seq_lens, out=d)
        kv.decode_noalloc(qd, wl.seq_lens, num_splits=2, out=dn)
    for _ in range(4):
        others()
        torch.cuda.synchronize()
        for t in outs:
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(bits(*outs), want):
            assert torch.equal(a, b)
        kv.decode(qd, wl.seq_lens)
