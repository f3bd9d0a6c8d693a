"""Plans read in place in the staging ring, or copied into the workspace (needs an MI355X).

A small call's kernel reads its work list where it was staged; debug checks and graph capture
keep the copy.  Both must give the same bits, over more calls than the ring has slots, and a
captured call must give them at every replay.
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


def test_in_place_equals_copied(case, monkeypatch):
    wl, kv, q, qd, k, v = case
    got = []
    for checks in ("0", "1"):
        monkeypatch.setenv("TIDE_DEBUG_CHECKS", checks)
        for _ in range(20):
            kv.append(k, v, wl.prefix_lens, wl.extend_lens)
            e = kv.extend(q, wl.prefix_lens, wl.extend_lens)
            d = kv.decode(qd, wl.seq_lens)
        got.append(bits(e, d, kv.k_pool, kv.v_pool))
    for a, b in zip(*got):
        assert torch.equal(a, b)


def test_captured_call_replays(case):
    wl, kv, q, qd, k, v = case
    want = bits(kv.extend(q, wl.prefix_lens, wl.extend_lens), kv.decode(qd, wl.seq_lens))
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    e, d = torch.empty_like(q), torch.empty_like(qd)
    with torch.cuda.stream(side):
        kv.extend(q, wl.prefix_lens, wl.extend_lens, out=e)
        kv.decode(qd, wl.seq_lens, out=d)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        kv.extend(q, wl.prefix_lens, wl.extend_lens, out=e)
        kv.decode(qd, wl.seq_lens, out=d)
    for _ in range(4):
        e.zero_()
        d.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(bits(e, d), want):
            assert torch.equal(a, b)
        kv.decode(qd, wl.seq_lens)  # eager work between the replays
        torch.cuda.synchronize()
