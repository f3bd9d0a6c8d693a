"""Shared-prefix decode with the chunk that fits one round of waves (between the shortest chunk
and 1,280 keys), which ends neither with the prompts nor with the trajectories' own keys.

Against the fp64 oracle and the log-sum-exp, and against a forced number of splits.
"""
import pytest
import torch

import oracle
import workloads as W
from gpu_harness import DeviceWorkload, assert_close, assert_lse, dev_bf16, log, oracle_pools

CASES = {  # heads, d, group sizes, prompts, own keys
    "g1_groups_of_8": (8, 8, 128, [8] * 8, [2048, 16, 4000, 992, 1008, 0, 2000, 3008],
                       [1 + (997 * i) % 5000 for i in range(64)]),
    "g7_groups_of_16": (28, 4, 64, [16] * 6, [160, 4096, 0, 1280, 1296, 688],
                        [1 + (1499 * i) % 7000 for i in range(96)]),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(CASES))
def test_one_round_chunk_parity(name):
    hq, hkv, d, sizes, prompts, own = CASES[name]
    log("shared decode in one round %s" % name)
    wl = W.custom_group_workload(hq, hkv, d, sizes, [p // 16 * 16 for p in prompts], own, seed=11)
    dw = DeviceWorkload(wl)
    dw.append_extend()
    kp, vp = oracle_pools(wl)
    q = wl.packed("q", wl.extend_ranges())
    ref, ref_lse = oracle.decode(q, kp, vp, wl.block_table, wl.seq_lens, hq, wl.sm_scale)
    for splits in (0, 2):
        lse = torch.empty((q.shape[0], hq), dtype=torch.float32, device="cuda")
        out = dw.kv.decode_shared(dev_bf16(q), wl.seq_lens, wl.group_start, wl.shared_lens,
                                  num_splits=splits, lse=lse)
        assert_close(out, ref, "%s splits=%d" % (name, splits))
        assert_lse(lse, ref_lse, "%s splits=%d" % (name, splits))
