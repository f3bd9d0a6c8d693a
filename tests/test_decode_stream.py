"""Decode with the library's own split: equal runs of key steps per wave.

CPU: stream_check.cpp walks the plan's runs and checks parts, slots and arrival counts.
GPU: against the fp64 oracle where runs and units meet in every way: one step per wave, units
that end on a run's last step, several units in a run, units over several workgroups, the
smallest call, both workgroup sizes, G over 8; and the fused append against append + decode,
bit for bit, over slots at both ends of a page and a step.
"""
import os
import subprocess

import numpy as np
import pytest
import torch

import oracle
import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_10402_amd", "csrc")


def test_runs_cover_the_call(tmp_path):
    exe = str(tmp_path / "stream_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, "-I",
                    os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "stream_check.cpp"),
                    os.path.join(CSRC, "plan.cpp"), "-o", exe], check=True)
    rng = np.random.default_rng(9)
    lines = []
    for _ in range(200):
        hq, hkv = [(28, 4), (32, 8), (8, 8), (16, 1), (64, 8), (12, 4)][rng.integers(6)]
        n = int(rng.choice([1, 2, 5, 64, 300]))
        kv = rng.integers(1, int(rng.choice([33, 400, 8000, 90000])), n)
        lines.append((hq, hkv, int(rng.choice([64, 128])), kv))
    lines += [(16, 1, 64, [1]), (8, 8, 128, [32] * 256), (8, 8, 128, [64] * 256),
              (32, 8, 128, [4096] * 16), (32, 8, 128, [5] * 4096), (16, 1, 64, [2_000_000])]
    text = "".join("%d %d %d %d %s\n" % (*x[:3], len(x[3]), " ".join(map(str, x[3]))) for x in lines)
    r = subprocess.run([exe], input=text, capture_output=True, text=True)
    out = r.stdout.strip().split("\n")
    assert r.returncode == 0 and len(out) == len(lines) and all(o.startswith("ok") for o in out), r.stdout[-500:]


@pytest.mark.parametrize("heads, kv", [((65536, 4096, 128), [28]), ((114452, 8804, 128), [900]),
                                       ((214592, 53648, 64), [21]), ((30720, 1920, 128), [2000] * 3)])
def test_one_run_needs_no_partials(heads, kv):
    """Over 1,024 kv heads make one run of the whole call, which cuts no task: the call needs the
    plan's bytes and fits the static scratch of tide_decode_attn_noalloc at any head count."""
    import paper_2608_10402_amd as tide
    dims = tide.make_dims(*heads, 0.1)
    size = tide.tide_workspace_size(tide.TIDE_OP_DECODE, np.array(kv, np.int32), None, dims)
    assert size <= 2048


def test_no_scratch_access_inside_loops(tmp_path):
    """A spill reload inside the step loop would wait for every K/V load in flight."""
    from test_codegen import _asm, loops_with_scratch
    found = loops_with_scratch(_asm(tmp_path, "attn_decode_stream.hip"))
    assert found and not [x for x in found if x[2]]


GPU_CASES = {
    "one_key": (16, 1, 64, [1]),
    "one_run_many_heads": (1100, 1100, 64, [5, 40, 16]),
    "page_and_step_ends": (28, 4, 128, [1, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65]),
    "several_units_a_run": (8, 8, 128, [17 + 5 * (i % 9) for i in range(400)]),
    "units_end_with_runs": (8, 8, 128, [64 * 32] * 16),   # 8192 steps: 4 a wave, 16 waves a unit
    "long_alone": (32, 2, 64, [20011]),
    "g16_d128": (16, 1, 128, [5000, 77, 3111]),
    "mixed": (12, 4, 64, [9000, 3, 700, 33, 4096, 2049]),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(GPU_CASES))
def test_decode_parity(name):
    from gpu_harness import DeviceWorkload, assert_close, assert_lse, dev_bf16, log, oracle_pools
    hq, hkv, d, kv = GPU_CASES[name]
    wl = W.custom_workload(hq, hkv, d, [x - 1 for x in kv], [1] * len(kv), seed=len(name))
    log("decode runs %s" % name)
    dw = DeviceWorkload(wl)
    q = dev_bf16(wl.packed("q", wl.extend_ranges()))
    k = dev_bf16(wl.packed("k", wl.extend_ranges()))
    v = dev_bf16(wl.packed("v", wl.extend_ranges()))
    lse = torch.empty((len(kv), hq), dtype=torch.float32, device="cuda")
    fused = dw.kv.decode_append(q, k, v, wl.seq_lens, lse=lse)
    pools = dw.kv.k_pool.clone(), dw.kv.v_pool.clone()
    other = DeviceWorkload(wl)
    other.append_extend()
    lse2 = torch.empty_like(lse)
    out = other.kv.decode(q, wl.seq_lens, lse=lse2)
    torch.cuda.synchronize()
    kp, vp = oracle_pools(wl)
    ref, ref_lse = oracle.decode(wl.packed("q", wl.extend_ranges()), kp, vp, wl.block_table,
                                 wl.seq_lens, hq, wl.sm_scale)
    assert_close(out, ref, name)
    assert_lse(lse2, ref_lse, name)
    assert torch.equal(out.view(torch.int16), fused.view(torch.int16)) and torch.equal(lse, lse2)
    for a, b in zip(pools, (other.kv.k_pool, other.kv.v_pool)):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    again = other.kv.decode(q, wl.seq_lens)
    assert torch.equal(again.view(torch.int16), out.view(torch.int16))
