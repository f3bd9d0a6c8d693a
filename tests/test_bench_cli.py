"""Host checks of the benchmark's command line (no GPU): the one-GPU contract."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused_with_a_message():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode != 0
    assert "one GPU" in r.stderr
    assert r.stdout.strip() == ""


def test_decode_label_follows_the_plan():
    """The kernel that the benchmark names is the one the library plans (tide_plan_info_get):
    runs, or chunks where the runs would be over 208 steps, from one task to 256."""
    from types import SimpleNamespace

    import numpy as np

    sys.path.insert(0, ROOT)
    import bench

    def label(hq, hkv, d, kv, fused=False):
        spec = SimpleNamespace(num_q_heads=hq, num_kv_heads=hkv, head_dim=d, decode_steps=8 * fused)
        return bench.kernel_label(SimpleNamespace(spec=spec, sm_scale=0.1, seq_lens=np.array(kv, np.int32)),
                                  "decode")

    assert label(32, 8, 128, [5000] * 256) == "decode_stream_kernel<128, false, 8>"
    assert label(8, 2, 64, [100] * 4, fused=True) == "decode_stream_kernel<64, true, 4>"
    assert label(32, 8, 128, [10000] * 256).startswith("decode_split_kernel<128, false, false, 8>")
    assert label(16, 1, 64, [1_000_000]).startswith("decode_stream_kernel")
    assert label(16, 1, 64, [60_000_000]).startswith("decode_split_kernel")


def test_help_lists_the_contract_flags():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--help"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0
    for flag in ("--gpus", "--steps", "--warmup", "--workload", "--cpu-seconds"):
        assert flag in r.stdout
