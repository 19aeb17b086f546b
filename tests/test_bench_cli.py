"""bench.py's command line on the CPU: the one-GPU guard answers before any
GPU work, and the help text lists the options the driver and the docs use."""
import json
import os
import shutil
import subprocess
import sys
import types

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _bench(*args, env=None):
    return subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), *args], capture_output=True,
                          text=True, timeout=120, env=env)


def test_more_than_one_gpu_is_refused():
    r = _bench("--gpus", "2")
    assert r.returncode == 2
    assert "exactly one GPU" in r.stderr
    assert r.stdout == ""


def test_distributed_launch_is_refused():
    env = dict(os.environ, WORLD_SIZE="4")
    r = _bench(env=env)
    assert r.returncode == 2
    assert "exactly one GPU" in r.stderr


def test_help_lists_options():
    r = _bench("--help")
    assert r.returncode == 0
    for opt in ("--steps", "--warmup", "--workload", "--no-cpu-baseline", "--remote-fraction", "--splits"):
        assert opt in r.stdout


@pytest.fixture
def bench_copy(tmp_path, monkeypatch):
    """bench.py looking at a copy of the kernel sources, with counters recorded on them."""
    monkeypatch.syspath_prepend(ROOT)
    import bench
    csrc = tmp_path / "paper_2606_22968_amd" / "csrc"
    shutil.copytree(os.path.join(ROOT, "paper_2606_22968_amd", "csrc"), csrc)
    (tmp_path / "profiles").mkdir()
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    rec = {"kernel_sources_sha256": bench.kernel_sources_sha256(), "avg_clock_ghz": 1.8}
    (tmp_path / "profiles" / "chunk_attn_x_counters.json").write_text(json.dumps(rec))
    return bench, csrc


@pytest.mark.parametrize("name,kept", [
    (None, True), ("chunk_attn.hip", False), ("attn_device.h", False), ("chunk_attn_short.hip", False),
    ("internal.h", False), ("kv_append.hip", True),
])
def test_recorded_counters_hold_for_the_sources_they_were_taken_on(bench_copy, name, kept):
    bench, csrc = bench_copy
    if name is not None:
        with open(csrc / name, "a") as f:
            f.write("// changed\n")
    assert (bench.recorded_counters("x") is not None) == kept
    assert bench.recorded_counters("another workload") is None


@pytest.mark.parametrize("h_q,d,lengths,two,want", [
    (32, 128, [2048] * 16, False, "chunk_attn_kernel<128, false>"),
    (32, 128, [2048] * 16, True, "chunk_attn_kernel<128, true>"),
    (32, 128, [2048, 0, 1024], False, "chunk_attn_kernel<128, false> or chunk_attn_short_kernel<128, false>"),
    (32, 128, [1025], False, "chunk_attn_kernel<128, false>"),
    (8, 64, [256] * 4, False, "chunk_attn_kernel<64, false> or chunk_attn_short_kernel<64, false>"),
])
def test_kernels_named_in_the_roofline(monkeypatch, h_q, d, lengths, two, want):
    monkeypatch.syspath_prepend(ROOT)
    import bench
    assert bench.attention_kernels(types.SimpleNamespace(h_q=h_q, head_dim=d), lengths, two, 256) == want
