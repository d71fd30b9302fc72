"""bench.py's command-line contract, checked without a GPU, and what its timed steps run."""
import json
import os
import subprocess
import sys

import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(*args):
    return subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), *args], capture_output=True, text=True,
                          timeout=120, cwd=ROOT)


def test_more_than_one_gpu_exits_with_a_message():
    r = _run("--gpus", "2", "--steps", "1", "--warmup", "0")
    assert r.returncode != 0
    assert "one GPU" in r.stderr and r.stdout.strip() == ""


def test_help_lists_the_contract_flags():
    r = _run("--help")
    assert r.returncode == 0
    for flag in ("--gpus", "--steps", "--warmup", "--workload", "--mode"):
        assert flag in r.stdout


def test_block_delivery_modes_need_a_shard():
    for mode in ("ring", "gather"):
        r = _run("--workload", "c3", "--mode", mode, "--steps", "1", "--warmup", "0", "--no-cpu-baseline")
        assert r.returncode == 2
        assert "no shard segments" in r.stderr and r.stdout.strip() == ""


@pytest.mark.gpu
@pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")
def test_timed_steps_run_unprofiled(monkeypatch, capsys):
    """The warm-up and the timed steps run as any caller's do; only a later pass is profiled."""
    import bench
    from paper_2608_01150_amd import api
    on, calls = [False], []
    enable, bwd = api.profile_enable, api.attn_bwd
    monkeypatch.setattr(api, "profile_enable", lambda x: (on.__setitem__(0, bool(x)), enable(x))[1])
    monkeypatch.setattr(api, "attn_bwd", lambda *a, **k: (calls.append(on[0]), bwd(*a, **k))[1])
    monkeypatch.setattr(sys, "argv", ["bench.py", "--workload", "c2", "--steps", "3", "--warmup", "2", "--merge-reps", "0",
                                      "--no-ceiling", "--no-cpu-baseline"])
    bench.main()
    rec = json.loads(capsys.readouterr().out.splitlines()[-1])
    assert calls == [False] * 5 + [True] * 3
    assert rec["steps"] == 3 and rec["ms_per_step"] > 0
    assert rec["kernel_ms"]["bwd_dkdv"] > 0 and rec["kernel_ms"]["bwd_dq"] > 0
