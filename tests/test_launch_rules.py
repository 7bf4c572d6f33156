"""The host-side launch rules of csrc/common.h and csrc/gemv_tiles.h, checked
without a GPU (built with g++ against the HIP headers), and the spread slice counters of the
plan-free forward where they just fit its scratch array and where they do not."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"),
                    reason="needs g++ and the HIP headers")
@pytest.mark.parametrize("check", ["launch_rules_check", "gemv_tiles_check"])
def test_launch_rules(check, tmp_path):
    exe = tmp_path / check
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "paper_2305_06942_amd", "csrc"), "-I" + os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", check + ".cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "bad=0" in r.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("n_flags", [1024, 1025, 65536])
def test_noalloc_counters_at_scratch_limits(n_flags):
    import torch
    import oracle
    import paper_2305_06942_amd as ebag
    import synth
    from synth import device as sdev
    from tests.gpu_util import check_full, flags_np, say
    w = synth.scaled(synth.TINY, rows=50, B=n_flags, T=2, R=1, C=1).with_(lengths="uniform:0:2")
    inp = synth.make_inputs(w)
    say("noalloc counters", n_flags)
    dev = sdev.to_device(inp)
    send = torch.full((w.B, w.sum_dim), float("nan"), device="cuda")
    flags = torch.zeros(n_flags, dtype=torch.int32, device="cuda")
    for _ in range(2):  # the second call finds what the first left in the counters
        ebag.forward_noalloc(w.rows, w.dims, w.dtype, w.C, dev.tables, dev.indices, dev.offsets, None, w.B, w.R, send,
                             flags)
    torch.cuda.synchronize()
    assert np.all(flags_np(flags) == 2)
    check_full(inp, send.cpu().numpy())
