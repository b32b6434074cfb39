"""The library's host side (allocations, choice of kernels, their grids and arguments) on a stand-in for the HIP runtime: no GPU."""
import importlib.util
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def host_test(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("host")
    spec = importlib.util.spec_from_file_location("_amusd_build", os.path.join(ROOT, "paper_2410_17375_amd", "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    csrc = os.path.join(ROOT, "paper_2410_17375_amd", "csrc")
    objs = []
    # (the test includes amusd_prefill.hip)
    for src in (os.path.join(csrc, "amusd_kernels.hip"), os.path.join(csrc, "amusd_host.hip"), os.path.join(ROOT, "tests", "cpu", "host_test.hip")):
        obj = str(tmp / os.path.basename(src).replace(".hip", ".o"))
        r = subprocess.run([build.HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-fPIC", "-Wno-unused-function", "--offload-host-only",
                            "-c", src, "-o", obj], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        objs.append(obj)
    # device code is not linked in: the stand-in takes no notice of where it would be
    undefined = subprocess.run(["nm", "-u"] + objs, capture_output=True, text=True, check=True).stdout
    absent = ["-Wl,--defsym=%s=0" % name for name in sorted(set(re.findall(r"__hip_fatbin_\w+", undefined)))]
    exe = str(tmp / "host_test")
    r = subprocess.run(["g++", "-no-pie"] + objs + absent + ["-o", exe, "-lpthread"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.mark.parametrize("scenario", ["logits_block", "logits_of_stretches", "shared_sums", "shares_against_measured_times", "timed_stages"])
def test_host_side(host_test, scenario):
    r = subprocess.run([host_test, scenario], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "OK\n", r.stdout + r.stderr


def _attention(host_test, over, max_ctx, lens, rows):
    args = [over["n_q_heads"], over["n_kv_heads"], over["head_dim"], max_ctx] + [x for pair in zip(rows, lens) for x in pair]
    r = subprocess.run([host_test, "form"] + [str(x) for x in args], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout.split()[0]


def test_windows_reach_the_attention_kernels_they_are_meant_for(host_test):
    import test_gpu_attention_heads as heads
    for over, max_ctx, blocks, lens, rows in heads.CASES:
        group = over["n_q_heads"] // over["n_kv_heads"]
        per_head = 256 // (over["n_kv_heads"] * (2 if len(lens) > 1 else 1)) * (8 // group) * 32   # keys of a head, one block a run
        assert blocks == -(-max_ctx // per_head), (over, max_ctx)
        assert _attention(host_test, over, max_ctx, lens, rows) == f"k_attention_g{group}", (over, max_ctx, lens, rows)
        for n in lens:
            assert _attention(host_test, over, max_ctx, (n,) * len(lens), (1,) * len(lens)) == "k_attention_packed", (over, max_ctx, n)
