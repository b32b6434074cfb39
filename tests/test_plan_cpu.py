"""Host-side choices between forms of a stage: against measured times, and what they mean for the sizes that other tests have."""
import ctypes
import os
import shutil
import subprocess

import pytest

from workload import SHAPES

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "cpu", "plan_test.cpp")
CUS = 256


def _compile(flags, out):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no g++")
    r = subprocess.run([gxx, "-std=c++17", "-O1"] + flags + [SRC, "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr


def test_attention_form_against_measured_times(tmp_path):
    exe = str(tmp_path / "plan_test")
    _compile([], exe)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


def test_sizes_reach_the_attention_kernels_they_are_meant_for(tmp_path):
    import test_gpu_prefill_attention as cases
    lib = str(tmp_path / "plan.so")
    _compile(["-shared", "-fPIC"], lib)
    whole_rows = ctypes.CDLL(lib).whole_rows
    for whole, name, over, before, n, blocks in [(0,) + c for c in cases.SPLIT] + [(1,) + c for c in cases.WHOLE]:
        s = SHAPES[name].with_(**over)
        runs, keys = 8 // s.group, 32 if s.dtype == "bf16" else 16             # a chunk's runs, a block's keys
        per_head = CUS // s.n_kv_heads * runs * keys                           # keys of a head, one block a run, on the whole chip
        assert blocks == -(-(before + n + 40) // per_head), (name, over, before, n)   # (models of that test hold 40 tokens more)
        chunk = runs * blocks * keys
        stretch = chunk * max(1, 256 // chunk)
        assert whole == whole_rows(s.dtype == "bf16", s.head_dim, s.group, s.n_kv_heads, n, before + n, CUS, chunk, blocks, stretch), (name, over, before, n)
