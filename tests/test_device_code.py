"""Properties of the prefill kernels that a run does not show: read off the assembly that the build's compiler and flags
make of them."""
import importlib.util
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NONE = 1 << 30          # no load is under way


def _compile(source, out):
    spec = importlib.util.spec_from_file_location("_amusd_build", os.path.join(ROOT, "paper_2410_17375_amd", "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    r = subprocess.run([build.HIPCC] + build.FLAGS + ["--cuda-device-only", "-S", source, "-o", str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return _kernels(open(out).read())


def _kernels(text):
    """name -> instructions and labels of every kernel."""
    names, out, body = set(re.findall(r"\.amdhsa_kernel (\S+)", text)), {}, None
    for line in text.splitlines():
        m = re.match(r"(\w+):", line)
        if m and m.group(1) in names:
            body = out.setdefault(m.group(1), [])
        elif line.startswith(".Lfunc_end"):
            body = None
        elif body is not None:
            line = line.split(";")[0].strip()
            if line and (not line.startswith(".") or line.startswith(".LBB")):
                body.append(line)
    return out


def _ends_with_load_in_flight(body):
    """Whether some path reaches the end of the program with a vector load that nothing has waited for.  The state is the
    least number of vector-memory instructions issued after the youngest such load (they return in order)."""
    label = {line[:-1]: i for i, line in enumerate(body) if line.endswith(":")}
    state, work = {}, [(0, NONE)]
    while work:
        i, s = work.pop()
        while i < len(body):
            if s >= state.get(i, NONE + 1):
                break
            state[i] = s
            op = body[i]
            if re.match(r"(global|buffer|flat|scratch)_(load|store|atomic)", op):
                s = 0 if "_load" in op.split()[0] else min(NONE, s + 1)
            wait = re.match(r"s_waitcnt .*vmcnt\((\d+)\)", op)
            if wait and int(wait.group(1)) <= s:
                s = NONE
            if op.startswith("s_endpgm"):
                if s < NONE:
                    return True
                break
            jump = re.match(r"s_(c?branch)\w*\s+(\S+)", op)
            if jump:
                work.append((label[jump.group(2)], s))
                if jump.group(1) == "branch":
                    break
            i += 1
    return False


def test_reading_of_the_assembly():
    code = ["global_load_dword v0, v[2:3], off", "s_cbranch_execz .LBB0_1", "s_waitcnt vmcnt(0)", ".LBB0_1:", "s_endpgm"]
    assert _ends_with_load_in_flight(code)
    code[1:1] = ["global_store_dword v[2:3], v1, off", "s_waitcnt vmcnt(1)"]
    assert not _ends_with_load_in_flight(code)
    code[2] = "s_waitcnt vmcnt(2)"
    assert _ends_with_load_in_flight(code)


@pytest.fixture(scope="module")
def prefill(tmp_path_factory):
    return _compile(os.path.join(ROOT, "paper_2410_17375_amd", "csrc", "amusd_prefill.hip"), tmp_path_factory.mktemp("asm") / "prefill.s")


def test_no_wave_ends_with_a_load_in_flight(prefill):
    assert len(prefill) > 50
    assert [k for k, body in prefill.items() if _ends_with_load_in_flight(body)] == []
