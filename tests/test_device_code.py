"""Properties of the kernels that a run does not show: read off the assembly that the build's compiler and flags
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


MIXED_LOADS = """
#include "%s"
extern "C" __global__ void mixed_loads(const char* a, const char* b, float* out) {     // compiled, never run
    extern __shared__ char smem[];
    auto own = [&](int at) {
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(b + at + threadIdx.x * 4),
                                         (__attribute__((address_space(3))) void*)(smem + 4096), 4, 0, 0);
    };
    own(0);
    amusd::load_to_lds(a, threadIdx.x * 16, 0);
    own(4096);
    amusd::wait_vm<0>();
    __syncthreads();
    out[threadIdx.x] = reinterpret_cast<float*>(smem)[threadIdx.x] + reinterpret_cast<float*>(smem + 4096)[threadIdx.x];
}
"""


def test_compiler_sets_m0_again_behind_the_written_out_load(tmp_path):
    """m0 is where a load into LDS delivers to: the compiler's own loads must not go where load_to_lds sent its."""
    src = tmp_path / "mixed.hip"
    src.write_text(MIXED_LOADS % os.path.join(ROOT, "paper_2410_17375_amd", "csrc", "amusd_math.h"))
    ops = [line for line in _compile(str(src), tmp_path / "mixed.s")["mixed_loads"] if re.search(r"\bm0\b|global_load_lds", line)]
    kinds = ["set" if "m0" in op else op.split()[0] for op in ops]
    assert kinds == ["set", "global_load_lds_dword", "set", "global_load_lds_dwordx4", "set", "global_load_lds_dword"], ops


@pytest.fixture(scope="module")
def prefill(tmp_path_factory):
    return _compile(os.path.join(ROOT, "paper_2410_17375_amd", "csrc", "amusd_prefill.hip"), tmp_path_factory.mktemp("asm") / "prefill.s")


def test_no_wave_ends_with_a_load_in_flight(prefill):
    assert len(prefill) > 50
    assert [k for k, body in prefill.items() if _ends_with_load_in_flight(body)] == []


def test_stores_of_a_chunk_are_as_many_as_its_waits_count(prefill):
    """k_pf_attention waits for loads that are older than a chunk's stores by a count that includes those (kStores): with
    one store fewer it would read a block that has not arrived.  It has no other vector-memory instruction in the loop."""
    seen = 0
    for name, body in prefill.items():
        m = re.search(r"14k_pf_attentionI.*ELi(64|128)ELi[48]E", name)
        if not m:
            continue
        seen += 1
        stores = [op.split()[0] for op in body if re.match(r"(global|buffer|flat|scratch)_(store|atomic)", op)]
        assert sorted(stores) == ["global_store_dwordx2"] + ["global_store_dwordx4"] * (int(m.group(1)) // 16), name
        assert not [op for op in body if op.startswith("scratch_")], name
        first = next(i for i, op in enumerate(body) if op.startswith("global_load_lds"))
        later = {op.split()[0] for op in body[first:] if re.match(r"(global|buffer|flat)_load", op)}
        assert later == {"global_load_lds_dwordx4"}, name
    assert seen == 8


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    return _compile(os.path.join(ROOT, "paper_2410_17375_amd", "csrc", "amusd_kernels.hip"), tmp_path_factory.mktemp("asm") / "kernels.s")


def test_one_form_of_attention_per_kernel(kernels):
    """Forms of the attention unit that share a kernel also share the largest one's registers and LDS."""
    forms = {name: {m.group(0) for op in body for m in re.finditer(r"^global_load_lds_dwordx4|^global_load_dwordx4", op)}
             for name, body in kernels.items() if re.search(r"\d+k_attention(_g[48])?I", name)}
    assert len(forms) == 24                    # 3 forms x 2 types x 2 head dims x (one sequence, several)
    for name, loads in forms.items():
        staged = "global_load_lds_dwordx4" in loads
        assert staged == ("k_attention_g" in name), name
    units = {name: sum("ds_write_b128" in op for op in body) for name, body in kernels.items() if name in forms}
    for name, writes in units.items():         # the runs' numerators go to LDS once, in the form's own merge
        assert writes == (8 if "ELi128E" in name else 4), (name, writes)


def test_attention_over_pairs_keeps_its_blocks_in_registers(kernels):
    """k_attention_packed and _whole hold two key blocks, up to 236 of 256 registers where two waves share a SIMD, and ask for the next
    ones under a condition: nothing of it may go to scratch, and no wave may end with a load under way."""
    forms = {name: body for name, body in kernels.items() if re.search(r"\d+k_attention_(packed|whole)I", name)}
    assert len(forms) == 32                    # 2 forms x 2 types x 2 head dims x (one sequence, several) x groups of 4 and 8
    for name, body in forms.items():
        assert not [op for op in body if op.startswith("scratch_")], name
        assert not _ends_with_load_in_flight(body), name


def test_no_kernel_of_a_verify_pass_spills(kernels):
    assert len(kernels) > 90
    assert [name for name, body in kernels.items() if any(op.startswith("scratch_") for op in body)] == []
