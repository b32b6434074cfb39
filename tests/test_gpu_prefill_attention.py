"""Every kernel of a prompt's attention, over runs of several key blocks, against the same tokens in verify passes, bit for bit.
tests/test_plan_cpu.py checks that the sizes reach the kernels that they are meant for."""
import pytest

import test_gpu_prefill as prefill

pytestmark = pytest.mark.gpu

_SMALL = {"d_model": 128, "d_ffn": 128}


def _heads(kv_heads, group, head_dim):
    return dict(_SMALL, n_q_heads=kv_heads * group, n_kv_heads=kv_heads, head_dim=head_dim)


# (shape, overrides, cached before, prompt, blocks a run): keys split into stretches.  Row tiles end after different numbers of a run's
# blocks; odd runs end in a step of one block
SPLIT = [
    ("tiny_gqa_bf16", _heads(16, 4, 64), 980, 24, 2), ("tiny_gqa_bf16", _heads(16, 4, 64), 1920, 104, 3), ("tiny_gqa_bf16", _heads(32, 4, 64), 1941, 71, 5),
    ("tiny_gqa_bf16", _heads(8, 4, 128), 1880, 136, 2), ("tiny_gqa_bf16", _heads(16, 4, 128), 1939, 73, 3),
    ("tiny_gqa_bf16", _heads(8, 8, 64), 920, 72, 2), ("tiny_gqa_bf16", _heads(16, 8, 64), 961, 39, 3), ("tiny_gqa_bf16", _heads(16, 8, 64), 1940, 72, 5),
    ("tiny_gqa_bf16", _heads(8, 8, 128), 960, 40, 2), ("tiny_gqa_bf16", _heads(8, 8, 128), 1880, 136, 3),
    ("tiny_gqa_fp32", _heads(16, 4, 64), 440, 40, 2), ("tiny_gqa_fp32", _heads(16, 4, 64), 899, 105, 3), ("tiny_gqa_fp32", _heads(16, 4, 64), 1920, 104, 5),
    ("tiny_gqa_fp32", _heads(8, 4, 128), 900, 104, 2), ("tiny_gqa_fp32", _heads(32, 4, 128), 920, 72, 5),
    ("tiny_gqa_fp32", _heads(8, 8, 64), 420, 104, 2), ("tiny_gqa_fp32", _heads(8, 8, 64), 900, 104, 3),
    ("tiny_gqa_fp32", _heads(8, 8, 128), 461, 23, 2), ("tiny_gqa_fp32", _heads(8, 8, 128), 960, 40, 3),
]
# .. and walked whole: the kernels that no other test has
WHOLE = [
    ("tiny_gqa_bf16", _heads(8, 8, 128), 0, 200, 1), ("tiny_gqa_bf16", _heads(16, 8, 128), 39, 901, 2), ("tiny_gqa_bf16", _heads(32, 8, 128), 0, 650, 3),
    ("tiny_gqa_fp32", _heads(8, 4, 128), 0, 150, 1), ("tiny_gqa_fp32", _heads(32, 4, 128), 5, 500, 3), ("tiny_gqa_fp32", _heads(8, 8, 128), 0, 150, 1),
    ("tiny_gqa_fp32", _heads(32, 8, 128), 17, 300, 3),
]


@pytest.mark.parametrize("name,over,before,n,blocks", SPLIT + WHOLE)
def test_prompt_attention_equals_short_passes(name, over, before, n, blocks):
    prefill.test_prefill_pass_equals_short_passes(name, over, before, n)
