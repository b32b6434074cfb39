"""Prompts at the sizes where the prefill pass changes form, against the same tokens in verify passes, bit for bit."""
import pytest

import test_gpu_prefill as prefill

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,over,before,n", [
    # sums of squares of fewer tiles than a row has partial sums (6), of a last round that is not full (46, 290) and of more than the
    # loads in front of the contraction take (290, 528); summed by the streaming form, by a tile's workgroups, by a launch of their own
    ("tiny_verify", {"d_model": 96}, 0, 40), ("tiny_wide_bf16", {"d_model": 736}, 3, 90), ("tiny_wide_bf16", {"d_model": 4640}, 0, 40),
    ("tiny_wide_bf16", {"d_model": 8448, "vocab": 16000}, 0, 1000), ("tiny_wide_fp32", {"d_model": 4640, "vocab": 16000}, 0, 700),
    # 8 column tiles x 2 row tiles: more groups of 4 than compute units
    ("one_layer_8b_width_bf16", {"d_ffn": 14336, "vocab": 16000}, 0, 24),
    # attention over runs of one block, taken in pairs, with an odd one at the end; heads of 64, groups of 4
    ("tiny_gqa_bf16", {"n_q_heads": 8, "n_kv_heads": 2}, 0, 90), ("tiny_gqa_bf16", {"n_q_heads": 8, "n_kv_heads": 2}, 16, 150),
])
def test_prefill_form_equals_short_passes(name, over, before, n):
    prefill.test_prefill_pass_equals_short_passes(name, over, before, n)
