"""Stages whose K slices are workgroups of their own and are added up by a launch of its own, against the same tokens in verify passes,
bit for bit: the down projection of one row group (33 to 64 rows, 65 to 128) in 16 slices, and at its edges; few column tiles of a long
contraction in 8 (O-projection, gate/up, LM head); a down projection of middling width in 2, 8 and 16 (float32)."""
import pytest

import test_gpu_prefill as prefill

pytestmark = pytest.mark.gpu

LONG = {"d_model": 8192, "d_ffn": 64, "vocab": 512}


@pytest.mark.parametrize("name,over,before,n", [
    ("one_layer_8b_width_bf16", {"vocab": 1024}, 0, 32), ("one_layer_8b_width_bf16", {"vocab": 1024}, 0, 33), ("one_layer_8b_width_bf16", {"vocab": 1024}, 5, 64),
    ("one_layer_8b_width_bf16", {"vocab": 1024}, 0, 65), ("one_layer_8b_width_bf16", {"vocab": 1024}, 0, 128), ("one_layer_8b_width_bf16", {"vocab": 1024}, 0, 129),
    ("tiny_wide_bf16", {"d_model": 2048, "vocab": 512}, 0, 49), ("tiny_wide_fp32", {"d_model": 2048, "vocab": 512}, 0, 49),
    ("tiny_gqa_bf16", LONG, 0, 90), ("tiny_gqa_fp32", LONG, 2, 150),
    ("tiny_gqa_bf16", {"d_model": 96, "n_q_heads": 64, "n_kv_heads": 16, "d_ffn": 96, "vocab": 512}, 0, 300),
    ("tiny_gqa_bf16", {"n_layers": 1, "d_model": 1024, "d_ffn": 4096, "vocab": 512}, 3, 577), ("tiny_gqa_bf16", {"n_layers": 1, "d_model": 3072, "d_ffn": 8192, "vocab": 512}, 0, 330),
    ("tiny_gqa_fp32", {"n_layers": 1, "d_model": 2048, "d_ffn": 8192, "vocab": 512}, 0, 270),
])
def test_slices_equal_short_passes(name, over, before, n):
    prefill.test_prefill_pass_equals_short_passes(name, over, before, n)
