"""Slices of masks whose rows are more than two 64-bit words long: the attention of a slice of at most 128 nodes reads its own
words of every row, wherever the full mask's rows end."""
import numpy as np
import pytest

from workloads import WORKLOADS, attention_inputs, scaled

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,lens", [("bf16", 128, (130, 70)), ("bf16", 64, (700, 0)), ("bf16", 128, (900, 1024)), ("f32", 64, (50, 33))])
@pytest.mark.parametrize("br,gamma", [((16, 2, 2, 2), 3), ((10, 2, 2, 2, 2), 3)])      # 112 of 240 nodes, 70 of 310
def test_slice_of_a_mask_with_long_rows(oracle, br, gamma, dtype, d, lens):
    import gpu_helpers as H
    from paper_2409_10644_amd import binding
    w = scaled(WORKLOADS["cfg2"], B=2, H=2, d=d, branching=br, prefix_min=0, prefix_max=max(lens), dtype=dtype, cfg_id=137)
    inp = attention_inputs(w, seed=4, lens=lens)
    view = binding.slice_mask(binding.build_mask(br), gamma)
    assert view.words_per_row > 2 and 64 < view.n_nodes <= 128
    got = H.run_attention(binding, view, H.AttnDevice(inp), fill=float("nan"))
    H.assert_close(got, oracle.tree_attention(inp, oracle.build_mask(br), view.n_nodes), dtype, f"{br} gamma {gamma}")
