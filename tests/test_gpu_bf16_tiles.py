"""bf16 attention at the edges of its key tiles: no full tile, one, two and three of them, a ragged one of 1 key to one key short
of full, one and two tree tiles, the tree's keys in a workgroup of their own or behind a split's, all query-block counts."""
import numpy as np
import pytest
import torch

from workloads import WORKLOADS, attention_inputs, scaled

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import gpu_helpers
    return gpu_helpers


@pytest.fixture(scope="module")
def binding():
    from paper_2409_10644_amd import binding as b
    return b


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("br", [(1,), (31,), (32,), (4, 15), (64,), (8, 7), (8, 2, 2, 1, 1), (2, 63)])
def test_tile_edges(binding, oracle, H, br, d):
    lens = (0, 1, 63, 64, 65, 127, 128, 129, 192, 255, 257, 400, 513)
    w = scaled(WORKLOADS["cfg2"], B=len(lens), H=3, d=d, branching=br, prefix_min=0, prefix_max=max(lens), cfg_id=131)
    inp = attention_inputs(w, seed=2, lens=lens)
    ad = H.AttnDevice(inp)
    view = binding.slice_mask(binding.build_mask(br), len(br))
    n, mp = view.n_nodes, ad.max_prefix
    want = oracle.tree_attention(inp, oracle.build_mask(br), n)
    for splits, tree_keys in ((0, 0), (1, 0), (2, 1), (3, 2), (5, 3)):
        tu = binding.AttentionTuning(key_splits=splits, tree_keys=tree_keys)
        ws = binding.new_workspace(binding.tree_attention_tuned_workspace(tu, 0, ad.B, 3, 3, d, n, 0, mp))
        ad.out.fill_(float("nan"))
        binding.tree_attention_tuned(tu, view, 1, 0, 1.0, 1.0, ad.B, 3, 3, d, 0, ad.q, ad.kt, ad.vt, ad.node_stride, ad.kp,
                                     ad.vp, ad.base, ad.lens, ad.head_stride, mp, ad.scale, ad.out, ws)
        got = ad.out[:, :, :n].float().cpu().numpy().astype(np.float64)
        H.assert_close(got, want, "bf16", f"{br} d={d} splits={splits} tree_keys={tree_keys}")
