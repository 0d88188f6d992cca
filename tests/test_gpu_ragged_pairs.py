"""bf16 attention where workgroups outnumber the compute units and come in pairs, a long and a short one: the long one keeps more
loads under way.  Every number of its full tiles from none on, partners from empty to nearly as long, grids with and without a
partner for every workgroup."""
import numpy as np
import pytest

from workloads import WORKLOADS, attention_inputs, scaled

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,br,H", [(64, (4, 2), 48), (64, (4, 15), 43), (128, (4, 15), 48), (128, (8, 4), 35), (128, (4, 2), 44)])
def test_pairs(oracle, d, br, H):
    import gpu_helpers as G
    from paper_2409_10644_amd import binding
    lens = (0, 70, 1029, 128, 640, 300, 513, 897, 64, 448)       # 350 to 480 workgroups of one split
    w = scaled(WORKLOADS["cfg2"], B=len(lens), H=H, d=d, branching=br, prefix_min=0, prefix_max=max(lens), cfg_id=133)
    inp = attention_inputs(w, seed=3, lens=lens)
    ad = G.AttnDevice(inp)
    view = binding.slice_mask(binding.build_mask(br), len(br))
    n, mp = view.n_nodes, ad.max_prefix
    want = oracle.tree_attention(inp, oracle.build_mask(br), n)
    tu = binding.AttentionTuning(key_splits=1)
    ws = binding.new_workspace(binding.tree_attention_tuned_workspace(tu, 0, ad.B, H, H, d, n, 0, mp))
    plan = binding.tree_attention_plan(tu, 1, 0, ad.B, H, H, d, n, 0, mp)
    assert plan.ordered_by_length and plan.query_blocks <= 2
    for order in (0, 1):                                         # 1: as they come, without pairs
        tu = binding.AttentionTuning(key_splits=1, natural_order=order)
        ad.out.fill_(float("nan"))
        binding.tree_attention_tuned(tu, view, 1, 0, 1.0, 1.0, ad.B, H, H, d, 0, ad.q, ad.kt, ad.vt, ad.node_stride, ad.kp,
                                     ad.vp, ad.base, ad.lens, ad.head_stride, mp, ad.scale, ad.out, ws)
        got = ad.out[:, :, :n].float().cpu().numpy().astype(np.float64)
        G.assert_close(got, want, "bf16", f"{br} d={d} H={H} order={order}")
