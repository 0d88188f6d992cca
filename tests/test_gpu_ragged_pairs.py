"""bf16 attention where workgroups outnumber the compute units and come in pairs, a long and a short one: the long one keeps more
loads under way.  Partners from empty to nearly as long and grids with and without a partner for every workgroup; every number of
full tiles from none to six, with and without a last one that is not full, in workgroups without a partner; query heads
that share keys, and the newest levels alone."""
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


@pytest.mark.parametrize("d,br,Hq,Hkv,row_begin", [(64, (4, 2), 26, 26, 0), (64, (4, 15), 26, 26, 0), (128, (4, 15), 26, 26, 0),
                                                   (64, (4, 2), 27, 9, 4), (64, (4, 15), 24, 8, 4), (128, (4, 15), 27, 9, 4), (128, (4, 15), 24, 8, 0),
                                                   (128, (4, 2), 48, 8, 4), (128, (4, 15), 26, 26, 4)])
def test_every_number_of_full_tiles(oracle, d, br, Hq, Hkv, row_begin):
    import gpu_helpers as G
    from paper_2409_10644_amd import binding
    grp, rows = Hq // Hkv, 4 * (1 + br[1]) - row_begin
    T = 128 if rows <= 32 and grp != 6 else 64                   # one query block or two (of two heads)
    lens = (0, T // 2, T, T + 9, 2 * T, 3 * T + 5, 4 * T, 5 * T + 1, 6 * T, 7 * T - 1, 2 * T - 3)     # 264 to 297 workgroups
    B, mp = len(lens), max(lens)
    w = scaled(WORKLOADS["cfg2"], B=B, H=Hq, d=d, branching=br, prefix_min=0, prefix_max=mp, cfg_id=134)
    qi, ki = attention_inputs(w, seed=3, lens=lens), attention_inputs(scaled(w, H=Hkv, cfg_id=135), seed=3, lens=lens)
    rep = dict(qi, **{k: np.repeat(ki[k], grp, axis=1) for k in ("k_tree", "v_tree", "k_prefix", "v_prefix")})
    aq, ak = G.AttnDevice(qi), G.AttnDevice(ki)
    view = binding.slice_mask(binding.build_mask(br), len(br))
    n = view.n_nodes
    tu = binding.AttentionTuning(key_splits=1)
    plan = binding.tree_attention_plan(tu, 1, 0, B, Hq, Hkv, d, n, row_begin, mp)
    assert plan.ordered_by_length and plan.key_splits == 1 and T == (128 if plan.query_blocks == 1 else 64)
    assert 256 < plan.workgroups <= 2 * 256                      # most have a compute unit to themselves, the longest share it with the shortest
    aq.out.fill_(float("nan"))
    binding.tree_attention_tuned(tu, view, 1, 0, 1.0, 1.0, B, Hq, Hkv, d, row_begin, aq.q, ak.kt, ak.vt, ak.node_stride, ak.kp, ak.vp,
                                 ak.base, ak.lens, ak.head_stride, mp, aq.scale, aq.out, None)
    got = aq.out[:, :, row_begin:n].float().cpu().numpy().astype(np.float64)
    G.assert_close(got, oracle.tree_attention(rep, oracle.build_mask(br), n)[:, :, row_begin:], "bf16", f"{br} d={d} {Hq}/{Hkv}")
