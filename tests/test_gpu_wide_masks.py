"""Slices of masks whose rows are more than two 64-bit words long: the attention of a slice of at most 128 nodes reads its own
words of every row, wherever the full mask's rows end."""
import numpy as np
import pytest
import torch

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


@pytest.mark.parametrize("kind,d,lens", [("bf16", 128, (900, 130)), ("bf16", 64, (70, 300)), ("fp8", 128, (900, 130)), ("fp8", 128, (64, 70)), ("f32", 64, (50, 33))])
@pytest.mark.parametrize("row_begin", [0, 16, 48])                # behind level 1, behind level 2 of 16 + 32 + 64 nodes
def test_levels_of_a_mask_with_long_rows(oracle, row_begin, kind, d, lens):
    import gpu_helpers as H
    from paper_2409_10644_amd import binding
    br, gamma, heads, fp8 = (16, 2, 2, 2), 3, 2, kind == "fp8"
    w = scaled(WORKLOADS["cfg2"], B=2, H=heads, d=d, branching=br, prefix_min=0, prefix_max=max(lens), dtype="f32" if kind == "f32" else "bf16", cfg_id=138)
    inp = attention_inputs(w, seed=4, lens=lens, kv_fp8=(1.0, 1.0) if fp8 else None)
    view = binding.slice_mask(binding.build_mask(br), gamma)
    n = view.n_nodes
    assert view.words_per_row > 2 and n == 112
    want = (oracle.tree_attention_fp8kv if fp8 else oracle.tree_attention)(inp, oracle.build_mask(br), n)
    none = dict(k_prefix=np.zeros(1, np.uint16), v_prefix=np.zeros(1, np.uint16)) if fp8 else {}
    ad = H.AttnDevice(dict(inp, **none))
    if fp8:
        ad.kp, ad.vp = (torch.from_numpy(inp[k]).cuda() for k in ("k_prefix", "v_prefix"))
    ws = binding.new_workspace(binding.tree_attention_tuned_workspace(None, int(fp8), 2, heads, heads, d, n, row_begin, max(lens)))
    ad.out.fill_(float("nan"))
    binding.tree_attention_tuned(None, view, ad.code, int(fp8), 1.0, 1.0, 2, heads, heads, d, row_begin, ad.q, ad.kt, ad.vt, ad.node_stride,
                                 ad.kp, ad.vp, ad.base, ad.lens, ad.head_stride, max(lens), ad.scale, ad.out, ws)
    got = ad.out[:, :, row_begin:n].float().cpu().numpy().astype(np.float64)
    H.assert_close(got, want[:, :, row_begin:], "f32" if kind == "f32" else "bf16", f"{kind} from row {row_begin}")
