"""Attention with an infinite value in the last key of a sequence or of the tree: the rows that see the key get that infinity in
that column and nothing else changes, whatever stands, or is read, behind the last key of a tile that is not full."""
import numpy as np
import pytest
import torch

from workloads import WORKLOADS, attention_inputs, scaled

pytestmark = pytest.mark.gpu

COL = 5


@pytest.fixture(scope="module")
def H():
    import gpu_helpers
    return gpu_helpers


@pytest.fixture(scope="module")
def binding():
    from paper_2409_10644_amd import binding as b
    return b


def _call(binding, tu, view, ad, heads, fp8, ws):
    kp, vp = (ad.kp8, ad.vp8) if fp8 else (ad.kp, ad.vp)
    ad.out.fill_(float("nan"))
    binding.tree_attention_tuned(tu, view, ad.code, fp8, 1.0, 1.0, ad.B, heads, heads, ad.d, 0, ad.q, ad.kt, ad.vt, ad.node_stride, kp, vp,
                                 ad.base, ad.lens, ad.head_stride, ad.max_prefix, ad.scale, ad.out, ws)
    return ad.out[:, :, :view.n_nodes].float().cpu().numpy()


@pytest.mark.parametrize("br", [(3,), (16,), (2, 19), (8, 2, 2, 1, 1)])
@pytest.mark.parametrize("dtype,d,splits,stages", [("f32", 64, 0, 0), ("f32", 128, 3, 0), ("bf16", 64, 1, 0), ("bf16", 128, 0, 0),
                                                   ("bf16", 128, 3, 4), ("fp8", 128, 0, 0), ("fp8", 128, 2, 0)])
def test_infinite_value_in_the_last_key(binding, H, br, dtype, d, splits, stages):
    lens, heads = (1, 15, 50, 64, 77, 129, 200, 383), 2
    w = scaled(WORKLOADS["cfg1" if dtype == "f32" else "cfg2"], B=len(lens), H=heads, d=d, branching=br, prefix_min=0, prefix_max=max(lens), cfg_id=140)
    ad = H.AttnDevice(attention_inputs(w, seed=3, lens=lens))
    view = binding.slice_mask(binding.build_mask(br), len(br))
    n, fp8 = view.n_nodes, int(dtype == "fp8")
    if fp8:
        ad.kp8, ad.vp8 = (t.to(torch.float8_e4m3fn).view(torch.uint8) for t in (ad.kp, ad.vp))
    tu = binding.AttentionTuning(key_splits=splits, stages=stages)
    ws = binding.new_workspace(binding.tree_attention_tuned_workspace(tu, fp8, ad.B, heads, heads, d, n, 0, ad.max_prefix))
    plain = _call(binding, tu, view, ad, heads, fp8, ws)
    others = np.arange(d) != COL
    if not fp8:                                         # (the 8-bit format has no infinity)
        vp = ad.vp.clone()
        flat = ad.vp.view(-1)
        for b, L in enumerate(lens):
            for h in range(heads):
                flat[int(ad.base[b]) + h * ad.head_stride + (L - 1) * d + COL] = float("inf")
        got = _call(binding, tu, view, ad, heads, fp8, ws)
        assert np.all(got[..., COL] == np.inf)
        assert np.array_equal(got[..., others], plain[..., others])
        ad.vp = vp
    ad.vt[:, :, n - 1, COL] = -float("inf")             # seen by the last node alone
    got = _call(binding, tu, view, ad, heads, fp8, ws)
    assert np.all(got[:, :, n - 1, COL] == -np.inf)
    assert np.array_equal(got[..., others], plain[..., others])
