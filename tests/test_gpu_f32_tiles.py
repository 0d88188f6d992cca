"""fp32 attention at the edges of its tiles: 16 query rows, 16-key blocks of the prefix and of the tree, four wavefronts, key
splits folded inside the kernel and by the second kernel, first rows inside a tile, grouped-query heads."""
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


def _check(binding, oracle, H, br, heads, d, lens, row0=0, tuning=None, cfg_id=130):
    w = scaled(WORKLOADS["cfg1"], B=len(lens), H=heads, d=d, branching=br, prefix_min=0, prefix_max=max(max(lens), 1), cfg_id=cfg_id)
    inp = attention_inputs(w, seed=1, lens=lens)
    ad = H.AttnDevice(inp)
    view = binding.slice_mask(binding.build_mask(br), len(br))
    n, mp = view.n_nodes, ad.max_prefix
    ws = binding.new_workspace(binding.tree_attention_tuned_workspace(tuning, 0, ad.B, heads, heads, d, n, row0, mp))
    for _ in range(2):                                  # the second call finds the workspace as the first left it
        ad.out.fill_(float("nan"))
        binding.tree_attention_tuned(tuning, view, 0, 0, 1.0, 1.0, ad.B, heads, heads, d, row0, ad.q, ad.kt, ad.vt, ad.node_stride, ad.kp,
                                     ad.vp, ad.base, ad.lens, ad.head_stride, mp, ad.scale, ad.out, ws)
        got = ad.out[:, :, row0:n].cpu().numpy().astype(np.float64)
        want = oracle.tree_attention(inp, oracle.build_mask(br), n)[:, :, row0:]
        H.assert_close(got, want, "f32", f"{br} d={d} lens={lens} row0={row0}")
        assert torch.isnan(ad.out[:, :, :row0]).all()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("br", [(1,), (3, 4), (4, 3), (16,), (17,), (2, 31), (8, 2, 2, 1, 1), (4, 31)])
def test_query_and_tree_tiles(binding, oracle, H, br, d):
    _check(binding, oracle, H, br, 3, d, (0, 1, 15, 16, 17, 63, 64, 65, 200))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("splits,fold", [(2, 0), (3, 0), (3, 1), (7, 0), (64, 0), (64, 1)])
def test_key_splits(binding, oracle, H, d, splits, fold):
    tu = binding.AttentionTuning(key_splits=splits, fold=fold)
    for heads in (8, 3):
        _check(binding, oracle, H, (4, 2, 2, 1), heads, d, (0, 5, 100, 1030), tuning=tu)
        _check(binding, oracle, H, (4, 2, 2, 1), heads, d, (77, 640), row0=21, tuning=tu)
