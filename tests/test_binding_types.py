"""The natively marshalled calls take the structures they are declared with and nothing that merely is as long (no GPU needed:
the argument is refused before anything is called)."""
import ctypes as C

import pytest
import torch

from paper_2409_10644_amd import binding as b

WRONG = [b.Mlp(), b.AttentionPlan(), (C.c_char * 4096)(), bytearray(4096), None, 7]


def _calls(structure):
    t = torch.zeros(8)
    head = (1, 1, 4, 64)
    tail = (t, t, 14, t, t, t, t, 64, 8, 0.1, t)
    return {
        "tree_attention": lambda: b.tree_attention(structure, 0, 1, 4, 64, t, *tail, t),
        "tree_attention_rows": lambda: b.tree_attention_rows(structure, 0, 1, 4, 64, 0, t, *tail, t),
        "tree_attention_gqa": lambda: b.tree_attention_gqa(structure, 0, 1, 4, 4, 64, 0, t, *tail, t),
        "tree_attention_static": lambda: b.tree_attention_static(structure, 0, 1, 4, 64, t, *tail),
        "tree_attention_fp8kv": lambda: b.tree_attention_fp8kv(structure, 1, 4, 4, 0, t, t, t, 14, t, t, 1.0, 1.0, t, t, 64, 8, 0.1, t, t),
        "verify_tree": lambda: b.verify_tree(structure, 0, 1, 8, t, t, t, 8, 8, t, t, 1, t, t, t, t),
        "verify_tree_sampling": lambda: b.verify_tree_sampling(structure, 0, 0, 1, 8, t, t, t, 8, 8, t, t, 1, t, t, t, t),
        "commit_path": lambda: b.commit_path(structure, 0, 1, 4, 64, [t], [t], 14, [t], [t], t, 64, 8, 16, t, t, t, t, 1, 1, t, t, t),
    }, {
        "early_stop_distribution": lambda: b.early_stop_distribution(structure, 1, 1, 8, 1, t, 8, 8, 0.4, None, t, t),
        "early_stop_hidden": lambda: b.early_stop_hidden(structure, 1, 1, t, 8, 8, 0.4, t, t),
    }


@pytest.mark.parametrize("wrong", WRONG, ids=lambda w: type(w).__name__)
def test_another_structure_is_refused(wrong):
    with_view, with_mlp = _calls(wrong)
    for name, call in with_view.items():
        with pytest.raises((C.ArgumentError, TypeError)):
            call()
    if not isinstance(wrong, b.Mlp):
        for name, call in with_mlp.items():
            with pytest.raises((C.ArgumentError, TypeError)):
                call()


def test_a_mask_view_is_no_network():
    view = b.slice_mask(b.build_mask((2, 2)), 2)         # 80 bytes, a network's description is 72
    for call in _calls(view)[1].values():
        with pytest.raises(C.ArgumentError):
            call()
